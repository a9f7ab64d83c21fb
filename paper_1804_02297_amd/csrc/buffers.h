// Buffers that belong together: all of them are there, or none is.
#pragma once

#include <cstddef>
#include <initializer_list>
#include <utility>

#include "../../include/ls.h"

namespace ls {

// Buf: alloc(bytes) releases what the buffer held before and reports LS_ENOMEM with
// nothing held; release() gives it back.

// Each buffer at its size; none of them if one fails, so that code which looks at one
// buffer (or at a mark it set) to see whether the group is there is never wrong.
template <class Buf>
ls_status alloc_all(std::initializer_list<std::pair<Buf*, size_t>> group) {
  for (const auto& a : group) {
    const ls_status st = a.first->alloc(a.second);
    if (st == LS_OK) continue;
    for (const auto& r : group) r.first->release();
    return st;
  }
  return LS_OK;
}

// Vectors of the GPU block solves, grown on demand.
template <class Buf>
struct SolveWork {
  Buf X, Z, U;        // the vectors [N][nrhs], the forward results, the fronts' update vectors
  int cap_rhs = 0;    // right-hand sides all three hold

  ls_status reserve(int nrhs, size_t vec_bytes, size_t update_bytes) {
    if (nrhs <= cap_rhs) return LS_OK;
    cap_rhs = 0;      // until all three are there
    const ls_status st =
        alloc_all<Buf>({{&X, vec_bytes * nrhs}, {&Z, vec_bytes * nrhs}, {&U, update_bytes * nrhs}});
    if (st == LS_OK) cap_rhs = nrhs;
    return st;
  }
};

}  // namespace ls
