// Vectors of the GPU block solves, grown on demand.
#pragma once

#include <cstddef>

#include "../../include/ls.h"

namespace ls {

// Buf: a buffer whose alloc(bytes) releases what it held before and reports LS_ENOMEM
// with nothing held.
template <class Buf>
struct SolveWork {
  Buf X, Z, U;        // the vectors [N][nrhs], the forward results, the fronts' update vectors
  int cap_rhs = 0;    // right-hand sides all three hold

  ls_status reserve(int nrhs, size_t vec_bytes, size_t update_bytes) {
    if (nrhs <= cap_rhs) return LS_OK;
    cap_rhs = 0;      // until all three are there: one that failed leaves the others of any size
    ls_status st = X.alloc(vec_bytes * nrhs);
    if (st == LS_OK) st = Z.alloc(vec_bytes * nrhs);
    if (st == LS_OK) st = U.alloc(update_bytes * nrhs);
    if (st == LS_OK) cap_rhs = nrhs;
    return st;
  }
};

}  // namespace ls
