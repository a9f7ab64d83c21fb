// GPU multifrontal LU of the sparsified system S and its block solves.
//
// Paper: the assembled local rows form a sparse system that is factored by
// nested dissection and used as the preconditioner (end of Section 3.1;
// costs in Section 3.3).  The dissection is the host solver's (nd_tree.h);
// here every front lives in HBM and a whole level of the tree is processed
// by each launch (grid.y or grid.z runs over the level's fronts).
//
// Factorisation of a level:
//   merge the children's update blocks (child 0, then child 1: their targets
//   overlap) into the fronts; assemble S's entries; then for each
//   48-column step kb of the pivot block:
//     diag_kernel   LU of the 48 x 48 diagonal tile, pivots searched among
//                   the tile's rows
//     panel_kernel  L below the tile (l U = f) and U right of it (L u = P f),
//                   by substitution
//     schur_kernel  F -= L U on the trailing block, complex product on
//                   MFMA (v_mfma_*_16x16x4, FP32 or FP64)
//   and copy the pivot rows and the boundary rows' pivot columns out.
// Pivoting inside 48-row tiles (a multiple of the three unknowns of a
// point) reproduces the host solver's partial pivoting over the whole pivot
// block to rounding on the tested media: the pivots of S sit in each
// point's own 3 x 3 diagonal block.
//
// Tile permutations are not applied to the L part left of the tile: the
// forward solve applies a tile's permutation to its rows right before the
// tile is solved, after every earlier tile has updated them.
//
// Solves (many right-hand sides): vectors in elimination order (each
// node's pivots contiguous), right-hand side fastest, real and imaginary
// parts in separate planes.  Forward by levels from the leaves: add the
// children's update vectors, then per tile z = L^-1 P x and a right-looking
// update of the rows below (pivot rows in place, boundary rows into the
// node's update vector).  Backward from the root: subtract U12 x_boundary,
// then per tile (last first) x = U^-1 z and the update of the rows above.
#include "buffers.h"
#include "gpu_solver.h"
#include "gpu_symbolic.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <limits>
#include <functional>
#include <memory>
#include <new>
#include <system_error>
#include <thread>
#include <utility>
#include <vector>

#include "nd_tree.h"

namespace ls {

namespace {

constexpr int kRB = 64;    // rows or columns per workgroup in the panel and solve kernels
constexpr int kSR = 64;    // right-hand sides per workgroup in the solve kernels
constexpr int kKC = 32;    // boundary columns per LDS chunk of the U12 product
constexpr int kKS = 512;   // boundary columns per workgroup of the U12 product (split over workgroups)


// ---- MFMA operand conventions -------------------------------------------------------
// v_mfma_{f32,f64}_16x16x4 (wave64): A lane l holds A[l % 16][l / 16], B lane l holds
// B[l / 16][l % 16].  The 16 x 16 result sits in 4 registers per lane: the f32 form
// holds D[4 (l / 16) + r][l % 16] in register r, the f64 form D[4 r + l / 16][l % 16].
template <typename R>
struct Mma;
template <>
struct Mma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 op(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <>
struct Mma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 op(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};

// ---- factorisation kernels ------------------------------------------------------------

// S's entries into the fronts of a level; each entry of S belongs to exactly
// one front position, so plain additions do not collide.
template <typename R, int NC>
__global__ __launch_bounds__(256) void assemble_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                       int nlvl, const int* __restrict__ ib,
                                                       const C<double>* __restrict__ rows, R* __restrict__ buf) {
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const int npp = d.np / NC, nbp = d.nb / NC;
    const long nf = d.nf;
    R* Fr = buf + d.f;
    R* Fi = Fr + nf * nf;
    const long work = (long)(npp + nbp) * 27;
    for (long w = (long)blockIdx.x * blockDim.x + threadIdx.x; w < work; w += (long)gridDim.x * blockDim.x) {
      const int a = (int)(w / 27), slot = (int)(w % 27);
      int pt, lj;
      if (a < npp) {
        pt = ib[d.e0 + NC * a];                         // perm (at offset 0): component 0 of point a
        lj = ib[d.am + 27L * a + slot];
      } else {
        pt = ib[d.bp + (a - npp)];
        lj = ib[d.ab + 27L * (a - npp) + slot];
      }
      if (lj < 0) continue;
#pragma unroll
      for (int r = 0; r < NC; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const C<double> v = rows[(((long)pt * NC + r) * 27 + slot) * NC + c];
          const long o = ((long)NC * a + r) * nf + (long)NC * lj + c;
          Fr[o] += (R)v.re;
          Fi[o] += (R)v.im;
        }
    }
  }
}

// The fronts of a level from their children's update blocks, child 0 then
// child 1, zero where neither reaches (child_map_kernel's cinv); every entry is
// written once, a row per wave.  Memory-bound: clearing the level and adding
// each child into it read and wrote the fronts twice more (complete n = 29
// set-up, FP64: 3.9 ms, now 2.6).
template <typename R, int NC>
__global__ __launch_bounds__(256) void merge_children_kernel(const FrontDev* __restrict__ fr,
                                                             const int* __restrict__ lvl, int nlvl,
                                                             const int* __restrict__ cinv, const R* __restrict__ cbuf,
                                                             R* __restrict__ buf) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const int nf = d.nf, np = nf / NC;
    const int* m0 = cinv + d.ci;
    const int* m1 = m0 + np;
    struct Child {
      const R *re, *im;   // the update block
      long ld;
    };
    const auto child = [&](int id) {
      if (id < 0) return Child{cbuf, cbuf, 0};
      const FrontDev c = fr[id];
      const long cnf = c.nf;
      const R* p = cbuf + c.f + c.np * cnf + c.np;
      return Child{p, p + cnf * cnf, cnf};
    };
    const Child a = child(d.child[0]), b = child(d.child[1]);
    R* Fr = buf + d.f;
    R* Fi = Fr + (long)nf * nf;
    for (int i = blockIdx.x * 4 + wv; i < nf; i += gridDim.x * 4) {
      const int ea = m0[i / NC], eb = m1[i / NC], k = i % NC;
      const long oa = (NC * (long)ea + k) * a.ld, ob = (NC * (long)eb + k) * b.ld;
#pragma unroll 4
      for (int j = lane; j < nf; j += 64) {
        const int p = j / NC, kj = j - p * NC;
        const int fa = ea < 0 ? -1 : m0[p], fb = eb < 0 ? -1 : m1[p];
        R vr = R(0), vi = R(0);
        if (fa >= 0) {
          vr = a.re[oa + NC * fa + kj];
          vi = a.im[oa + NC * fa + kj];
        }
        if (fb >= 0) {
          vr += b.re[ob + NC * fb + kj];
          vi += b.im[ob + NC * fb + kj];
        }
        Fr[(long)i * nf + j] = vr;
        Fi[(long)i * nf + j] = vi;
      }
    }
  }
}

// Lane-swap instructions: swap32 exchanges lanes 32.. of a with lanes 0..31 of b,
// swap16 the odd rows of 16 lanes of a with the even rows of b.
__device__ __forceinline__ void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
template <typename F>
__device__ __forceinline__ void swap_halves(double& a, double& b, F f) {
  float al = __int_as_float(__double2loint(a)), ah = __int_as_float(__double2hiint(a));
  float bl = __int_as_float(__double2loint(b)), bh = __int_as_float(__double2hiint(b));
  f(al, bl);
  f(ah, bh);
  a = __hiloint2double(__float_as_int(ah), __float_as_int(al));
  b = __hiloint2double(__float_as_int(bh), __float_as_int(bl));
}
__device__ __forceinline__ void swap32(double& a, double& b) {
  swap_halves(a, b, [](float& x, float& y) { swap32(x, y); });
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  swap_halves(a, b, [](float& x, float& y) { swap16(x, y); });
}

// Largest of v over a wave, in every lane: rotations inside the rows of 16
// lanes, then the two lane-swap instructions across rows.
template <int ROT>
__device__ __forceinline__ float row_ror(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + ROT, 0xF, 0xF, false));
}
template <int ROT>
__device__ __forceinline__ double row_ror(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + ROT, 0xF, 0xF, false),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + ROT, 0xF, 0xF, false));
}
template <typename R>
__device__ __forceinline__ R wave_max(R v) {
  v = fmax(v, row_ror<8>(v));
  v = fmax(v, row_ror<4>(v));
  v = fmax(v, row_ror<2>(v));
  v = fmax(v, row_ror<1>(v));
  R w = v;
  swap16(v, w);
  v = fmax(v, w);
  w = v;
  swap32(v, w);
  return fmax(v, w);
}

__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// LU with partial pivoting of the diagonal tile [kb, kb + tw)^2 of every front
// of a level, one workgroup per front.
// What bounds it: 48 dependent elimination steps in one workgroup, launched
// 126 times one after another in an n = 29 factor; a step's time is its
// instruction count, one wave per SIMD.  So the tile is taken in three panels
// of 16 columns, a lane per row and the panel's columns in registers: a step
// needs no LDS and no barrier (the pivot row is read from its lane, rows are
// exchanged by renaming, lpos, instead of moving them).  Every wave factors the panel for
// itself and updates four columns of each later panel; the panels meet in
// LDS, two barriers each.  The tile's inverses, which only the solves need,
// are formed for a whole level at once (tile_inverse_kernel).  FP64, average
// launch of the n = 29 factor: 36 us (204 us with the tile in LDS, six barriers
// a step and the inverses in the same launch); FP32 30 us (219 us).
template <typename R>
__global__ __launch_bounds__(256) void diag_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl, int nlvl,
                                                   int kb, R* __restrict__ buf, int* __restrict__ ib) {
  static_assert(kT == 48, "three panels of 16 columns, 48 rows in the lanes of a wave");
  __shared__ R Sr[kT][kT + 1], Si[kT][kT + 1];   // the tile, rows as loaded
  __shared__ int rowof[kT];                      // position in pivot order -> row as loaded
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = min(lane, kT - 1);
  for (int q = blockIdx.x; q < nlvl; q += gridDim.x) {
    const FrontDev d = fr[lvl[q]];
    if (kb >= d.np) continue;
    const int tw = min(kT, d.np - kb);
    const long nf = d.nf;
    R* Fr = buf + d.f + kb * nf + kb;
    R* Fi = Fr + nf * nf;
    __syncthreads();                             // the previous front's LDS reads are done
#pragma unroll
    for (int u = 0; u < kT * kT / 256; ++u) {
      const int o = tid + 256 * u, i = o / kT, c = o % kT;
      const bool in = i < tw && c < tw;
      Sr[i][c] = in ? Fr[i * nf + c] : R(0);
      Si[i][c] = in ? Fi[i * nf + c] : R(0);
    }
    __syncthreads();
    R tr[2][4], ti[2][4];                        // this wave's columns of panels 1 and 2
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        tr[g][c] = Sr[row][16 * (g + 1) + 4 * wave + c];
        ti[g][c] = Si[row][16 * (g + 1) + 4 * wave + c];
      }
    int lpos = lane;                             // place of this lane's row in pivot order
    for (int pb = 0; pb < 3; ++pb) {
      R ar[16], ai[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        ar[c] = Sr[row][16 * pb + c];
        ai[c] = Si[row][16 * pb + c];
      }
      static_for<0, 16>([&](auto JJ) {              // a constant column index keeps the panel in registers
        constexpr int jj = decltype(JJ)::value;
        const int j = 16 * pb + jj;
        if (j >= tw) return;
        // the pivot: largest |x|^2 among the rows not yet used, the first of them in pivot order
        const R xr = ar[jj], xi = ai[jj];
        const bool cand = lpos >= j && lpos < tw;
        const R v = cand ? xr * xr + xi * xi : R(-1);
        const R best = wave_max(v);
        unsigned long long eq = __ballot(cand && v == best);
        if (eq == 0) eq = __ballot(lpos == j);   // NaN only
        int prow = __ffsll(eq) - 1;
        for (unsigned long long m = eq & (eq - 1); m; m &= m - 1) {
          const int o = __ffsll(m) - 1;
          if (__builtin_amdgcn_readlane(lpos, o) < __builtin_amdgcn_readlane(lpos, prow)) prow = o;
        }
        prow = __builtin_amdgcn_readfirstlane(prow);
        const int pp = __builtin_amdgcn_readlane(lpos, prow);
        lpos = lpos == j ? pp : lpos == pp ? j : lpos;
        R pr = lane_value(xr, prow), pi = lane_value(xi, prow);
        if (pr == R(0) && pi == R(0)) {          // exactly singular tile: perturb (FGMRES absorbs it)
          pr = sqrt(std::numeric_limits<R>::min());
          if (lane == prow) ar[jj] = pr;
        }
        const R den = pr * pr + pi * pi;
        const R ir = pr / den, ii = -pi / den;
        const bool below = lpos > j;
        const R lr = below ? xr * ir - xi * ii : R(0), li = below ? xr * ii + xi * ir : R(0);
        ar[jj] = below ? lr : ar[jj];
        ai[jj] = below ? li : ai[jj];
        auto update = [&](R& xr, R& xi) {        // x -= l u, u this column's value in the pivot row
          const R ur = lane_value(xr, prow), ui = lane_value(xi, prow);
          xr = fma(li, ui, fma(-lr, ur, xr));
          xi = fma(-li, ur, fma(-lr, ui, xi));
        };
#pragma unroll
        for (int c = jj + 1; c < 16; ++c) update(ar[c], ai[c]);
        if (pb < 1)
#pragma unroll
          for (int c = 0; c < 4; ++c) update(tr[0][c], ti[0][c]);
        if (pb < 2)
#pragma unroll
          for (int c = 0; c < 4; ++c) update(tr[1][c], ti[1][c]);
      });
      __syncthreads();                           // every wave has read this panel
      if (lane < kT) {
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if (c >> 2 == wave) {                  // the finished panel, and the next one as updated
            Sr[lane][16 * pb + c] = ar[c];
            Si[lane][16 * pb + c] = ai[c];
          }
        if (pb < 2)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            Sr[lane][16 * (pb + 1) + 4 * wave + c] = pb == 0 ? tr[0][c] : tr[1][c];
            Si[lane][16 * (pb + 1) + 4 * wave + c] = pb == 0 ? ti[0][c] : ti[1][c];
          }
      }
      __syncthreads();
    }
    if (wave == 0 && lane < kT) {
      rowof[lpos] = lane;
      if (lane < tw) ib[d.pv + kb + lpos] = lane;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kT * kT / 256; ++u) {
      const int o = tid + 256 * u, i = o / kT, c = o % kT;
      if (i < tw && c < tw) {
        Fr[i * nf + c] = Sr[rowof[i]][c];
        Fi[i * nf + c] = Si[rowof[i]][c];
      }
    }
  }
}

// L^-1 (unit lower) and U^-1 (upper) of every factored 48 x 48 tile of a
// level's fronts (grid.x fronts, grid.y tiles), for the solves' super-blocks.
// Both advance together, one row of each per barrier, as rank-1 updates of
// register tiles (thread (ti, tj) of 16 x 16 owns rows ti + 16 a, columns
// tj + 16 b).  48 dependent steps: about 45 us for a
// launch that the chip holds at once, one a level (FP64, the nine levels of an
// n = 29 factor: 54 us on average).  40 KB of LDS in FP64 let four workgroups
// share a CU, so a level of more than about 1000 tiles takes that several times
// over (2-D n = 959: 268 us on average).
template <typename R>
__global__ __launch_bounds__(256) void tile_inverse_kernel(const FrontDev* __restrict__ fr,
                                                           const int* __restrict__ lvl, int nlvl,
                                                           const R* __restrict__ buf, R* __restrict__ fac) {
  __shared__ R Dr[kT][kT + 1], Di[kT][kT + 1];
  __shared__ R xlr[2][kT], xli[2][kT], xur[2][kT], xui[2][kT];
  const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
  const int kb = blockIdx.y * kT;
  for (int q = blockIdx.x; q < nlvl; q += gridDim.x) {
    const FrontDev d = fr[lvl[q]];
    if (kb >= d.np) continue;
    const int tw = min(kT, d.np - kb);
    const long nf = d.nf;
    const R* Fr = buf + d.f + kb * nf + kb;
    const R* Fi = Fr + nf * nf;
    __syncthreads();                             // the previous front's LDS reads are done
    for (int o = tid; o < kT * kT; o += 256) {
      const int i = o / kT, c = o % kT;
      const bool in = i < tw && c < tw;
      Dr[i][c] = in ? Fr[i * nf + c] : R(0);
      Di[i][c] = in ? Fi[i * nf + c] : R(0);
    }
    // L^-1 rows k ascending: X[k][c] = -sum_{c <= l < k} L[k][l] X[l][c]; U^-1 rows e descending:
    // X[e][c] = (delta_ec - sum_{e < l <= c} U[e][l] X[l][c]) / U[e][e].  sl, su: the running sums.
    R slr[3][3] = {}, sli[3][3] = {}, sur[3][3] = {}, sui[3][3] = {};
    R* T = fac + d.t + (long)(kb / kT) * 4 * kTileElems;
    __syncthreads();
#pragma unroll
    for (int ka = 0; ka < 3; ++ka) {
      for (int kt = 0; kt < 16; ++kt) {
        const int k = 16 * ka + kt, e = tw - 1 - k, p = k & 1;
        if (k >= tw) break;
        if (ti == kt) {
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const int c = tj + 16 * b;
            const R vr = c < k ? -slr[ka][b] : c == k ? R(1) : R(0);
            const R vi = c < k ? -sli[ka][b] : R(0);
            xlr[p][c] = vr;
            xli[p][c] = vi;
            if (c < tw) {
              T[k * kT + c] = vr;
              T[kTileElems + k * kT + c] = vi;
            }
          }
        }
        if (ti == (e & 15)) {
          const R ur = Dr[e][e], ui = Di[e][e];
          const R dd = ur * ur + ui * ui;
          const R gr = ur / dd, gi = -ui / dd;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const int c = tj + 16 * b, ea = e >> 4;
            const R sr = ea == 0 ? sur[0][b] : ea == 1 ? sur[1][b] : sur[2][b];
            const R si = ea == 0 ? sui[0][b] : ea == 1 ? sui[1][b] : sui[2][b];
            const R nr = c == e ? R(1) : -sr, ni = c == e ? R(0) : -si;
            const R vr = c < e ? R(0) : nr * gr - ni * gi;
            const R vi = c < e ? R(0) : nr * gi + ni * gr;
            xur[p][c] = c < tw ? vr : R(0);
            xui[p][c] = c < tw ? vi : R(0);
            if (c < tw) {
              T[2 * kTileElems + e * kT + c] = vr;
              T[3 * kTileElems + e * kT + c] = vi;
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int r = ti + 16 * a;
          const bool lo = r > k && r < tw, up = r < e;
          const R dlr = lo ? Dr[r][k] : R(0), dli = lo ? Di[r][k] : R(0);
          const R dur = up ? Dr[r][e] : R(0), dui = up ? Di[r][e] : R(0);
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const int c = tj + 16 * b;
            slr[a][b] += dlr * xlr[p][c] - dli * xli[p][c];
            sli[a][b] += dlr * xli[p][c] + dli * xlr[p][c];
            sur[a][b] += dur * xur[p][c] - dui * xui[p][c];
            sui[a][b] += dur * xui[p][c] + dui * xur[p][c];
          }
        }
      }
    }
  }
}

// Rows (columns) per workgroup of the panel kernel.
constexpr int kPR = 64;   // 256 threads load kPR x kT values in kT / 4 rounds

// Workgroups [0, half): the L part below the tile by substitution, l U = f
// for kPR rows (U the tile's upper factor).  Workgroups [half, 2 half): the U
// part right of it, L u = P f for kPR columns (L the tile's unit lower factor,
// P its row permutation).  Substitution rather than the tile's explicit
// inverse keeps the panel backward stable.
// What bounds it: the 48 dependent steps of a row.  Four neighbouring lanes
// share a row (column) in registers, lane q the unknowns 4 m + q, so a step is
// one lane's product, a broadcast inside the quad and at most twelve updates a
// lane; the tile is read from LDS a quad's 4 values at a time, the reciprocals
// of the diagonal are formed once, and every load is in flight before the first
// wait.  FP64, average launch of the n = 29 factor: 38 us (152 us with one
// thread per row and the row in LDS).
// A reciprocal is held as the sum of two values (recip): a product with the
// rounded reciprocal alone has one rounding more per entry of L than a division.
// A lane forms each once, while the rows are on their way through LDS (formed
// where the tile is stored, by the lane that holds the value, 40 us).
template <int Q>
__device__ __forceinline__ float quad_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), Q * 0x55, 0xF, 0xF, false));
}
template <int Q>
__device__ __forceinline__ double quad_bcast(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), Q * 0x55, 0xF, 0xF, false),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), Q * 0x55, 0xF, 0xF, false));
}
// 1 / u to about twice the precision of R: g, and the rest h = g (1 - g u).
template <typename R>
__device__ __forceinline__ void recip(R ur, R ui, C<R>& g, C<R>& h) {
#pragma clang fp contract(off)
  const R den = ur * ur + ui * ui;
  g = cmk(ur / den, -ui / den);
  // 1 - g u: exact products, the larger part of the sum taken from 1 first
  const R a = g.re * ur, b = -g.im * ui, c = g.re * ui, d = g.im * ur;
  const R ea = fma(g.re, ur, -a), eb = fma(-g.im, ui, -b), ec = fma(g.re, ui, -c), ed = fma(g.im, ur, -d);
  const bool al = a >= b;
  const R er = ((R(1) - (al ? a : b)) - (al ? b : a)) - (ea + eb), ei = -(c + d) - (ec + ed);
  h = cmk(g.re * er - g.im * ei, g.re * ei + g.im * er);
}

template <typename R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 3 : 2))) void panel_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                    int nlvl, int kb, int half, R* __restrict__ buf,
                                                    const int* __restrict__ ib) {
  // T[j][c]: U[j][c] for the rows, L[c][j] for the columns, zero at and left of the diagonal
  // and past the tile; g, h: 1 / U[j][j] (rows) and its rest
  __shared__ R Tr[kT][kT], Ti[kT][kT];
  __shared__ C<R> g[kT], h[kT];
  __shared__ R Bs[kPR][kT + 1];                  // one plane of the rows at a time (two workgroups per CU in FP64)
  const int tid = threadIdx.x, row = tid >> 2, qd = tid & 3;
  const bool lrole = (int)blockIdx.x < half;
  const long blk = lrole ? blockIdx.x : blockIdx.x - half;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    if (kb >= d.np) continue;
    const int tw = min(kT, d.np - kb);
    const long ke = kb + tw, nf = d.nf;
    const long x0 = ke + blk * kPR;
    if (x0 >= nf) continue;
    const int cnt = (int)min((long)kPR, nf - x0);
    R* Fr = buf + d.f;
    R* Fi = Fr + nf * nf;
    // every load is issued before the first wait: the rows (columns) and the tile
    R br[kT / 4], bi[kT / 4], vr[kT * kT / 256], vi[kT * kT / 256];
    int pk[kT / 4];
#pragma unroll
    for (int m = 0; m < kT / 4; ++m) pk[m] = lrole ? 0 : ib[d.pv + kb + min((tid >> 6) + 4 * m, tw - 1)];
#pragma unroll
    for (int u = 0; u < kT * kT / 256; ++u) {
      const int o = tid + 256 * u, i = o / kT, c = o % kT;
      const long src = min(i, tw - 1) * nf + min(c, tw - 1);
      vr[u] = Fr[kb * nf + kb + src];
      vi[u] = Fi[kb * nf + kb + src];
    }
#pragma unroll
    for (int m = 0; m < kT / 4; ++m) {
      // rows: 48 values each, kPR * kT / 256 = 12 loads a thread; columns: row (tid >> 6) + 4 m, column tid & 63
      const int o = tid + 256 * m, i = lrole ? o / kT : tid & 63, k = lrole ? o % kT : (tid >> 6) + 4 * m;
      const long src = lrole ? (x0 + min(i, cnt - 1)) * nf + kb + min(k, tw - 1)
                             : (kb + pk[m]) * nf + x0 + min(i, cnt - 1);
      br[m] = Fr[src];
      bi[m] = Fi[src];
    }
    __syncthreads();                              // the previous front's LDS reads are done
#pragma unroll
    for (int u = 0; u < kT * kT / 256; ++u) {
      const int o = tid + 256 * u, i = o / kT, c = o % kT;   // F row i, column c
      const int j = lrole ? i : c, k = lrole ? c : i;
      const bool in = k > j && k < tw;
      Tr[j][k] = in ? vr[u] : R(0);
      Ti[j][k] = in ? vi[u] : R(0);
      if (k == j) g[k] = cmk(vr[u], vi[u]);
    }
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
#pragma unroll
      for (int m = 0; m < kT / 4; ++m) {
        const int o = tid + 256 * m, i = lrole ? o / kT : tid & 63, k = lrole ? o % kT : (tid >> 6) + 4 * m;
        Bs[i][k] = i < cnt && k < tw ? (pl ? bi : br)[m] : R(0);
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < kT / 4; ++m) (pl ? bi : br)[m] = Bs[row][4 * m + qd];
      if (pl == 0 && tid < kT) {                  // the diagonal's reciprocals, a lane each
        C<R> gk = cmk(tid < tw ? R(1) : R(0), R(0)), hk = cmk(R(0), R(0));
        if (lrole && tid < tw) recip(g[tid].re, g[tid].im, gk, hk);
        g[tid] = gk;
        h[tid] = hk;
      }
      __syncthreads();
    }
    // step j = 4 M + Q: x_j = f_j / T_jj, then f_c -= x_j T[j][c] for c > j (T is zero elsewhere)
    auto step = [&](auto M, auto Q) {
      constexpr int m0 = decltype(M)::value, q0 = decltype(Q)::value, j = 4 * m0 + q0;
      const R zr = quad_bcast<q0>(br[m0]), zi = quad_bcast<q0>(bi[m0]);
      const C<R> w = g[j], e = h[j];
      const R xr = fma(zr, w.re, fma(-zi, w.im, fma(zr, e.re, -(zi * e.im))));
      const R xi = fma(zr, w.im, fma(zi, w.re, fma(zr, e.im, zi * e.re)));
      if (qd == q0) {
        br[m0] = xr;
        bi[m0] = xi;
      }
#pragma unroll
      for (int m = m0; m < kT / 4; ++m) {
        const R tr = Tr[j][4 * m + qd], t2 = Ti[j][4 * m + qd];
        br[m] -= xr * tr - xi * t2;
        bi[m] -= xr * t2 + xi * tr;
      }
    };
    static_for<0, kT / 4>([&](auto M) { static_for<0, 4>([&](auto Q) { step(M, Q); }); });
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
      R* F = pl ? Fi : Fr;
      if (pl) __syncthreads();
#pragma unroll
      for (int m = 0; m < kT / 4; ++m) Bs[row][4 * m + qd] = (pl ? bi : br)[m];
      __syncthreads();
      if (lrole) {
        for (int o = tid; o < cnt * kT; o += 256) {
          const int i = o / kT, k = o % kT;
          if (k < tw) F[(x0 + i) * nf + kb + k] = Bs[i][k];
        }
      } else {
        for (int o = tid; o < kPR * tw; o += 256) {
          const int k = o / kPR, j = o % kPR;
          if (j < cnt) F[(kb + k) * nf + x0 + j] = Bs[j][k];
        }
      }
    }
  }
}

// Complex tile product acc += A B on MFMA: A [..][lda] (rows x K) and B
// [K][ldb] in LDS, K a multiple of 4; a wave owns the 16 NA x 16 NB part at
// (wm, wn).  The two products of one accumulator are issued apart (back to
// back the second waits for the first).
template <typename R, int NA, int NB>
__device__ __forceinline__ void cmma64(const R* Ar, const R* Ai, int lda, const R* Br, const R* Bi, int ldb, int K,
                                       int wm, int wn, int lane, typename Mma<R>::v4 (&cr)[NA][NB],
                                       typename Mma<R>::v4 (&ci)[NA][NB]) {
  for (int k4 = 0; k4 < K; k4 += 4) {
    const int kr = k4 + (lane >> 4);
    R ar[NA], ai[NA], br[NB], bi[NB];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      ar[a] = Ar[(wm + 16 * a + (lane & 15)) * lda + kr];
      ai[a] = Ai[(wm + 16 * a + (lane & 15)) * lda + kr];
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      br[b] = Br[kr * ldb + wn + 16 * b + (lane & 15)];
      bi[b] = Bi[kr * ldb + wn + 16 * b + (lane & 15)];
    }
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        cr[a][b] = Mma<R>::op(ar[a], br[b], cr[a][b]);
        ci[a][b] = Mma<R>::op(ar[a], bi[b], ci[a][b]);
      }
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        cr[a][b] = Mma<R>::op(-ai[a], bi[b], cr[a][b]);
        ci[a][b] = Mma<R>::op(ai[a], br[b], ci[a][b]);
      }
  }
}

// The same 64 x 64 complex product for the solve kernels, accumulated in a
// form chosen by precision: FP32 takes three real products per complex
// multiply-add (ArBr, AiBi and (Ar + Ai)(Br + Bi); re = ArBr - AiBi, im = the
// third minus the other two), three quarters of the MFMAs; FP64 keeps the
// four products of cmma64 (and its rounding).
template <typename R, int NBW = 2, int NAW = 2>   // 16-column B tiles, 16-row A tiles per wave
struct CAcc {
  typedef typename Mma<R>::v4 v4;
  static constexpr bool G3 = sizeof(R) == 4;
  v4 p[3][NAW][NBW];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int a = 0; a < NAW; ++a)
#pragma unroll
        for (int b = 0; b < NBW; ++b) p[q][a][b] = v4{R(0), R(0), R(0), R(0)};
  }
  __device__ __forceinline__ void mma(const R* Ar, const R* Ai, int lda, const R* Br, const R* Bi, int ldb, int K,
                                      int wm, int wn, int lane) {
    if constexpr (!G3) {
      cmma64<R, NAW, NBW>(Ar, Ai, lda, Br, Bi, ldb, K, wm, wn, lane, p[0], p[1]);
    } else {
      // two k steps at a time: a full unroll hoists every LDS load of the
      // chunk and leaves no registers for a second wave per SIMD
#pragma unroll 2
      for (int k4 = 0; k4 < K; k4 += 4) {
        const int kr = k4 + (lane >> 4);
        R ar[NAW], ai[NAW], br[NBW], bi[NBW];
#pragma unroll
        for (int a = 0; a < NAW; ++a) {
          ar[a] = Ar[(wm + 16 * a + (lane & 15)) * lda + kr];
          ai[a] = Ai[(wm + 16 * a + (lane & 15)) * lda + kr];
        }
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
          br[b] = Br[kr * ldb + wn + 16 * b + (lane & 15)];
          bi[b] = Bi[kr * ldb + wn + 16 * b + (lane & 15)];
        }
#pragma unroll
        for (int a = 0; a < NAW; ++a)
#pragma unroll
          for (int b = 0; b < NBW; ++b) {
            p[0][a][b] = Mma<R>::op(ar[a], br[b], p[0][a][b]);
            p[1][a][b] = Mma<R>::op(ai[a], bi[b], p[1][a][b]);
            p[2][a][b] = Mma<R>::op(ar[a] + ai[a], br[b] + bi[b], p[2][a][b]);
          }
      }
    }
  }
  __device__ __forceinline__ void result(v4 (&cr)[NAW][NBW], v4 (&ci)[NAW][NBW]) const {
#pragma unroll
    for (int a = 0; a < NAW; ++a)
#pragma unroll
      for (int b = 0; b < NBW; ++b) {
        if constexpr (G3) {
          cr[a][b] = p[0][a][b] - p[1][a][b];
          ci[a][b] = p[2][a][b] - p[0][a][b] - p[1][a][b];
        } else {
          cr[a][b] = p[0][a][b];
          ci[a][b] = p[1][a][b];
        }
      }
  }
};

// Schur updates F[rows][cols] -= F[rows][K] F[K][cols] on a TS x TS tile per
// workgroup (four waves of TS/2 x TS/2, the complex product as CAcc forms it:
// three real MFMA products in FP32, four in FP64).  With the 48-column step kb
// inside the outer block starting at kb0 (obe = min(kb0 + kOB, np)):
//   step:  rows [ke, nf), cols [ke, obe) (the first nbx x nby tiles) and
//          rows [ke, obe), cols [obe, nf) (as many again, x and y exchanged),
//          K = the step's columns
//   block: rows [obe, nf), cols [obe, nf), K = [kb0, obe)   (once per block)
// The steps keep the block's own columns and rows current for the next
// step; the rest of the trailing matrix is read by nothing inside the block,
// so its update waits and is applied once with K up to kOB.
// What bounds it: the block update the FP64 matrix cores, the step a chain of
// latencies at the top of the tree, so both its parts are one launch.  Why TS = 32:
// 112 VGPRs and 17 KB of LDS let four workgroups share a CU, and few tiles
// spread wider; with 64 x 64 tiles (226 VGPRs, two) the block update of two
// fronts of 3741 took 844 us (52 TFLOP/s) against 806, that of one of 2300 185
// against 146, the root's steps 2 x 20 against 8 to 16.  64 x 32 and 32 x 64 lie
// between; tile rows padded to a multiple of the eight XCDs lost 2%.  A complete
// n = 29 set-up's FP64 updates: 25.9 to 20.8 ms; FP32, n = 32: 20.5 to 18.2.  On
// larger fronts TS = 64 (kSchurCols): a 32 x 32 tile reads twice as much per product.
template <typename R, int TS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void schur_kernel(
    const FrontDev* __restrict__ fr, const int* __restrict__ lvl, int nlvl, int kb, int kb0, int nbx, int nby, bool step,
    R* __restrict__ buf) {
  typedef typename Mma<R>::v4 v4;
  constexpr int W = TS / 32;   // 16-tiles of a wave per dimension
  constexpr int U = TS / 16;   // chunk elements per thread and plane
  __shared__ R Ar[TS][17], Ai[TS][17];
  __shared__ R Br[16][TS + 1], Bi[16][TS + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (TS / 2), wn = (wave & 1) * (TS / 2);
  const int tiles = nbx * nby;
  const bool second = step && (int)blockIdx.x >= tiles;
  const int tile = second ? blockIdx.x - tiles : blockIdx.x;
  const int bx = tile % (second ? nby : nbx), by = tile / (second ? nby : nbx);
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const long nf = d.nf, obe = min((long)kb0 + kOB, (long)d.np);
    long r0, r1, c0, c1, k0, k1;
    if (!step) {
      if (kb0 >= d.np) continue;
      r0 = c0 = obe;
      r1 = c1 = nf;
      k0 = kb0;
      k1 = obe;
    } else {
      if (kb >= d.np) continue;
      k0 = kb;
      k1 = min((long)kb + kT, (long)d.np);
      r0 = k1;
      r1 = second ? obe : nf;
      c0 = second ? obe : k1;
      c1 = second ? nf : obe;
    }
    const long i0 = r0 + (long)TS * by, j0 = c0 + (long)TS * bx;
    if (i0 >= r1 || j0 >= c1) continue;
    const int tw = (int)(k1 - k0);
    const long kb_ = k0;
    R* Fr = buf + d.f;
    R* Fi = Fr + nf * nf;
    CAcc<R, W, W> acc;
    acc.zero();
    // the next 16-deep K chunk is loaded into registers while the MFMAs
    // consume the current one from LDS
    R par[U], pai[U], pbr[U], pbi[U];
    auto fetch = [&](int kc) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int o = tid + 256 * u;
        const int ii = o >> 4, kk = o & 15;
        const bool ok = i0 + ii < r1 && kc + kk < tw;
        const long src = (i0 + ii) * nf + kb_ + kc + kk;
        par[u] = ok ? Fr[src] : R(0);
        pai[u] = ok ? Fi[src] : R(0);
        const int kr = o / TS, jj = o % TS;
        const bool okb = kc + kr < tw && j0 + jj < c1;
        const long srcb = (kb_ + kc + kr) * nf + j0 + jj;
        pbr[u] = okb ? Fr[srcb] : R(0);
        pbi[u] = okb ? Fi[srcb] : R(0);
      }
    };
    fetch(0);
    for (int kc = 0; kc < tw; kc += 16) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int o = tid + 256 * u;
        Ar[o >> 4][o & 15] = par[u];
        Ai[o >> 4][o & 15] = pai[u];
        Br[o / TS][o % TS] = pbr[u];
        Bi[o / TS][o % TS] = pbi[u];
      }
      __syncthreads();
      if (kc + 16 < tw) fetch(kc + 16);
      acc.mma(&Ar[0][0], &Ai[0][0], 17, &Br[0][0], &Bi[0][0], TS + 1, 16, wm, wn, lane);
      __syncthreads();
    }
    v4 cr[W][W], ci[W][W];
    acc.result(cr, ci);
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
      for (int b = 0; b < W; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const long gi = i0 + wm + 16 * a + Mma<R>::row(lane, r), gj = j0 + wn + 16 * b + (lane & 15);
          if (gi < r1 && gj < c1) {
            Fr[gi * nf + gj] -= cr[a][b][r];
            Fi[gi * nf + gj] -= ci[a][b][r];
          }
        }
  }
}

// pivot rows and the boundary rows' pivot columns into the factor
template <typename R>
__global__ __launch_bounds__(256) void copyout_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                      int nlvl, const R* __restrict__ buf, R* __restrict__ fac) {
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const long nf = d.nf, np = d.np, nb = d.nb;
    const R* Fr = buf + d.f;
    const R* Fi = Fr + nf * nf;
    const long c1 = np * nf, c2 = nb * np;
    for (long w = (long)blockIdx.x * blockDim.x + threadIdx.x; w < c1; w += (long)gridDim.x * blockDim.x) {
      fac[d.p + w] = Fr[w];
      fac[d.p + c1 + w] = Fi[w];
    }
    for (long i = blockIdx.x; i < nb; i += gridDim.x)
      for (long j = threadIdx.x; j < np; j += blockDim.x) {
        fac[d.l + i * np + j] = Fr[(np + i) * nf + j];
        fac[d.l + c2 + i * np + j] = Fi[(np + i) * nf + j];
      }
  }
}

// ---- solve kernels --------------------------------------------------------------------

// b (complex128 [nrhs][N]) -> X ([N][nrhs] in elimination order, split planes);
// four unknowns per workgroup pass, the right-hand sides across 64 lanes
// Lanes of a 256-thread workgroup given to one row's right-hand sides (the
// smallest power of two >= nrhs, at most 64); the workgroup covers 256 / lanes
// rows per pass.  One rhs: a row per thread.
__host__ __device__ inline int rhs_lanes(int nrhs) {
  int l = 1;
  while (l < nrhs && l < 64) l *= 2;
  return l;
}

template <typename R>
__global__ __launch_bounds__(256) void sol_in_kernel(const C<double>* __restrict__ b, long N, int nrhs,
                                                     const int* __restrict__ perm, R* __restrict__ Xr,
                                                     R* __restrict__ Xi) {
  const int lanes = rhs_lanes(nrhs), rpp = 256 / lanes;
  for (long e = (long)blockIdx.x * rpp + threadIdx.x / lanes; e < N; e += (long)gridDim.x * rpp) {
    const long pe = perm[e];
    for (int r = threadIdx.x % lanes; r < nrhs; r += lanes) {
      const C<double> v = b[r * N + pe];
      Xr[e * nrhs + r] = (R)v.re;
      Xi[e * nrhs + r] = (R)v.im;
    }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void sol_out_kernel(C<double>* __restrict__ b, long N, int nrhs,
                                                      const int* __restrict__ perm, const R* __restrict__ Xr,
                                                      const R* __restrict__ Xi) {
  const int lanes = rhs_lanes(nrhs), rpp = 256 / lanes;
  for (long e = (long)blockIdx.x * rpp + threadIdx.x / lanes; e < N; e += (long)gridDim.x * rpp) {
    const long pe = perm[e];
    for (int r = threadIdx.x % lanes; r < nrhs; r += lanes)
      b[r * N + pe] = cmk((double)Xr[e * nrhs + r], (double)Xi[e * nrhs + r]);
  }
}

// The same two copies as tiled transposes through LDS, for many right-hand
// sides: a workgroup takes 64 natural unknowns p and 64 rhs r, reads b[r][p]
// along p and writes row ipm[p] of X along r, so both sides are whole runs
// (the per-row kernels above read or write 64 separate lines per row).
// ipm is the inverse of the elimination order: ipm[ib[e]] = e.
constexpr int kTP = 64;
constexpr int kSolTileRhs = 16;    // from this many rhs on the copies take the tiled kernels
__global__ void inv_perm_kernel(const int* __restrict__ perm, long N, int* __restrict__ ipm) {
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x)
    ipm[perm[e]] = (int)e;
}

template <typename R>
__global__ __launch_bounds__(256) void sol_in_tile_kernel(const C<double>* __restrict__ b, long N, int nrhs,
                                                          const int* __restrict__ ipm, R* __restrict__ Xr,
                                                          R* __restrict__ Xi) {
  __shared__ R tr[kTP][kTP + 1], ti[kTP][kTP + 1];   // [p][r]
  const long p0 = (long)blockIdx.x * kTP;
  const int r0 = blockIdx.y * kTP;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int rr = wv; rr < kTP; rr += 4) {
    const int r = r0 + rr;
    const long p = p0 + lane;
    C<double> v = cmk(0.0, 0.0);
    if (r < nrhs && p < N) v = b[(long)r * N + p];
    tr[lane][rr] = (R)v.re;
    ti[lane][rr] = (R)v.im;
  }
  __syncthreads();
  for (int pp = wv; pp < kTP; pp += 4) {
    const long p = p0 + pp;
    const int r = r0 + lane;
    if (p < N && r < nrhs) {
      const long e = ipm[p];
      Xr[e * nrhs + r] = tr[pp][lane];
      Xi[e * nrhs + r] = ti[pp][lane];
    }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void sol_out_tile_kernel(C<double>* __restrict__ b, long N, int nrhs,
                                                           const int* __restrict__ ipm, const R* __restrict__ Xr,
                                                           const R* __restrict__ Xi) {
  __shared__ R tr[kTP][kTP + 1], ti[kTP][kTP + 1];   // [p][r]
  const long p0 = (long)blockIdx.x * kTP;
  const int r0 = blockIdx.y * kTP;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int pp = wv; pp < kTP; pp += 4) {
    const long p = p0 + pp;
    const int r = r0 + lane;
    R vr = R(0), vi = R(0);
    if (p < N && r < nrhs) {
      const long e = ipm[p];
      vr = Xr[e * nrhs + r];
      vi = Xi[e * nrhs + r];
    }
    tr[pp][lane] = vr;
    ti[pp][lane] = vi;
  }
  __syncthreads();
  for (int rr = wv; rr < kTP; rr += 4) {
    const int r = r0 + rr;
    const long p = p0 + lane;
    if (r < nrhs && p < N) b[(long)r * N + p] = cmk((double)tr[lane][rr], (double)ti[lane][rr]);
  }
}

// Where each front's rows get their children's updates from: cinv[d.ci + slot
// (nf / NC) + p] = the boundary point of child `slot` at front point p, or -1.
template <int NC>
__global__ __launch_bounds__(256) void child_map_kernel(const FrontDev* __restrict__ fr, int nfronts,
                                                        const int* __restrict__ ib, int* __restrict__ cinv) {
  for (int q = blockIdx.x; q < nfronts; q += gridDim.x) {
    const FrontDev d = fr[q];
    const int np = d.nf / NC;
    for (int e = threadIdx.x; e < 2 * np; e += blockDim.x) cinv[d.ci + e] = -1;
    __syncthreads();
    for (int slot = 0; slot < 2; ++slot) {
      const int cid = slot ? d.child[1] : d.child[0];
      if (cid < 0) continue;
      const FrontDev c = fr[cid];
      for (int e = threadIdx.x; e < c.nb / NC; e += blockDim.x) cinv[d.ci + (long)slot * np + ib[c.xm + e]] = e;
    }
  }
}

// The children's update vectors added to the pivot rows (x) and set as the
// update vector (u; zero where no child reaches) of every front of a level:
// each row takes child 0's value, then child 1's, through cinv, in one launch
// and with nothing to clear beforehand (adding the children in turn took two
// launches of about 5 us a level and a clearing pass over u).
// 256 / rhs_lanes(nrhs) rows per workgroup pass.
template <typename R, int NC>
__global__ __launch_bounds__(256) void fwd_child_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                        int nlvl, const int* __restrict__ cinv, int nrhs,
                                                        R* __restrict__ Xr, R* __restrict__ Xi, R* __restrict__ Ur,
                                                        R* __restrict__ Ui) {
  const int lanes = rhs_lanes(nrhs), rpp = 256 / lanes;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const int* ci = cinv + d.ci;
    const int np = d.nf / NC;
    for (int row = blockIdx.x * rpp + threadIdx.x / lanes; row < d.nf; row += gridDim.x * rpp) {
      const int p = row / NC, e0 = ci[p], e1 = ci[np + p];
      const bool piv = row < d.np;
      if (piv && e0 < 0 && e1 < 0) continue;
      const long s0 = (d.cu[0] + (long)NC * e0 + row % NC) * nrhs, s1 = (d.cu[1] + (long)NC * e1 + row % NC) * nrhs;
      const long dst = (piv ? (long)d.e0 + row : d.u + row - d.np) * nrhs;
      for (int r = threadIdx.x % lanes; r < nrhs; r += lanes) {
        R vr = piv ? Xr[dst + r] : R(0), vi = piv ? Xi[dst + r] : R(0);
        if (e0 >= 0) {
          vr += Ur[s0 + r];
          vi += Ui[s0 + r];
        }
        if (e1 >= 0) {
          vr += Ur[s1 + r];
          vi += Ui[s1 + r];
        }
        (piv ? Xr : Ur)[dst + r] = vr;
        (piv ? Xi : Ui)[dst + r] = vi;
      }
    }
  }
}

// acc[rt] (rows 16 rt.., rt < 3; the 16 columns col0..col0+15) = A B for a
// 48 x 48 block A read from global memory (A(i, k) = Ag[i * lda + k] for
// i < arows and k < acols, zero elsewhere) and B rows of an LDS array
// (B(k, c) = Bs[bidx(k) * ldb + c] for k < acols, zero elsewhere).
template <typename R>
__device__ __forceinline__ void mma48_gl(const R* __restrict__ Agr, const R* __restrict__ Agi, long lda, int arows,
                                         int acols, const R* Bsr, const R* Bsi, int ldb, const int* bperm, int brow0,
                                         int col0, int lane, typename Mma<R>::v4 (&yr)[3],
                                         typename Mma<R>::v4 (&yi)[3]) {
  typedef typename Mma<R>::v4 v4;
#pragma unroll
  for (int rt = 0; rt < 3; ++rt) {
    yr[rt] = v4{R(0), R(0), R(0), R(0)};
    yi[rt] = v4{R(0), R(0), R(0), R(0)};
  }
  const int c = col0 + (lane & 15);
#pragma unroll 4
  for (int k4 = 0; k4 < kT; k4 += 4) {
    const int k = k4 + (lane >> 4);
    R br = R(0), bi = R(0);
    if (k < acols) {
      const int row = brow0 + (bperm ? bperm[k] : k);
      br = Bsr[row * ldb + c];
      bi = Bsi[row * ldb + c];
    }
#pragma unroll
    for (int rt = 0; rt < 3; ++rt) {
      const int i = 16 * rt + (lane & 15);
      const bool ok = i < arows && k < acols;
      const R ar = ok ? Agr[i * lda + k] : R(0);
      const R ai = ok ? Agi[i * lda + k] : R(0);
      yr[rt] = Mma<R>::op(ar, br, yr[rt]);
      yr[rt] = Mma<R>::op(-ai, bi, yr[rt]);
      yi[rt] = Mma<R>::op(ar, bi, yi[rt]);
      yi[rt] = Mma<R>::op(ai, br, yi[rt]);
    }
  }
}

constexpr int kLX = kSR + 1;                 // row stride of right-hand-side blocks in LDS
constexpr int kLL = kT + 1;                  // row stride of a 64 x 48 factor block in LDS
template <typename R>
struct SolveCfg {
  static constexpr int RZ = sizeof(R) == 4 ? 64 : 32;   // rhs per super-tile workgroup (LDS: 192 x RZ)
};

// Selective inversion of each super-block [kb0, kb0 + sw) of a front's pivot
// block, at factor time (the front still in its level buffer F):
//   FWD: M with z_block = M x_block for the forward tile procedure (for each
//        48-row tile t: x_t <- L_t^-1 P_t x_t, then x_t' -= L[t'][t] x_t for
//        the later tiles t' of the block);
//   BWD: H = U_block^-1 (tiles from last to first: x_t <- U_t^-1 x_t, then
//        x_t' -= U[t'][t] x_t for the earlier tiles).
// Each workgroup runs one procedure on RZ columns of the identity in LDS
// (grid.y: super-blocks, grid.z: column chunks of M, then of H), products on MFMA.
// What bounds it: the chain of tiles, so M and H are one launch, the tiles whose
// part of the columns is still zero are not visited, and in FP64 (RZ = 32) the
// four waves share the later tiles as two columns of waves: n = 29 set-up 4.6 to
// 2.0 ms, 2-D n = 479 12.5 to 7.5 ms.
template <typename R>
__global__ __launch_bounds__(256) void sb_inverse_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                         int nlvl, const R* __restrict__ buf, R* __restrict__ fac,
                                                         const int* __restrict__ ib) {
  typedef typename Mma<R>::v4 v4;
  constexpr int RZ = SolveCfg<R>::RZ, LD = RZ + 1;
  __shared__ R Sr[kSB * LD], Si[kSB * LD];
  __shared__ int perm[kT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int CW = RZ / 16, UW = 4 / CW;   // waves by columns, and by the tiles of an update
  const int c16 = 16 * (wave % CW), uwave = wave / CW;
  const auto run = [&](auto FW) {
  constexpr bool FWD = decltype(FW)::value;
  const int chunk = blockIdx.z % (kSB / RZ);
  for (int q = blockIdx.x; q < nlvl; q += gridDim.x) {
    const FrontDev d = fr[lvl[q]];
    const long nf = d.nf;
    const R* Fr = buf + d.f;
    const R* Fi = Fr + nf * nf;
    for (int sb = blockIdx.y; (long)sb * kSB < d.np; sb += gridDim.y) {
      const int kb0 = sb * kSB;
      const int sw = min(kSB, d.np - kb0);
      const int c0 = chunk * RZ;
      if (c0 >= sw) continue;
      for (int o = tid; o < kSB * RZ; o += blockDim.x) {
        const int k = o / RZ, r = o % RZ;
        Sr[k * LD + r] = (k == c0 + r && k < sw) ? R(1) : R(0);
        Si[k * LD + r] = R(0);
      }
      __syncthreads();
      const int nt = (sw + kT - 1) / kT;
      // M is lower, H upper triangular by tiles: the columns are zero before their first / after their last tile
      for (int s = FWD ? c0 / kT : nt - 1 - min(c0 + RZ - 1, sw - 1) / kT; s < nt; ++s) {
        const int t0 = FWD ? s * kT : (nt - 1 - s) * kT;
        const int tw = min(kT, sw - t0);
        const long kb = kb0 + t0;
        if (FWD && tid < tw) perm[tid] = ib[d.pv + kb + tid];
        __syncthreads();
        if (uwave == 0) {   // x_t <- L_t^-1 P_t x_t  or  U_t^-1 x_t, in place
          v4 yr[3], yi[3];
          const R* T = fac + d.t + (kb / kT) * 4 * kTileElems + (FWD ? 0 : 2 * kTileElems);
          mma48_gl<R>(T, T + kTileElems, kT, tw, tw, Sr, Si, LD, FWD ? perm : nullptr, t0, c16, lane, yr, yi);
#pragma unroll
          for (int rt = 0; rt < 3; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int i = 16 * rt + Mma<R>::row(lane, r);
              if (i < tw) {
                Sr[(t0 + i) * LD + c16 + (lane & 15)] = yr[rt][r];
                Si[(t0 + i) * LD + c16 + (lane & 15)] = yi[rt][r];
              }
            }
        }
        __syncthreads();
        {   // the other tiles of the block: x_t' -= F[t'][t] x_t
          const int ua = FWD ? t0 + kT : 0, ue = FWD ? sw : t0;
          for (int u0 = ua + kT * uwave; u0 < ue; u0 += kT * UW) {
            const int uw = min(kT, sw - u0);
            v4 yr[3], yi[3];
            const long a0 = (kb0 + u0) * nf + kb;
            mma48_gl<R>(Fr + a0, Fi + a0, nf, uw, tw, Sr, Si, LD, nullptr, t0, c16, lane, yr, yi);
#pragma unroll
            for (int rt = 0; rt < 3; ++rt)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int i = 16 * rt + Mma<R>::row(lane, r);
                if (i < uw) {
                  Sr[(u0 + i) * LD + c16 + (lane & 15)] -= yr[rt][r];
                  Si[(u0 + i) * LD + c16 + (lane & 15)] -= yi[rt][r];
                }
              }
          }
        }
        __syncthreads();
      }
      R* Mr = fac + (FWD ? d.m : d.h) + (long)sb * 2 * kSB * kSB;
      R* Mi = Mr + kSB * kSB;
      for (int o = tid; o < sw * RZ; o += blockDim.x) {
        const int k = o / RZ, r = o % RZ;
        if (c0 + r < sw) {
          Mr[k * kSB + c0 + r] = Sr[k * LD + r];
          Mi[k * kSB + c0 + r] = Si[k * LD + r];
        }
      }
      __syncthreads();
    }
  }
  };
  if (blockIdx.z < kSB / RZ)
    run(std::true_type{});
  else
    run(std::false_type{});
}

// The factor entries outside a super-block that multiply its unknowns, folded
// with the block's map: LU = 0: Lhat[i][block] = L[i][block] M for the rows
// below the block (pivot rows after it and boundary rows); LU = 1:
// Uhat[i][block] = U[i][block] H for the pivot rows above it.  Read from the
// front F, written into the factor; 64 x 64 output tile per workgroup (grid.y:
// super-block x three column tiles), K = the block width in chunks of 48.
template <typename R, int LU>
__global__ __launch_bounds__(256) void hat_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                  int nlvl, const R* __restrict__ buf, R* __restrict__ fac) {
  typedef typename Mma<R>::v4 v4;
  __shared__ R Ar_[kRB * kLL], Ai_[kRB * kLL];
  __shared__ R Br_[kT * kLX], Bi_[kT * kLX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  constexpr int NCT = kSB / 64;
  for (int q = blockIdx.z; q < nlvl; q += gridDim.z) {
    const FrontDev d = fr[lvl[q]];
    const long nf = d.nf, np = d.np;
    const R* Fr = buf + d.f;
    const R* Fi = Fr + nf * nf;
    for (int y = blockIdx.y; (long)(y / NCT) * kSB < np; y += gridDim.y) {
      const int sb = y / NCT, ct = y % NCT;
      const long kb0 = (long)sb * kSB;
      const int sw = (int)min((long)kSB, np - kb0);
      const int j0 = ct * 64;
      if (j0 >= sw) continue;
      const long r0 = LU == 0 ? kb0 + sw : 0, r1 = LU == 0 ? nf : kb0;
      const long i0 = r0 + (long)blockIdx.x * kRB;
      if (i0 >= r1) continue;
      const int cnt = (int)min((long)kRB, r1 - i0);
      const R* Br = fac + (LU == 0 ? d.m : d.h) + (long)sb * 2 * kSB * kSB;
      const R* Bi = Br + kSB * kSB;
      v4 cr[2][2], ci[2][2];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          cr[a][b] = v4{R(0), R(0), R(0), R(0)};
          ci[a][b] = v4{R(0), R(0), R(0), R(0)};
        }
      for (int kc = 0; kc < sw; kc += kT) {
        const int kw = min(kT, sw - kc);
        {  // all loads issued before the LDS stores
          constexpr int NU = (kRB * kT) / 256;
          R ld0_[NU], ld1_[NU];
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const int o = tid + 256 * u;
            const int i = o / kT, k = o % kT;
            const bool ok = i < cnt && k < kw;
            const long src = (i0 + i) * nf + kb0 + kc + k;
            ld0_[u] = ok ? Fr[src] : R(0);
            ld1_[u] = ok ? Fi[src] : R(0);
          }
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const int o = tid + 256 * u;
            const int i = o / kT, k = o % kT;
            Ar_[i * kLL + k] = ld0_[u];
            Ai_[i * kLL + k] = ld1_[u];
          }
        }
        {  // all loads issued before the LDS stores
          constexpr int NU = (kT * 64) / 256;
          R ld0_[NU], ld1_[NU];
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const int o = tid + 256 * u;
            const int k = o / 64, c = o % 64;
            const bool ok = k < kw && j0 + c < sw;
            ld0_[u] = ok ? Br[(kc + k) * kSB + j0 + c] : R(0);
            ld1_[u] = ok ? Bi[(kc + k) * kSB + j0 + c] : R(0);
          }
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const int o = tid + 256 * u;
            const int k = o / 64, c = o % 64;
            Br_[k * kLX + c] = ld0_[u];
            Bi_[k * kLX + c] = ld1_[u];
          }
        }
        __syncthreads();
        cmma64<R, 2, 2>(Ar_, Ai_, kLL, Br_, Bi_, kLX, kT, wm, wn, lane, cr, ci);
        __syncthreads();
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = wm + 16 * a + Mma<R>::row(lane, r), col = wn + 16 * b + (lane & 15);
            if (row < cnt && j0 + col < sw) {
              const long gi = i0 + row, gc = kb0 + j0 + col;
              if (gi < np) {
                fac[d.p + gi * nf + gc] = cr[a][b][r];
                fac[d.p + np * nf + gi * nf + gc] = ci[a][b][r];
              } else {
                fac[d.l + (gi - np) * np + gc] = cr[a][b][r];
                fac[d.l + (long)d.nb * np + (gi - np) * np + gc] = ci[a][b][r];
              }
            }
          }
    }
  }
}

// Forward solve step of super-block [kb0, kb0 + sw) of every front of a
// level.  Workgroups [0, 3): z_block (64 rows each) = M x_block, written to Z.
// The others: 64 rows i below the block: x_i -= Lhat[i][block] x_block (pivot
// rows in X, boundary rows in the node's update vector).  Both read only the
// block's x rows, which no workgroup writes.  SR rhs per workgroup (64, or
// 32 in FP32 launches of few workgroups).
template <typename R, int SR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 3 : 1, 8))) void fwd_sb_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                     int nlvl, int kb0, const R* __restrict__ fac, int nrhs,
                                                     R* __restrict__ Xr, R* __restrict__ Xi, R* __restrict__ Zr,
                                                     R* __restrict__ Zi, R* __restrict__ Ur, R* __restrict__ Ui) {
  typedef typename Mma<R>::v4 v4;
  constexpr int LX = SR + 1, NBW = SR / 32;
  constexpr int NZB = kSB / kRB;
  __shared__ R Ar_[kRB * kLL], Ai_[kRB * kLL];
  __shared__ R Br_[kT * LX], Bi_[kT * LX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * (SR / 2);
  const int r0 = blockIdx.z * SR;
  const int nr = min(SR, nrhs - r0);
  const bool zrole = (int)blockIdx.x < NZB;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    if (kb0 >= d.np) continue;
    const int sw = min(kSB, d.np - kb0);
    const long nf = d.nf, np = d.np;
    long i0;
    int cnt;
    if (zrole) {
      i0 = (long)blockIdx.x * kRB;                       // rows of the block
      if (i0 >= sw) continue;
      cnt = (int)min((long)kRB, sw - i0);
    } else {
      i0 = kb0 + sw + (long)(blockIdx.x - NZB) * kRB;    // rows below it
      if (i0 >= nf) continue;
      cnt = (int)min((long)kRB, nf - i0);
    }
    const R* Mr = fac + d.m + (long)(kb0 / kSB) * 2 * kSB * kSB;
    const R* Mi = Mr + kSB * kSB;
    CAcc<R, NBW> acc;
    acc.zero();
    // the next K chunk is loaded into registers while the MFMAs consume the current one
    constexpr int NUA = (kRB * kT) / 256, NUB = (kT * SR) / 256;
    R pa0[NUA], pa1[NUA], pb0[NUB], pb1[NUB];
    auto fetch = [&](int kc) {
      // addresses formed per chunk from an opaque thread index, not kept live
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int kw = min(kT, sw - kc);
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        const int i = o / kT, k = o % kT;
        R vr = R(0), vi = R(0);
        if (i < cnt && k < kw) {
          if (zrole) {
            vr = Mr[(i0 + i) * kSB + kc + k];
            vi = Mi[(i0 + i) * kSB + kc + k];
          } else {
            const long gi = i0 + i, col = kb0 + kc + k;
            if (gi < np) {
              vr = fac[d.p + gi * nf + col];
              vi = fac[d.p + np * nf + gi * nf + col];
            } else {
              vr = fac[d.l + (gi - np) * np + col];
              vi = fac[d.l + (long)d.nb * np + (gi - np) * np + col];
            }
          }
        }
        pa0[u] = vr;
        pa1[u] = vi;
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        const int k = o / SR, r = o % SR;
        R vr = R(0), vi = R(0);
        if (k < kw && r < nr) {
          vr = Xr[(d.e0 + kb0 + kc + k) * (long)nrhs + r0 + r];
          vi = Xi[(d.e0 + kb0 + kc + k) * (long)nrhs + r0 + r];
        }
        pb0[u] = vr;
        pb1[u] = vi;
      }
    };
    fetch(0);
    for (int kc = 0; kc < sw; kc += kT) {
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        Ar_[(o / kT) * kLL + o % kT] = pa0[u];
        Ai_[(o / kT) * kLL + o % kT] = pa1[u];
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        Br_[(o / SR) * LX + o % SR] = pb0[u];
        Bi_[(o / SR) * LX + o % SR] = pb1[u];
      }
      __syncthreads();
      if (kc + kT < sw) fetch(kc + kT);
      acc.mma(Ar_, Ai_, kLL, Br_, Bi_, LX, kT, wm, wn, lane);
      __syncthreads();
    }
    v4 cr[2][NBW], ci[2][NBW];
    acc.result(cr, ci);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wm + 16 * a + Mma<R>::row(lane, r), col = wn + 16 * b + (lane & 15);
          if (row < cnt && col < nr) {
            if (zrole) {
              Zr[(d.e0 + kb0 + i0 + row) * nrhs + r0 + col] = cr[a][b][r];
              Zi[(d.e0 + kb0 + i0 + row) * nrhs + r0 + col] = ci[a][b][r];
            } else {
              const long gi = i0 + row;
              const long dst = gi < np ? (d.e0 + gi) * nrhs + r0 + col : (d.u + gi - np) * nrhs + r0 + col;
              R* Tr = gi < np ? Xr : Ur;
              R* Ti = gi < np ? Xi : Ui;
              Tr[dst] -= cr[a][b][r];
              Ti[dst] -= ci[a][b][r];
            }
          }
        }
  }
}

// z_i -= sum_j U12[i][j] x_bnd(j) for 64 pivot rows and kKS boundary columns
// per workgroup (grid.z = column split + splits * rhs chunk).  A node with
// one split subtracts in place; with more, each split writes its partial sum
// and u12_reduce_kernel adds them in split order.
template <typename R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 4 : 1, 8))) void bwd_u12_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                      int nlvl, int nks_max, long np_max,
                                                      const R* __restrict__ fac, const int* __restrict__ ib, int nrhs,
                                                      const R* __restrict__ Xr, const R* __restrict__ Xi,
                                                      R* __restrict__ Zr, R* __restrict__ Zi, R* __restrict__ Pr,
                                                      R* __restrict__ Pi) {
  typedef typename Mma<R>::v4 v4;
  constexpr int LA = kKC + 1;
  __shared__ R Ar_[kRB * LA], Ai_[kRB * LA];   // U12 block [64][kKC]
  __shared__ R Br_[kKC * kLX], Bi_[kKC * kLX]; // gathered x_bnd [kKC][kSR]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int ks = blockIdx.z % nks_max;
  const int r0 = (blockIdx.z / nks_max) * kSR;
  const int nr = min(kSR, nrhs - r0);
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const long np = d.np, nf = d.nf, nb = d.nb;
    const int nks = (int)((nb + kKS - 1) / kKS);
    if (ks >= nks) continue;
    const long i0 = (long)blockIdx.x * kRB;
    if (i0 >= np) continue;
    const int cnt = (int)min((long)kRB, np - i0);
    const long j0 = (long)ks * kKS, j1 = min(nb, j0 + kKS);
    CAcc<R> acc;
    acc.zero();
    // the next chunk is loaded into registers while the MFMAs consume the current one
    constexpr int NUA = (kRB * kKC) / 256, NUB = (kKC * kSR) / 256;
    R pa0[NUA], pa1[NUA], pb0[NUB], pb1[NUB];
    auto fetch = [&](long jc) {
      // addresses formed per chunk from an opaque thread index, not kept live
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int nj = (int)min((long)kKC, j1 - jc);
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        const int i = o / kKC, j = o % kKC;
        R vr = R(0), vi = R(0);
        if (i < cnt && j < nj) {
          vr = fac[d.p + (i0 + i) * nf + np + jc + j];
          vi = fac[d.p + np * nf + (i0 + i) * nf + np + jc + j];
        }
        pa0[u] = vr;
        pa1[u] = vi;
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        const int j = o / kSR, r = o % kSR;
        R vr = R(0), vi = R(0);
        if (j < nj && r < nr) {
          const long e = ib[d.bm + jc + j];
          vr = Xr[e * nrhs + r0 + r];
          vi = Xi[e * nrhs + r0 + r];
        }
        pb0[u] = vr;
        pb1[u] = vi;
      }
    };
    fetch(j0);
    for (long jc = j0; jc < j1; jc += kKC) {
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        Ar_[(o / kKC) * LA + o % kKC] = pa0[u];
        Ai_[(o / kKC) * LA + o % kKC] = pa1[u];
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        Br_[(o / kSR) * kLX + o % kSR] = pb0[u];
        Bi_[(o / kSR) * kLX + o % kSR] = pb1[u];
      }
      __syncthreads();
      if (jc + kKC < j1) fetch(jc + kKC);
      acc.mma(Ar_, Ai_, LA, Br_, Bi_, kLX, kKC, wm, wn, lane);
      __syncthreads();
    }
    v4 cr[2][2], ci[2][2];
    acc.result(cr, ci);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wm + 16 * a + Mma<R>::row(lane, r), col = wn + 16 * b + (lane & 15);
          if (row < cnt && col < nr) {
            if (nks == 1) {
              Zr[(d.e0 + i0 + row) * nrhs + r0 + col] -= cr[a][b][r];
              Zi[(d.e0 + i0 + row) * nrhs + r0 + col] -= ci[a][b][r];
            } else {
              const long o = (((long)q * nks_max + ks) * np_max + i0 + row) * nrhs + r0 + col;
              Pr[o] = cr[a][b][r];
              Pi[o] = ci[a][b][r];
            }
          }
        }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void u12_reduce_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                         int nlvl, int nks_max, long np_max, int nrhs,
                                                         const R* __restrict__ Pr, const R* __restrict__ Pi,
                                                         R* __restrict__ Zr, R* __restrict__ Zi) {
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    const int nks = (int)((d.nb + kKS - 1) / kKS);
    if (nks < 2) continue;
    for (long i = (long)blockIdx.x * 4 + (threadIdx.x >> 6); i < d.np; i += (long)gridDim.x * 4)
      for (int r = threadIdx.x & 63; r < nrhs; r += 64) {
        R sr = R(0), si = R(0);
        for (int ks = 0; ks < nks; ++ks) {
          const long o = (((long)q * nks_max + ks) * np_max + i) * nrhs + r;
          sr += Pr[o];
          si += Pi[o];
        }
        Zr[(d.e0 + i) * nrhs + r] -= sr;
        Zi[(d.e0 + i) * nrhs + r] -= si;
      }
  }
}

// Backward solve step of super-block [kb0, kb0 + sw).  Workgroups [0, 3):
// x_block (64 rows each) = H y_block, written to X.  The others: 64 rows
// i < kb0: y_i -= Uhat[i][block] y_block.  Both read only the block's y rows.
// SR rhs per workgroup, as in fwd_sb_kernel.
template <typename R, int SR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? (SR == 32 ? 4 : 3) : 1, 8))) void bwd_sb_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                     int nlvl, int kb0, const R* __restrict__ fac, int nrhs,
                                                     R* __restrict__ Xr, R* __restrict__ Xi, R* __restrict__ Zr,
                                                     R* __restrict__ Zi) {
  typedef typename Mma<R>::v4 v4;
  constexpr int LX = SR + 1, NBW = SR / 32;
  constexpr int NZB = kSB / kRB;
  __shared__ R Ar_[kRB * kLL], Ai_[kRB * kLL];
  __shared__ R Br_[kT * LX], Bi_[kT * LX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * (SR / 2);
  const int r0 = blockIdx.z * SR;
  const int nr = min(SR, nrhs - r0);
  const bool xrole = (int)blockIdx.x < NZB;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    if (kb0 >= d.np) continue;
    const int sw = min(kSB, d.np - kb0);
    const long nf = d.nf, np = d.np;
    long i0;
    int cnt;
    if (xrole) {
      i0 = (long)blockIdx.x * kRB;
      if (i0 >= sw) continue;
      cnt = (int)min((long)kRB, sw - i0);
    } else {
      i0 = (long)(blockIdx.x - NZB) * kRB;
      if (i0 >= kb0) continue;
      cnt = (int)min((long)kRB, kb0 - i0);
    }
    const R* Hr = fac + d.h + (long)(kb0 / kSB) * 2 * kSB * kSB;
    const R* Hi = Hr + kSB * kSB;
    CAcc<R, NBW> acc;
    acc.zero();
    // the next K chunk is loaded into registers while the MFMAs consume the current one
    constexpr int NUA = (kRB * kT) / 256, NUB = (kT * SR) / 256;
    R pa0[NUA], pa1[NUA], pb0[NUB], pb1[NUB];
    auto fetch = [&](int kc) {
      // addresses formed per chunk from an opaque thread index, not kept live
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int kw = min(kT, sw - kc);
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        const int i = o / kT, k = o % kT;
        R vr = R(0), vi = R(0);
        if (i < cnt && k < kw) {
          if (xrole) {
            vr = Hr[(i0 + i) * kSB + kc + k];
            vi = Hi[(i0 + i) * kSB + kc + k];
          } else {
            vr = fac[d.p + (i0 + i) * nf + kb0 + kc + k];
            vi = fac[d.p + np * nf + (i0 + i) * nf + kb0 + kc + k];
          }
        }
        pa0[u] = vr;
        pa1[u] = vi;
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        const int k = o / SR, r = o % SR;
        R vr = R(0), vi = R(0);
        if (k < kw && r < nr) {
          vr = Zr[(d.e0 + kb0 + kc + k) * (long)nrhs + r0 + r];
          vi = Zi[(d.e0 + kb0 + kc + k) * (long)nrhs + r0 + r];
        }
        pb0[u] = vr;
        pb1[u] = vi;
      }
    };
    fetch(0);
    for (int kc = 0; kc < sw; kc += kT) {
#pragma unroll
      for (int u = 0; u < NUA; ++u) {
        const int o = tid + 256 * u;
        Ar_[(o / kT) * kLL + o % kT] = pa0[u];
        Ai_[(o / kT) * kLL + o % kT] = pa1[u];
      }
#pragma unroll
      for (int u = 0; u < NUB; ++u) {
        const int o = tid + 256 * u;
        Br_[(o / SR) * LX + o % SR] = pb0[u];
        Bi_[(o / SR) * LX + o % SR] = pb1[u];
      }
      __syncthreads();
      if (kc + kT < sw) fetch(kc + kT);
      acc.mma(Ar_, Ai_, kLL, Br_, Bi_, LX, kT, wm, wn, lane);
      __syncthreads();
    }
    v4 cr[2][NBW], ci[2][NBW];
    acc.result(cr, ci);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wm + 16 * a + Mma<R>::row(lane, r), col = wn + 16 * b + (lane & 15);
          if (row < cnt && col < nr) {
            if (xrole) {
              Xr[(d.e0 + kb0 + i0 + row) * nrhs + r0 + col] = cr[a][b][r];
              Xi[(d.e0 + kb0 + i0 + row) * nrhs + r0 + col] = ci[a][b][r];
            } else {
              Zr[(d.e0 + i0 + row) * nrhs + r0 + col] -= cr[a][b][r];
              Zi[(d.e0 + i0 + row) * nrhs + r0 + col] -= ci[a][b][r];
            }
          }
        }
  }
}

// Five to kThinRhs right-hand sides: the products of fwd_sb_kernel (KIND 0),
// bwd_sb_kernel (KIND 1) and bwd_u12_kernel (KIND 2) with 16 rows and CT tiles
// of 16 rhs per wave, four row tiles per workgroup.
// What bounds it: with a few rhs the factor streams through once (memory) at
// the wide levels, and at the top of the tree each launch is a chain of
// latencies.  The 64 x 64 LDS tiles of the kernels above multiplied mostly
// zero columns at 16 rhs (four times the FP64 MFMAs), kept a 6912-row front to
// 108 workgroups, and staged every factor value through LDS between two
// barriers.  Here the right-hand sides go to LDS once (KST of them at a time:
// 48 KB in FP64, three workgroups per CU) and each lane loads its factor
// operands itself, D chunks of 16 columns ahead; the rows a wave updates are
// read before its products.  A lane loads four consecutive columns of its row
// and to_mfma turns them into one column of each of four MFMA steps: loaded
// straight in the MFMA layout (neighbouring lanes in different rows, one value
// each) the address unit took 64 cycles per instruction for a quarter of the
// data, 10 of the 17 us of a top-of-tree launch.
// Blocks of M right of a row's own 48-row tile and entries of H left of the
// diagonal are exact zeros and are skipped.  SPLIT (FP64 launches of about a
// wave per SIMD): two waves per row tile, one the real, one the imaginary
// part, because four dependent FP64 MFMAs per four columns are what such a
// launch waits for.  Every output keeps the order of products of the LDS
// kernels (K ascending in steps of four into the same accumulators), so blocks
// of any size above kGemvRhs agree bit for bit.
// Measured, preconditioner apply (us), with this kernel and with the LDS kernels:
//              n = 48 complex128   n = 48 complex64   2-D n = 479 complex128
//   5 rhs        7506 / 24729        3988 / 10100       2263 / 7427
//   16 rhs       8159 / 25311        4341 / 10455       2836 / 7967
//   17 rhs      10678 / 26159        6352 / 10890       3597 / 8408
//   32 rhs      11127 / 27362        6639 / 11179       4047 / 9093
// so every count from 5 to 32 takes it (17 and up two tiles of 16); 33 rhs take
// the LDS kernels, 27409 / 11653 / 9204.  A launch at the top of the tree, 16
// rhs: 23.5 (FP64) and 17 us (FP32) -> 14.7 and 8 us.
constexpr int kThinRhs = 32;
constexpr int kThinPad = 256;   // factor values past the end that thin_kernel may read
// Four consecutive values from p (aligned to one value only), 16 bytes a load.
__device__ __forceinline__ void load4(const float* p, float (&v)[4]) {
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  const f4 t = *reinterpret_cast<const f4*>(p);
  v[0] = t.x;
  v[1] = t.y;
  v[2] = t.z;
  v[3] = t.w;
}
__device__ __forceinline__ void load4(const double* p, double (&v)[4]) {
  typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
  const d2 a = reinterpret_cast<const d2*>(p)[0], b = reinterpret_cast<const d2*>(p)[1];
  v[0] = a.x;
  v[1] = a.y;
  v[2] = b.x;
  v[3] = b.y;
}
// v[j] of lane group g (lanes 16 g ..) and v[g] of lane group j change places:
// from four consecutive columns per lane to one column of each MFMA step.
template <typename R>
__device__ __forceinline__ void to_mfma(R (&v)[4]) {
  swap32(v[0], v[2]);
  swap32(v[1], v[3]);
  swap16(v[0], v[1]);
  swap16(v[2], v[3]);
}

template <typename R, int KIND, int CT, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 128 : 256) __attribute__((amdgpu_waves_per_eu(SPLIT ? 1 : 2))) void thin_kernel(
    const FrontDev* __restrict__ fr, const int* __restrict__ lvl, int nlvl, int kb0, int nks_max, long np_max,
    const R* __restrict__ fac, const int* __restrict__ ib, int nrhs, R* __restrict__ Xr, R* __restrict__ Xi,
    R* __restrict__ Zr, R* __restrict__ Zi, R* __restrict__ Ur, R* __restrict__ Ui, R* __restrict__ Pr,
    R* __restrict__ Pi) {
  typedef typename Mma<R>::v4 v4;
  constexpr bool G3 = sizeof(R) == 4;    // three real products per complex one, as CAcc
  static_assert(!(G3 && SPLIT), "the three-product form needs all its sums in one wave");
  constexpr int NZ = kSB / 16;           // row tiles of the block itself (KIND 0, 1)
  constexpr int NT = SPLIT ? 128 : 256;
  constexpr int TPW = SPLIT ? 1 : 4;     // row tiles per workgroup
  constexpr int D = SPLIT && CT == 1 ? 6 : !G3 && CT == 2 ? 2 : 4;   // chunks of 16 columns in flight
  constexpr int KST = kSB / CT, W = 16 * CT;
  static_assert(NZ % TPW == 0, "a workgroup's tiles are all of the block or all outside it");
  __shared__ R Bsr[KST * W], Bsi[KST * W];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, g = lane >> 4;
  const int part = SPLIT ? (tid >> 6) & 1 : 0;
  const int tile0 = blockIdx.x * TPW, tile = tile0 + (SPLIT ? 0 : tid >> 6);
  const int ks = blockIdx.z;
  bool first = true;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    // the whole descriptor in one go: read where they are used, its fields
    // would be a chain of dependent scalar loads
    asm volatile("" ::"s"(d.np), "s"(d.nb), "s"(d.nf), "s"(d.e0), "s"(d.p), "s"(d.l), "s"(d.u), "s"(d.m), "s"(d.h),
                 "s"(d.bm));
    const long nf = d.nf, np = d.np, nb = d.nb;
    const bool own = KIND != 2 && tile0 < NZ;   // rows of the block: z = M x or x = H y
    long rb, re;                                // rows of this launch part: [rb, re)
    int K, nks = 1;
    if (KIND == 2) {
      nks = (int)((nb + kKS - 1) / kKS);
      if (ks >= nks) continue;
      K = (int)min((long)kKS, nb - (long)ks * kKS);
      rb = 0;
      re = np;
    } else {
      if (kb0 >= np) continue;
      K = (int)min((long)kSB, np - kb0);
      rb = own || KIND == 1 ? 0 : kb0 + K;
      re = own ? K : (KIND == 0 ? nf : kb0);
    }
    const int toff = KIND == 2 || own ? 0 : NZ;
    if (rb + 16L * (tile0 - toff) >= re) continue;
    const long i0 = rb + 16L * (tile - toff);
    const bool active = i0 < re;
    const int cnt = active ? (int)min(16L, re - i0) : 1;
    int k0 = 0, k1 = K;
    if (own && KIND == 0) k1 = min(K, ((int)i0 / kT + 1) * kT);
    if (own && KIND == 1) k0 = (int)i0;
    // this lane's factor row (rows past cnt repeat the last, unused)
    const long gi = active ? i0 + min(lr, cnt - 1) : rb;
    const R* ar;
    long im;                                    // distance to the imaginary plane
    if (KIND == 2) {
      ar = fac + d.p + gi * nf + np + (long)ks * kKS;
      im = np * nf;
    } else if (own) {
      ar = fac + (KIND == 0 ? d.m : d.h) + (long)(kb0 / kSB) * 2 * kSB * kSB + gi * kSB;
      im = (long)kSB * kSB;
    } else if (KIND == 1 || gi < np) {
      ar = fac + d.p + gi * nf + kb0;
      im = np * nf;
    } else {
      ar = fac + d.l + (gi - np) * np + kb0;
      im = nb * np;
    }
    // Chunks of 16 columns from kc on, up to D past the row's end (never used;
    // the factor's allocation is kThinPad longer for the last row): no bounds,
    // so the loads in flight are counted exactly.
    ar += 4 * g;
    const R* ai = ar + im;
    R fr_[D][4], fi_[D][4];
    auto fetch = [&](int u, int kc) {
      load4(ar + kc, fr_[u]);
      load4(ai + kc, fi_[u]);
    };
    const long eb = d.e0 + kb0;
    // destinations; the rows updated in place are read ahead of the products
    long dst[4];
    const bool upd = KIND == 2 ? nks == 1 : !own;
    R* const Tr = KIND == 2 ? (nks > 1 ? Pr : Zr) : (KIND == 0) == own ? Zr : Xr;
    R* const Ti = KIND == 2 ? (nks > 1 ? Pi : Zi) : (KIND == 0) == own ? Zi : Xi;
    bool bnd[4];
    R or_[CT][4], oi_[CT][4];
    int col[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) col[c] = min(16 * c + lr, nrhs - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const long row = active ? i0 + min(Mma<R>::row(lane, r), cnt - 1) : rb;
      bnd[r] = KIND == 0 && !own && row >= np;
      if (KIND == 2 && nks > 1)
        dst[r] = (((long)q * nks_max + ks) * np_max + row) * nrhs;
      else if (own)
        dst[r] = (eb + row) * nrhs;
      else
        dst[r] = (bnd[r] ? d.u + row - np : d.e0 + row) * nrhs;
      if (upd)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          or_[c][r] = (bnd[r] ? Ur : Tr)[dst[r] + col[c]];
          oi_[c][r] = (bnd[r] ? Ui : Ti)[dst[r] + col[c]];
        }
    }
    v4 p[3][CT];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int c = 0; c < CT; ++c) p[m][c] = v4{R(0), R(0), R(0), R(0)};
    for (int st = 0; st < K; st += KST) {
      const int se = min(K, st + KST);
      const int a0 = max(k0, st), a1 = min(k1, se);
      if (active && a0 < a1)
#pragma unroll
        for (int u = 0; u < D; ++u) fetch(u, a0 + 16 * u);
      __builtin_amdgcn_sched_barrier(0);
      // this stage's right-hand sides, zeros past its last column
      constexpr int NU = KST * W / NT;
      R vr[NU], vi[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int kk = min(st + (tid + NT * u) / W, K - 1), c = (tid + NT * u) % W;
        const long e = KIND == 2 ? (long)ib[d.bm + (long)ks * kKS + kk] : eb + kk;
        const long o = e * nrhs + min(c, nrhs - 1);
        vr[u] = (KIND == 1 ? Zr : Xr)[o];
        vi[u] = (KIND == 1 ? Zi : Xi)[o];
      }
      __builtin_amdgcn_sched_barrier(0);
      if (!first) __syncthreads();              // the previous stage's reads are done
      first = false;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const bool in = st + (tid + NT * u) / W < se;
        Bsr[tid + NT * u] = in ? vr[u] : R(0);
        Bsi[tid + NT * u] = in ? vi[u] : R(0);
      }
      __syncthreads();
      if (!active) continue;
      R br_[2][CT][4], bi_[2][CT][4];           // LDS operands, one chunk ahead
      auto rhs = [&](int b, int kc) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const int o = min(kc - st + 4 * s + g, KST - 1) * W + lr + 16 * c;
            br_[b][c][s] = Bsr[o];
            bi_[b][c][s] = Bsi[o];
          }
      };
      auto mul = [&](int u, int b) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const R br = br_[b][c][s], bi = bi_[b][c][s];
            if constexpr (G3) {
              p[0][c] = Mma<R>::op(fr_[u][s], br, p[0][c]);
              p[1][c] = Mma<R>::op(fi_[u][s], bi, p[1][c]);
              p[2][c] = Mma<R>::op(fr_[u][s] + fi_[u][s], br + bi, p[2][c]);
            } else if constexpr (SPLIT) {       // re: ar br - ai bi; im: ar bi + ai br
              p[0][c] = Mma<R>::op(fr_[u][s], part ? bi : br, p[0][c]);
              p[0][c] = Mma<R>::op(part ? fi_[u][s] : -fi_[u][s], part ? br : bi, p[0][c]);
            } else {
              p[0][c] = Mma<R>::op(fr_[u][s], br, p[0][c]);
              p[0][c] = Mma<R>::op(-fi_[u][s], bi, p[0][c]);
              p[1][c] = Mma<R>::op(fr_[u][s], bi, p[1][c]);
              p[1][c] = Mma<R>::op(fi_[u][s], br, p[1][c]);
            }
          }
      };
      static_assert(D % 2 == 0, "the LDS operands alternate between two sets");
      int kc = a0;
      rhs(0, kc);
      for (; kc + 16 * D < a1; kc += 16 * D)
#pragma unroll
        for (int u = 0; u < D; ++u) {
          rhs((u + 1) & 1, kc + 16 * (u + 1));
          to_mfma(fr_[u]);
          to_mfma(fi_[u]);
          __builtin_amdgcn_sched_barrier(0);
          mul(u, u & 1);
          fetch(u, kc + 16 * (u + D));
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int u = 0; u < D; ++u)
        if (kc + 16 * u < a1) {
          to_mfma(fr_[u]);
          to_mfma(fi_[u]);
#pragma unroll
          for (int s = 0; s < 4; ++s)           // columns past the end of the last chunk
            if (kc + 16 * u + 4 * s + g >= a1) fr_[u][s] = fi_[u][s] = R(0);
          if (u + 1 < D) rhs((u + 1) & 1, kc + 16 * (u + 1));
          __builtin_amdgcn_sched_barrier(0);
          mul(u, u & 1);
        }
    }
    if (!active) continue;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      v4 cr = p[0][c], ci = SPLIT ? p[0][c] : p[1][c];
      if constexpr (G3) {
        cr = p[0][c] - p[1][c];
        ci = p[2][c] - p[0][c] - p[1][c];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (Mma<R>::row(lane, r) < cnt && 16 * c + lr < nrhs) {
          if (!SPLIT || part == 0) (bnd[r] ? Ur : Tr)[dst[r] + col[c]] = upd ? or_[c][r] - cr[r] : cr[r];
          if (!SPLIT || part == 1) (bnd[r] ? Ui : Ti)[dst[r] + col[c]] = upd ? oi_[c][r] - ci[r] : ci[r];
        }
    }
  }
}

// Up to kGemvRhs right-hand sides: the products of fwd_sb_kernel (FWD) and
// bwd_sb_kernel as matrix-vector products, kGemvLanes lanes per row with the
// block's vector in LDS (the MFMA tiles would compute mostly zero columns).
// Same grid and the same rows read and written as those kernels.
// What bounds it: memory at the wide levels (the 4096 leaf fronts of a 2-D
// n = 479 factor: about 3 TB/s on row pieces of 0.5 to 0.7 KB), a chain of
// latencies at the top of the tree (4 to 5 us a launch).  Every factor value of
// a row (sw <= 192: twelve a lane and plane) is loaded before the first wait,
// ahead of the vector's staging, and the descriptor in one go; the steps' count
// is uniform, so loads and LDS reads are addressed by constant offsets (with a
// clamp per load the kernels were bound by issuing address arithmetic); the
// zero blocks of M and H are not read (thin_kernel).  2-D preconditioner apply, n = 479,
// one rhs: 1450 to 923 us, the leaf level's three launches 525 to 355 us.  Up to
// four rhs, where thin_kernel multiplies mostly zero columns: apply at n = 48,
// complex128 / complex64, one rhs 4102 / 2483 us (thin_kernel 7300 / 3780), four
// 5398 / 3309 (7465 / 3895), five by thin_kernel 7506 / 3988; 2-D n = 479
// complex128 one rhs 935 (2104), four 1249 (2220), five 2263.
constexpr int kGemvRhs = 4;
constexpr int kGemvLanes = 16;   // lanes per row: four rows per wave, 128-byte row segments per load
constexpr int kGemvRows = 256 / kGemvLanes;   // rows per workgroup: more workgroups per front

// A lane's factor values of up to UN whole steps of kGemvLanes columns of a
// row (n of them used, the same n in the whole wave): every load is issued
// before the first wait and addressed by a constant offset.
template <typename R, int NR, int UN>
struct GemvRow {
  R a[UN], b[UN];
  __device__ __forceinline__ void load(const R* p, const R* q, int n) {
    static_for<0, UN>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if (i < n) {
        a[i] = p[i * kGemvLanes];
        b[i] = q[i * kGemvLanes];
      }
    });
  }
  // s[r] += sum over the steps, columns ascending, of the row times the vector in LDS ([column][rhs], re and im)
  __device__ __forceinline__ void add(const C<R>* v, int n, R (&sr)[NR], R (&si)[NR]) {
    static_for<0, UN>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if (i < n)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const C<R> x = v[i * kGemvLanes * NR + r];
          sr[r] += a[i] * x.re - b[i] * x.im;
          si[r] += a[i] * x.im + b[i] * x.re;
        }
    });
  }
};

template <typename R>
__device__ __forceinline__ R row_sum(R x) {
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  return x + row_ror<1>(x);
}

// The row's sums over its kGemvLanes lanes; lane r < NR ends with rhs r's.
template <typename R, int NR>
__device__ __forceinline__ void gemv_reduce(const R (&sr)[NR], const R (&si)[NR], int sub, R& vr, R& vi) {
  static_assert(kGemvLanes == 16, "a DPP row");
  vr = row_sum(sr[0]);
  vi = row_sum(si[0]);
#pragma unroll
  for (int r = 1; r < NR; ++r) {
    const R tr = row_sum(sr[r]), ti = row_sum(si[r]);
    if (sub == r) {
      vr = tr;
      vi = ti;
    }
  }
}

// UN * kGemvLanes: the widest super-block of the level, at most kSB.  Workgroup
// blockIdx.x takes the 16-row tiles blockIdx.x + i gridDim.x of the block
// (M or H) and of the rows outside it.
template <typename R, bool FWD, int NR, int UN>
__global__ __launch_bounds__(256) void sb_gemv_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                      int nlvl, int kb0, const R* __restrict__ fac,
                                                      R* __restrict__ Xr, R* __restrict__ Xi, R* __restrict__ Zr,
                                                      R* __restrict__ Zi, R* __restrict__ Ur, R* __restrict__ Ui) {
  __shared__ C<R> v_[UN * kGemvLanes * NR];
  const int tid = threadIdx.x, sub = tid % kGemvLanes, row = tid / kGemvLanes;
  // the block's vector: x rows (forward) or y rows (backward) of the block
  const R* Vr = FWD ? Xr : Zr;
  const R* Vi = FWD ? Xi : Zi;
  bool first = true;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    asm volatile("" ::"s"(d.np), "s"(d.nb), "s"(d.nf), "s"(d.e0), "s"(d.p), "s"(d.l), "s"(d.u), "s"(d.m), "s"(d.h));
    if (kb0 >= d.np) continue;
    const int sw = min(kSB, d.np - kb0), mt = (sw + kGemvRows - 1) / kGemvRows;
    const int out0 = FWD ? kb0 + sw : 0, outs = (FWD ? d.nf : kb0) - out0;   // rows below (forward) or above the block
    const int nt = mt + (outs + kGemvRows - 1) / kGemvRows;
    const long nf = d.nf, np = d.np;
    bool staged = false;
    for (int t = blockIdx.x; t < nt; t += gridDim.x) {
      const bool brole = t < mt;
      const int i0 = (brole ? t : t - mt) * kGemvRows, cnt = min(kGemvRows, (brole ? sw : outs) - i0);
      const long gi = (brole ? 0 : out0) + i0 + min(row, cnt - 1);
      const R* ar;
      long im;
      int k0 = 0, k1 = sw;
      if (brole) {
        ar = fac + (FWD ? d.m : d.h) + (long)(kb0 / kSB) * 2 * kSB * kSB + gi * kSB;   // M (forward) or H
        im = (long)kSB * kSB;
        if (FWD)
          k1 = min(sw, (i0 / kT + 1) * kT);
        else
          k0 = i0;
      } else if (!FWD || gi < np) {
        ar = fac + d.p + gi * nf + kb0;
        im = np * nf;
      } else {
        ar = fac + d.l + (gi - np) * np + kb0;
        im = (long)d.nb * np;
      }
      ar += k0 + sub;
      const int ns = (k1 - k0) / kGemvLanes, kt = k0 + ns * kGemvLanes + sub;   // whole steps, then a part of one
      GemvRow<R, NR, UN> g;
      g.load(ar, ar + im, ns);
      GemvRow<R, NR, 1> tail;
      if (kt < k1) tail.load(ar + ns * kGemvLanes, ar + im + ns * kGemvLanes, 1);
      // the row this lane updates, read ahead of the products
      const bool bnd = FWD && !brole && gi >= np;
      R* const Tr = brole ? (FWD ? Zr : Xr) : bnd ? Ur : FWD ? Xr : Zr;
      R* const Ti = brole ? (FWD ? Zi : Xi) : bnd ? Ui : FWD ? Xi : Zi;
      const long dst = (brole ? d.e0 + kb0 + gi : bnd ? d.u + gi - np : d.e0 + gi) * NR + min(sub, NR - 1);
      const C<R> old = brole ? C<R>{} : C<R>{Tr[dst], Ti[dst]};
      if (!staged) {
        if (!first) __syncthreads();   // the previous front's reads of the vector are done
        first = false;
        for (int e = tid; e < sw * NR; e += 256)
          v_[e] = {Vr[(d.e0 + kb0) * (long)NR + e], Vi[(d.e0 + kb0) * (long)NR + e]};
        __syncthreads();
        staged = true;
      }
      R sr[NR] = {}, si[NR] = {};
      g.add(v_ + (k0 + sub) * NR, ns, sr, si);
      if (kt < k1) tail.add(v_ + kt * NR, 1, sr, si);
      R vr, vi;
      gemv_reduce<R, NR>(sr, si, sub, vr, vi);
      if (sub < NR && row < cnt) {
        Tr[dst] = brole ? vr : old.re - vr;
        Ti[dst] = brole ? vi : old.im - vi;
      }
    }
  }
}

// Up to kGemvRhs right-hand sides: bwd_u12_kernel as matrix-vector products,
// kGemvLanes lanes per pivot row over the split's kKS boundary columns
// (gathered x in LDS), in rounds of UN kGemvLanes columns with two rounds'
// loads in flight; the same outputs (in place with one split, else the split's
// partial sums).  The boundary's indices are loaded ahead of the factor, so the
// gather does not wait for it.
template <typename R, int NR, int UN>
__global__ __launch_bounds__(256) void u12_gemv_kernel(const FrontDev* __restrict__ fr, const int* __restrict__ lvl,
                                                       int nlvl, int nks_max, long np_max,
                                                       const R* __restrict__ fac, const int* __restrict__ ib,
                                                       const R* __restrict__ Xr, const R* __restrict__ Xi,
                                                       R* __restrict__ Zr, R* __restrict__ Zi, R* __restrict__ Pr,
                                                       R* __restrict__ Pi) {
  constexpr int RK = UN * kGemvLanes, GI = kKS * NR / 256;
  __shared__ C<R> v_[kKS * NR];
  const int tid = threadIdx.x, sub = tid % kGemvLanes, row = tid / kGemvLanes;
  const int ks = blockIdx.z;
  bool first = true;
  for (int q = blockIdx.y; q < nlvl; q += gridDim.y) {
    const FrontDev d = fr[lvl[q]];
    asm volatile("" ::"s"(d.np), "s"(d.nb), "s"(d.nf), "s"(d.e0), "s"(d.p), "s"(d.bm));
    const long np = d.np, nf = d.nf, nb = d.nb;
    const int nks = (int)((nb + kKS - 1) / kKS);
    if (ks >= nks) continue;
    const long j0 = (long)ks * kKS;
    const int nj = (int)min((long)kKS, nb - j0), ns = nj / kGemvLanes, jt = ns * kGemvLanes + sub;
    bool staged = false;
    for (long i0 = (long)blockIdx.x * kGemvRows; i0 < np; i0 += (long)gridDim.x * kGemvRows) {
      int bi[GI];
      if (!staged)
#pragma unroll
        for (int i = 0; i < GI; ++i) bi[i] = ib[d.bm + j0 + min((tid + 256 * i) / NR, nj - 1)];
      const int cnt = (int)min((long)kGemvRows, np - i0);
      const long gi = i0 + min(row, cnt - 1);
      const R* ar = fac + d.p + gi * nf + np + j0 + sub;
      const R* ai = ar + np * nf;
      GemvRow<R, NR, UN> g, h;
      GemvRow<R, NR, 1> tail;
      g.load(ar, ai, ns);
      h.load(ar + RK, ai + RK, ns - UN);
      if (jt < nj) tail.load(ar + ns * kGemvLanes, ai + ns * kGemvLanes, 1);
      const long dst = (d.e0 + gi) * NR + min(sub, NR - 1);
      const R tr = nks == 1 ? Zr[dst] : R(0), ti = nks == 1 ? Zi[dst] : R(0);
      if (!staged) {
        if (!first) __syncthreads();   // the previous front's reads of the vector are done
        first = false;
#pragma unroll
        for (int i = 0; i < GI; ++i) {
          const int e = tid + 256 * i;
          if (e < nj * NR) {
            const long x = (long)bi[i] * NR + e % NR;
            v_[e] = {Xr[x], Xi[x]};
          }
        }
        __syncthreads();
        staged = true;
      }
      R sr[NR] = {}, si[NR] = {};
      const C<R>* v = v_ + sub * NR;
      for (int k = 0; k < ns; k += 2 * UN, v += 2 * RK * NR) {
        ar += 2 * RK;
        ai += 2 * RK;
        g.add(v, ns - k, sr, si);
        g.load(ar, ai, ns - k - 2 * UN);
        h.add(v + RK * NR, ns - k - UN, sr, si);
        h.load(ar + RK, ai + RK, ns - k - 3 * UN);
      }
      if (jt < nj) tail.add(v_ + jt * NR, 1, sr, si);
      R vr, vi;
      gemv_reduce<R, NR>(sr, si, sub, vr, vi);
      if (sub < NR && row < cnt) {
        if (nks == 1) {
          Zr[dst] = tr - vr;
          Zi[dst] = ti - vi;
        } else {
          const long o = (((long)q * nks_max + ks) * np_max + gi) * NR + sub;
          Pr[o] = vr;
          Pi[o] = vi;
        }
      }
    }
  }
}

inline unsigned grid_for(long work, long per = 256, long cap = 65535) {
  long g = (work + per - 1) / per;
  return (unsigned)std::max(1L, std::min(g, cap));
}

}  // namespace

struct GpuSolver {
  int n = 0;
  int dims[3] = {0, 0, 0};             // grid extents (n, n, n) in 3-D, (n, n, 1) in 2-D
  int nc = 3;                          // unknowns per point (field components)
  long npts = 0;
  bool fp32 = false;
  long N = 0;                          // nc * npts unknowns
  std::vector<FrontDev> fh;            // per node (host copy)
  std::vector<std::vector<int>> levels;   // node ids per depth
  std::vector<long> lvl_off;           // offset of each level's list in lvl_d
  std::vector<int> lvl_np, lvl_nf;     // largest np / nf per level
  std::vector<size_t> lvl_elems;       // level buffer elements (R) per level
  DevBuf fd, lvl_d, ib, fac;
  DevBuf cinv;                         // children's rows per front point (child_map_kernel)
  DevBuf ipm;                          // inverse of the final elimination order (natural -> position)
  long u_rows = 0;                     // sum of nb over the nodes
  SolveWork<DevBuf> work;              // vectors of the solves
  DevBuf P;                            // split-K partial sums of the U12 products
  size_t bytes = 0;
  double flops = 0.0;
};

namespace {

// Extents from which the updates take 64 x 64 tiles (schur_kernel): the factor at
// n = 64, complex64 / complex128, spends 929 / 1981 ms in them with 4096, 929 / 1987
// with 3072, 942 / 1984 with 6144, 1085 / 2160 with 32 x 32 tiles only.
constexpr long kSchurCols = 4096;
// cols x rows: extents of the (first) part, at most
template <typename R>
void launch_schur(long cols, long rows, bool step, unsigned gy, hipStream_t s, const FrontDev* fr, const int* lvl,
                  int nl, int kb, int kb0, R* buf) {
  const auto go = [&](auto TS) {
    constexpr int ts = decltype(TS)::value;
    const long nbx = std::max(1L, (cols + ts - 1) / ts), nby = std::max(1L, (rows + ts - 1) / ts);
    hipLaunchKernelGGL((schur_kernel<R, ts>), dim3((unsigned)((step ? 2 : 1) * nbx * nby), gy), dim3(256), 0, s, fr, lvl,
                       nl, kb, kb0, (int)nbx, (int)nby, step, buf);
  };
  if (cols <= kSchurCols || rows <= kSchurCols)
    go(std::integral_constant<int, 32>{});
  else
    go(std::integral_constant<int, 64>{});
}

template <typename R>
ls_status factor_numeric(GpuSolver& g, const C<double>* rows, hipStream_t s) {
  const int L = (int)g.levels.size();
  size_t cap[2] = {0, 0};
  for (int dep = 0; dep < L; ++dep) cap[dep & 1] = std::max(cap[dep & 1], g.lvl_elems[dep]);
  DevBuf lb[2];
  LS_TRY(lb[0].alloc(cap[0] * sizeof(R)));
  LS_TRY(lb[1].alloc(cap[1] * sizeof(R)));
  const FrontDev* fr = g.fd.as<FrontDev>();
  int* ib = g.ib.as<int>();
  const int* cinv = g.cinv.as<int>();
  R* fac = g.fac.as<R>();
  for (int dep = L - 1; dep >= 0; --dep) {
    const int nl = (int)g.levels[dep].size();
    const int* lvl = g.lvl_d.as<int>() + g.lvl_off[dep];
    R* buf = lb[dep & 1].as<R>();
    const R* cbuf = lb[(dep + 1) & 1].as<R>();
    const unsigned gy = (unsigned)std::min(nl, 65535);
    const long mnf = g.lvl_nf[dep], mnp = g.lvl_np[dep];
    const dim3 gm((unsigned)std::max(1L, std::min((mnf + 3) / 4, 4096L)), gy);
    if (g.nc == 3) {
      hipLaunchKernelGGL((merge_children_kernel<R, 3>), gm, dim3(256), 0, s, fr, lvl, nl, cinv, cbuf, buf);
      hipLaunchKernelGGL((assemble_kernel<R, 3>), dim3(grid_for(mnf / 3 * 27), gy), dim3(256), 0, s, fr, lvl, nl, ib,
                         rows, buf);
    } else {
      hipLaunchKernelGGL((merge_children_kernel<R, 2>), gm, dim3(256), 0, s, fr, lvl, nl, cinv, cbuf, buf);
      hipLaunchKernelGGL((assemble_kernel<R, 2>), dim3(grid_for(mnf / 2 * 27), gy), dim3(256), 0, s, fr, lvl, nl, ib,
                         rows, buf);
    }
    for (long kb0 = 0; kb0 < mnp; kb0 += kOB) {
      const long kbe = std::min(mnp, kb0 + kOB);
      for (long kb = kb0; kb < kbe; kb += kT) {
        hipLaunchKernelGGL(diag_kernel<R>, dim3(gy), dim3(256), 0, s, fr, lvl, nl, (int)kb, buf, ib);
        const long rest = mnf - kb - 1;           // rows right of / below the tile, at most
        const int half = (int)std::max(1L, (rest + kPR - 1) / kPR);
        hipLaunchKernelGGL(panel_kernel<R>, dim3(2 * half, gy), dim3(256), 0, s, fr, lvl, nl, (int)kb, half, buf,
                           (const int*)ib);
        if (kb + kT < kbe) launch_schur<R>(kbe - kb - 1, rest, true, gy, s, fr, lvl, nl, (int)kb, (int)kb0, buf);
      }
      launch_schur<R>(mnf - kb0 - 1, mnf - kb0 - 1, false, gy, s, fr, lvl, nl, (int)kb0, (int)kb0, buf);
    }
    hipLaunchKernelGGL(copyout_kernel<R>, dim3(grid_for(mnf * mnf, 256, 8192), std::min(gy, 64u)), dim3(256), 0, s,
                       fr, lvl, nl, (const R*)buf, fac);
    // selective inversion of the super-blocks, then the folded L and U entries
    hipLaunchKernelGGL(tile_inverse_kernel<R>, dim3(gy, (unsigned)((mnp + kT - 1) / kT)), dim3(256), 0, s, fr, lvl, nl,
                       (const R*)buf, fac);
    const unsigned nsb = (unsigned)((mnp + kSB - 1) / kSB);
    const unsigned ncc = (unsigned)(kSB / SolveCfg<R>::RZ);
    hipLaunchKernelGGL(sb_inverse_kernel<R>, dim3(gy, nsb, 2 * ncc), dim3(256), 0, s, fr, lvl, nl, (const R*)buf, fac,
                       (const int*)ib);
    const unsigned hy = std::min(65535u, nsb * (unsigned)(kSB / 64));
    const unsigned hx = (unsigned)std::max(1L, (mnf + kRB - 1) / kRB);
    hipLaunchKernelGGL((hat_kernel<R, 0>), dim3(hx, hy, gy), dim3(256), 0, s, fr, lvl, nl, (const R*)buf, fac);
    hipLaunchKernelGGL((hat_kernel<R, 1>), dim3(hx, hy, gy), dim3(256), 0, s, fr, lvl, nl, (const R*)buf, fac);
    LS_HIP(hipGetLastError());
  }
  // the elimination order is final once the pivots are chosen
  hipLaunchKernelGGL(inv_perm_kernel, dim3(grid_for(g.N, 256, 1 << 16)), dim3(256), 0, s, (const int*)ib, g.N,
                     g.ipm.as<int>());
  LS_HIP(hipGetLastError());
  LS_HIP(hipStreamSynchronize(s));
  return LS_OK;
}

// FP32 super-block launches with fewer than this many 64-rhs workgroups (the
// few large fronts at the top of the tree) take 32-rhs tiles on twice the
// workgroups; the factor blocks are then read once per 32 rhs.
constexpr long kSplitWg = 512;

// FP64 launches of fewer row tiles than this (about a wave per SIMD) take
// thin_kernel's SPLIT form.
constexpr long kSplitTiles = 1024;

// tiles: 16-row tiles of the launch, those of the super-block itself included.
template <typename R, int KIND>
void launch_thin(long tiles, unsigned gy, unsigned gz, hipStream_t s, const FrontDev* fr, const int* lvl, int nl,
                 int kb0, int nks, long np_max, const R* fac, const int* ib, int nrhs, R* Xr, R* Xi, R* Zr, R* Zi,
                 R* Ur, R* Ui, R* Pr, R* Pi) {
  if constexpr (sizeof(R) == 8) {
    if (tiles * gy * gz < kSplitTiles) {
      const auto kern = nrhs <= 16 ? thin_kernel<R, KIND, 1, true> : thin_kernel<R, KIND, 2, true>;
      hipLaunchKernelGGL(kern, dim3((unsigned)std::max(1L, tiles), gy, gz), dim3(128), 0, s, fr, lvl, nl, kb0, nks,
                         np_max, fac, ib, nrhs, Xr, Xi, Zr, Zi, Ur, Ui, Pr, Pi);
      return;
    }
  }
  const auto kern = nrhs <= 16 ? thin_kernel<R, KIND, 1, false> : thin_kernel<R, KIND, 2, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)std::max(1L, (tiles + 3) / 4), gy, gz), dim3(256), 0, s, fr, lvl, nl, kb0,
                     nks, np_max, fac, ib, nrhs, Xr, Xi, Zr, Zi, Ur, Ui, Pr, Pi);
}

template <typename R>
void launch_sb(bool fwd, unsigned gx, unsigned gy, int nrhs, hipStream_t s, const FrontDev* fr, const int* lvl,
               int nl, int kb0, const R* fac, R* Xr, R* Xi, R* Zr, R* Zi, R* Ur, R* Ui) {
  const unsigned gz = (unsigned)((nrhs + kSR - 1) / kSR);
  if (nrhs <= kThinRhs) {
    if (fwd)
      launch_thin<R, 0>(gx * (kRB / 16L), gy, 1, s, fr, lvl, nl, kb0, 1, 0, fac, nullptr, nrhs, Xr, Xi, Zr, Zi, Ur,
                        Ui, nullptr, nullptr);
    else
      launch_thin<R, 1>(gx * (kRB / 16L), gy, 1, s, fr, lvl, nl, kb0, 1, 0, fac, nullptr, nrhs, Xr, Xi, Zr, Zi, Ur,
                        Ui, nullptr, nullptr);
    return;
  }
  if constexpr (sizeof(R) == 4) {
    if ((long)gx * gy * gz < kSplitWg) {
      const unsigned gz2 = (unsigned)((nrhs + 31) / 32);
      if (fwd)
        hipLaunchKernelGGL((fwd_sb_kernel<R, 32>), dim3(gx, gy, gz2), dim3(256), 0, s, fr, lvl, nl, kb0, fac, nrhs,
                           Xr, Xi, Zr, Zi, Ur, Ui);
      else
        hipLaunchKernelGGL((bwd_sb_kernel<R, 32>), dim3(gx, gy, gz2), dim3(256), 0, s, fr, lvl, nl, kb0, fac, nrhs,
                           Xr, Xi, Zr, Zi);
      return;
    }
  }
  if (fwd)
    hipLaunchKernelGGL((fwd_sb_kernel<R, kSR>), dim3(gx, gy, gz), dim3(256), 0, s, fr, lvl, nl, kb0, fac, nrhs, Xr,
                       Xi, Zr, Zi, Ur, Ui);
  else
    hipLaunchKernelGGL((bwd_sb_kernel<R, kSR>), dim3(gx, gy, gz), dim3(256), 0, s, fr, lvl, nl, kb0, fac, nrhs, Xr,
                       Xi, Zr, Zi);
}

// f(integral_constant<int, NR>) for nrhs = NR <= kGemvRhs
template <typename F>
void with_rhs(int nrhs, F&& f) {
  static_assert(kGemvRhs == 4, "one kernel per count");
  switch (nrhs) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    default: f(std::integral_constant<int, 4>{}); break;
  }
}

// Workgroups per front of the matrix-vector kernels: a row tile each where the
// level's fronts are few, else about kGemvGrid in all, so that a workgroup of a
// wide level keeps its front's descriptor and vector for several tiles.
// Same apply with 2048 / 4096 / 8192 / a tile each: 936 / 923 / 948 / 1262 us
// (the last before the constant offsets: the levels of 2048 fronts and fewer
// took 10 to 45 us a launch, now 5 to 24).
constexpr long kGemvGrid = 4096;
inline unsigned gemv_grid(long tiles, int nl) {
  return (unsigned)std::max(1L, std::min(tiles, (kGemvGrid + nl - 1) / nl));
}

template <typename R, bool FWD>
void launch_sb_gemv(long tiles, unsigned gy, long sw, int nrhs, hipStream_t s, const FrontDev* fr, const int* lvl,
                    int nl, int kb0, const R* fac, R* Xr, R* Xi, R* Zr, R* Zi, R* Ur, R* Ui) {
  with_rhs(nrhs, [&](auto NR) {
    constexpr int nr = decltype(NR)::value;
    auto* k = sw <= 8 * kGemvLanes ? sb_gemv_kernel<R, FWD, nr, 8> : sb_gemv_kernel<R, FWD, nr, kSB / kGemvLanes>;
    hipLaunchKernelGGL(k, dim3(gemv_grid(tiles, nl), gy), dim3(256), 0, s, fr, lvl, nl, kb0, fac, Xr, Xi, Zr, Zi, Ur,
                       Ui);
  });
}

template <typename R>
ls_status solve_numeric(GpuSolver& g, const C<double>* b, C<double>* xo, int nrhs, hipStream_t s) {
  const int L = (int)g.levels.size();
  // split-K partial sums of the U12 products: levels whose widest boundary
  // needs more than one split
  std::vector<int> nks(L, 1);
  size_t pelems = 1;
  for (int dep = 0; dep < L; ++dep) {
    for (int id : g.levels[dep]) nks[dep] = std::max(nks[dep], (int)((g.fh[id].nb + kKS - 1) / kKS));
    if (nks[dep] > 1)
      pelems = std::max(pelems, (size_t)g.levels[dep].size() * nks[dep] * (size_t)g.lvl_np[dep] * nrhs);
  }
  LS_TRY(g.work.reserve(nrhs, 2 * (size_t)g.N * sizeof(R), 2 * (size_t)std::max(1L, g.u_rows) * sizeof(R)));
  if (g.P.bytes < 2 * pelems * sizeof(R)) LS_TRY(g.P.alloc(2 * pelems * sizeof(R)));
  R* Pr = g.P.as<R>();
  R* Pi = Pr + pelems;
  const long N = g.N;
  R* Xr = g.work.X.as<R>();
  R* Xi = Xr + N * nrhs;
  R* Zr = g.work.Z.as<R>();
  R* Zi = Zr + N * nrhs;
  R* Ur = g.work.U.as<R>();
  R* Ui = Ur + std::max(1L, g.u_rows) * nrhs;
  const FrontDev* fr = g.fd.as<FrontDev>();
  const int* ib = g.ib.as<int>();
  const R* fac = g.fac.as<R>();
  const int* cinv = g.cinv.as<int>();
  const unsigned gz = (unsigned)((nrhs + kSR - 1) / kSR);
  const int rpp = 256 / rhs_lanes(nrhs);     // rows per workgroup pass of the gather kernels
  if (nrhs >= kSolTileRhs)
    hipLaunchKernelGGL(sol_in_tile_kernel<R>, dim3((unsigned)((N + kTP - 1) / kTP), (unsigned)((nrhs + kTP - 1) / kTP)),
                       dim3(256), 0, s, b, N, nrhs, (const int*)g.ipm.as<int>(), Xr, Xi);
  else
    hipLaunchKernelGGL(sol_in_kernel<R>, dim3(grid_for(N, rpp, 65535)), dim3(256), 0, s, b, N, nrhs, ib, Xr, Xi);
  for (int dep = L - 1; dep >= 0; --dep) {
    const int nl = (int)g.levels[dep].size();
    const int* lvl = g.lvl_d.as<int>() + g.lvl_off[dep];
    const unsigned gy = (unsigned)std::min(nl, 65535);
    const long mnf = g.lvl_nf[dep], mnp = g.lvl_np[dep];
    {
      // one front per workgroup row (a front loop would chain descriptor loads)
      const long gxc = std::max(1L, std::min((mnf + rpp - 1) / rpp, std::max(1L, 65536L / nl)));
      if (g.nc == 3)
        hipLaunchKernelGGL((fwd_child_kernel<R, 3>), dim3((unsigned)gxc, gy), dim3(256), 0, s, fr, lvl, nl, cinv, nrhs,
                           Xr, Xi, Ur, Ui);
      else
        hipLaunchKernelGGL((fwd_child_kernel<R, 2>), dim3((unsigned)gxc, gy), dim3(256), 0, s, fr, lvl, nl, cinv, nrhs,
                           Xr, Xi, Ur, Ui);
    }
    for (long kb0 = 0; kb0 < mnp; kb0 += kSB) {
      const unsigned gx = (unsigned)(kSB / kRB + std::max(0L, (mnf - kb0 - 1 + kRB - 1) / kRB));
      if (nrhs <= kGemvRhs)
        launch_sb_gemv<R, true>((mnf - kb0 + kGemvRows - 1) / kGemvRows + 1, gy, mnp - kb0, nrhs, s, fr, lvl, nl,
                                (int)kb0, fac, Xr, Xi, Zr, Zi, Ur, Ui);
      else
        launch_sb<R>(true, gx, gy, nrhs, s, fr, lvl, nl, (int)kb0, fac, Xr, Xi, Zr, Zi, Ur, Ui);
    }
  }
  for (int dep = 0; dep < L; ++dep) {
    const int nl = (int)g.levels[dep].size();
    const int* lvl = g.lvl_d.as<int>() + g.lvl_off[dep];
    const unsigned gy = (unsigned)std::min(nl, 65535);
    const long mnp = g.lvl_np[dep];
    const unsigned gu = (unsigned)std::max(1L, (mnp + kRB - 1) / kRB);
    if (nrhs <= kGemvRhs)
      with_rhs(nrhs, [&](auto NR) {
        constexpr int nr = decltype(NR)::value;
        auto* k = g.lvl_nf[dep] <= 12 * kGemvLanes ? u12_gemv_kernel<R, nr, 4> : u12_gemv_kernel<R, nr, 8>;
        hipLaunchKernelGGL(k, dim3(gemv_grid((mnp + kGemvRows - 1) / kGemvRows, nl), gy, nks[dep]), dim3(256), 0, s, fr,
                           lvl, nl, nks[dep], mnp, fac, ib, (const R*)Xr, (const R*)Xi, Zr, Zi, Pr, Pi);
      });
    else if (nrhs <= kThinRhs)
      launch_thin<R, 2>((mnp + 15) / 16, gy, (unsigned)nks[dep], s, fr, lvl, nl, 0, nks[dep], mnp, fac, ib, nrhs, Xr,
                        Xi, Zr, Zi, Ur, Ui, Pr, Pi);
    else
      hipLaunchKernelGGL(bwd_u12_kernel<R>, dim3(gu, gy, gz * nks[dep]), dim3(256), 0, s, fr, lvl, nl, nks[dep],
                         mnp, fac, ib, nrhs, (const R*)Xr, (const R*)Xi, Zr, Zi, Pr, Pi);
    if (nks[dep] > 1)
      hipLaunchKernelGGL(u12_reduce_kernel<R>, dim3(grid_for(mnp, 4, 4096), gy), dim3(256), 0, s, fr, lvl, nl,
                         nks[dep], mnp, nrhs, (const R*)Pr, (const R*)Pi, Zr, Zi);
    for (long kb0 = ((mnp - 1) / kSB) * kSB; kb0 >= 0; kb0 -= kSB) {
      const unsigned gx = (unsigned)(kSB / kRB + (kb0 + kRB - 1) / kRB);
      if (nrhs <= kGemvRhs) {
        const long sw = std::min((long)kSB, mnp - kb0);
        launch_sb_gemv<R, false>((sw + kb0 + kGemvRows - 1) / kGemvRows, gy, sw, nrhs, s, fr, lvl, nl, (int)kb0, fac, Xr,
                                 Xi, Zr, Zi, Ur, Ui);
      } else
        launch_sb<R>(false, gx, gy, nrhs, s, fr, lvl, nl, (int)kb0, fac, Xr, Xi, Zr, Zi, Ur, Ui);
    }
  }
  if (nrhs >= kSolTileRhs)
    hipLaunchKernelGGL(sol_out_tile_kernel<R>, dim3((unsigned)((N + kTP - 1) / kTP), (unsigned)((nrhs + kTP - 1) / kTP)),
                       dim3(256), 0, s, xo, N, nrhs, (const int*)g.ipm.as<int>(), (const R*)Xr, (const R*)Xi);
  else
    hipLaunchKernelGGL(sol_out_kernel<R>, dim3(grid_for(N, rpp, 65535)), dim3(256), 0, s, xo, N, nrhs, ib,
                       (const R*)Xr, (const R*)Xi);
  LS_HIP(hipGetLastError());
  return LS_OK;
}

}  // namespace

ls_status gpu_factor(int n, const C<double>* rows_dev, bool fp32, hipStream_t s, GpuSolver** out) {
  const int dims[3] = {n, n, n};
  return gpu_factor_grid(dims, 3, rows_dev, fp32, s, out);
}

ls_status gpu_factor_grid(const int dims[3], int nc, const C<double>* rows_dev, bool fp32, hipStream_t s,
                          GpuSolver** out) {
  if (!out) return LS_EINVAL;
  *out = nullptr;
  if (!dims || dims[0] < 1 || dims[1] < 1 || dims[2] < 1 || (nc != 2 && nc != 3) || !rows_dev) return LS_EINVAL;
  std::unique_ptr<GpuSolver> g(new GpuSolver());
  g->n = dims[0];
  for (int d = 0; d < 3; ++d) g->dims[d] = dims[d];
  g->nc = nc;
  g->npts = (long)dims[0] * dims[1] * dims[2];
  g->fp32 = fp32;
  GpuSymbolic sym;
  LS_TRY(gpu_symbolic(dims, nc, sym));
  g->N = sym.N;
  g->fh = std::move(sym.fh);
  g->levels = std::move(sym.levels);
  g->lvl_off = std::move(sym.lvl_off);
  g->lvl_np = std::move(sym.lvl_np);
  g->lvl_nf = std::move(sym.lvl_nf);
  g->lvl_elems = std::move(sym.lvl_elems);
  g->u_rows = sym.u_rows;
  g->flops = sym.flops;
  const long fac_elems = sym.fac_elems;
  const IntMap& ibh = sym.ibh;
  long cinv_elems = 0;
  for (FrontDev& d : g->fh) {
    d.ci = cinv_elems;
    cinv_elems += 2L * (d.nf / nc);
    for (int slot = 0; slot < 2; ++slot) d.cu[slot] = d.child[slot] >= 0 ? g->fh[d.child[slot]].u : 0;
  }
  const size_t rs = fp32 ? sizeof(float) : sizeof(double);
  LS_TRY(g->cinv.alloc((size_t)cinv_elems * sizeof(int)));
  LS_TRY(g->fac.alloc((size_t)(fac_elems + kThinPad) * rs));
  LS_TRY(g->ib.alloc(ibh.size() * sizeof(int)));
  LS_TRY(g->ipm.alloc((size_t)std::max(1L, g->N) * sizeof(int)));
  LS_TRY(g->fd.alloc(g->fh.size() * sizeof(FrontDev)));
  std::vector<int> lv;
  for (const auto& l : g->levels) lv.insert(lv.end(), l.begin(), l.end());
  LS_TRY(g->lvl_d.alloc(lv.size() * sizeof(int)));
  LS_HIP(hipMemcpyAsync(g->ib.p, ibh.data(), ibh.size() * sizeof(int), hipMemcpyHostToDevice, s));
  LS_HIP(hipMemcpyAsync(g->fd.p, g->fh.data(), g->fh.size() * sizeof(FrontDev), hipMemcpyHostToDevice, s));
  LS_HIP(hipMemcpyAsync(g->lvl_d.p, lv.data(), lv.size() * sizeof(int), hipMemcpyHostToDevice, s));
  g->bytes = (size_t)fac_elems * rs;
  const int nfr = (int)g->fh.size();
  if (nc == 3)
    hipLaunchKernelGGL(child_map_kernel<3>, dim3(std::min(nfr, 65535)), dim3(256), 0, s, g->fd.as<FrontDev>(), nfr,
                       g->ib.as<int>(), g->cinv.as<int>());
  else
    hipLaunchKernelGGL(child_map_kernel<2>, dim3(std::min(nfr, 65535)), dim3(256), 0, s, g->fd.as<FrontDev>(), nfr,
                       g->ib.as<int>(), g->cinv.as<int>());
  LS_HIP(hipGetLastError());
  if (fp32)
    LS_TRY(factor_numeric<float>(*g, rows_dev, s));
  else
    LS_TRY(factor_numeric<double>(*g, rows_dev, s));
  *out = g.release();
  return LS_OK;
}

ls_status gpu_solve(GpuSolver* gs, const C<double>* b_dev, C<double>* x_dev, int nrhs, hipStream_t s) {
  if (!gs || !b_dev || !x_dev || nrhs < 1) return LS_EINVAL;
  return gs->fp32 ? solve_numeric<float>(*gs, b_dev, x_dev, nrhs, s)
                  : solve_numeric<double>(*gs, b_dev, x_dev, nrhs, s);
}

size_t gpu_factor_bytes(const GpuSolver* gs) { return gs ? gs->bytes : 0; }
double gpu_factor_flops(const GpuSolver* gs) { return gs ? gs->flops : 0.0; }
bool gpu_factor_is_fp32(const GpuSolver* gs) { return gs && gs->fp32; }
void gpu_free(GpuSolver* gs) { delete gs; }

}  // namespace ls
