// row_ops.h -- sixteen lanes sharing one cell: building blocks of the kernels that hold a
// cell's field polynomials in the registers of a row of lanes (point.hip).
//
// Inside one cell a field of the spline of degree SH is a polynomial sum_p F_p X^i/i! Y^j/j!
// Z^k/k!, p = i + (SH+1) (j + (SH+1) k), in the offset from the cell's base node (the nearest
// node for SH = 2, the node below for SH = 1).  A gather is a contraction of the coefficients
// F_p with the monomials at the particle.  A deposit sums the particles' node values over the
// cell before a node is touched, as exact integers.
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include "cell.h"
#include "fixsum.h"
#include "gmhc_internal.h"

namespace gmhc {
namespace {

// acc += (lane L of the row's c) * w: an FP64 multiply-add whose first factor is read
// from lane L of each row of sixteen lanes (DPP row broadcast), at the full rate and without
// LDS.  Every lane of the wave must be active.  The wait states cover a VALU write of c just
// before (two are needed ahead of a DPP read) and a transcendental result in w.
#define GMHC_FMAC(ACC, L) "v_fmac_f64_dpp " ACC ", %3, %4 row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
template <int L>
__device__ __forceinline__ void row_fma3(double& a0, double& a1, double& a2, double c, double w) {
  asm("s_nop 1\n\t" GMHC_FMAC("%0", "%5") GMHC_FMAC("%1", "%6") GMHC_FMAC("%2", "%7")
      : "+v"(a0), "+v"(a1), "+v"(a2)
      : "v"(c), "v"(w), "n"(L), "n"(L + 1), "n"(L + 2));
}
#undef GMHC_FMAC

template <int D, int SH>
constexpr int powers() {
  return D == 1 ? SH + 1 : (D == 2 ? (SH + 1) * (SH + 1) : (SH + 1) * (SH + 1) * (SH + 1));
}

// Row-wide read of lane 0 of each row.
__device__ __forceinline__ int row_first(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150, 0xF, 0xF, true); }

// The monomials at the point f times u.
template <int D, int SH, class R>
__device__ __forceinline__ void monomials(const R* f, R u, R* m) {
  constexpr int N = SH + 1;
  m[0] = u;
  m[1] = u * f[0];
  if constexpr (SH == 2) m[2] = R(0.5) * f[0] * m[1];
  if constexpr (D > 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      m[N + i] = f[1] * m[i];
      if constexpr (SH == 2) m[2 * N + i] = R(0.5) * f[1] * m[N + i];
    }
  }
  if constexpr (D > 2) {
#pragma unroll
    for (int i = 0; i < N * N; ++i) {
      m[N * N + i] = f[2] * m[i];
      if constexpr (SH == 2) m[2 * N * N + i] = R(0.5) * f[2] * m[N * N + i];
    }
  }
}

// Node values along one axis (v[0], v[st], v[2 st]) of the spline of degree SH into the
// coefficients of the cell's polynomial, in place.
template <int SH, class T>
__device__ __forceinline__ void to_powers(T* v, int st) {
  if constexpr (SH == 1) {
    v[st] = v[st] - v[0];
  } else {
    const T a = v[0], b = v[st], c = v[2 * st];
    const T s = (a - b) + (c - b);
    v[0] = b + T(0.125) * s;
    v[st] = T(0.5) * (c - a);
    v[2 * st] = s;
  }
}
template <int D, int SH, class T>
__device__ __forceinline__ void all_to_powers(T* v) {
  constexpr int N = SH + 1, NP = powers<D, SH>();
#pragma unroll
  for (int l = 0, st = 1; l < D; ++l, st *= N)
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if ((p / st) % N == 0) to_powers<SH>(v + p, st);
}

// ---- batches of one cell
//
// A wave cuts a window of wn consecutive particles, at most MAX, into batches: runs of one cell cut
// every sixteen particles, so that each batch fits a row of lanes.  list[b] is the first particle of
// batch b, list[(the number returned)] the end; cell(r) is the cell of particle r of the window (any
// r < wn).  All 64 lanes call it.
template <int MAX, class Cell>
__device__ __forceinline__ int list_batches(int wn, uint16_t* list, Cell&& cell) {
  static_assert(MAX <= 65535, "list holds 16-bit indices");
  const int lane = threadIdx.x & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  int nb = 0, carry = INT_MIN, run = 0;  // the last particle's cell and the start of its run
  for (int c0 = 0; c0 < wn; c0 += 64) {
    const int r = c0 + lane;
    const bool in = r < wn;
    const int g = cell(in ? r : wn - 1);
    int prev = __shfl_up(g, 1);
    if (lane == 0) prev = carry;
    const uint64_t starts = __ballot(in && g != prev);
    const uint64_t upto = starts & (below | (1ull << lane));
    const int first = upto ? c0 + 63 - __builtin_clzll(upto) : run;
    const bool bs = in && ((r - first) & 15) == 0;
    const uint64_t bm = __ballot(bs);
    if (bs) list[nb + __popcll(bm & below)] = (uint16_t)r;
    nb += __popcll(bm);
    carry = __builtin_amdgcn_readlane(g, 63);
    if (starts) run = c0 + 63 - __builtin_clzll(starts);
  }
  if (lane == 0) list[nb] = (uint16_t)wn;
  __syncthreads();
  return nb;
}

// Base cell of a position (linear index) and the offset from its base node.
template <int D, int SH>
__device__ __forceinline__ int base_cell(const Mesh& M, const double* x, double* f0) {
  int cell = 0;
#pragma unroll
  for (int l = 0; l < D; ++l) {
    const int j = (int)axis_node(M, l, SH == 1, x[l], f0[l]);
    cell |= (j & (M.n[l] - 1)) << (l == 0 ? 0 : (l == 1 ? M.ln[0] : M.ln[0] + M.ln[1]));
  }
  return cell;
}

// Mesh index of the node at offset (k0, k1, k2) from the base node of a cell.
template <int D>
__device__ __forceinline__ int cell_node(const Mesh& M, int cell, int k0, int k1, int k2) {
  const int s1 = M.ln[0], s2 = M.ln[0] + M.ln[1];
  int g = (cell + k0) & (M.n[0] - 1);
  if (D > 1) g |= (((cell >> s1) + k1) & (M.n[1] - 1)) << s1;
  if (D > 2) g |= (((cell >> s2) + k2) & (M.n[2] - 1)) << s2;
  return g;
}

// ---- sums over a row
//
// Sixteen values of every lane at a time go through LDS; the padding of the buffer puts the
// sixteen lanes that read one row in distinct banks.  (A reduce-scatter through DPP moves
// takes about 7 instructions per value, this about 2.)
struct RowBuffer {
  double v[16][66];
};

// Exact sums of FP64 values rounded to the fixed-point resolution q = 2^-s (fixsum.h), in two FP64
// numbers.  hi, offset by 3 2^91 q = 3 B, keeps every partial sum in one binade, so that adding v
// rounds it to a multiple of 2^40 q and the part left over, at most 2^39 q, is exact; that part is
// rounded to a multiple of q (to nearest, ties to even, as fix_add rounds v) and summed in lo, exactly
// for up to 2^13 values.  What reaches a node is therefore what its values would add one by one,
// whatever the order and the rows: particles that are mirror images leave mirror images.
constexpr int kExactSumMax = 1 << 13;
struct ExactScale {
  double hi0, lo0, hi_inv, lo_inv;
  __device__ __forceinline__ explicit ExactScale(const FixScale& f)
      : hi0(f.lo * (3.0 * 0x1p91)), lo0(f.lo * (1.5 * 0x1p52)), hi_inv(f.up * 0x1p-10), lo_inv(f.up * 0x1p30) {}
};
static_assert(kFixK == 30, "the limbs of ExactSum::add_to and the scale");
struct ExactSum {
  double hi, lo;
  __device__ __forceinline__ void clear(const ExactScale& x) {
    hi = x.hi0;
    lo = 0.0;
  }
  __device__ __forceinline__ void add(const ExactScale& x, double v) {
    const double h = hi + v;
    const double r = v - (h - hi);
    hi = h;
    lo += (r + x.lo0) - x.lo0;
  }
  __device__ __forceinline__ void add_to(const ExactScale& x, unsigned long long* acc, int64_t i) const {
    const long long h = (long long)((hi - x.hi0) * x.hi_inv), l = (long long)(lo * x.lo_inv);
    const long long H = (h << 10) + (l >> kFixK), L = l & ((1ll << kFixK) - 1);
    if (H) atomicAdd(acc + 2 * i, (unsigned long long)H);
    if (L) atomicAdd(acc + 2 * i + 1, (unsigned long long)L);
  }
};

// t[c] += the row's values 16 c + (lane of the row), for the NV values val(o).
template <int NV, class Val>
__device__ __forceinline__ void row_sums(RowBuffer& b, ExactSum* t, const ExactScale& x, Val&& val) {
  const int lane = threadIdx.x & 63, rl = lane & 15;
#pragma unroll
  for (int c = 0; c < (NV + 15) / 16; ++c) {
    __syncthreads();
#pragma unroll
    for (int o = 16 * c; o < 16 * c + 16 && o < NV; ++o) b.v[o - 16 * c][lane] = val(o);
    __syncthreads();
    // every lane sums a row of the buffer; those past the NV values are not used
    const double2* v = reinterpret_cast<const double2*>(&b.v[rl][lane & 48]);
    double2 u[8];
#pragma unroll
    for (int l = 0; l < 8; ++l) u[l] = v[l];
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      t[c].add(x, u[l].x);
      t[c].add(x, u[l].y);
    }
    // in place: sums left for later would hold every chunk's values in registers
    asm volatile("" : "+v"(t[c].hi), "+v"(t[c].lo));
  }
}

}  // namespace
}  // namespace gmhc
