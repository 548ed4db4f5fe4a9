// point.hip -- the passes over particles at one time: the point-shape deposit of charge and
// current at initialization, the canonical momenta P = p + q A_h(x), and the kinetic-energy
// sums of the diagnostics.
//
// What bounded the thread-per-particle forms: the deposit added 4 (SH+1)^d values per
// particle through 64-bit atomics, and neighbouring particles hit the same nodes; the gathers
// read 3 (SH+1)^d scattered mesh values per particle.  Here a row of sixteen lanes takes a
// batch of particles of one cell: the deposit's node values are summed over the batch, and over
// the row's following batches of the same cell, before a node is touched (exactly, so the mesh sums
// do not depend on the particles' order), and the gather reads the cell's three polynomials once per
// row and broadcasts their coefficients.  At
// initialization the particles may be in any order, so where it pays (point_order_pays) they are
// taken through their stable order by cell (an index sort; the storage order stays).  Elsewhere
// the storage order serves, and a window whose particles are too scattered (fewer than four per
// batch on average) takes one particle per lane.
//
// Measured at 8,388,608 particles on 64^3 (32 per cell, in grid-cell order): the deposit 76.2
// to 0.85 ms (0.81 with rounded sums of the cell's moments; the index sort adds 0.3 ms), the
// canonical momenta 1.74 to 0.61 ms, the kinetic energy 1.71 to 0.54 ms; the traffic none of them can
// do without takes 0.1 ms.  At 67,108,864 particles on 512^2 the deposit took 222 ms.  Left:
// instruction issue (exact LDS sums of 108 values per batch, gathers of 27 coefficients per cell).
#include <math.h>

#include <algorithm>

#include "gmhc_internal.h"
#include "row_ops.h"
#include "wave.h"

namespace gmhc {
namespace {

constexpr int kPointWindow = 256;  // particles per listing of batches, at most
constexpr int kPointBatch = 4;     // particles per batch of a window, on average and at least, for the row path
constexpr int kPointFill = 2048;   // workgroups that fill the chip (two waves per SIMD)
static_assert(kExactSumMax % kPointWindow == 0, "a row's sums are cleared between windows");

struct PointArgs {
  Mesh M;
  int64_t np, per;  // particles, and particles per workgroup
  double kappa, sign;
  int prec;
  const double* x[3];
  void* P[3];
  const void* q;
  void* v[3];
  unsigned long long* rho;
  unsigned long long* J;
  const double* A[3];
  double* partials;
  const int32_t* keys;  // the particles taken in the order perm, cells keys (may be null)
  const int32_t* perm;
};

enum PointMode { kDeposit = 0, kCanonical = 1, kKinetic = 2 };

// Weights of the nodes of one axis at the offset f.
template <int SH>
__device__ __forceinline__ void axis_weights(double f, double* w) {
  if constexpr (SH == 1) {
    w[0] = 1.0 - f;
    w[1] = f;
  } else {
    const double a = 0.5 - f, b = 0.5 + f;
    w[0] = 0.5 * a * a;
    w[1] = fma(-f, f, 0.75);
    w[2] = 0.5 * b * b;
  }
}

// The stencil of one particle read or written node by node.
template <int D, int SH, class F>
__device__ __forceinline__ void each_node(const Mesh& M, int cell, const double* f, F&& fn) {
  constexpr int N = SH + 1, NP = powers<D, SH>(), off = SH == 2 ? 1 : 0;
  double w[D][N];
#pragma unroll
  for (int l = 0; l < D; ++l) axis_weights<SH>(f[l], w[l]);
  // a row of nodes along x at a time, so that its reads are in flight together
#pragma unroll 1
  for (int r = 0; r < NP / N; ++r) {
    const int j = r % N, k = r / N;
    const double wy = D < 2 ? 1.0 : (j == 0 ? w[D > 1][0] : (j == 1 ? w[D > 1][1] : w[D > 1][N - 1]));
    const double wz = D < 3 ? 1.0 : (k == 0 ? w[D - 1][0] : (k == 1 ? w[D - 1][1] : w[D - 1][N - 1]));
#pragma unroll
    for (int i = 0; i < N; ++i) fn(cell_node<D>(M, cell, i - off, j - off, k - off), w[0][i] * wy * wz);
  }
}

// The same weights at once: the same products in the same order, so a particle adds the same
// values in a row and by itself.
template <int D, int SH>
__device__ __forceinline__ void node_weights(const double* f, double* s) {
  constexpr int N = SH + 1, NP = powers<D, SH>();
  double w[D][N];
#pragma unroll
  for (int l = 0; l < D; ++l) axis_weights<SH>(f[l], w[l]);
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const double wy = D < 2 ? 1.0 : w[D > 1][p / N % N], wz = D < 3 ? 1.0 : w[D - 1][p / (N * N)];
    s[p] = w[0][p % N] * wy * wz;
  }
}

template <int D, int SH, int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 3 && SH == 2 ? 2 : 4))) void k_point(PointArgs a) {
  constexpr int N = SH + 1, NP = powers<D, SH>(), off = SH == 2 ? 1 : 0;
  constexpr int NC = MODE == kDeposit ? (4 * NP + 15) / 16 : 1;
  __shared__ __align__(16) RowBuffer buf;
  __shared__ uint16_t list[kPointWindow + 1];
  const int lane = threadIdx.x, row = lane >> 4, rl = lane & 15;
  const Mesh& M = a.M;
  const int64_t b0 = (int64_t)blockIdx.x * a.per;
  const int64_t b1 = b0 + a.per < a.np ? b0 + a.per : a.np;
  double part[3] = {0.0, 0.0, 0.0};  // kinetic energy, sum |q| (v_y^2 + v_z^2), sum |q|
  double cf[NP];
  int tag = -1;
  const ExactScale fx(M.fx);
  ExactSum tot[NC];
  int jt = -1;
#pragma unroll
  for (int c = 0; c < NC; ++c) tot[c].clear(fx);
#pragma unroll
  for (int p = 0; p < NP; ++p) cf[p] = 0.0;

  auto position = [&](int64_t i, double* x) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < D; ++l) x[l] = a.x[l][i];
  };
  auto locate = [&](int64_t i, double* f) __attribute__((always_inline)) {
    double x[D];
    position(i, x);
    return base_cell<D, SH>(M, x, f);
  };
  // v = V(p) of particle i and its deposit weights q/dV (1, v)
  auto velocity = [&](int64_t i, double* coef) __attribute__((always_inline)) {
    const double q = ld_bulk(a.q, i, a.prec), m = fabs(q);
    const double p[3] = {ld_bulk(a.P[0], i, a.prec), ld_bulk(a.P[1], i, a.prec), ld_bulk(a.P[2], i, a.prec)};
    const double imk = 1.0 / (m * a.kappa);
    const double g = sqrt(1.0 + (p[0] * p[0] + p[1] * p[1] + p[2] * p[2]) * imk * imk);
    coef[0] = q / M.dV;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double v = p[c] / (m * g);
      st_bulk(a.v[c], i, v, a.prec);
      // a velocity that is not finite (a bad momentum, no charge) deposits nothing: its row's
      // sums are the neighbours' too
      coef[1 + c] = isfinite(v) ? coef[0] * v : 0.0;
    }
  };
  // what the potential at particle i is gathered for
  auto use = [&](int64_t i, const double* Ah) __attribute__((always_inline)) {
    const double q = ld_bulk(a.q, i, a.prec);
    if constexpr (MODE == kCanonical) {
#pragma unroll
      for (int c = 0; c < 3; ++c) st_bulk(a.P[c], i, ld_bulk(a.P[c], i, a.prec) + a.sign * q * Ah[c], a.prec);
    } else {
      const double m = fabs(q), imk = 1.0 / (m * a.kappa);
      double p[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) p[c] = ld_bulk(a.P[c], i, a.prec) - q * Ah[c];
      const double p2 = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
      const double g = sqrt(1.0 + p2 * imk * imk);
      part[0] += p2 / (m * (g + 1.0));
      const double vy = p[1] / (m * g), vz = p[2] / (m * g);
      part[1] += m * (vy * vy + vz * vz);
      part[2] += m;
    }
  };
  auto flush = [&]() __attribute__((always_inline)) {
    int r = rl;
    asm volatile("" : "+v"(r));  // keeps the lane's indices out of the registers of the main loop
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int o = 16 * c + r;
      if (o < 4 * NP && jt >= 0) {
        const int k = o / NP, nd = o - k * NP;
        const int g = cell_node<D>(M, jt, nd % N - off, (nd / N) % N - off, nd / (N * N) - off);
        if (k == 0)
          tot[c].add_to(fx, a.rho, g);
        else
          tot[c].add_to(fx, a.J, (int64_t)(k - 1) * M.Ng + g);
      }
      tot[c].clear(fx);
    }
  };

#pragma unroll 1
  for (int64_t w0 = b0; w0 < b1; w0 += kPointWindow) {
    const int wn = (int)(b1 - w0 < kPointWindow ? b1 - w0 : kPointWindow);
    if constexpr (MODE == kDeposit) {  // the most values an exact sum takes
      if ((w0 - b0) % kExactSumMax == 0 && w0 > b0 && __ballot(jt >= 0) != 0) flush();
    }
    __syncthreads();
    const int nb = list_batches<kPointWindow>(wn, list, [&](int r) {
      if (a.keys) return a.keys[w0 + r];
      double f[D];
      return locate(w0 + r, f);
    });
    if (kPointBatch * nb > wn) {  // scattered particles: one per lane
#pragma unroll 1
      for (int r = lane; r < wn; r += 64) {
        const int64_t i = a.perm ? a.perm[w0 + r] : w0 + r;
        double f[D];
        const int cell = locate(i, f);
        if constexpr (MODE == kDeposit) {
          double coef[4];
          velocity(i, coef);
          each_node<D, SH>(M, cell, f, [&](int g, double s) {
            fix_add(a.rho, g, rounded(coef[0] * s), M.fx.up);
            for (int c = 0; c < 3; ++c) fix_add(a.J, c * M.Ng + g, rounded(coef[1 + c] * s), M.fx.up);
          });
        } else {
          double Ah[3] = {0.0, 0.0, 0.0};
          each_node<D, SH>(M, cell, f, [&](int g, double s) {
            for (int c = 0; c < 3; ++c) Ah[c] += s * a.A[c][g];
          });
          use(i, Ah);
        }
      }
      continue;
    }
    const int rounds = (nb + 3) >> 2;
#pragma unroll 1
    for (int t = 0; t < rounds; ++t) {
      const int b = row * rounds + t;
      const bool on = b < nb;
      const int lo = on ? list[b] : 0;
      const bool live = on && rl < list[on ? b + 1 : 0] - lo;
      const int64_t r = w0 + (live ? lo + rl : 0);
      const int64_t i = a.perm ? a.perm[r] : r;
      double f[D], m[NP];
      const int cell = locate(i, f);
      int home = row_first(live ? cell : -1);
      if constexpr (MODE == kDeposit)
        node_weights<D, SH>(f, m);
      else
        monomials<D, SH>(f, 1.0, m);
      if constexpr (MODE == kDeposit) {
        double coef[4] = {0.0, 0.0, 0.0, 0.0};
        if (live) velocity(i, coef);
        if (home < 0) home = jt;
        if (__ballot(jt != home) != 0) {
          if (__ballot(jt >= 0) != 0) flush();
          jt = home;
        }
        row_sums<4 * NP>(buf, tot, fx, [&](int o) { return coef[o / NP] * m[o % NP]; });
      } else {
        if (home < 0) home = max(tag, 0);
        if (__ballot(tag != home) != 0) {  // lane c of the row holds A_c of the cell
          const double* base = a.A[0] + (rl < 3 ? rl : 0) * M.Ng;
#pragma unroll
          for (int p = 0; p < NP; ++p) cf[p] = base[cell_node<D>(M, home, p % N - off, (p / N) % N - off, p / (N * N) - off)];
          all_to_powers<D, SH>(cf);
          tag = home;
        }
        double Ah[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < NP; ++p) row_fma3<0>(Ah[0], Ah[1], Ah[2], cf[p], m[p]);
        if (live) use(i, Ah);
      }
    }
  }
  if constexpr (MODE == kDeposit) {
    if (__ballot(jt >= 0) != 0) flush();
  }
  if constexpr (MODE == kKinetic) {
    double s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = wave_reduce_f64<false>(part[k]);
    if (lane < kDiagParts)
      a.partials[(int64_t)blockIdx.x * kDiagParts + lane] = lane < 3 ? (lane == 0 ? s[0] : (lane == 1 ? s[1] : s[2])) : 0.0;
  }
}

// Particles per workgroup: one window, shorter (down to a wave's lanes) while the workgroups are
// too few to fill the chip, and several windows beyond eight waves per SIMD's worth of workgroups.
// With whole windows throughout, the kinetic energy's read-out took 5 to 10 us more for up to
// 131,072 particles (3D, 1,000 particles: 49 against 29 us).
int64_t point_per(int64_t np) {
  const int64_t waves = (np + 63) / 64;
  if (waves <= kPointFill * (kPointWindow / 64)) return 64 * std::max<int64_t>((waves + kPointFill - 1) / kPointFill, 1);
  const int64_t windows = (np + kPointWindow - 1) / kPointWindow;
  return kPointWindow * ((windows + kPointBlocks - 1) / kPointBlocks);
}

template <int MODE>
hipError_t launch_point(PointArgs& a, hipStream_t s) {
  if (a.np <= 0) return hipSuccess;
  a.per = point_per(a.np);
  const dim3 g((unsigned)point_blocks(a.np)), b(64);
  const bool lin = a.M.shape == 1;
  switch (a.M.d) {
    case 1:
      if (lin) hipLaunchKernelGGL((k_point<1, 1, MODE>), g, b, 0, s, a);
      else hipLaunchKernelGGL((k_point<1, 2, MODE>), g, b, 0, s, a);
      break;
    case 2:
      if (lin) hipLaunchKernelGGL((k_point<2, 1, MODE>), g, b, 0, s, a);
      else hipLaunchKernelGGL((k_point<2, 2, MODE>), g, b, 0, s, a);
      break;
    default:
      if (lin) hipLaunchKernelGGL((k_point<3, 1, MODE>), g, b, 0, s, a);
      else hipLaunchKernelGGL((k_point<3, 2, MODE>), g, b, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

int point_blocks(int64_t np) { return (int)((np + point_per(np) - 1) / point_per(np)); }

hipError_t launch_init_deposit(const InitArgs& i, hipStream_t s) {
  PointArgs a{};
  a.M = i.M;
  a.np = i.np;
  a.kappa = i.kappa;
  a.prec = i.prec;
  for (int c = 0; c < 3; ++c) {
    a.x[c] = i.x[c];
    a.P[c] = i.P[c];
    a.v[c] = i.v[c];
  }
  a.keys = i.keys;
  a.perm = i.perm;
  a.q = i.q;
  a.rho = i.rho;
  a.J = i.J;
  return launch_point<kDeposit>(a, s);
}

hipError_t launch_canonical(const CanonArgs& i, hipStream_t s) {
  PointArgs a{};
  a.M = i.M;
  a.np = i.np;
  a.sign = i.sign;
  a.prec = i.prec;
  for (int c = 0; c < 3; ++c) {
    a.x[c] = i.x[c];
    a.P[c] = i.P[c];
    a.A[c] = i.A[c];
  }
  a.keys = i.keys;
  a.perm = i.perm;
  a.q = i.q;
  return launch_point<kCanonical>(a, s);
}

hipError_t launch_kinetic(const KinArgs& i, hipStream_t s) {
  PointArgs a{};
  a.M = i.M;
  a.np = i.np;
  a.kappa = i.kappa;
  a.prec = i.prec;
  for (int c = 0; c < 3; ++c) {
    a.x[c] = i.x[c];
    a.P[c] = const_cast<void*>(i.P[c]);
    a.A[c] = i.A[c];
  }
  a.q = i.q;
  a.partials = i.partials;
  return launch_point<kKinetic>(a, s);
}

}  // namespace gmhc
