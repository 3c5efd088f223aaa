// Smooth particle-mesh Ewald for point charges, gfx950.  Paper: CabanaMD's
// long-range path -- real-space energies and forces through the neighbor
// parallel loops, and for reciprocal space spline spreading of charge onto a
// uniform grid, 3-D FFTs and a gradient gather back to the particles
// (CabanaMD subsection; Cabana "Long Range Solvers", "Particle-Grid
// Interpolation").  The paper prints no equation; the method is SPME as
// defined by Essmann et al. (1995, J. Chem. Phys. 103, 8577), Gaussian units:
//
//   real space:  E_dir = 1/2 sum_i sum_{j, r < rc} q_i q_j erfc(alpha r)/r
//                F_i   = sum_j q_i q_j [erfc(alpha r)/r + 2 alpha/sqrt(pi) e^{-alpha^2 r^2}] d_ij / r^2
//   reciprocal:  u_a = K_a x_a / L_a; cardinal B-splines M_n of even order n
//                Q(k) = sum_i q_i prod_a M_n(u_ai - k_a)   (k_a = floor(u_ai) - j mod K_a)
//                E_rec = 1/2 sum_m B(m) C(m) |F(Q)(m)|^2,
//                B = prod_a |sum_{k<n-1} M_n(k+1) e^{2 pi i m_a k/K_a}|^-2,
//                C = e^{-pi^2 |m'|^2/alpha^2} / (pi V |m'|^2), C(0) = 0
//                phi = unnormalised inverse transform of B C F(Q);
//                F_i = -q_i sum_k grad_i[prod_a M_n(u_ai - k_a)] phi(k)
//   self:        E_self = -alpha/sqrt(pi) sum_i q_i^2
//
// Kernels: the real-space pair loop walks the tiled full list with four lanes
// per particle over packed (x, y, z, q) records (the LJ traversal), erfc(x) and e^{-x^2}
// from polynomials (two forms, by alpha rc and by whether energies are wanted);
// charge is spread into boxes of grid tiles in LDS, which the x pass adds up as it
// reads its rows (or onto the grid by FP64 atomics); the 3-D transform is real-to-complex: the x pass turns each row of
// K0 reals into K0/2 + 1 coefficients through one complex FFT of length K0/2
// plus a split step, and the y and z passes run on that half grid, each pass two
// register transforms per row with one exchange through LDS (rows along y and z
// loaded with consecutive x across lanes, so every pass reads and writes whole cache
// lines).  The z pass multiplies by the influence function between its forward and
// inverse transforms, each coefficient with 0 < m_0 < K0/2 counted twice in the
// energy (Hermitian symmetry of a real input); the inverse mirrors it and leaves phi
// real; the gather reads boxes of phi from LDS (or the grid).
#include <type_traits>

#include "common.h"

namespace ljmd {

void launch_scan(int32_t m, const int32_t *counts, int32_t *start, hipStream_t st);

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kMaxGrid = 256;  // points per edge
constexpr int kThreads = 256;
constexpr int kGatherAtoms = 256;  // particles per gather block
constexpr int kGatherTeam = 2;     // lanes per particle
constexpr int kEwAtoms = 128;  // real space: particles per block
constexpr int kEwTeam = 4;      // lanes per particle
constexpr int kEwThreads = kEwAtoms * kEwTeam;
// Two forms of the pair's erfc(x) and e^{-x^2}, x = alpha r:
//   table   (forces without energies, alpha rc up to kTableReach) the force's kernel
//           G(x) = erfc(x) + 2/sqrt(pi) x e^{-x^2} by Taylor polynomials about the centres of
//           128 equal intervals of [0, alpha rc]: no exponential per pair;
//   erfcx   (everything else) erfc(x) = e^{-x^2} erfcx(x), erfcx by degree-10 Taylor
//           polynomials about the centres of 32 equal intervals, relative error ~1e-15: as
//           accurate for each pair's own value wherever the pair lies.
// Why the line lies there: a polynomial's remainder is a fraction of G(0) = 1, not of the
// far pairs' G.  Largest relative error of a pair's force over (0.2 rc, rc), erfcx / table:
// alpha rc = 3 1.4e-15 / 1.2e-15, 3.5 1.4e-15 / 1.5e-15, 4 2.4e-15 / 3.4e-15, 5 5.8e-16 /
// 4.2e-13, 6 4.9e-15 / 1.8e-11, 10 8.8e-16 / 4.5e-7; of a pair's energy at 3 1.5e-15 / 5.4e-15.
constexpr double kTableReach = 3.5;
constexpr int kErfcIntervals = 128;
constexpr int kErfcCoefs = 9;   // degree 8
constexpr int kErfcStride = 10;  // doubles per interval in LDS: 16 of 80-byte rows share no bank
constexpr int kErfcSeeds = 384;  // doubles of the workspace: G(c) and e^{-c^2} per interval, or
                                 // the erfcx polynomials
constexpr int kErfcxIntervals = 32;
constexpr int kErfcxDegree = 10;
constexpr int kErfcxStride = 12;  // coefficients per interval, padded
static_assert(kErfcxIntervals * kErfcxStride <= kErfcSeeds, "erfcx polynomials");
static_assert(2 * kErfcIntervals <= kErfcSeeds, "seeds of G");

// Slots per group and lane, four lanes per particle.  500,000 / 32,000 particles (us): table
// 103.8 / 15.0 (with r rounded once more, which doubles the error, 101.7 / 14.8; erfcx with two
// lanes per particle and 6 slots 136.5 / 21.1); erfcx without energies 2, 3, 4 slots 140 / 16.4,
// 136 / 15.8, 140 / 15.9; with energies 2, 3, 4 slots 137 / 19.2, 145 / 18.6, 142 / 19.4 (two
// lanes and 6 slots 145 / 23.4; the table and one for erfc 150 / 19.8).
template <bool EV, bool TABLE>
constexpr int ew_unroll() { return EV || TABLE ? 2 : 3; }

// ------------------------------------------------------------ real space --

struct RealArgs {
  BoxK b;
  double alpha, a2, c2a;  // alpha, alpha^2, 2 alpha / sqrt(pi) (the last two: erfcx)
  double rc2, margin;
  int32_t n;
  const int32_t *nbr;
  const int32_t *nnbr;
  int32_t maxn;
  const double4 *xq;  // packed (x, y, z, q)
  double *F;
  int accumulate;
  double *partial;  // per-block E_dir, or null
  const double *seeds;  // [kErfcIntervals] G(c), then e^{-c^2}; or [kErfcxIntervals][kErfcxStride]
  double dx, u_scale;   // table: interval width in alpha r; intervals per unit length
  double inv_dx, half_dx;  // erfcx: intervals of width dx = alpha rc / kErfcxIntervals
};

// Packs (x, y, z, q) records; block 0 also writes, for the form TABLE or not,
//   the table's seeds G(c) and e^{-c^2} at every interval's centre c, or
//   the erfcx polynomials: about each centre c, a_n = erfcx^(n)(c) / n! from erfcx(c) =
//   e^{c^2} erfc(c) and y' = 2 x y - 2/sqrt(pi), y^(n+1) = 2 x y^(n) + 2 n y^(n-1).
template <bool TABLE>
__global__ __launch_bounds__(kThreads) void k_pack_xq(RealArgs a, const double *x, const double *q,
                                                      double4 *xq, double *seeds) {
  if (TABLE && blockIdx.x == 0 && threadIdx.x < kErfcIntervals) {
    // c = alpha (k + 1/2) / u_scale with what its rounding leaves, lo, and c^2 likewise:
    // G changes by 2 c^2 times a relative change of c
    const double k = threadIdx.x + 0.5, h = k / a.u_scale;
    const double c = a.alpha * h;
    const double lo =
        __builtin_fma(a.alpha, h, -c) + a.alpha * (__builtin_fma(-h, a.u_scale, k) / a.u_scale);
    const double cc = c * c;
    const double e0 = exp(-cc), e = __builtin_fma(-e0, __builtin_fma(c, c, -cc), e0);
    constexpr double two = 1.1283791670955126, two_lo = 1.533545961316588e-17;  // 2/sqrt(pi)
    const double ce = c * e;
    seeds[threadIdx.x] =
        __builtin_fma(two, ce, erfc(c)) + (two_lo * ce - 2.0 * two * cc * e * lo);
    seeds[kErfcIntervals + threadIdx.x] = __builtin_fma(-2.0 * c * lo, e, e);
  }
  if (!TABLE && blockIdx.x == 0 && threadIdx.x < kErfcxIntervals) {
    const double c = (2 * threadIdx.x + 1) * a.half_dx;
    double *p = seeds + threadIdx.x * kErfcxStride;
    double ym1 = exp(c * c) * erfc(c);
    double y = 2.0 * c * ym1 - 2.0 / sqrt(kPi);
    double fact = 1.0;
    p[0] = ym1;
    p[1] = y;
    for (int k = 1; k < kErfcxDegree; ++k) {
      const double yn = 2.0 * c * y + 2.0 * k * ym1;
      fact *= (k + 1);
      p[k + 1] = yn / fact;
      ym1 = y;
      y = yn;
    }
  }
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  xq[i] = make_double4(x[3 * i], x[3 * i + 1], x[3 * i + 2], q[i]);
}

// The block's polynomials in LDS.  TABLE: from the seeds; with e_n the Taylor coefficients
// of e^{-x^2} about c, e_{n+1} = -2 (c e_n + e_{n-1}) / (n+1), the coefficients are
//   G(c), then -4/sqrt(pi) (c^2 e_{n-1} + 2 c e_{n-2} + e_{n-3}) / n  (G' = -4/sqrt(pi) x^2 e^{-x^2})
// times dx^n.  Else a copy of the erfcx polynomials.
template <bool TABLE>
__device__ __forceinline__ void erfc_tables(const RealArgs &a, double *tab) {
  if constexpr (!TABLE) {
    for (int k = threadIdx.x; k < kErfcxIntervals * kErfcxStride; k += kEwThreads)
      if (k % kErfcxStride <= kErfcxDegree) tab[k] = a.seeds[k];
    return;
  }
  const int k0 = threadIdx.x;
  if (k0 >= kErfcIntervals) return;
  constexpr double two = 1.1283791670955126;  // 2 / sqrt(pi)
  const double c = (k0 + 0.5) * a.dx;
  double *g = tab + k0 * kErfcStride;
  double e0 = a.seeds[kErfcIntervals + k0], e1 = 0.0, e2 = 0.0;  // e_{n-1}, e_{n-2}, e_{n-3}
  g[0] = a.seeds[k0];
  double pw = -two;
#pragma unroll
  for (int k = 1; k < kErfcCoefs; ++k) {
    pw *= a.dx;
    const double f = pw * (1.0 / k);
    g[k] = 2.0 * f * ((c * c) * e0 + 2.0 * c * e1 + e2);
    const double en = (-2.0 / k) * (c * e0 + e1);
    e2 = e1;
    e1 = e0;
    e0 = en;
  }
}

template <bool WIDE>
__device__ __forceinline__ const double4 *xq_of(const double4 *p, int32_t j) {
  if constexpr (WIDE)
    return p + j;
  else
    return (const double4 *)((const char *)p + ((uint32_t)j << 5));
}

template <int DEGREE>
__device__ __forceinline__ double horner(const double *cf, double t) {
  double p = cf[DEGREE];
#pragma unroll
  for (int k = DEGREE - 1; k >= 0; --k) p = __builtin_fma(p, t, cf[k]);
  return p;
}

// One pair: adds q_j-weighted force scalar times d and (EV) the energy kernel.
template <bool WRAP, bool EV, bool TABLE>
__device__ __forceinline__ void real_pair(const RealArgs &a, const double *tab, const double4 &me,
                                          const double4 &o, bool ok, double &fx, double &fy,
                                          double &fz, double &e) {
  static_assert(!(EV && TABLE), "energies come from erfcx");
  double dx = me.x - o.x, dy = me.y - o.y, dz = me.z - o.z;
  if constexpr (WRAP) {
    dx = min_image(dx, a.b.L[0], a.b.invL[0]);
    dy = min_image(dy, a.b.L[1], a.b.invL[1]);
    dz = min_image(dz, a.b.L[2], a.b.invL[2]);
  }
  const double r2 = dist2(dx, dy, dz);
  const bool in = ok && r2 < a.rc2;
  double qs;
  if constexpr (TABLE) {
    // r^2 with fewer roundings than the cutoff's, and r to half a unit: a relative error
    // of r enters the force 2 (alpha r)^2 times over; 1 keeps padding and far pairs finite
    const double rr2 = in ? __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx)) : 1.0;
    const double ir = rsqrt64(rr2);
    double r = rr2 * ir;
    const double u = a.u_scale * r;  // the interval, before r's last refinement
    int it = (int)u;
    it = it < kErfcIntervals - 1 ? it : kErfcIntervals - 1;
    r = __builtin_fma(0.5 * ir, __builtin_fma(-r, r, rr2), r);
    const double t = __builtin_fma(a.u_scale, r, -((double)it + 0.5));
    qs = (in ? o.w * ir : 0.0) * (ir * ir) * horner<kErfcCoefs - 1>(tab + it * kErfcStride, t);
  } else {
    const double rr2 = in ? r2 : 1.0;  // keeps padding and far pairs finite
    // 1/r from one refined reciprocal square root of r^2 and r = r^2 / r: about
    // 9 % faster at 500k atoms than a square root followed by a reciprocal
    const double ir = rsqrt64(rr2);
    const double xa = a.alpha * (rr2 * ir);
    int it = (int)(xa * a.inv_dx);
    it = it < kErfcxIntervals - 1 ? it : kErfcxIntervals - 1;
    const double t = xa - (2 * it + 1) * a.half_dx;
    const double ex = exp(-a.a2 * rr2);
    const double er = ex * horner<kErfcxDegree>(tab + it * kErfcxStride, t) * ir;  // erfc(alpha r) / r
    qs = in ? o.w * ((er + a.c2a * ex) * (ir * ir)) : 0.0;
    if constexpr (EV) e += in ? o.w * er : 0.0;
  }
  fx = __builtin_fma(qs, dx, fx);
  fy = __builtin_fma(qs, dy, fy);
  fz = __builtin_fma(qs, dz, fz);
}

// Lane t's entries of the row, in masked groups of U (slots beyond cnt repeat the
// group's first entry).
template <bool WRAP, bool WIDE, bool EV, bool TABLE>
__device__ __forceinline__ void real_row(const RealArgs &a, const double *tab, const int32_t *row,
                                         int32_t cnt, const double4 &me, double &fx, double &fy,
                                         double &fz, double &e) {
  constexpr int U = ew_unroll<EV, TABLE>();
  constexpr int kStep = kEwTeam * kWave;
#pragma unroll 1
  for (int32_t k = 0; k < cnt; k += U, row += U * kStep) {
    int32_t j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = row[(k + u < cnt ? u : 0) * kStep];
    double4 o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) o[u] = *xq_of<WIDE>(a.xq, j[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      real_pair<WRAP, EV, TABLE>(a, tab, me, o[u], k + u < cnt, fx, fy, fz, e);
  }
}

template <bool WIDE, bool EV, bool TABLE>
__global__ __launch_bounds__(kEwThreads) void k_ewald_real(RealArgs a) {
  __shared__ double red[kRedRows * kEwThreads / kWave];
  __shared__ __align__(16) double
      tab[TABLE ? kErfcIntervals * kErfcStride : kErfcxIntervals * kErfcxStride];
  const int blk = flat_block<WIDE>(), nblk = flat_blocks<WIDE>(a.n, kEwAtoms);
  if (WIDE && blk >= nblk) return;
  erfc_tables<TABLE>(a, tab);
  __syncthreads();
  const int t = (int)threadIdx.x % kEwTeam;
  const int32_t i = xcd_block(blk, nblk) * kEwAtoms + (int)threadIdx.x / kEwTeam;
  const bool live = i < a.n;
  double4 me = make_double4(0.0, 0.0, 0.0, 0.0);
  if (live) me = a.xq[i];
  const double m = a.margin;
  const bool inside = !live || (me.x >= m && me.x <= a.b.L[0] - m && me.y >= m &&
                                me.y <= a.b.L[1] - m && me.z >= m && me.z <= a.b.L[2] - m);
  const bool interior = __ballot(!inside) == 0;
  double fx = 0.0, fy = 0.0, fz = 0.0, e = 0.0;
  if (live) {
    const int32_t ctot = a.nnbr[i];
    const int32_t cnt = ctot > t ? (ctot - t + kEwTeam - 1) / kEwTeam : 0;
    const int32_t *row =
        a.nbr + (int64_t)(i >> 6) * a.maxn * kWave + (i & (kWave - 1)) + (int64_t)t * kWave;
    if (interior)
      real_row<false, WIDE, EV, TABLE>(a, tab, row, cnt, me, fx, fy, fz, e);
    else
      real_row<true, WIDE, EV, TABLE>(a, tab, row, cnt, me, fx, fy, fz, e);
  }
  fx = team_sum<kEwTeam>(fx);
  fy = team_sum<kEwTeam>(fy);
  fz = team_sum<kEwTeam>(fz);
  if (live && t < 3) {  // lane t of the team writes component t
    double *F = a.F + 3 * (int64_t)i + t;
    const double f = me.w * (t == 0 ? fx : (t == 1 ? fy : fz));
    *F = a.accumulate ? *F + f : f;
  }
  if constexpr (EV) {
    double v[1] = {live ? 0.5 * me.w * e : 0.0};  // per lane: the team's lanes add up
    block_sum<kEwThreads / kWave, 1>(v, red, a.partial + blk);
  }
}

// ------------------------------------------------------------- B-splines --

// M_n(w + j) for j = 0..n-1 (w in [0, 1)) by the recursion
//   M_k(v) = (v M_{k-1}(v) + (k - v) M_{k-1}(v - 1)) / (k - 1),  M_2(w) = w, M_2(w+1) = 1 - w;
// dm receives dM_n(w + j)/dv = M_{n-1}(w + j) - M_{n-1}(w + j - 1) when requested.
template <int N, bool DERIV>
__device__ __forceinline__ void spline_weights(double w, double (&m)[N], double (&dm)[N]) {
  double a[N];
  a[0] = w;
  a[1] = 1.0 - w;
#pragma unroll
  for (int j = 2; j < N; ++j) a[j] = 0.0;
#pragma unroll
  for (int k = 3; k <= N; ++k) {
    if (DERIV && k == N) {
#pragma unroll
      for (int j = 0; j < N; ++j) dm[j] = a[j] - (j > 0 ? a[j - 1] : 0.0);
    }
    const double inv = 1.0 / (k - 1);
#pragma unroll
    for (int j = k - 1; j >= 0; --j) {
      const double v = w + j;
      const double lo = j > 0 ? a[j - 1] : 0.0;
      a[j] = (v * a[j] + (k - v) * lo) * inv;
    }
  }
#pragma unroll
  for (int j = 0; j < N; ++j) m[j] = a[j];
}

struct RecArgs {
  BoxK b;
  int32_t K[3];
  double scale[3];  // K_a / L_a
  double alpha;
  int32_t n;
  const double *x;
  const double *q;
  double *grid;        // [K2][K1][K0] real: Q, later phi; x fastest
  double2 *half;       // [K2][K1][K0/2 + 1] complex transform of the grid
  double *bmod;        // axis factors of the influence function at bmod + a * kMaxGrid
  double *partial;     // reciprocal energy, then gather blocks
  double *F;
  int accumulate;
};

// k mod K for a grid edge K, a power of two.
__device__ __forceinline__ int wrapi(int k, int K) { return k & (K - 1); }

// |b_a(m)|^2 e^{-pi^2 (m'/L_a)^2 / alpha^2} for every axis a, m < K_a (m' = m, or m - K_a
// above K_a/2), with |b_a(m)|^2 = |sum_{k=0}^{n-2} M_n(k+1) e^{2 pi i m k / K_a}|^-2: the
// influence function's factors of one axis (its Gaussian is a product over the axes).
// The blocks beyond those of the tables set z[0..nz) to zero.
constexpr int kBmodBlocks = 3 * kMaxGrid / kThreads;
template <int N>
__global__ __launch_bounds__(kThreads) void k_bmod(RecArgs a, double *z, int64_t nz) {
  if (blockIdx.x >= kBmodBlocks) {
    const int64_t k = (int64_t)(blockIdx.x - kBmodBlocks) * kThreads + threadIdx.x;
    if (k < nz) z[k] = 0.0;
    return;
  }
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int ax = t / kMaxGrid, m = t % kMaxGrid;
  if (ax >= 3 || m >= a.K[ax]) return;
  double mk[N], dk[N];
  spline_weights<N, false>(0.0, mk, dk);  // mk[j] = M_n(j): M_n(k+1) = mk[k+1]
  double re = 0.0, im = 0.0;
  for (int k = 0; k <= N - 2; ++k) {
    double s, c;
    sincospi(2.0 * (double)((int64_t)m * k % a.K[ax]) / a.K[ax], &s, &c);
    re += mk[k + 1] * c;
    im += mk[k + 1] * s;
  }
  const double f = (m <= a.K[ax] / 2 ? m : m - a.K[ax]) * a.b.invL[ax];
  a.bmod[ax * kMaxGrid + m] =
      exp(-kPi * kPi * (f * f) / (a.alpha * a.alpha)) / (re * re + im * im);
}

// ------------------------------------------------- charge and force tiles --
//
// The grid is cut into tiles; a particle belongs to the tile of its base point
// floor(u).  Its support reaches N - 1 points below the base in every dimension, so a
// tile's particles touch a box of E = T + N - 1 points per dimension.  Particles are
// sorted by tile (count, then scan and scatter of their indices, one launch for up to
// 4,096 tiles); one block per tile (more for a crowded one) then adds its particles'
// weights into the box in LDS and writes the box out, and the x pass adds up the (one to
// eight) boxes that cover each point as it reads its rows: no atomics on the grid, no
// clearing of it, and the same cost in whatever order the particles come.  The gather takes
// the box of phi into LDS once per tile.
//
// Why: FP64 atomics on the grid run at about 190 per ns whatever their locality, and one
// box per 64 consecutive particles needs 21 of them per particle (96 us at 500,000
// particles and 128^3, 41 of them without the atomics); the gather's 16-byte reads of
// single rows are bound at one lane per cycle.  Measured (us, 500,000 particles and
// 128^3 / 32,000 and 64^3): clearing and spreading 102 / 41 -> count, scan, scatter,
// boxes and their sums in the x pass 8.7 + 5.5 + 4.1 + 26.1 + 6.2 / 4.1 + 3.9 + 2.6 +
// 6.9 + 2.7; gather 35 / 6.9 -> 22.8 / 5.6.  The boxes are bound by the LDS atomics
// (about 30 cycles per 64 additions), the same with 1, 2 or 4 lanes per particle.
struct TileK {
  int32_t lg[3];  // log2 of the tile's edge T
  int32_t nt[3];  // tiles per dimension
  int32_t e[3];   // box edge T + N - 1
  int32_t ntiles, box;  // box: points per box
  int32_t crowd, chunk;  // most particles of a tile's own block; particles per chunk
  int32_t *count, *start, *key, *rank, *order;  // count[ntiles]: number of crowded tiles
  double *boxes;
};

// A tile of more than `crowd` particles is crowded: its block leaves them to other blocks,
// two for every `chunk` consecutive particles in tile order (a chunk meets at most two
// crowded tiles, its first particle's and its last's, as crowd >= chunk), each adding its
// box to the tile's by FP64 atomics (the tile's box is cleared when the particles are
// ordered).  So a droplet or a slab spreads over the chip too.  The whole reciprocal call at
// order 4 (us), spreading by atomics / one block per tile whatever it holds / this: 262,144
// particles in a 20th, an 8th, a quarter of the edge of a 128^3 grid 290 / 882 / 182, 266 /
// 2,205 / 177, 191 / 626 / 151, in a slab of a tenth 174 / 237 / 150; 32,768 in an 8th of 64^3
// 69 / 350 / 57, in a 20th of 32^3 60 / 785 / 48.  Uniform systems: 121.9 / 47.2 without
// this, 121.8 / 47.4 with it at 500,000 and 128^3 / 32,000 and 64^3.
constexpr int kTileCrowd = 1024;  // at least: four passes of a block
constexpr int kTileChunk = 256;   // at least: one pass

// The tile of block `blk` and its particles in tile order [p0, end): all of tile blk's for
// blk < ntiles (the caller leaves when they are more than crowd), else the part of a chunk
// in a crowded tile; false when there is none.  Block-uniform.
__device__ __forceinline__ bool tile_work(const TileK &t, int n, int blk, int &tile, int &p0,
                                          int &end) {
  if (blk < t.ntiles) {
    tile = xcd_block(blk, t.ntiles);
    p0 = t.start[tile];
    end = t.start[tile + 1];
    return true;
  }
  if (t.count[t.ntiles] == 0) return false;  // no crowded tile
  const int c0 = (blk - t.ntiles) / 2 * t.chunk, c1 = n - c0 > t.chunk ? c0 + t.chunk : n;
  const int first = t.key[t.order[c0]];
  tile = (blk - t.ntiles) % 2 == 0 ? first : t.key[t.order[c1 - 1]];
  if ((blk - t.ntiles) % 2 != 0 && tile == first) return false;
  p0 = t.start[tile];
  end = t.start[tile + 1];
  if (end - p0 <= t.crowd) return false;
  p0 = p0 > c0 ? p0 : c0;
  end = end < c1 ? end : c1;
  return true;
}

// Clears the box of every crowded tile whose particle of rank 0 is this thread's (live
// threads: a particle of tile `key` with m particles) and counts those tiles; the whole
// block calls it.
template <int THREADS>
__device__ __forceinline__ void clear_crowded(const TileK &t, bool live, int key, int rank, int m) {
  __shared__ int32_t crowded[THREADS], ncrowded;
  if (threadIdx.x == 0) ncrowded = 0;
  __syncthreads();
  if (live && rank == 0 && m > t.crowd) {
    crowded[atomicAdd(&ncrowded, 1)] = key;
    atomicAdd(&t.count[t.ntiles], 1);
  }
  __syncthreads();
  for (int k = 0; k < ncrowded; ++k) {
    double *box = t.boxes + (int64_t)crowded[k] * t.box;
    for (int q = threadIdx.x; q < t.box; q += THREADS) box[q] = 0.0;
  }
}

// Tile of a base point, and the point's place in it.
__device__ __forceinline__ int tile_of(const TileK &t, const int (&b)[3]) {
  return ((b[2] >> t.lg[2]) * t.nt[1] + (b[1] >> t.lg[1])) * t.nt[0] + (b[0] >> t.lg[0]);
}

// Tile and rank in it (in order of counting) of every particle, tile counts, and per
// block the self energy -alpha/sqrt(pi) q_i^2.  Lanes of a wavefront in the same tile
// share one atomic add, as in the cell sort.
__global__ __launch_bounds__(kGatherAtoms) void k_tile_count(RecArgs a, TileK tk,
                                                            double *self_partial) {
  __shared__ double red[kRedRows * kGatherAtoms / kWave];
  const int64_t i = (int64_t)blockIdx.x * kGatherAtoms + threadIdx.x;
  const bool live = i < a.n;
  double v[1] = {0.0};
  int tile = -1;
  if (live) {
    int b[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) b[d] = wrapi((int)floor(a.x[3 * i + d] * a.scale[d]), a.K[d]);
    tile = tile_of(tk, b);
    const double qi = a.q[i];
    v[0] = -a.alpha / __builtin_sqrt(kPi) * qi * qi;
  }
  const int r = count_ranks(live, tile, tk.count);
  if (live) {
    tk.key[i] = tile;
    tk.rank[i] = r;
  }
  block_sum<kGatherAtoms / kWave, 1>(v, red, self_partial + blockIdx.x);
}

__global__ __launch_bounds__(kThreads) void k_tile_scatter(int32_t n, TileK tk) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const bool live = i < n;
  const int32_t key = live ? tk.key[i] : 0, rank = live ? tk.rank[i] : 0;
  const int32_t s = tk.start[key];
  if (live) tk.order[s + rank] = (int32_t)i;
  const int32_t m = tk.start[key + 1] - s;
  if (__syncthreads_or(live && m > tk.crowd)) clear_crowded<kThreads>(tk, live, key, rank, m);
}

// As the scan of the counts into tk.start and k_tile_scatter, in one launch, for up to
// kOrderTiles tiles: every block scans all counts (four per thread) into LDS, block 0
// also writes them.  The
// whole reciprocal call, replayed from a graph (us): 32,000 particles and 64^3 47.1 ->
// 45.7, 500,000 and 128^3 120.9 -> 120.6.
constexpr int kOrderThreads = 1024;
constexpr int kOrderTiles = 4 * kOrderThreads;
__global__ __launch_bounds__(kOrderThreads) void k_tile_order(int32_t n, TileK tk) {
  constexpr int kWaves = kOrderThreads / kWave;
  __shared__ int32_t start[kOrderTiles + 1];
  __shared__ int32_t wsum[kWaves], wfull[kWaves];
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  const int64_t i = (int64_t)blockIdx.x * kOrderThreads + t;
  const int32_t key = i < n ? tk.key[i] : 0, rank = i < n ? tk.rank[i] : 0;
  int32_t v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = 4 * t + q < tk.ntiles ? tk.count[4 * t + q] : 0;
  const int32_t s = v[0] + v[1] + v[2] + v[3];
  const int32_t inc = wave_inclusive_scan(s);
  const bool full = __ballot(max(max(v[0], v[1]), max(v[2], v[3])) > tk.crowd) != 0;
  if (lane == kWave - 1) {
    wsum[w] = inc;
    wfull[w] = full;
  }
  __syncthreads();
  int32_t run = inc - s, crowded = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    run += k < w ? wsum[k] : 0;
    crowded |= wfull[k];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = 4 * t + q;
    start[c] = run;
    if (blockIdx.x == 0 && c < tk.ntiles) tk.start[c] = run;
    run += v[q];
    if (blockIdx.x == 0 && c == tk.ntiles - 1) tk.start[tk.ntiles] = run;
    if (c == kOrderTiles - 1) start[kOrderTiles] = run;
  }
  __syncthreads();
  if (i < n) tk.order[start[key] + rank] = (int32_t)i;
  if (crowded) clear_crowded<kOrderThreads>(tk, i < n, key, rank, start[key + 1] - start[key]);
}

// Origin of tile `tile` (first base point).
__device__ __forceinline__ void tile_origin(const TileK &t, int tile, int (&o)[3]) {
  const int q = tile / t.nt[0];
  o[0] = (tile - q * t.nt[0]) << t.lg[0];
  o[2] = (q / t.nt[1]) << t.lg[2];
  o[1] = (q % t.nt[1]) << t.lg[1];
}

constexpr int kTileThreads = 512;
constexpr int kTileTeam = 2;  // lanes per particle

// TEAM lanes per particle, lane t the planes jz = t, t + TEAM, ...
template <int N, int TX, int TY, int TZ, int TEAM>
__global__ __launch_bounds__(kTileThreads) void k_spread_tile(RecArgs a, TileK tk) {
  constexpr int EX = TX + N - 1, EY = TY + N - 1, EZ = TZ + N - 1;
  __shared__ double box[EX * EY * EZ];
  int tile, p0, end;
  if (!tile_work(tk, a.n, blockIdx.x, tile, p0, end)) return;  // block-uniform
  const int t = (int)threadIdx.x % TEAM;
  for (int k = threadIdx.x; k < EX * EY * EZ; k += kTileThreads) box[k] = 0.0;
  __syncthreads();
  const bool own = (int)blockIdx.x < tk.ntiles;
  if (own && end - p0 > tk.crowd) return;
  for (uint32_t p = p0 + threadIdx.x / TEAM; p < (uint32_t)end; p += kTileThreads / TEAM) {
    const int64_t i = tk.order[p];
    double w[3][N], dw[N];
    int b[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = a.x[3 * i + d] * a.scale[d];
      const double fl = floor(u);
      b[d] = (int)fl & ((d == 0 ? TX : (d == 1 ? TY : TZ)) - 1);  // place in the tile
      spline_weights<N, false>(u - fl, w[d], dw);
    }
    const double qi = a.q[i];
#pragma unroll
    for (int z = 0; z < N; z += TEAM) {
      double wz = w[2][z];
#pragma unroll
      for (int s = 1; s < TEAM; ++s) wz = t == s ? w[2][z + s] : wz;
      wz *= qi;
#pragma unroll
      for (int jy = 0; jy < N; ++jy) {
        const double wyz = wz * w[1][jy];
        double *row =
            box + ((b[2] + N - 1 - (z + t)) * EY + (b[1] + N - 1 - jy)) * EX + b[0] + N - 1;
#pragma unroll
        for (int jx = 0; jx < N; ++jx) unsafeAtomicAdd(row - jx, wyz * w[0][jx]);
      }
    }
  }
  __syncthreads();
  double *out = tk.boxes + (int64_t)tile * (EX * EY * EZ);
  if (own) {
    for (int k = threadIdx.x; k < EX * EY * EZ; k += kTileThreads) out[k] = box[k];
  } else {
    for (int k = threadIdx.x; k < EX * EY * EZ; k += kTileThreads)
      if (box[k] != 0.0) unsafeAtomicAdd(&out[k], box[k]);
  }
}

// The forces of a tile's particles from the box of phi (k_gather's sums).
template <int N, int TX, int TY, int TZ, int TEAM>
__global__ __launch_bounds__(kTileThreads) void k_gather_tile(RecArgs a, TileK tk) {
  constexpr int EX = TX + N - 1, EY = TY + N - 1, EZ = TZ + N - 1;
  __shared__ double box[EX * EY * EZ];
  int tile, p0, end;
  if (!tile_work(tk, a.n, blockIdx.x, tile, p0, end) || p0 == end ||
      ((int)blockIdx.x < tk.ntiles && end - p0 > tk.crowd))
    return;  // block-uniform
  const int t = (int)threadIdx.x % TEAM;
  int o[3];
  tile_origin(tk, tile, o);
  for (int k = threadIdx.x; k < EX * EY * EZ; k += kTileThreads) {
    const int r = k / EX, lx = k - r * EX, lz = r / EY, ly = r - lz * EY;
    const int x = wrapi(o[0] + lx - (N - 1), a.K[0]), y = wrapi(o[1] + ly - (N - 1), a.K[1]),
              z = wrapi(o[2] + lz - (N - 1), a.K[2]);
    box[k] = a.grid[((int64_t)z * a.K[1] + y) * a.K[0] + x];
  }
  __syncthreads();
  for (uint32_t p = p0 + threadIdx.x / TEAM; p < (uint32_t)end; p += kTileThreads / TEAM) {
    const int64_t i = tk.order[p];
    double w[3][N], dw[3][N];
    int b[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = a.x[3 * i + d] * a.scale[d];
      const double fl = floor(u);
      b[d] = (int)fl & ((d == 0 ? TX : (d == 1 ? TY : TZ)) - 1);
      spline_weights<N, true>(u - fl, w[d], dw[d]);
    }
    const double qi = a.q[i];
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
#pragma unroll
    for (int z = 0; z < N; z += TEAM) {
      double wz = w[2][z], dz = dw[2][z];
#pragma unroll
      for (int s = 1; s < TEAM; ++s) {
        wz = t == s ? w[2][z + s] : wz;
        dz = t == s ? dw[2][z + s] : dz;
      }
#pragma unroll
      for (int jy = 0; jy < N; ++jy) {
        const double *row =
            box + ((b[2] + N - 1 - (z + t)) * EY + (b[1] + N - 1 - jy)) * EX + b[0] + N - 1;
        double sx = 0.0, sdx = 0.0;
#pragma unroll
        for (int jx = 0; jx < N; ++jx) {
          const double ph = row[-jx];
          sx = __builtin_fma(w[0][jx], ph, sx);
          sdx = __builtin_fma(dw[0][jx], ph, sdx);
        }
        g0 = __builtin_fma(sdx * w[1][jy], wz, g0);
        g1 = __builtin_fma(sx * dw[1][jy], wz, g1);
        g2 = __builtin_fma(sx * w[1][jy], dz, g2);
      }
    }
    g0 = team_sum<TEAM>(g0);
    g1 = team_sum<TEAM>(g1);
    g2 = team_sum<TEAM>(g2);
    if (t == 0) {
      double *F = a.F + 3 * i;
      const double f0 = -qi * g0 * a.scale[0], f1 = -qi * g1 * a.scale[1],
                   f2 = -qi * g2 * a.scale[2];
      if (a.accumulate) {
        F[0] += f0;
        F[1] += f1;
        F[2] += f2;
      } else {
        F[0] = f0;
        F[1] = f1;
        F[2] = f2;
      }
    }
  }
}

// Points (x, x + 1), x even, of row (y, z) of the charge grid from the boxes that
// cover them: per dimension the point's own tile, and the next one when the point is
// among the last N - 1 of its tile.
template <int COUNT, int STRIDE>
__device__ __forceinline__ void row_from_boxes(const TileK &t, int y, int z, int n2,
                                               double2 (&v)[COUNT]) {
  const int ty = 1 << t.lg[1], tz = 1 << t.lg[2], tx = 1 << t.lg[0];
  const int h = t.e[0] - tx;  // N - 1
  const int ry = y & (ty - 1), rz = z & (tz - 1);
  const int my = ry >= ty - h ? 2 : 1, mz = rz >= tz - h ? 2 : 1;
#pragma unroll
  for (int k = 0; k < COUNT; ++k) v[k] = make_double2(0.0, 0.0);
  for (int iz = 0; iz < mz; ++iz) {
    const int qz = ((z >> t.lg[2]) + iz) & (t.nt[2] - 1), lz = rz + h - iz * tz;
    for (int iy = 0; iy < my; ++iy) {
      const int qy = ((y >> t.lg[1]) + iy) & (t.nt[1] - 1), ly = ry + h - iy * ty;
      const double *rows = t.boxes + (int64_t)(qz * t.nt[1] + qy) * t.nt[0] * t.box +
                           (lz * t.e[1] + ly) * t.e[0];
      // every load before the first sum, so that all are in flight together
      double own[COUNT][2], next[COUNT][2];
#pragma unroll
      for (int k = 0; k < COUNT; ++k) {
        const int x = 2 * (n2 + STRIDE * k);
        const double *p = rows + (x >> t.lg[0]) * t.box + (x & (tx - 1)) + h;
        own[k][0] = p[0];
        own[k][1] = p[1];
      }
#pragma unroll
      for (int k = 0; k < COUNT; ++k) {
        const int x = 2 * (n2 + STRIDE * k), rx = x & (tx - 1), qx = (x >> t.lg[0]) + 1;
        next[k][0] = next[k][1] = 0.0;
        if (rx + 1 >= tx - h) {  // x + 1, and x too except at the first such pair
          const double *p = rows + (qx & (t.nt[0] - 1)) * t.box + rx + h - tx;
          next[k][0] = p[rx >= tx - h ? 0 : 1];
          next[k][1] = p[1];
        }
      }
#pragma unroll
      for (int k = 0; k < COUNT; ++k) {
        const int rx = (2 * (n2 + STRIDE * k)) & (tx - 1);
        v[k].x += own[k][0] + (rx >= tx - h ? next[k][0] : 0.0);
        v[k].y += own[k][1] + next[k][1];
      }
    }
  }
}

// Charge spreading without tiles (order 8, the smaller workspace), one wavefront of 64
// consecutive particles per block.  The wavefront first adds its n^3 weights per
// particle into a private box of grid points in LDS (LDS atomics), then adds every
// non-zero point of that box to the grid with one global FP64 atomic: ~4x fewer
// global atomics than adding each weight directly, which is what bounds this kernel.
// Per axis the box is taken in whichever of two cyclic frames (indices as they are, or
// shifted by K/2) gives the smaller extent, so groups that straddle a periodic face
// stay compact.  A group whose box exceeds the LDS capacity adds its weights straight
// to the grid.
constexpr int kSpreadCap = 2048;  // grid points (doubles) in the LDS box

__device__ __forceinline__ int wave_min_i(int v) { return -wave_max(-v); }

template <int N>
__global__ __launch_bounds__(kWave) void k_spread(RecArgs a) {
  __shared__ double box[kSpreadCap];
  const int lane = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * kWave + lane;
  const bool live = i < a.n;
  double w[3][N], dw[N];
  int b[3] = {0, 0, 0};
  double qi = 0.0;
  if (live) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = a.x[3 * i + d] * a.scale[d];
      const double fl = floor(u);
      b[d] = wrapi((int)fl, a.K[d]);
      spline_weights<N, false>(u - fl, w[d], dw);
    }
    qi = a.q[i];
  }
  int lo[3], ext[3], sh[3], sb[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int K = a.K[d];
    const int s0 = b[d], s1 = wrapi(b[d] + K / 2, K);
    const int mn0 = wave_min_i(live ? s0 : 1 << 30), mx0 = wave_max(live ? s0 : -(1 << 30));
    const int mn1 = wave_min_i(live ? s1 : 1 << 30), mx1 = wave_max(live ? s1 : -(1 << 30));
    const bool shift = mx1 - mn1 < mx0 - mn0;
    sh[d] = shift ? K / 2 : 0;
    lo[d] = shift ? mn1 : mn0;
    ext[d] = (shift ? mx1 - mn1 : mx0 - mn0) + N;
    sb[d] = shift ? s1 : s0;
  }
  const int64_t vol = (int64_t)ext[0] * ext[1] * ext[2];
  if (vol > kSpreadCap) {  // wavefront-uniform
    if (!live) return;
    for (int jz = 0; jz < N; ++jz) {
      const int kz = wrapi(b[2] - jz, a.K[2]);
      for (int jy = 0; jy < N; ++jy) {
        const int ky = wrapi(b[1] - jy, a.K[1]);
        const double wyz = qi * w[2][jz] * w[1][jy];
        double *line = a.grid + ((int64_t)kz * a.K[1] + ky) * a.K[0];
#pragma unroll
        for (int jx = 0; jx < N; ++jx)
          unsafeAtomicAdd(&line[wrapi(b[0] - jx, a.K[0])], wyz * w[0][jx]);
      }
    }
    return;
  }
  for (int p = lane; p < vol; p += kWave) box[p] = 0.0;
  __syncthreads();
  if (live) {
    const int c0 = sb[0] - lo[0] + N - 1, c1 = sb[1] - lo[1] + N - 1, c2 = sb[2] - lo[2] + N - 1;
    for (int jz = 0; jz < N; ++jz) {
      for (int jy = 0; jy < N; ++jy) {
        const double wyz = qi * w[2][jz] * w[1][jy];
        double *row = box + ((int64_t)(c2 - jz) * ext[1] + (c1 - jy)) * ext[0] + c0;
#pragma unroll
        for (int jx = 0; jx < N; ++jx) unsafeAtomicAdd(row - jx, wyz * w[0][jx]);
      }
    }
  }
  __syncthreads();
  for (int p = lane; p < vol; p += kWave) {
    const double v = box[p];
    if (v == 0.0) continue;
    const int l0 = p % ext[0], l1 = (p / ext[0]) % ext[1], l2 = p / (ext[0] * ext[1]);
    const int k0 = wrapi(lo[0] + l0 - (N - 1) - sh[0], a.K[0]);
    const int k1 = wrapi(lo[1] + l1 - (N - 1) - sh[1], a.K[1]);
    const int k2 = wrapi(lo[2] + l2 - (N - 1) - sh[2], a.K[2]);
    unsafeAtomicAdd(&a.grid[((int64_t)k2 * a.K[1] + k1) * a.K[0] + k0], v);
  }
}

// ------------------------------------------------------------------ FFTs --
//
// A row of NP = R1 R2 points is transformed in two register steps with one
// exchange through LDS.  With input index n = n2 + R2 n1 and output index
// k = k1 + R1 k2,
//   X[k1 + R1 k2] = sum_n2 W_NP^(n2 k1) W_R2^(n2 k2) sum_n1 v[n2 + R2 n1] W_R1^(n1 k1):
// a thread transforms the R1 points of one n2 in registers, multiplies by the
// twiddles and leaves them in LDS; then it takes the R2 points of R1 / R2 values of
// k1.  The inverse runs the same two sums in the other order, so a pass that
// transforms forward and back needs no reordering in between.  M rows per block, one
// wavefront (two for NP = 256); rows are the fast index of the block's LDS, padded
// by one point per k1 against bank conflicts.
//
// These passes are bound by the latency of their one round trip over the grid
// (17 + 17 MB at 128^3): every thread has R1 16-byte loads in flight before it
// computes.  With radix-2 stages over LDS (a barrier and an LDS round trip each) and
// 64-bit divisions for every element's place -> now (us): 128^3 x 12.1 -> 9.4, y
// 19.6 -> 7.8, z 27.0 -> 15.7, inverse y 19.6 -> 10.0 (with the energy sum), inverse x
// 13.5 -> 10.9; 64^3 5.6 -> 4.9, 7.2 -> 4.8, 9.9 -> 5.6, 7.2 -> 4.3, 6.2 -> 5.6.

// e^(2 pi i j / 16), j = 0..3 (cos, sin)
constexpr double kC16[4] = {1.0, 0.92387953251128674, 0.70710678118654752, 0.38268343236508977};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }

// In-register transform of R points (R = 1, 2, 4, 8, 16), sign S (-1 forward, +1
// unnormalised inverse), natural order in and out; all twiddles are constants.
template <int R, int S>
__device__ __forceinline__ void fft_reg(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = make_double2(a.x + b.x, a.y + b.y);
    v[1] = make_double2(a.x - b.x, a.y - b.y);
  } else if constexpr (R > 2) {
    double2 e[R / 2], o[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      e[k] = v[2 * k];
      o[k] = v[2 * k + 1];
    }
    fft_reg<R / 2, S>(e);
    fft_reg<R / 2, S>(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      const int j = k * (16 / R);  // e^(S 2 pi i j / 16), j < 8
      double2 t;
      if (j == 0) {
        t = o[k];
      } else if (j == 4) {
        t = make_double2(-S * o[k].y, S * o[k].x);
      } else {
        const double c = j < 4 ? kC16[j] : -kC16[8 - j];
        const double s = j < 4 ? kC16[4 - j] : kC16[j - 4];
        t = cmul(o[k], make_double2(c, S * s));
      }
      v[k] = make_double2(e[k].x + t.x, e[k].y + t.y);
      v[k + R / 2] = make_double2(e[k].x - t.x, e[k].y - t.y);
    }
  }
}

template <int NP>
struct Fft {
  static constexpr int R1 = NP <= 8 ? NP : NP == 16 ? 4 : NP <= 64 ? 8 : 16;
  static constexpr int R2 = NP / R1;
  static constexpr int T = NP > 128 ? 128 : 64;  // threads
  static constexpr int M = T / R2;               // rows
  static constexpr int J = R1 / R2;              // values of k1 per thread in the second step
  static constexpr int kPitch = R2 * M + 1;      // LDS points per k1
  static constexpr int kLds = R2 > 1 ? R1 * kPitch : 1;

  // v[n1] = element n2 + R2 n1 of row m  ->  out[q R2 + k2] = element k1 + R1 k2
  // of row mo, k1 = kk + R2 q.  tw[TS j] = e^(-2 pi i j / NP); every thread of the
  // block calls it, buf may be written again after the caller's next barrier.
  template <int S, int TS>
  static __device__ __forceinline__ void forward(double2 (&v)[R1], double2 (&out)[R1], double2 *buf,
                                                 const double2 *tw, int m, int n2, int mo,
                                                 int kk) {
    fft_reg<R1, S>(v);
    if constexpr (R2 == 1) {
#pragma unroll
      for (int k = 0; k < R1; ++k) out[k] = v[k];  // J = R1: k1 = q, one point each
    } else {
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) {
        const double2 w = tw[TS * n2 * k1];
        buf[k1 * kPitch + n2 * M + m] = cmul(v[k1], S < 0 ? w : conj2(w));
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < J; ++q) {
        double2 u[R2];
#pragma unroll
        for (int j = 0; j < R2; ++j) u[j] = buf[(kk + R2 * q) * kPitch + j * M + mo];
        fft_reg<R2, S>(u);
#pragma unroll
        for (int j = 0; j < R2; ++j) out[q * R2 + j] = u[j];
      }
    }
  }

  // The inverse of forward's layout: in[q R2 + k2] of row m (k1 = kk + R2 q) ->
  // v[n1] = element n2 + R2 n1 of the same row, n2 = kk.
  template <int S, int TS>
  static __device__ __forceinline__ void backward(double2 (&in)[R1], double2 (&v)[R1],
                                                  double2 *buf, const double2 *tw, int m, int kk) {
    if constexpr (R2 == 1) {
#pragma unroll
      for (int k = 0; k < R1; ++k) v[k] = in[k];
    } else {
      __syncthreads();  // forward's reads of buf
#pragma unroll
      for (int q = 0; q < J; ++q) {
        double2 u[R2];
        const int k1 = kk + R2 * q;
#pragma unroll
        for (int j = 0; j < R2; ++j) u[j] = in[q * R2 + j];
        fft_reg<R2, S>(u);
#pragma unroll
        for (int j = 0; j < R2; ++j) {
          const double2 w = tw[TS * j * k1];
          buf[k1 * kPitch + j * M + m] = cmul(u[j], S < 0 ? w : conj2(w));
        }
      }
      __syncthreads();
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) v[k1] = buf[k1 * kPitch + kk * M + m];
    }
    fft_reg<R1, S>(v);
  }
};

// tw[j] = e^(-2 pi i j / NP), j < NP
template <int NP, int T>
__device__ __forceinline__ void fill_twiddles(double2 *tw) {
  for (int j = threadIdx.x; j < NP; j += T) {
    double s, c;
    sincospi(2.0 * (double)j / (double)NP, &s, &c);
    tw[j] = make_double2(c, -s);
  }
}

// Points per stored row of the half grid: K0/2 + 1 coefficients, rounded up to whole
// 128-byte lines where the region (K0/2 + K0/8 points per row) has room for it.
__host__ __device__ __forceinline__ int half_pitch(int K0) {
  return K0 >= 64 ? (K0 / 2 + 8) / 8 * 8 : K0 / 2 + 1;
}

// Point k of a column: `off` (the lane's 32-bit byte offset; the half grid has at most
// 142 MB) from a wavefront-uniform base, so the 16 addresses of a thread share one
// vector register.
__device__ __forceinline__ double2 *column_at(double2 *g, int64_t uniform, uint32_t off) {
  return (double2 *)((char *)(g + uniform) + off);
}

// y pass over the half grid: block (bx, z) transforms the columns x0 = bx M .. of
// plane z, in place.  Inverse (S = 1): the first block also sums the z pass's energy
// partials part[0..nparts) into *sum, in a fixed order.
template <int NP, int S>
__global__ __launch_bounds__(Fft<NP>::T) void k_fft_y(double2 *g, int W, int P, const double *part,
                                                      int nparts, double *sum) {
  using F = Fft<NP>;
  __shared__ double2 buf[F::kLds];
  __shared__ double2 tw[NP];
  const int t = threadIdx.x, m = t % F::M, n2 = t / F::M;
  if constexpr (S > 0) {
    if (blockIdx.x == 0 && blockIdx.y == 0) {  // block-uniform
      __shared__ double red[kRedRows * F::T / kWave];
      double e[1] = {0.0};
#pragma unroll 8
      for (int k = t; k < nparts; k += F::T) e[0] += part[k];
      block_sum<F::T / kWave, 1>(e, red, sum);
    }
  }
  const int x = blockIdx.x * F::M + m;
  double2 *plane = g + (int64_t)blockIdx.y * NP * P;
  const uint32_t off = (uint32_t)(n2 * P + (x < W ? x : W - 1)) * (uint32_t)sizeof(double2);
  double2 v[F::R1], out[F::R1];
#pragma unroll
  for (int k = 0; k < F::R1; ++k) v[k] = *column_at(plane, (int64_t)(F::R2 * k) * P, off);
  fill_twiddles<NP, F::T>(tw);
  __syncthreads();
  F::template forward<S, 1>(v, out, buf, tw, m, n2, m, n2);
  if (x < W) {
#pragma unroll
    for (int q = 0; q < F::J; ++q)
#pragma unroll
      for (int j = 0; j < F::R2; ++j)
        *column_at(plane, (int64_t)(F::R2 * q + F::R1 * j) * P, off) = out[q * F::R2 + j];
  }
}

// x pass, real to complex: row r of NP reals -> NP/2 + 1 coefficients X_m =
// sum_k v_k e^{-2 pi i m k / NP}.  With z_k = v_2k + i v_2k+1 and Z its
// transform of length NH = NP/2: X_m = E_m + e^{-2 pi i m/NP} O_m, where
// E_m = (Z_m + conj Z_{NH-m}) / 2 and O_m = (Z_m - conj Z_{NH-m}) / (2i) are the
// transforms of the even and odd samples (indices of Z mod NH).  rows is a multiple
// of the M rows of a block (K1 K2 >= 64).  BOXES: the rows are read from the tiles'
// boxes instead of the grid (lgK1 = log2 K1).
template <int NP, bool BOXES>
__global__ __launch_bounds__(Fft<NP / 2>::T) void k_fft_x_r2c(const double *rg, TileK tk, int lgK1,
                                                             double2 *h) {
  constexpr int NH = NP / 2;
  using F = Fft<NH>;
  constexpr int P = NP >= 64 ? (NP / 2 + 8) / 8 * 8 : NP / 2 + 1;
  constexpr int kRow = NH + 1;  // pitch of Z rows in LDS
  __shared__ double2 buf[F::kLds > F::M * kRow ? F::kLds : F::M * kRow];
  __shared__ double2 tw[NP];
  double2 *z = buf;  // Z rows, once the transform has read the exchanged points
  const int t = threadIdx.x, n2 = t % F::R2, m = t / F::R2;
  const int64_t r0 = (int64_t)blockIdx.x * F::M;
  double2 v[F::R1], out[F::R1];
  if constexpr (BOXES) {
    const int r = (int)r0 + m;
    row_from_boxes<F::R1, F::R2>(tk, r & ((1 << lgK1) - 1), r >> lgK1, n2, v);
  } else {
    const double2 *row = (const double2 *)(rg + (r0 + m) * NP);
#pragma unroll
    for (int k = 0; k < F::R1; ++k) v[k] = row[n2 + F::R2 * k];
  }
  fill_twiddles<NP, F::T>(tw);
  __syncthreads();
  F::template forward<-1, 2>(v, out, buf, tw, m, n2, m, n2);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < F::J; ++q)
#pragma unroll
    for (int j = 0; j < F::R2; ++j) z[m * kRow + n2 + F::R2 * q + F::R1 * j] = out[q * F::R2 + j];
  __syncthreads();
  for (int idx = t; idx < F::M * kRow; idx += F::T) {
    const int mr = idx / kRow, k = idx % kRow;
    const double2 zm = z[mr * kRow + (k & (NH - 1))], zc = z[mr * kRow + ((NH - k) & (NH - 1))];
    const double er = 0.5 * (zm.x + zc.x), ei = 0.5 * (zm.y - zc.y);
    const double orr = 0.5 * (zm.y + zc.y), oi = -0.5 * (zm.x - zc.x);
    const double c = tw[k].x, s = tw[k].y;
    h[(r0 + mr) * P + k] = make_double2(er + (c * orr - s * oi), ei + (c * oi + s * orr));
  }
}

// x pass, complex to real: the NP/2 + 1 coefficients X_m of a Hermitian row
// -> v_k = sum_{m<NP} X_m e^{+2 pi i m k / NP}.  With A_m = X_m + conj X_{NH-m},
// B_m = (X_m - conj X_{NH-m}) e^{+2 pi i m/NP} for m < NH, the inverse transform
// of length NH of A + iB is z_k = v_2k + i v_2k+1.
template <int NP>
__global__ __launch_bounds__(Fft<NP / 2>::T) void k_fft_x_c2r(const double2 *h, double *rg) {
  constexpr int NH = NP / 2;
  using F = Fft<NH>;
  constexpr int P = NP >= 64 ? (NP / 2 + 8) / 8 * 8 : NP / 2 + 1;
  __shared__ double2 buf[F::kLds > F::M * (NH + 1) ? F::kLds : F::M * (NH + 1)];
  __shared__ double2 tw[NP];
  double2 *xin = buf;  // X rows, until they are in registers
  const int t = threadIdx.x, n2 = t % F::R2, m = t / F::R2;
  const int64_t r0 = (int64_t)blockIdx.x * F::M;
  for (int idx = t; idx < F::M * (NH + 1); idx += F::T) {
    const int mr = idx / (NH + 1), k = idx % (NH + 1);
    xin[idx] = h[(r0 + mr) * P + k];
  }
  fill_twiddles<NP, F::T>(tw);
  __syncthreads();
  double2 v[F::R1], out[F::R1];
#pragma unroll
  for (int q = 0; q < F::R1; ++q) {
    const int k = n2 + F::R2 * q;
    const double2 x1 = xin[m * (NH + 1) + k], x2 = xin[m * (NH + 1) + NH - k];
    const double ar = x1.x + x2.x, ai = x1.y - x2.y;  // X_m + conj X_{NH-m}
    const double dr = x1.x - x2.x, di = x1.y + x2.y;  // X_m - conj X_{NH-m}
    const double c = tw[k].x, s = -tw[k].y;
    const double br = c * dr - s * di, bi = c * di + s * dr;
    v[q] = make_double2(ar - bi, ai + br);
  }
  __syncthreads();
  F::template forward<1, 2>(v, out, buf, tw, m, n2, m, n2);
  double2 *row = (double2 *)(rg + (r0 + m) * NP);
#pragma unroll
  for (int q = 0; q < F::J; ++q)
#pragma unroll
    for (int j = 0; j < F::R2; ++j) row[n2 + F::R2 * q + F::R1 * j] = out[q * F::R2 + j];
}

// z pass with the influence function between its two transforms: block (bx, y)
// takes the columns x0 = bx M .. of row y (element m2 at m2 P K1 points), transforms
// them forward, multiplies by G(m) = B(m) C(m) and transforms back, so the half grid
// makes one round trip instead of three.  Per block the reciprocal energy
// 1/2 sum G |F(Q)|^2 (fixed order) goes to the real grid's region, which is free
// between the x passes; the inverse y pass sums it.
template <int NP>
__global__ __launch_bounds__(Fft<NP>::T, 2) void k_fft_z_influence(RecArgs a) {
  using F = Fft<NP>;
  __shared__ double2 buf[F::kLds];
  __shared__ double2 tw[NP];
  __shared__ double red[kRedRows * F::T / kWave];
  const int t = threadIdx.x, m = t % F::M, n2 = t / F::M;
  const int W = a.K[0] / 2 + 1, P = half_pitch(a.K[0]);
  const int m0 = blockIdx.x * F::M + m, m1 = blockIdx.y;
  const int64_t plane = (int64_t)P * a.K[1];
  double2 *row = a.half + (int64_t)m1 * P;
  const uint32_t off =
      (uint32_t)(n2 * (int)plane + (m0 < W ? m0 : W - 1)) * (uint32_t)sizeof(double2);
  double2 v[F::R1], out[F::R1];
#pragma unroll
  for (int k = 0; k < F::R1; ++k) v[k] = *column_at(row, F::R2 * k * plane, off);
  fill_twiddles<NP, F::T>(tw);
  __syncthreads();
  F::template forward<-1, 1>(v, out, buf, tw, m, n2, m, n2);
  const double piV = kPi * (a.b.L[0] * a.b.L[1] * a.b.L[2]);
  const double f0 = m0 * a.b.invL[0];
  const double f1 = (m1 <= a.K[1] / 2 ? m1 : m1 - a.K[1]) * a.b.invL[1];
  const double b01 = m0 < W ? a.bmod[m0] * a.bmod[kMaxGrid + m1] : 0.0;
  const double mult = (m0 == 0 || 2 * m0 == a.K[0]) ? 0.5 : 1.0;
  double e[1] = {0.0};
#pragma unroll
  for (int q = 0; q < F::J; ++q)
#pragma unroll
    for (int j = 0; j < F::R2; ++j) {
      const int m2 = n2 + F::R2 * q + F::R1 * j;
      const double f2 = (m2 <= NP / 2 ? m2 : m2 - NP) * a.b.invL[2];
      const double msq = (f0 * f0 + f1 * f1) + f2 * f2;
      double G = 0.0;
      if (m0 < W && (m0 | m1 | m2) != 0) {
        G = b01 * a.bmod[2 * kMaxGrid + m2] * recip64(piV * msq);
      }
      double2 &z = out[q * F::R2 + j];
      // 1/2 G |F|^2, doubled for the columns 0 < m0 < K0/2 whose mirror -m0 is not stored
      e[0] += mult * G * (z.x * z.x + z.y * z.y);
      z = make_double2(G * z.x, G * z.y);
    }
  F::template backward<1, 1>(out, v, buf, tw, m, n2);
  if (m0 < W) {
#pragma unroll
    for (int k = 0; k < F::R1; ++k) *column_at(row, F::R2 * k * plane, off) = v[k];
  }
  block_sum<F::T / kWave, 1>(e, red, a.grid + (int64_t)blockIdx.y * gridDim.x + blockIdx.x);
}

// F_i = -q_i grad sum_k theta_i(k) phi(k); per block the self energy -alpha/sqrt(pi) q_i^2.
//
// TEAM lanes per particle, lane t the planes jz = t, t + TEAM, ... of its support;
// blocks renumbered per XCD (the particles' order is spatial).  A row of the support
// is N consecutive points read with 16-byte loads unless some lane's row wraps
// around the box.  Bound by those loads (16 rows of 32 bytes per particle at order 4).
// Integer divisions for every point's place and 8-byte loads, one lane per particle,
// took 42 us at 500,000 particles and 128^3; now 35.
template <int N, int TEAM>
__global__ __launch_bounds__(kGatherAtoms * TEAM) void k_gather(RecArgs a, double *self_partial) {
  __shared__ double red[kRedRows * kGatherAtoms * TEAM / kWave];
  const int t = (int)threadIdx.x % TEAM;
  const int64_t i =
      (int64_t)xcd_block(blockIdx.x, gridDim.x) * kGatherAtoms + (int)threadIdx.x / TEAM;
  const bool live = i < a.n;
  const int64_t ii = live ? i : 0;  // the last block's spare lanes repeat particle 0
  double w[3][N], dw[3][N];
  int base[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double u = a.x[3 * ii + d] * a.scale[d];
    const double fl = floor(u);
    base[d] = wrapi((int)fl, a.K[d]);
    spline_weights<N, true>(u - fl, w[d], dw[d]);
  }
  const double qi = a.q[ii];
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  const bool wraps = base[0] < N - 1;
  auto planes = [&](auto whole) {
#pragma unroll
    for (int z = 0; z < N; z += TEAM) {
      double wz = w[2][z], dz = dw[2][z];
#pragma unroll
      for (int s = 1; s < TEAM; ++s) {  // this lane's plane jz = z + t
        wz = t == s ? w[2][z + s] : wz;
        dz = t == s ? dw[2][z + s] : dz;
      }
      const double *plane =
          a.grid + (int64_t)wrapi(base[2] - (z + t), a.K[2]) * a.K[1] * a.K[0];
#pragma unroll
      for (int jy = 0; jy < N; ++jy) {
        const double *line = plane + (int64_t)wrapi(base[1] - jy, a.K[1]) * a.K[0];
        double ph[N];
        if constexpr (decltype(whole)::value) {
          const double *p = line + (base[0] - (N - 1));
#pragma unroll
          for (int jx = 0; jx < N; ++jx) ph[jx] = p[N - 1 - jx];
        } else {
#pragma unroll
          for (int jx = 0; jx < N; ++jx) ph[jx] = line[wrapi(base[0] - jx, a.K[0])];
        }
        double sx = 0.0, sdx = 0.0;
#pragma unroll
        for (int jx = 0; jx < N; ++jx) {
          sx = __builtin_fma(w[0][jx], ph[jx], sx);
          sdx = __builtin_fma(dw[0][jx], ph[jx], sdx);
        }
        g0 = __builtin_fma(sdx * w[1][jy], wz, g0);
        g1 = __builtin_fma(sx * dw[1][jy], wz, g1);
        g2 = __builtin_fma(sx * w[1][jy], dz, g2);
      }
    }
  };
  if (__ballot(wraps) == 0)
    planes(std::true_type{});
  else
    planes(std::false_type{});
  g0 = team_sum<TEAM>(g0);
  g1 = team_sum<TEAM>(g1);
  g2 = team_sum<TEAM>(g2);
  double v[1] = {0.0};
  if (live && t == 0) {
    double *F = a.F + 3 * i;
    const double f0 = -qi * g0 * a.scale[0], f1 = -qi * g1 * a.scale[1],
                 f2 = -qi * g2 * a.scale[2];
    if (a.accumulate) {
      F[0] += f0;
      F[1] += f1;
      F[2] += f2;
    } else {
      F[0] = f0;
      F[1] = f1;
      F[2] = f2;
    }
    v[0] = -a.alpha / __builtin_sqrt(kPi) * qi * qi;
  }
  if (self_partial) block_sum<kGatherAtoms * TEAM / kWave, 1>(v, red, self_partial + blockIdx.x);
}

// nparts: energy partials of the z pass (inverse pass only).
template <int NP>
void y_pass(const RecArgs &a, bool forward, int nparts, hipStream_t st) {
  using F = Fft<NP>;
  const int W = a.K[0] / 2 + 1, P = half_pitch(a.K[0]);
  const dim3 nb((W + F::M - 1) / F::M, a.K[2]);
  if (forward)
    k_fft_y<NP, -1><<<nb, F::T, 0, st>>>(a.half, W, P, nullptr, 0, nullptr);
  else
    k_fft_y<NP, 1><<<nb, F::T, 0, st>>>(a.half, W, P, a.grid, nparts, a.partial);
}

void fft_y(const RecArgs &a, bool forward, int nparts, hipStream_t st) {
  switch (a.K[1]) {
    case 8: y_pass<8>(a, forward, nparts, st); break;
    case 16: y_pass<16>(a, forward, nparts, st); break;
    case 32: y_pass<32>(a, forward, nparts, st); break;
    case 64: y_pass<64>(a, forward, nparts, st); break;
    case 128: y_pass<128>(a, forward, nparts, st); break;
    default: y_pass<256>(a, forward, nparts, st); break;
  }
}

// Returns the number of energy partials (one per block, fewer than the grid's points).
template <int NP>
int z_influence_pass(const RecArgs &a, hipStream_t st) {
  using F = Fft<NP>;
  const dim3 nb((a.K[0] / 2 + 1 + F::M - 1) / F::M, a.K[1]);
  k_fft_z_influence<NP><<<nb, F::T, 0, st>>>(a);
  return (int)(nb.x * nb.y);
}

int fft_z_influence(const RecArgs &a, hipStream_t st) {
  switch (a.K[2]) {
    case 8: return z_influence_pass<8>(a, st);
    case 16: return z_influence_pass<16>(a, st);
    case 32: return z_influence_pass<32>(a, st);
    case 64: return z_influence_pass<64>(a, st);
    case 128: return z_influence_pass<128>(a, st);
    default: return z_influence_pass<256>(a, st);
  }
}

int log2_of(int k) { return __builtin_ctz((unsigned)k); }

// tk: read the charge rows from the tiles' boxes (forward pass), or null.
template <int NP>
void x_pass(const RecArgs &a, bool forward, const TileK *tk, hipStream_t st) {
  using F = Fft<NP / 2>;
  // K1 K2 >= 64, M a power of two <= 64
  const unsigned nb = (unsigned)((int64_t)a.K[1] * a.K[2] / F::M);
  if (!forward)
    k_fft_x_c2r<NP><<<nb, F::T, 0, st>>>(a.half, a.grid);
  else if (tk)
    k_fft_x_r2c<NP, true><<<nb, F::T, 0, st>>>(a.grid, *tk, log2_of(a.K[1]), a.half);
  else
    k_fft_x_r2c<NP, false><<<nb, F::T, 0, st>>>(a.grid, TileK{}, 0, a.half);
}

void fft_x(const RecArgs &a, bool forward, const TileK *tk, hipStream_t st) {
  switch (a.K[0]) {
    case 8: x_pass<8>(a, forward, tk, st); break;
    case 16: x_pass<16>(a, forward, tk, st); break;
    case 32: x_pass<32>(a, forward, tk, st); break;
    case 64: x_pass<64>(a, forward, tk, st); break;
    case 128: x_pass<128>(a, forward, tk, st); break;
    default: x_pass<256>(a, forward, tk, st); break;
  }
}

int64_t grid_points(const int32_t K[3]) { return (int64_t)K[0] * K[1] * K[2]; }
unsigned blocks_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per > 0 ? (n + per - 1) / per : 1); }

// Large tiles (16 x 16 x 8) where the grid has at least 512 of them -- two per compute
// unit --, else 8 x 8 x 8; their boxes hold 1.94 and 2.60 points per grid point at
// order 4.  Order 6 takes the large ones only (2.80; small ones 4.29), order 8 none
// (3.87, 6.59): there, and in the smaller of the two workspaces that the call accepts,
// charge is spread by wavefront boxes and atomics.
constexpr double kBoxPoints = 2.8;  // largest box points per grid point of a shape taken

bool large_tiles(const int32_t K[3]) {
  return K[0] >= 16 && K[1] >= 16 && (int64_t)K[0] * K[1] * K[2] >= 512 * 2048;
}
bool tiled(int order, const int32_t K[3]) { return order == 4 || (order == 6 && large_tiles(K)); }

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Bytes of the tiles' part of the workspace, at most.
size_t tile_workspace(int64_t n, int64_t npts) {
  const size_t ints = align256((size_t)(npts / 512 + 2) * sizeof(int32_t));
  const size_t per = align256((size_t)(n > 0 ? n : 0) * sizeof(int32_t));
  return 256 + 2 * ints + 3 * per + (size_t)(kBoxPoints * (double)npts) * sizeof(double);
}

TileK make_tiles(int order, const int32_t K[3], int64_t n, char *p) {
  TileK t{};
  const bool large = large_tiles(K);
  t.ntiles = t.box = 1;
  for (int d = 0; d < 3; ++d) {
    t.lg[d] = large && d < 2 ? 4 : 3;
    t.nt[d] = K[d] >> t.lg[d];
    t.e[d] = (1 << t.lg[d]) + order - 1;
    t.ntiles *= t.nt[d];
    t.box *= t.e[d];
  }
  // Up to 512 chunks.  Where the tiles fill the chip a tile is crowded only above twice the
  // mean, since a uniform system of any density is then balanced as it is.
  const int64_t part = (n / 512 + kTileChunk - 1) / kTileChunk * kTileChunk;
  t.chunk = (int32_t)(part > kTileChunk ? part : kTileChunk);
  const int64_t twice = t.ntiles >= 512 ? 2 * n / t.ntiles : 0;
  t.crowd = (int32_t)(twice > kTileCrowd ? twice : kTileCrowd);
  if (t.crowd < t.chunk) t.crowd = t.chunk;
  p = (char *)align256((size_t)p);
  const size_t ints = align256((size_t)(t.ntiles + 2) * sizeof(int32_t));
  const size_t per = align256((size_t)n * sizeof(int32_t));
  t.count = (int32_t *)p, p += ints;
  t.start = (int32_t *)p, p += ints;
  t.key = (int32_t *)p, p += per;
  t.rank = (int32_t *)p, p += per;
  t.order = (int32_t *)p, p += per;
  t.boxes = (double *)p;
  return t;
}

// A block per tile and, where there can be crowded tiles, two per chunk (up to 1,026).
unsigned tile_blocks(const RecArgs &a, const TileK &t) {
  return (unsigned)t.ntiles + (a.n > t.crowd ? 2 * blocks_of(a.n, t.chunk) : 0);
}

template <int N>
void spread_tiles(const RecArgs &a, const TileK &t, bool large, hipStream_t st) {
  const unsigned nb = tile_blocks(a, t);
  if (large)
    k_spread_tile<N, 16, 16, 8, kTileTeam><<<nb, kTileThreads, 0, st>>>(a, t);
  else if constexpr (N == 4)
    k_spread_tile<N, 8, 8, 8, kTileTeam><<<nb, kTileThreads, 0, st>>>(a, t);
}

template <int N>
void gather_tiles(const RecArgs &a, const TileK &t, bool large, hipStream_t st) {
  const unsigned nb = tile_blocks(a, t);
  if (large)
    k_gather_tile<N, 16, 16, 8, kTileTeam><<<nb, kTileThreads, 0, st>>>(a, t);
  else if constexpr (N == 4)
    k_gather_tile<N, 8, 8, 8, kTileTeam><<<nb, kTileThreads, 0, st>>>(a, t);
}

// tk: the tiles, or null for spreading by atomics.
template <int N>
void launch_rec_order(const RecArgs &a, const TileK *tk, double *self_partial, hipStream_t st) {
  const int64_t npts = grid_points(a.K);
  // one launch for the tables and the zeros: tile counts (in pairs), or the grid
  double *zero = tk ? (double *)tk->count : a.grid;
  const int64_t nzero = tk ? tk->ntiles / 2 + 1 : npts;  // with count[ntiles]
  k_bmod<N><<<kBmodBlocks + blocks_of(nzero, kThreads), kThreads, 0, st>>>(a, zero, nzero);
  const bool large = large_tiles(a.K);
  if (tk) {
    k_tile_count<<<blocks_of(a.n, kGatherAtoms), kGatherAtoms, 0, st>>>(a, *tk, self_partial);
    if (tk->ntiles <= kOrderTiles) {
      k_tile_order<<<blocks_of(a.n, kOrderThreads), kOrderThreads, 0, st>>>(a.n, *tk);
    } else {
      launch_scan(tk->ntiles, tk->count, tk->start, st);
      k_tile_scatter<<<blocks_of(a.n, kThreads), kThreads, 0, st>>>(a.n, *tk);
    }
    if constexpr (N <= 6) spread_tiles<N>(a, *tk, large, st);
  } else if (a.n > 0) {
    k_spread<N><<<blocks_of(a.n, kWave), kWave, 0, st>>>(a);
  }
  fft_x(a, true, tk, st);
  fft_y(a, true, 0, st);
  const int nparts = fft_z_influence(a, st);
  fft_y(a, false, nparts, st);
  fft_x(a, false, nullptr, st);
  if (tk) {
    if constexpr (N <= 6) gather_tiles<N>(a, *tk, large, st);
  } else if (a.n > 0) {
    k_gather<N, kGatherTeam>
        <<<blocks_of(a.n, kGatherAtoms), kGatherAtoms * kGatherTeam, 0, st>>>(a, self_partial);
  }
}

}  // namespace

size_t ewald_real_workspace(int64_t n) {
  return (size_t)(n > 0 ? n : 0) * sizeof(double4) +
         (size_t)blocks_of(n, kEwAtoms) * sizeof(double) + kErfcSeeds * sizeof(double) + 256;
}

// real grid, half grid (at most npts/2 + npts/8 complex points: K0 >= 8), tables,
// partials (one for the reciprocal energy, one per gather block)
// -- enough for every call, spreading by atomics; spme_workspace adds the tiles' part.
size_t spme_min_workspace(int64_t n, int64_t npts) {
  const int64_t half = npts / 2 + npts / 8;
  return (size_t)npts * sizeof(double) + (size_t)half * sizeof(double2) +
         3 * kMaxGrid * sizeof(double) +
         ((size_t)blocks_of(half, 512) + blocks_of(n, kGatherAtoms)) * sizeof(double) + 256;
}

size_t spme_workspace(int64_t n, int64_t npts) {
  return spme_min_workspace(n, npts) + tile_workspace(n, npts);
}

int launch_ewald_real(const BoxK &b, double alpha, double rc, int64_t n, const double *x,
                      const double *q, const int32_t *nbr, const int32_t *nnbr, int32_t maxn,
                      double *F, double *e_total, int accumulate, void *ws, hipStream_t st) {
  RealArgs a{};
  a.b = b;
  a.alpha = alpha;
  a.a2 = alpha * alpha;
  a.c2a = 2.0 * alpha / sqrt(kPi);
  a.rc2 = rc * rc;
  a.margin = rc;
  a.n = (int32_t)n;
  a.nbr = nbr;
  a.nnbr = nnbr;
  a.maxn = maxn;
  a.xq = (const double4 *)ws;
  a.F = F;
  a.accumulate = accumulate;
  const unsigned nblk = blocks_of(n, kEwAtoms);
  a.partial = (double *)((char *)ws + (size_t)(n > 0 ? n : 0) * sizeof(double4));
  double *seeds = a.partial + nblk;
  a.seeds = seeds;
  // rc within the range of the 24-bit intervals per unit length below
  const bool table = !e_total && alpha * rc <= kTableReach && rc > 1e-30 && rc < 1e30;
  if (table) {
    // intervals per unit length, cut to 24 bits: r in interval widths then carries no
    // error common to all pairs (G's relative sensitivity to it is ~2 (alpha r)^2)
    float per = (float)(kErfcIntervals / rc);
    if ((double)per * rc > kErfcIntervals) per = nextafterf(per, 0.0f);
    a.u_scale = per;
    a.dx = alpha / a.u_scale;
  } else {
    const double dx = alpha * rc / kErfcxIntervals;
    a.inv_dx = 1.0 / dx;
    a.half_dx = 0.5 * dx;
  }
  if (n > 0) {
    const unsigned npack = blocks_of(n, kThreads);
    if (table) k_pack_xq<true><<<npack, kThreads, 0, st>>>(a, x, q, (double4 *)ws, seeds);
    else k_pack_xq<false><<<npack, kThreads, 0, st>>>(a, x, q, (double4 *)ws, seeds);
    const bool wide = n > kNarrowAtoms;
#define LJMD_REAL(EV, TABLE)                                                       \
  wide ? k_ewald_real<true, EV, TABLE>                                             \
             <<<wide_grid(nblk, kEwThreads), kEwThreads, 0, st>>>(a)               \
       : k_ewald_real<false, EV, TABLE><<<nblk, kEwThreads, 0, st>>>(a)
    if (e_total) LJMD_REAL(true, false);
    else if (table) LJMD_REAL(false, true);
    else LJMD_REAL(false, false);
#undef LJMD_REAL
  }
  if (e_total)
    k_colsum<1024><<<1, 1024, 0, st>>>(n > 0 ? nblk : 0, 1, 1, a.partial, e_total, 1.0, 0);
  return check_launch("ljmd_ewald_real");
}

int launch_spme_recip(const BoxK &b, double alpha, int32_t order, const int32_t K[3], int64_t n,
                      const double *x, const double *q, double *F, double *e_total,
                      int accumulate, void *ws, size_t ws_bytes, hipStream_t st) {
  RecArgs a{};
  a.b = b;
  for (int d = 0; d < 3; ++d) {
    a.K[d] = K[d];
    a.scale[d] = (double)K[d] / b.L[d];
  }
  a.alpha = alpha;
  a.n = (int32_t)n;
  a.x = x;
  a.q = q;
  a.F = F;
  a.accumulate = accumulate;
  const int64_t npts = grid_points(K);
  char *p = (char *)ws;
  a.grid = (double *)p;
  p += (size_t)npts * sizeof(double);
  a.half = (double2 *)p;
  p += (size_t)(npts / 2 + npts / 8) * sizeof(double2);
  a.bmod = (double *)p;
  p += 3 * kMaxGrid * sizeof(double);
  a.partial = (double *)p;
  const unsigned ngat = blocks_of(n, kGatherAtoms);
  double *self_partial = n > 0 ? a.partial + 1 : nullptr;
  TileK tiles{};
  const TileK *tk = nullptr;
  if (n > 0 && tiled(order, K) && ws_bytes >= spme_workspace(n, npts)) {
    tiles = make_tiles(order, K, n, (char *)ws + spme_min_workspace(n, npts));
    tk = &tiles;
  }
  switch (order) {
    case 4: launch_rec_order<4>(a, tk, self_partial, st); break;
    case 6: launch_rec_order<6>(a, tk, self_partial, st); break;
    default: launch_rec_order<8>(a, tk, self_partial, st); break;
  }
  if (e_total)
    k_colsum<1024><<<1, 1024, 0, st>>>((int64_t)1 + (n > 0 ? ngat : 0), 1, 1, a.partial, e_total,
                                     1.0, 0);
  return check_launch("ljmd_spme_recip");
}

}  // namespace ljmd
