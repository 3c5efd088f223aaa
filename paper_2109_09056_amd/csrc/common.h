// Internal helpers shared by the gfx950 kernels of libljmd (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ljmd.h"

namespace ljmd {

constexpr int kWave = 64;

// Box constants handed to kernels by value.
struct BoxK {
  double L[3];
  double invL[3];
};

// Binning grid: nc cells per dimension, edge h = L/nc.
struct GridK {
  int32_t nc[3];
  double h[3];
  int32_t ncells;
};

// Representative of d modulo L nearest zero.  For |d| < L this equals the
// single shift "d > L/2: d - L; d < -L/2: d + L" bit for bit except when
// |d| is within rounding of L/2, where both representatives lie at ~L/2,
// beyond any list cutoff the ABI accepts.
__device__ __forceinline__ double min_image(double d, double L, double invL) {
  double k = __builtin_rint(d * invL);
  return __builtin_fma(-k, L, d);
}

// Atom j's 3-vector in an [n][3] FP64 array.  Narrow form (every index below
// kNarrowAtoms): a 32-bit byte offset from the array base, formed with the
// full-rate 24-bit multiply; wide form: 64-bit index arithmetic.
constexpr int64_t kNarrowAtoms = int64_t(1) << 24;
template <bool WIDE>
__device__ __forceinline__ const double *pos_of(const double *x, int32_t j) {
  if constexpr (WIDE)
    return x + 3 * (int64_t)j;
  else
    return (const double *)((const char *)x + __umul24((uint32_t)j, 24u));
}

// r^2 in the fixed order (dx*dx + dy*dy) + dz*dz; the library is compiled
// with -ffp-contract=off so no FMA is formed here.
__device__ __forceinline__ double dist2(double dx, double dy, double dz) {
  return (dx * dx + dy * dy) + dz * dz;
}

// Reciprocal by the hardware estimate refined with Newton-Raphson steps
// y <- y + y (1 - a y), each of which squares the relative error.
__device__ __forceinline__ double recip64(double a) {
  double y = __builtin_amdgcn_rcp(a);
  double e = __builtin_fma(-a, y, 1.0);
  y = __builtin_fma(y, e, y);
  e = __builtin_fma(-a, y, 1.0);
  return __builtin_fma(y, e, y);
}

// a^(-1/2) by the hardware estimate refined with Newton-Raphson steps
// y <- y (3/2 - (a/2) y^2), each of which squares the relative error.
__device__ __forceinline__ double rsqrt64(double a) {
  const double h = 0.5 * a;
  double y = __builtin_amdgcn_rsq(a);
  y = __builtin_fma(y, __builtin_fma(-h * y, y, 0.5), y);
  return __builtin_fma(y, __builtin_fma(-h * y, y, 0.5), y);
}

__device__ __forceinline__ float recip32(float a) {
  float y = __builtin_amdgcn_rcpf(a);
  float e = __builtin_fmaf(-a, y, 1.0f);
  return __builtin_fmaf(y, e, y);
}

// Value of v in lane `src` (wavefront-uniform src), through two scalar readlanes.
__device__ __forceinline__ double readlane_f64(double v, int src) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    int o = __shfl_xor(v, off, kWave);
    v = o > v ? o : v;
  }
  return v;
}

// v of the lane that DPP control CTRL reads (quad_perm, row rotation, ...): two
// VALU moves, where a shuffle through ds_bpermute would take two LDS round trips.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
  const uint32_t l2 = (uint32_t)__builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, true);
  const uint32_t h2 = (uint32_t)__builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)h2 << 32) | l2);
}
constexpr int kDppXor1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;  // quad_perm [2, 3, 0, 1]
constexpr int kDppRor4 = 0x124;  // row (16 lanes) rotated by 4
constexpr int kDppRor8 = 0x128;  // by 8: lane ^ 8

// v summed over the aligned group of TEAM lanes (TEAM a power of two up to
// 16) by a butterfly, widest exchange first: both lanes of every exchange add
// the same two numbers, so every lane ends with the same, order-fixed sum.
template <int TEAM>
__device__ __forceinline__ double team_sum(double v) {
  static_assert(TEAM == 1 || TEAM == 2 || TEAM == 4 || TEAM == 8 || TEAM == 16, "team of lanes");
  if constexpr (TEAM >= 16) v += dpp_f64<kDppRor8>(v);
  if constexpr (TEAM >= 8) v += __shfl_xor(v, 4, kWave);
  if constexpr (TEAM >= 4) v += dpp_f64<kDppXor2>(v);
  if constexpr (TEAM >= 2) v += dpp_f64<kDppXor1>(v);
  return v;
}

// Sums of NV (up to 8) values over each row of 16 lanes.  With P = NV rounded
// up to a power of two, two exchanges inside the quad halve the values a lane
// carries (lane bit 0 keeps the even or odd ones, bit 1 likewise), then the four
// quads of the row are added: 8 values take 6 exchanged doubles and 10 adds per lane
// instead of the 48 of a butterfly per value.  On return lane l < 16 of the
// row's first min(P, 4) lanes holds columns l % 4, l % 4 + 4 in out[0], out[1].
template <int NV>
__device__ __forceinline__ void row_sums(const double (&v)[NV], double (&out)[2]) {
  constexpr int P = NV > 4 ? 8 : (NV > 2 ? 4 : NV);
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
  double a[P];
#pragma unroll
  for (int q = 0; q < P; ++q) a[q] = q < NV ? v[q < NV ? q : 0] : 0.0;
  constexpr int H = P > 1 ? P / 2 : 1;
  double r[H];
  if constexpr (P > 1) {
#pragma unroll
    for (int k = 0; k < H; ++k)
      r[k] = (b0 ? a[2 * k + 1] : a[2 * k]) + dpp_f64<kDppXor1>(b0 ? a[2 * k] : a[2 * k + 1]);
  } else {
    r[0] = a[0] + dpp_f64<kDppXor1>(a[0]);
  }
  constexpr int G = H > 1 ? H / 2 : 1;
#pragma unroll
  for (int k = 0; k < G; ++k) {
    double t;
    if constexpr (H > 1)
      t = (b1 ? r[2 * k + 1] : r[2 * k]) + dpp_f64<kDppXor2>(b1 ? r[2 * k] : r[2 * k + 1]);
    else
      t = r[k] + dpp_f64<kDppXor2>(r[k]);
    t += dpp_f64<kDppRor4>(t);
    out[k] = t + dpp_f64<kDppRor8>(t);
  }
}

// Block of `NW` waves: sums NV (up to 8) values per thread into out[0..NV)
// for the block, in a fixed order (rows of 16 lanes by row_sums, then the rows).
// Every thread of the block must call it.  `red` is __shared__ storage of
// kRedRows * NW * NV doubles.  HALVES = 2: the sum of the first half of the block's
// rows plus the sum of the second, as two blocks of half the size would leave.
constexpr int kRedRows = kWave / 16;
template <int NW, int NV, int HALVES = 1>
__device__ __forceinline__ void block_sum(const double (&v)[NV], double *red, double *out) {
  constexpr int P = NV > 4 ? 8 : (NV > 2 ? 4 : NV);
  constexpr int kRows = kRedRows * NW;
  double s[2];
  row_sums<NV>(v, s);
  const int l = threadIdx.x & 15;
  double *row = red + (threadIdx.x >> 4) * NV;
  if (l < (P < 4 ? P : 4)) {
    if (l < NV) row[l] = s[0];
    if (P == 8 && l + 4 < NV) row[l + 4] = s[1];
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double t[HALVES];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
      t[h] = 0.0;
#pragma unroll
      for (int k = 0; k < kRows / HALVES; ++k)
        t[h] += red[(h * (kRows / HALVES) + k) * NV + threadIdx.x];
    }
    out[threadIdx.x] = HALVES == 2 ? t[0] + t[HALVES - 1] : t[0];
  }
}

// Column sums over `rows` partial rows of `stride` doubles (stride a power of
// two dividing THREADS) by one block of THREADS threads, left in LDS:
// part[q] = sum_r p[r*stride + q] for q < stride.  Thread t reads the flat
// array at t, t + THREADS, ... (coalesced), so it always sees column
// t % stride; the THREADS/stride threads of a column are then added by a tree
// in `part` (THREADS doubles of LDS).  Fixed order throughout; every thread of
// the block calls it and part[0..stride) is visible to all of them on return.
// PAIRS: the sums of the rows 2r and 2r + 1 (the second absent at an odd end) take
// the place of the rows.
template <int THREADS, bool PAIRS = false>
__device__ __forceinline__ void colsum_lds(int64_t rows, int stride, const double *__restrict__ p,
                                           double *part) {
  const int t = threadIdx.x;
  double s = 0.0;
  const int64_t all = rows * stride;
  const int64_t total = PAIRS ? (rows + 1) / 2 * stride : all;
  constexpr int B = 16;  // loads in flight per thread
  for (int64_t f0 = t; f0 < total; f0 += (int64_t)B * THREADS) {
    double v[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int64_t f = f0 + (int64_t)k * THREADS;
      if constexpr (PAIRS) {
        const int64_t g = 2 * f - (f & (stride - 1));  // row 2r, the same column
        v[k] = f < total ? p[g] : 0.0;
        if (g + stride < all) v[k] += p[g + stride];
      } else {
        v[k] = f < total ? p[f] : 0.0;
      }
    }
#pragma unroll
    for (int k = 0; k < B; ++k) s += v[k];
  }
  part[t] = s;
  __syncthreads();
  for (int off = THREADS / 2; off >= stride; off >>= 1) {
    if (t < off) part[t] += part[t + off];
    __syncthreads();
  }
}

// One launch of colsum_lds: out[q] = scale * column q for q < ncols (+= when
// accumulate).
template <int THREADS, bool PAIRS = false>
__global__ __launch_bounds__(THREADS) void k_colsum(int64_t rows, int stride, int ncols,
                                                   const double *__restrict__ p,
                                                   double *__restrict__ out, double scale,
                                                   int accumulate) {
  __shared__ double part[THREADS];
  colsum_lds<THREADS, PAIRS>(rows, stride, p, part);
  const int t = threadIdx.x;
  if (t < ncols) out[t] = accumulate ? out[t] + scale * part[t] : scale * part[t];
}

// Inclusive prefix sum of v over the lanes of the wavefront (shuffles only).
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t o = __shfl_up(v, off, kWave);
    if (lane >= off) v += o;
  }
  return v;
}

// One counting step of a counting sort for the lanes of a wavefront: counts[c] grows by
// the number of live lanes with key c, and every live lane gets its rank among all
// elements of its key counted so far.  Lanes with the same key (the common case: the
// input is usually in some spatial order) share one atomic add.  The groups are found
// first, in registers, and all their leaders add in one instruction: a wavefront waits
// for one atomic round trip instead of one per group.
__device__ __forceinline__ int32_t count_ranks(bool live, int32_t key, int32_t *counts) {
  const int lane = threadIdx.x & (kWave - 1);
  bool pending = live;
  int lead = lane, size = 0;
  int32_t r = 0;
  for (uint64_t act = __ballot(pending); act != 0; act = __ballot(pending)) {
    const int leader = __builtin_ctzll(act);
    const bool mine = pending && key == __builtin_amdgcn_readlane(key, leader);
    const uint64_t grp = __ballot(mine);
    if (mine) {
      lead = leader;
      size = (int)__popcll(grp);
      r = (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(grp >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)grp, 0u));
      pending = false;
    }
  }
  int32_t base = 0;
  if (live && lane == lead) base = atomicAdd(&counts[key], size);
  return r + __shfl(base, lead, kWave);
}

// Workgroups are handed to the 8 XCDs round-robin (block b runs on XCD b % 8),
// and each XCD has its own L2.  Renumbering so that XCD x gets one contiguous
// run of logical blocks keeps spatially adjacent tiles -- and the neighbor
// positions they gather -- inside one L2.  A bijection on [0, nblk).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_block(int b, int nblk) {
  const int q = nblk / kXcds, r = nblk % kXcds;
  const int x = b % kXcds, k = b / kXcds;
  return x * q + (x < r ? x : r) + k;
}

// A launch takes fewer than 2^32 threads per grid dimension: kernels for systems of any size
// (WIDE) get their blocks in rows (wide_grid).  A block's number and the number of blocks for
// n atoms, `per` of them each; the last row's spare blocks have numbers beyond and leave.
template <bool WIDE>
__device__ __forceinline__ int flat_block() {
  return WIDE ? (int)(blockIdx.y * gridDim.x + blockIdx.x) : (int)blockIdx.x;
}
template <bool WIDE>
__device__ __forceinline__ int flat_blocks(int32_t n, int per) {
  return WIDE ? (int)(((int64_t)n + per - 1) / per) : (int)gridDim.x;
}
inline dim3 wide_grid(int64_t nblk, int threads) {
  const int64_t row = (((int64_t)1 << 32) - 1) / threads, rows = (nblk + row - 1) / row;
  return rows <= 1 ? dim3((unsigned)nblk)
                   : dim3((unsigned)((nblk + rows - 1) / rows), (unsigned)rows);
}

// Packed upper-triangle index of the type pair (a, b).
__host__ __device__ __forceinline__ int packed_index(int a, int b, int T) {
  if (a > b) {
    int t = a;
    a = b;
    b = t;
  }
  return a * T - a * (a - 1) / 2 + (b - a);
}

// ---- host side ----
int set_error(int code, const char *fmt, ...);
int check_launch(const char *what);
BoxK make_box(const ljmd_box *b);
int make_grid(const ljmd_box *b, double rlist, GridK *g);

}  // namespace ljmd
