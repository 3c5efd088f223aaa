// Counting sort of atoms into binning cells (cell-major, ascending id inside a
// cell), gfx950.  Paper: Cabana "Particle Sorting" (geometric binning) and the
// re-sort that begins each MD timestep (Introduction).
//
// Four launches:
//   1. cell id + histogram   one thread per atom; lanes of a wavefront in the
//                            same cell share one atomic add and get ranks
//   2. exclusive scan        a 1024-thread block per chunk of cells (three launches
//                            beyond 65,536 cells)
//   3. scatter               one thread per atom to slot start[cell] + rank
//   4. in-cell rank + permute  one wavefront per cell: ids of the cell are
//                            staged in LDS, each lane ranks its atom among
//                            them, then copies x, v, type, id to the ranked slot.
// The rank order of step 1 depends on atomic timing; step 4 replaces it by
// the id order, so the output permutation is deterministic.
#include "common.h"

namespace ljmd {

namespace {

constexpr int kScanThreads = 1024;
constexpr int kPermWaves = 4;
constexpr int kStage = 256;  // ids per wavefront staged in LDS

__device__ __forceinline__ int32_t cell_of(const double *xi, const GridK &g) {
  int32_t c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    int32_t ck = (int32_t)floor(xi[k] / g.h[k]);
    ck = ck > g.nc[k] - 1 ? g.nc[k] - 1 : ck;
    c[k] = ck < 0 ? 0 : ck;
  }
  return (c[2] * g.nc[1] + c[1]) * g.nc[0] + c[0];
}

__global__ void k_fill_i32(int32_t *p, int64_t m, int32_t val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) p[i] = val;
}

// Cell of every atom and its rank among the atoms of its cell that were
// counted before it (count_ranks).
__global__ void k_count(int64_t n, const double *__restrict__ x, GridK g,
                        int32_t *__restrict__ cell, int32_t *__restrict__ rank,
                        int32_t *__restrict__ counts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < n;
  const int32_t c = live ? cell_of(x + 3 * i, g) : -1;
  const int32_t r = count_ranks(live, c, counts);
  if (live) {
    cell[i] = c;
    rank[i] = r;
  }
}

// Exclusive scan of counts[0..m) into start[0..m] (start[m] = total), kScanChunk counts per
// block, four consecutive ones per thread.
// SUMMED = false, one launch, no flags between blocks: every block sums the counts before
// its chunk by itself (coalesced, before the one barrier).  That is m^2 / (2 kScanChunk)
// reads, so only up to kScanOnce counts; beyond, k_scan_sums and k_scan_tops leave every
// chunk's prefix in its first place of start (SUMMED).
// Whole binning of a sparse gas (us), one block over all chunks with its carry / every block
// sums for itself / three launches: 32,768 cells 56 / 22 / -, 64,000 74 / 26 / 26, 125,000
// 110 / 33.7 / 30.5, 1,000,000 603 / 150 / 86, 8,000,000 4,546 / 2,539 / 509, 16,777,216
// 9,492 / 11,220 / 1,036.
constexpr int32_t kScanChunk = 4 * kScanThreads;
constexpr int32_t kScanOnce = 16 * kScanChunk;

template <bool SUMMED>
__global__ __launch_bounds__(kScanThreads) void k_scan(int32_t m, const int32_t *__restrict__ counts,
                                                     int32_t *start) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ int32_t wsum[kWaves], wbefore[kWaves];
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), w = t / kWave;
  const int32_t c0 = blockIdx.x * kScanChunk;
  int32_t v[4], part[4] = {0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = c0 + 4 * t + q < m ? counts[c0 + 4 * t + q] : 0;
  if constexpr (SUMMED) {
    if (t == 0) part[0] = start[c0];
  } else {
#pragma unroll 2
    for (int32_t c = t; c < c0; c += kScanChunk)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[q] += counts[c + q * kScanThreads];
  }
  const int32_t s = v[0] + v[1] + v[2] + v[3];
  const int32_t inc = wave_inclusive_scan(s);
  const int32_t bef = wave_inclusive_scan(part[0] + part[1] + part[2] + part[3]);
  if (lane == kWave - 1) {
    wsum[w] = inc;
    wbefore[w] = bef;
  }
  __syncthreads();
  int32_t run = inc - s;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) run += wbefore[k] + (k < w ? wsum[k] : 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t c = c0 + 4 * t + q;
    if (c < m) start[c] = run;
    run += v[q];
    if (c == m - 1) start[m] = run;
  }
}

// The sum of every chunk into its first place of start.
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int32_t m,
                                                          const int32_t *__restrict__ counts,
                                                          int32_t *__restrict__ start) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ int32_t wsum[kWaves];
  const int t = threadIdx.x;
  const int32_t c0 = blockIdx.x * kScanChunk;
  int32_t s = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) s += c0 + 4 * t + q < m ? counts[c0 + 4 * t + q] : 0;
  const int32_t inc = wave_inclusive_scan(s);
  if ((t & (kWave - 1)) == kWave - 1) wsum[t / kWave] = inc;
  __syncthreads();
  if (t != 0) return;
  s = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) s += wsum[k];
  start[c0] = s;
}

// Those sums replaced by their exclusive prefix sums, one block, a run of chunks per thread.
__global__ __launch_bounds__(kScanThreads) void k_scan_tops(int32_t nchunks,
                                                          int32_t *__restrict__ start) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ int32_t wsum[kWaves];
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), w = t / kWave;
  const int32_t per = (nchunks + kScanThreads - 1) / kScanThreads;
  const int32_t a = t * per < nchunks ? t * per : nchunks;
  const int32_t b = a + per < nchunks ? a + per : nchunks;
  int32_t s = 0;
#pragma unroll 8
  for (int32_t c = a; c < b; ++c) s += start[(int64_t)c * kScanChunk];
  const int32_t inc = wave_inclusive_scan(s);
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  int32_t run = inc - s;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) run += k < w ? wsum[k] : 0;
  for (int32_t c = a; c < b; ++c) {
    const int32_t v = start[(int64_t)c * kScanChunk];
    start[(int64_t)c * kScanChunk] = run;
    run += v;
  }
}

// Slot of atom i: start of its cell plus its rank (no atomics).
__global__ void k_scatter(int64_t n, const int32_t *__restrict__ cell,
                          const int32_t *__restrict__ rank, const int32_t *__restrict__ start,
                          int32_t *__restrict__ src) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  src[start[cell[i]] + rank[i]] = (int32_t)i;
}

__device__ __forceinline__ int64_t id_at(const int64_t *id_in, int32_t s) {
  return id_in ? id_in[s] : (int64_t)s;
}

__global__ __launch_bounds__(kPermWaves *kWave) void k_permute(
    int32_t ncells, const int32_t *__restrict__ start, const int32_t *__restrict__ src,
    const double *__restrict__ x_in, const double *__restrict__ v_in,
    const int32_t *__restrict__ type_in, const int64_t *__restrict__ id_in,
    double *__restrict__ x_out, double *__restrict__ v_out, int32_t *__restrict__ type_out,
    int64_t *__restrict__ id_out) {
  __shared__ int64_t ids[kPermWaves][kStage];
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  const int32_t c = blockIdx.x * kPermWaves + w;
  if (c >= ncells) return;  // whole wavefront leaves together; no block barrier below
  const int32_t s0 = start[c];
  const int32_t m = start[c + 1] - s0;
  const bool staged = m <= kStage;
  if (staged) {
    for (int32_t k = lane; k < m; k += kWave) ids[w][k] = id_at(id_in, src[s0 + k]);
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  for (int32_t k0 = 0; k0 < m; k0 += kWave) {
    const int32_t k = k0 + lane;
    if (k < m) {
      const int32_t s = src[s0 + k];
      const int64_t my = id_at(id_in, s);
      int32_t rank = 0;
      if (staged) {
        for (int32_t q = 0; q < m; ++q) rank += ids[w][q] < my;
      } else {
        for (int32_t q = 0; q < m; ++q) rank += id_at(id_in, src[s0 + q]) < my;
      }
      const int64_t o = (int64_t)s0 + rank;
      x_out[3 * o] = x_in[3 * (int64_t)s];
      x_out[3 * o + 1] = x_in[3 * (int64_t)s + 1];
      x_out[3 * o + 2] = x_in[3 * (int64_t)s + 2];
      if (v_in) {
        v_out[3 * o] = v_in[3 * (int64_t)s];
        v_out[3 * o + 1] = v_in[3 * (int64_t)s + 1];
        v_out[3 * o + 2] = v_in[3 * (int64_t)s + 2];
      }
      if (type_in) type_out[o] = type_in[s];
      id_out[o] = my;
    }
  }
}

inline unsigned blocks_for(int64_t n, int threads) {
  return (unsigned)((n + threads - 1) / threads);
}

}  // namespace

// start[0..m] = exclusive prefix sums of counts[0..m) and their total.
void launch_scan(int32_t m, const int32_t *counts, int32_t *start, hipStream_t st) {
  const unsigned nb = blocks_for(m, kScanChunk);
  if (m <= kScanOnce) {
    k_scan<false><<<nb, kScanThreads, 0, st>>>(m, counts, start);
  } else {
    k_scan_sums<<<nb, kScanThreads, 0, st>>>(m, counts, start);
    k_scan_tops<<<1, kScanThreads, 0, st>>>((int32_t)nb, start);
    k_scan<true><<<nb, kScanThreads, 0, st>>>(m, counts, start);
  }
}

size_t bin_workspace(int64_t n, int64_t ncells) {
  // counts[ncells] + cell[n] + rank[n] + src[n], int32, 256-byte aligned
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  return al((size_t)ncells * 4) + 3 * al((size_t)n * 4);
}

int launch_bin(const GridK &g, int64_t n, const double *x_in, const double *v_in,
               const int32_t *type_in, const int64_t *id_in, double *x_out, double *v_out,
               int32_t *type_out, int64_t *id_out, int32_t *cell_start, void *ws,
               hipStream_t st) {
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  char *p = (char *)ws;
  int32_t *counts = (int32_t *)p;
  p += al((size_t)g.ncells * 4);
  int32_t *cell = (int32_t *)p;
  p += al((size_t)n * 4);
  int32_t *rank = (int32_t *)p;
  p += al((size_t)n * 4);
  int32_t *src = (int32_t *)p;

  k_fill_i32<<<blocks_for(g.ncells, 256), 256, 0, st>>>(counts, g.ncells, 0);
  if (n > 0) k_count<<<blocks_for(n, 256), 256, 0, st>>>(n, x_in, g, cell, rank, counts);
  launch_scan(g.ncells, counts, cell_start, st);
  if (n > 0) {
    k_scatter<<<blocks_for(n, 256), 256, 0, st>>>(n, cell, rank, cell_start, src);
    k_permute<<<blocks_for(g.ncells, kPermWaves), kPermWaves * kWave, 0, st>>>(
        g.ncells, cell_start, src, x_in, v_in, type_in, id_in, x_out, v_out, type_out, id_out);
  }
  return check_launch("ljmd_bin");
}

}  // namespace ljmd
