// Verlet neighbor lists over the 27-cell stencil, gfx950.  Paper: Cabana
// "Neighbor List Creation" (distance-criterion lists built by binning, dense
// storage, thread-parallel creation).
//
// One wavefront per home cell (on grids of fewer than 2,048 cells, per part of
// a cell's home atoms: a 32,000-atom liquid has 1,331 cells, one wavefront per
// SIMD or fewer).  The candidates -- every atom of the stencil
// cells (offsets -1, 0, +1 per dimension modulo nc, with repeats removed when
// nc < 3) -- are loaded once into registers, 64 per register slot (lane t of
// slot r holds candidate 64 r + t).  The wavefront then walks the home atoms
// one at a time: every lane tests its candidates against the (uniform) home
// atom, a ballot + mbcnt prefix compacts the hits, and each hit is stored in
// the home atom's row of the tiled-ELL list:
//   nbr[((i / 64) * maxn + k) * 64 + (i % 64)].
// On grids of 3 or more cells per dimension the candidates are staged as
// 16-bit lattice coordinates and tested with packed integer arithmetic
// (QuantK below); only pairs within the lattice's error band of rlist take the
// FP64 test, so the lists are exactly those of the FP64 test everywhere.
// Cells with more candidates than the register slots hold fall back to
// reading candidates from global memory per home atom.
#include "common.h"
#include "stencil.h"

namespace ljmd {

namespace {

// Two shapes of the build kernel.  Standard: 12 register slots (up to 768
// candidates staged) and rows of up to 128 entries buffered in LDS.  Dense
// (chosen when maxn > 128, i.e. long rows and so crowded stencils, or when the mean
// stencil has more than 11 slots' candidates): 16 slots (1024 candidates) and rows of up
// to 256 entries, at twice the LDS.
// Stencils beyond the slots read every candidate from memory for every home atom.  Small
// boxes reach that at liquid densities, as their cells are up to 4/3 of the cutoff wide:
// tiled lists (us), standard -> dense, 864 atoms (27 cells) 59.0 -> 16.7, 2,048 59.3 ->
// 17.1, 4,000 69.6 -> 18.4, 13,500 (mean stencil of 11.1 slots, some cells above 12)
// 65.8 -> 21.0; where the standard shape holds all, the dense one costs 20 %
// (110,447 atoms 56.1 -> 68.5), on the smallest grids 5 % (256 and 500 atoms, 8 cells, half
// lists 9.8 -> 10.3 and 17.0 -> 17.6).
constexpr int kSlots = 12;
constexpr int kRowCap = 128;
constexpr int kDenseSlots = 16;
constexpr int kDenseRowCap = 256;
constexpr int64_t kStandardCandidates = (kSlots - 1) * kWave;
// Home atoms whose rows are buffered in LDS at once.  8 rather than 16 halves
// the one-wavefront block's LDS, so more blocks fit on a compute unit: at 500,000
// atoms 189.4 -> 171.2 us (full list), 159.3 -> 143.6 (half), 362.6 -> 261.3 (dense
// shape, 512,000 particles); batches that end at multiples of 8 atoms 174.1 / 145.8 / 265.6.
constexpr int kBatch = 8;
// Grids of at least this many cells (and so no split cells) have code for 2 and 4 (dense: 6
// and 8) slots too, for gases; smaller ones, whose launches are mostly instruction fetch, take
// the next larger.  With / without that code, two launches apart (us): 200,000 atoms at
// density 0.02, 0.05, 0.1, 0.3 (142,000 to 29,800 cells) 230 / 246, 167 / 181, 119 / 130,
// 72.8 / 79.4; 20,000 at 0.1 (8,000 cells) 30.7 / 29.3, at 0.2 (4,096) 30.0 / 26.6, at 0.05
// (17,576) 37.4 / 37.5.
constexpr unsigned kFewSlotGrid = 16384;
constexpr int kFlushRows = kWave / kBatch;  // list rows of a batch written per store instruction
// LDS row stride ROWCAP + 1 (odd): lanes reading entry k of different rows hit distinct banks

__global__ void k_fill_scalar(int32_t *p, int32_t val) { *p = val; }

// What a build pass writes: the tiled list (rows cut at maxn, counts in nnbr),
// only the true row lengths (into nnbr), or compressed rows at csr[offsets[i]..]
// (entries at or beyond cap dropped).
enum BuildMode { kTiled = 0, kCount = 1, kCsr = 2 };

// Output of a build pass.
struct BuildOut {
  int32_t *nbr;            // tiled list (kTiled)
  int32_t *nnbr;           // row lengths (kTiled: cut at maxn; kCount: true)
  int32_t maxn;
  const int64_t *offsets;  // kCsr: row starts
  int32_t *csr;            // kCsr: rows
  int64_t cap;             // kCsr: capacity of csr
  uint16_t *hits;          // bit r of [64 i + lane]: slot r's candidate of that lane is in row i
                           // (kCount writes, kCsr reads), or NULL
};

// Integer pre-test of the candidate distances (grids of at least 3 cells per
// dimension).  Each staged position is taken relative to the home cell's
// centre, minimum-imaged there and rounded to a lattice of spacing q: u =
// rint(min_image(x - centre) / q), |u| <= kQuantMax (the 27 stencil cells lie
// within 1.5 cell edges of the centre).  A pair's lattice displacement then
// differs from the true one by at most q per axis, so its length by at most
// sqrt(3) q, and with R = rlist / q the integer r2q = |u_i - u_j|^2 decides
//   r2q < t_in  = floor((R - 1.75)^2): inside rlist,
//   r2q > t_out = ceil((R + 1.75)^2):  outside rlist,
// and only the pairs between (about 0.08 per atom in the dense liquid) take
// the FP64 test with the minimum image.  The image of a candidate nearest the
// centre is the one nearest the home atom for every pair within rlist when
// the home atom lies within L/2 - rlist of the centre per axis (the pair is
// then within L/2 of the centre); atoms inside their cell always do (cell
// edges exceed rlist and nc >= 3), and a wavefront whose home atoms do not
// (positions outside the box) takes the unstaged FP64 path.  So the lists are
// exactly those of the FP64 test.
struct QuantK {
  double invq;     // 1 / q
  int32_t t_in;    // r2q below: inside rlist
  int32_t t_out;   // r2q above: outside rlist
  double home[3];  // bound on |home atom - centre| per axis: L/2 - rlist, rounded down
};
constexpr double kQuantSpan = 16000.0;  // lattice steps per 1.5 cell edges
constexpr int32_t kQuantMax = 16380;    // |u| of a staged coordinate
// r2q <= 3 * 32,760^2 = 3.22e9 and t_in <= (10,667 - 1.75)^2 = 1.14e8: r2q - t_in modulo
// 2^32 is at or above 2^32 - t_in exactly when r2q < t_in.
// z of an empty slot: 15,620 <= |dz| <= 48,380, so r2q is between 2.4e8 (above t_out)
// and 2.9e9
constexpr int32_t kQuantEmpty = 32000;

typedef short short2v __attribute__((ext_vector_type(2)));

// Lattice coordinates of x relative to the centre cc; false when a coordinate
// is out of range (or not finite).
__device__ __forceinline__ bool quantize(const double *p, const double *cc, const BoxK &b,
                                         double invq, int32_t &uxy, int32_t &uz) {
  int32_t u[3];
  bool in = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double d = min_image(p[k] - cc[k], b.L[k], b.invL[k]) * invq;
    in = in && __builtin_fabs(d) <= (double)kQuantMax;
    u[k] = in ? (int32_t)__builtin_rint(d) : 0;
  }
  uxy = (int32_t)((uint32_t)(uint16_t)u[0] | ((uint32_t)u[1] << 16));
  uz = u[2];
  return in;
}

// Stencil of cell c: its candidate ranges [rs[s], rs[s] + len) in sorted order
// and the prefix pre[s] of their lengths.  Returns the number of ranges.
__device__ __forceinline__ int stencil_ranges(const GridK &g, int32_t c, const int32_t *cell_start,
                                              int32_t *rs, int32_t *pre) {
  const int lane = threadIdx.x & (kWave - 1);
  int32_t cc[3] = {c % g.nc[0], (c / g.nc[0]) % g.nc[1], c / (g.nc[0] * g.nc[1])};
  // y and z: the distinct cells among c-1, c, c+1 (mod nc)
  int32_t cells[2][3];
  int cnt[2];
#pragma unroll
  for (int k = 1; k < 3; ++k) {
    const int32_t m = g.nc[k];
    if (m >= 3) {
      cells[k - 1][0] = cc[k] == 0 ? m - 1 : cc[k] - 1;
      cells[k - 1][1] = cc[k];
      cells[k - 1][2] = cc[k] == m - 1 ? 0 : cc[k] + 1;
      cnt[k - 1] = 3;
    } else {
      cells[k - 1][0] = 0;
      cells[k - 1][1] = 1;
      cells[k - 1][2] = 0;
      cnt[k - 1] = m;
    }
  }
  // x: runs of consecutive cells, which are consecutive in sorted order too
  const int32_t mx = g.nc[0];
  int32_t run0[2], runlen[2];
  int nrun;
  if (mx < 3) {
    run0[0] = 0, runlen[0] = mx, nrun = 1;
  } else if (cc[0] == 0) {
    run0[0] = 0, runlen[0] = 2, run0[1] = mx - 1, runlen[1] = 1, nrun = 2;
  } else if (cc[0] == mx - 1) {
    run0[0] = mx - 2, runlen[0] = 2, run0[1] = 0, runlen[1] = 1, nrun = 2;
  } else {
    run0[0] = cc[0] - 1, runlen[0] = 3, nrun = 1;
  }
  const int S = nrun * cnt[0] * cnt[1];
  int32_t len = 0;
  if (lane < S) {
    const int ir = lane % nrun;
    const int iy = (lane / nrun) % cnt[0];
    const int iz = lane / (nrun * cnt[0]);
    const int32_t row = (cells[1][iz] * g.nc[1] + cells[0][iy]) * mx;
    const int32_t a = cell_start[row + run0[ir]];
    rs[lane] = a;
    len = cell_start[row + run0[ir] + runlen[ir]] - a;
  }
  // inclusive prefix of len over the first S lanes (S <= 18 < 32)
  int32_t inc = len;
#pragma unroll
  for (int off = 1; off < 32; off <<= 1) {
    int32_t o = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += o;
  }
  if (lane < S) pre[lane + 1] = inc;
  if (lane == 0) pre[0] = 0;
  __syncthreads();  // the block is this one wavefront
  return S;
}

// Sorted index of candidate t (t < pre[S]).
__device__ __forceinline__ int32_t locate(int32_t t, const int32_t *rs, const int32_t *pre) {
  int r = 0;
  while (t >= pre[r + 1]) ++r;
  return rs[r] + (t - pre[r]);
}

// Register-staged build of one cell's rows (candidates <= SLOTS * 64).  BUF:
// rows are compacted in LDS (maxn <= ROWCAP) rather than stored directly.
template <bool HALF, bool WRAP, bool BUF, int SLOTS, int ROWCAP, int MODE>
__device__ __forceinline__ void build_staged(const BoxK &b, double rl2, const double *__restrict__ x,
                                             int32_t h0, int32_t h1, int32_t total, int nslot,
                                             const int32_t *rs, const int32_t *pre,
                                             const BuildOut &o, int32_t *rowbuf, int32_t *rowcnt,
                                             int32_t &maxc) {
  const int32_t maxn = o.maxn;
  int32_t *__restrict__ nbr = o.nbr;
  int32_t *__restrict__ nnbr = o.nnbr;
  static_assert(!BUF || MODE == kTiled, "rows are buffered only for the tiled list");
  const int lane = threadIdx.x & (kWave - 1);
  const double L0 = b.L[0], L1 = b.L[1], L2 = b.L[2];
  const double iL0 = b.invL[0], iL1 = b.invL[1], iL2 = b.invL[2];
  constexpr int kRowStride = ROWCAP + 1;
  double qx[SLOTS], qy[SLOTS], qz[SLOTS];
  int32_t qj[SLOTS];
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    const int32_t t = r * kWave + lane;
    qj[r] = -1;
    qx[r] = qy[r] = qz[r] = 0.0;
    if (r < nslot && t < total) {
      const int32_t j = locate(t, rs, pre);
      qj[r] = j;
      qx[r] = x[3 * (int64_t)j];
      qy[r] = x[3 * (int64_t)j + 1];
      qz[r] = x[3 * (int64_t)j + 2];
    }
  }
  // Rows of up to kBatch home atoms are compacted into LDS first (when they fit)
  // and then written out k by k: the atoms of a batch are consecutive, so each
  // store instruction covers one contiguous run of a tile row instead of
  // scattering 4-byte entries 256 bytes apart.
  constexpr bool buffered = BUF;
  // home positions: lane l holds atom c0 + l of the current chunk of 64, read
  // back by every lane with a scalar readlane (no load latency per home atom)
  double hx = 0.0, hy = 0.0, hz = 0.0;
  for (int32_t b0 = h0; b0 < h1; b0 += kBatch) {
    const int nb = h1 - b0 < kBatch ? h1 - b0 : kBatch;
    if ((b0 - h0) % kWave == 0) {
      const int32_t ih = b0 + lane;
      if (ih < h1) {
        hx = x[3 * (int64_t)ih];
        hy = x[3 * (int64_t)ih + 1];
        hz = x[3 * (int64_t)ih + 2];
      }
    }
    for (int bi = 0; bi < nb; ++bi) {
      const int32_t i = b0 + bi;
      const int src = (b0 - h0) % kWave + bi;
      const double xi = readlane_f64(hx, src), yi = readlane_f64(hy, src),
                   zi = readlane_f64(hz, src);
      int32_t *row = MODE == kTiled ? nbr + (int64_t)(i >> 6) * maxn * kWave + (i & (kWave - 1))
                                    : nullptr;
      const int64_t off = MODE == kCsr ? o.offsets[i] : 0;
      int32_t base = 0;
#pragma unroll
      for (int r = 0; r < SLOTS; ++r) {
        if (r < nslot) {
          double dx = xi - qx[r], dy = yi - qy[r], dz = zi - qz[r];
          if constexpr (WRAP) {
            dx = min_image(dx, L0, iL0);
            dy = min_image(dy, L1, iL1);
            dz = min_image(dz, L2, iL2);
          }
          const double r2 = dist2(dx, dy, dz);
          const bool ok = qj[r] >= 0 && r2 < rl2 && (HALF ? qj[r] > i : qj[r] != i);
          const uint64_t m = __builtin_amdgcn_ballot_w64(ok);
          if (MODE != kCount && ok) {
            const int32_t k = base + (int32_t)__builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if constexpr (MODE == kCsr) {
              if (off + k < o.cap) o.csr[off + k] = qj[r];
            } else if (k < maxn) {
              if (buffered)
                rowbuf[bi * kRowStride + k] = qj[r];
              else
                row[(int64_t)k * kWave] = qj[r];
            }
          }
          base += (int32_t)__popcll(m);
        }
      }
      if (lane == 0) rowcnt[bi] = MODE == kTiled ? (base < maxn ? base : maxn) : base;
      maxc = base > maxc ? base : maxc;
    }
    __syncthreads();  // rowbuf / rowcnt written by other lanes of this one-wavefront block
    if (MODE != kCsr && lane < nb) nnbr[b0 + lane] = rowcnt[lane];
    if (buffered) {
      // lane (a, h) = (lane % kBatch, lane / kBatch) stores rows k = h, h + kFlushRows,
      // ... of batch atom a: every store instruction covers kFlushRows list rows of
      // the whole batch
      const int a = lane % kBatch;
      const int32_t mine = a < nb ? rowcnt[a] : 0;
      const int32_t kmax = wave_max(mine);
      const int32_t i = b0 + a;
      int32_t *row = nbr + (int64_t)(i >> 6) * maxn * kWave + (i & (kWave - 1));
      for (int32_t k = lane / kBatch; k < kmax; k += kFlushRows)
        if (k < mine) row[(int64_t)k * kWave] = rowbuf[a * kRowStride + k];
    }
    __syncthreads();  // before the next batch overwrites rowbuf / rowcnt
  }
}

// The rows of the cell's home atoms from NS staged slots (slots from nslot on are
// empty: they never hit).  Per home atom, in two passes over the slots:
//   1. the integer test of every candidate; the lane masks of the hits stay in scalar
//      registers, and one running minimum notes whether any pair fell between the two
//      thresholds (then, about once in thirteen atoms, those pairs take the FP64 test);
//   2. with every mask known, and so the row's length and every slot's place in it, the
//      stores, without a capacity test per slot.
// What bounds it: the scalar unit, one instruction per cycle for the compute unit's
// four SIMDs, issued 100 M instructions against 76 M vector ones when each slot was
// tested, corrected, counted, checked against maxn and stored before the next (22
// scalar instructions per slot, now about 10).  Tiled lists (us), that -> this with the
// grouped staging of build_quant: 500,000 atoms full 211.8 -> 171.1, half 176.9 -> 144.4,
// 110,447 70.4 -> 56.1, 32,000 39.3 -> 31.3, 512,000 SPH particles (dense shape) 323 -> 263;
// compressed rows of 131,072 atoms (count and fill) 119 -> 99.5.
template <bool HALF, bool BUF, int NS, int SLOTS, int ROWCAP, int MODE>
__device__ __forceinline__ void quant_rows(const BoxK &b, const QuantK &q, const double *cc,
                                           double rl2, const double *__restrict__ x, int32_t h0,
                                           int32_t h1, int32_t tc, const int32_t (&qxy)[SLOTS],
                                           const int32_t (&qz)[SLOTS],
                                           const int32_t (&qj)[SLOTS], const BuildOut &o,
                                           int32_t *rowbuf, int32_t *rowcnt, int32_t &maxc) {
  const int32_t maxn = o.maxn;
  int32_t *__restrict__ nbr = o.nbr;
  int32_t *__restrict__ nnbr = o.nnbr;
  const int lane = threadIdx.x & (kWave - 1);
  constexpr int kRowStride = ROWCAP + 1;
  const uint32_t band = (uint32_t)(q.t_out - q.t_in), inside = 0u - (uint32_t)q.t_in;
  int32_t hxy = 0, huz = 0;  // lattice coordinates of home atom c0 + lane
  int32_t c0 = h0 - kWave;
  for (int32_t b0 = h0; b0 < h1; b0 += kBatch) {
    const int nb = h1 - b0 < kBatch ? h1 - b0 : kBatch;
    if (b0 + kBatch - c0 > kWave) {
      c0 = b0;
      const int32_t ih = b0 + lane;
      if (ih < h1)  // a staged candidate: in range
        quantize(x + 3 * (int64_t)ih, cc, b, q.invq, hxy, huz);
    }
    for (int bi = 0; bi < nb; ++bi) {
      const int32_t i = b0 + bi;
      const int src = i - c0;
      const short2v ui = __builtin_bit_cast(short2v, __builtin_amdgcn_readlane(hxy, src));
      const int32_t uzi = __builtin_amdgcn_readlane(huz, src);
      const int32_t tself = tc + (i - h0);  // candidate number of atom i
      const uint64_t self = 1ull << (tself & (kWave - 1));
      // squared lattice distance of slot r's candidate minus t_in (modulo 2^32)
      auto above_in = [&](int r) {
        const short2v d = __builtin_bit_cast(short2v, qxy[r]) - ui;
        const int32_t dz = qz[r] - uzi;
        return (uint32_t)__builtin_amdgcn_sdot2(d, d, __mul24(dz, dz) - q.t_in, false);
      };
      uint64_t m[NS];
      uint32_t least = ~0u;
#pragma unroll
      for (int r = 0; r < NS; ++r) {
        const uint32_t v = above_in(r);
        m[r] = __builtin_amdgcn_ballot_w64(v >= inside);
        least = v < least ? v : least;
      }
      if (__builtin_amdgcn_ballot_w64(least <= band) != 0) {
        // the FP64 test with the minimum image for the pairs near rlist: each lane's
        // such slots, one per round (a second round is rare)
        uint32_t left = 0, hit = 0;
#pragma unroll
        for (int r = 0; r < NS; ++r) left |= above_in(r) <= band ? 1u << r : 0u;
        const double xi = x[3 * (int64_t)i], yi = x[3 * (int64_t)i + 1],
                     zi = x[3 * (int64_t)i + 2];
        do {
          const uint32_t bit = left & (0u - left);
          int32_t j = i;
#pragma unroll
          for (int r = 0; r < NS; ++r) j = bit == 1u << r ? qj[r] : j;
          const double *p = x + 3 * (int64_t)j;
          const double dx = min_image(xi - p[0], b.L[0], b.invL[0]);
          const double dy = min_image(yi - p[1], b.L[1], b.invL[1]);
          const double dzz = min_image(zi - p[2], b.L[2], b.invL[2]);
          hit |= dist2(dx, dy, dzz) < rl2 ? bit : 0u;
          left ^= bit;
        } while (__builtin_amdgcn_ballot_w64(left != 0) != 0);
#pragma unroll
        for (int r = 0; r < NS; ++r) m[r] |= __builtin_amdgcn_ballot_w64((hit & 1u << r) != 0);
      }
      // the candidates that may be neighbours at all: j > i, or all but atom i itself
#pragma unroll
      for (int r = 0; r < NS; ++r) {
        if constexpr (HALF)
          m[r] &= __builtin_amdgcn_ballot_w64(qj[r] > i);
        else
          m[r] &= r == (tself >> 6) ? ~self : ~0ull;
      }
      int32_t total = 0;
#pragma unroll
      for (int r = 0; r < NS; ++r) total += (int32_t)__popcll(m[r]);
      if constexpr (MODE == kCount) {
        if (o.hits) {  // uniform
          uint32_t mine = 0;
#pragma unroll
          for (int r = 0; r < NS; ++r)
            mine |= __builtin_amdgcn_inverse_ballot_w64(m[r]) ? 1u << r : 0u;
          o.hits[(int64_t)i * kWave + lane] = (uint16_t)mine;
        }
      }
      if constexpr (MODE != kCount) {
        int32_t *row = MODE == kTiled ? nbr + (int64_t)(i >> 6) * maxn * kWave + (i & (kWave - 1))
                                      : nullptr;
        const int64_t off = MODE == kCsr ? o.offsets[i] : 0;
        // entry of this lane's hit in slot r of a row that starts at `first`
        auto entry = [&](int r, int32_t first) {
          return (int32_t)__builtin_amdgcn_mbcnt_hi(
              (uint32_t)(m[r] >> 32),
              __builtin_amdgcn_mbcnt_lo((uint32_t)m[r], (uint32_t)first));
        };
        const bool room = MODE == kCsr ? off + total <= o.cap : total <= maxn;  // uniform
        int32_t base = 0;
        if (room) {
          int32_t *out = BUF ? rowbuf + bi * kRowStride : (MODE == kCsr ? o.csr + off : row);
#pragma unroll
          for (int r = 0; r < NS; ++r) {
            if (__builtin_amdgcn_inverse_ballot_w64(m[r])) {
              const int32_t k = entry(r, base);
              out[BUF || MODE == kCsr ? (int64_t)k : (int64_t)k * kWave] = qj[r];
            }
            base += (int32_t)__popcll(m[r]);
          }
        } else {
#pragma unroll
          for (int r = 0; r < NS; ++r) {
            if (__builtin_amdgcn_inverse_ballot_w64(m[r])) {
              const int32_t k = entry(r, base);
              if constexpr (MODE == kCsr) {
                if (off + k < o.cap) o.csr[off + k] = qj[r];
              } else if (k < maxn) {
                if (BUF)
                  rowbuf[bi * kRowStride + k] = qj[r];
                else
                  row[(int64_t)k * kWave] = qj[r];
              }
            }
            base += (int32_t)__popcll(m[r]);
          }
        }
      }
      if (lane == 0) rowcnt[bi] = MODE == kTiled ? (total < maxn ? total : maxn) : total;
      maxc = total > maxc ? total : maxc;
    }
    __syncthreads();  // rowbuf / rowcnt written by other lanes of this one-wavefront block
    if (MODE != kCsr && lane < nb) nnbr[b0 + lane] = rowcnt[lane];
    if (BUF) {
      const int a = lane % kBatch;
      const int32_t mine = a < nb ? rowcnt[a] : 0;
      const int32_t kmax = wave_max(mine);
      const int32_t i = b0 + a;
      int32_t *row = nbr + (int64_t)(i >> 6) * maxn * kWave + (i & (kWave - 1));
      for (int32_t k = lane / kBatch; k < kmax; k += kFlushRows)
        if (k < mine) row[(int64_t)k * kWave] = rowbuf[a * kRowStride + k];
    }
    __syncthreads();  // before the next batch overwrites rowbuf / rowcnt
  }
}

// Register-staged build with the integer pre-test (QuantK): three registers
// per slot (packed x/y lattice coordinates, z, index) instead of seven.  Same
// rows in the same order as build_staged.  Returns false, having written
// nothing, when a staged coordinate or a home atom is outside the bounds the
// pre-test needs (positions outside the box); the caller then takes the
// unstaged path.
template <bool HALF, bool BUF, int SLOTS, int ROWCAP, int MODE>
__device__ __forceinline__ bool build_quant(const BoxK &b, const QuantK &q, const double *cc,
                                            double rl2, const double *__restrict__ x, int32_t h0,
                                            int32_t h1, int32_t total, int nslot,
                                            const int32_t *rs, const int32_t *pre,
                                            const BuildOut &o, int32_t *rowbuf, int32_t *rowcnt,
                                            int32_t &maxc) {
  static_assert(!BUF || MODE == kTiled, "rows are buffered only for the tiled list");
  const int lane = threadIdx.x & (kWave - 1);
  int32_t qxy[SLOTS], qz[SLOTS], qj[SLOTS];
  bool good = true;
  // Slots are staged in pairs, the loads of a pair in flight together (fours take as long
  // in a liquid and 4 to 7 % longer in a gas); a lane's candidate numbers grow by 64 per
  // slot, so its range is found from the last one.
  constexpr int kGroup = 2;
  int sr = 0;
#pragma unroll
  for (int r0 = 0; r0 < SLOTS; r0 += kGroup) {
    if (r0 < nslot) {  // uniform
      double p[kGroup][3];
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const int32_t t = (r0 + u) * kWave + lane;
        const int32_t tt = t < total ? t : total - 1;
        while (tt >= pre[sr + 1]) ++sr;
        const int32_t j = rs[sr] + (tt - pre[sr]);
        const double *xj = x + 3 * (int64_t)j;
        p[u][0] = xj[0];
        p[u][1] = xj[1];
        p[u][2] = xj[2];
        qj[r0 + u] = t < total ? j : -1;
      }
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const int r = r0 + u;
        const bool in = quantize(p[u], cc, b, q.invq, qxy[r], qz[r]);
        good = good && in;  // spare lanes repeat the last candidate
        qz[r] = qj[r] >= 0 ? qz[r] : kQuantEmpty;
        qxy[r] = qj[r] >= 0 ? qxy[r] : 0;
      }
    } else {
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        qj[r0 + u] = -1;
        qxy[r0 + u] = 0;
        qz[r0 + u] = kQuantEmpty;
      }
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u)  // keep the groups apart: fewer registers
      asm volatile("" : "+v"(qxy[r0 + u]), "+v"(qz[r0 + u]), "+v"(qj[r0 + u]));
  }
  for (int32_t c0 = h0; c0 < h1; c0 += kWave) {
    const int32_t ih = c0 + lane;
    if (ih < h1) {
      const double *p = x + 3 * (int64_t)ih;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        good = good && __builtin_fabs(min_image(p[k] - cc[k], b.L[k], b.invL[k])) <= q.home[k];
    }
  }
  if (__builtin_amdgcn_ballot_w64(!good) != 0) return false;
  // candidate number of home atom h0: the home cell lies in one stencil range
  // (ranges are disjoint on grids of 3 or more cells per dimension)
  int32_t tc = 0;
  for (int sr = 0; pre[sr] < total; ++sr)
    if (rs[sr] <= h0 && h0 < rs[sr] + (pre[sr + 1] - pre[sr])) tc = pre[sr] + (h0 - rs[sr]);
  tc = __builtin_amdgcn_readfirstlane(tc);
  // the code for the fewest slots that hold the stencil: no test of every slot's number
  const bool few = gridDim.x >= kFewSlotGrid;
#define LJMD_ROWS(NS)                                                                          \
  quant_rows<HALF, BUF, NS, SLOTS, ROWCAP, MODE>(b, q, cc, rl2, x, h0, h1, tc, qxy, qz, qj, o, \
                                                 rowbuf, rowcnt, maxc)
  if (few && nslot <= SLOTS - 10)
    LJMD_ROWS(SLOTS - 10);
  else if (few && nslot <= SLOTS - 8)
    LJMD_ROWS(SLOTS - 8);
  else if (nslot <= SLOTS - 6)
    LJMD_ROWS(SLOTS - 6);
  else if (nslot <= SLOTS - 4)
    LJMD_ROWS(SLOTS - 4);
  else if (nslot == SLOTS - 3)
    LJMD_ROWS(SLOTS - 3);
  else if (nslot == SLOTS - 2)
    LJMD_ROWS(SLOTS - 2);
  else
    LJMD_ROWS(SLOTS);
#undef LJMD_ROWS
  return true;
}

// Compressed rows from the hits that the counting pass noted: no positions, no tests.
// Count, scan and fill together (us), testing twice -> this: 32,000 atoms 55.7 -> 46.3,
// 131,072 99.2 -> 86.3, 500,000 282 -> 229 (4,000, whose stencils take the dense
// shape, 125 -> 28.5).  With a capacity test at every store instead
// of ROOM 91.7 and 248.
// ROOM: all rows of the block end within cap.
template <int NS, bool ROOM, int SLOTS>
__device__ __forceinline__ void fill_rows(const int32_t (&qj)[SLOTS], int32_t h0, int32_t h1,
                                          const BuildOut &o) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint16_t *__restrict__ hits = o.hits + (int64_t)h0 * kWave + lane;
  uint32_t next = *hits;
  int64_t at = o.offsets[h0];
  for (int32_t i = h0; i < h1; ++i) {
    const uint32_t mine = next;
    hits += kWave;
    if (i + 1 < h1) next = *hits;  // in flight while this row is written
    int32_t *row = o.csr + at;
    int32_t base = 0;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const bool hit = (mine >> r & 1u) != 0;
      const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
      if (hit) {
        const uint32_t k = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
        if (ROOM || at + k < o.cap) row[k] = qj[r];
      }
      base += (int32_t)__popcll(m);
    }
    at += base;
  }
}

// The candidates' indices, then fill_rows with the code for the fewest slots.
template <int SLOTS>
__device__ __forceinline__ void fill_from_hits(int32_t h0, int32_t h1, int32_t total, int nslot,
                                                const int32_t *rs, const int32_t *pre,
                                                const BuildOut &o) {
  const int lane = threadIdx.x & (kWave - 1);
  int32_t qj[SLOTS];
  int sr = 0;
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    const int32_t t = r * kWave + lane, tt = t < total ? t : total - 1;
    while (tt >= pre[sr + 1]) ++sr;
    qj[r] = rs[sr] + (tt - pre[sr]);
  }
  const bool room = o.offsets[h1] <= o.cap;  // uniform
  const bool few = gridDim.x >= kFewSlotGrid;
#define LJMD_FILL(NS) \
  room ? fill_rows<NS, true>(qj, h0, h1, o) : fill_rows<NS, false>(qj, h0, h1, o)
  if (few && nslot <= SLOTS - 10)
    LJMD_FILL(SLOTS - 10);
  else if (few && nslot <= SLOTS - 8)
    LJMD_FILL(SLOTS - 8);
  else if (nslot <= SLOTS - 6)
    LJMD_FILL(SLOTS - 6);
  else if (nslot <= SLOTS - 4)
    LJMD_FILL(SLOTS - 4);
  else if (nslot == SLOTS - 3)
    LJMD_FILL(SLOTS - 3);
  else if (nslot == SLOTS - 2)
    LJMD_FILL(SLOTS - 2);
  else
    LJMD_FILL(SLOTS);
#undef LJMD_FILL
}

// Block -> (home cell, part): part p of nsplit takes the cell's home atoms
// [len p / nsplit, len (p + 1) / nsplit) (each part stages the whole stencil).
// QUANT: integer pre-test (grids of 3 or more cells per dimension).
// FP64-staged kernel (smaller grids): the standard shape asks for 4 resident
// wavefronts per SIMD (at most 128 VGPRs: the full-list build needs 131 and
// keeps 3 otherwise; 2 registers spill), which took the 500k build from 299.5
// to 259.6 us when this kernel served every grid; the dense shape asks for 3
// (179 VGPRs otherwise, no spills at 166).
// QUANT asks for 6 (80 VGPRs instead of 84), its count-only and compressed-row passes for
// 7, the dense shape for 5: 500,000 atoms full 181.6 -> 172.7 us, dense 274.7 -> 267;
// counting and filling 131,072 atoms 110 -> 99; 7 for the tiled rows spills and loses on
// small grids.
constexpr int quant_occupancy(int slots, int mode) {
  return slots > kSlots ? 5 : (mode == kTiled ? 6 : 7);
}
template <int SLOTS>
constexpr int build_occupancy() { return SLOTS <= kSlots ? 4 : 3; }

template <bool HALF, int SLOTS, int ROWCAP, int MODE = kTiled, bool QUANT = false>
__global__ __launch_bounds__(kWave, QUANT ? quant_occupancy(SLOTS, MODE) : build_occupancy<SLOTS>())
void k_build(GridK g, BoxK b, double rl2, const double *__restrict__ x,
             const int32_t *__restrict__ cell_start, BuildOut o, int32_t *__restrict__ max_count,
             int nsplit, QuantK q) {
  const int32_t maxn = o.maxn;
  __shared__ int32_t rs[27];
  __shared__ int32_t pre[28];
  __shared__ int32_t rowbuf[kBatch * (ROWCAP + 1)];
  __shared__ int32_t rowcnt[kBatch];
  const int lane = threadIdx.x;
  const int32_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int32_t c = blk / nsplit;
  const int part = blk - c * nsplit;
  const int32_t c0 = cell_start[c], clen = cell_start[c + 1] - c0;
  const int32_t h0 = c0 + (int32_t)(((int64_t)clen * part) / nsplit);
  const int32_t h1 = c0 + (int32_t)(((int64_t)clen * (part + 1)) / nsplit);
  if (h0 == h1) return;
  const int S = stencil_ranges(g, c, cell_start, rs, pre);
  const int32_t total = pre[S];
  const int nslot = (total + kWave - 1) / kWave;
  int32_t maxc = 0;
  if constexpr (MODE == kCsr && QUANT) {
    if (o.hits && nslot <= SLOTS) {
      fill_from_hits<SLOTS>(h0, h1, total, nslot, rs, pre, o);
      return;
    }
  }
  // A home cell whose stencil does not wrap (nc >= 4 and the cell is not on a
  // face) pairs atoms at most two cell edges = L/2 apart per dimension: the raw
  // displacement is then the minimum image for every pair that can be inside
  // rlist, and any pair at ~L/2 is beyond rlist whichever image is taken.
  bool wrap = false;
  {
    const int32_t cc[3] = {c % g.nc[0], (c / g.nc[0]) % g.nc[1], c / (g.nc[0] * g.nc[1])};
    for (int k = 0; k < 3; ++k)
      wrap |= g.nc[k] < 4 || cc[k] == 0 || cc[k] == g.nc[k] - 1;
  }
  bool staged = false;
  if constexpr (QUANT) {
    if (nslot <= SLOTS) {
      const int32_t cc3[3] = {c % g.nc[0], (c / g.nc[0]) % g.nc[1], c / (g.nc[0] * g.nc[1])};
      const double cc[3] = {(cc3[0] + 0.5) * g.h[0], (cc3[1] + 0.5) * g.h[1],
                            (cc3[2] + 0.5) * g.h[2]};
#define LJMD_QUANT(B)                                                                            \
  build_quant<HALF, B, SLOTS, ROWCAP, MODE>(b, q, cc, rl2, x, h0, h1, total, nslot, rs, pre, o, \
                                            rowbuf, rowcnt, maxc)
      if constexpr (MODE == kTiled)
        staged = maxn <= ROWCAP ? LJMD_QUANT(true) : LJMD_QUANT(false);
      else
        staged = LJMD_QUANT(false);
#undef LJMD_QUANT
    }
  } else if (nslot <= SLOTS) {
    staged = true;
#define LJMD_STAGED(W, B)                                                                     \
  build_staged<HALF, W, B, SLOTS, ROWCAP, MODE>(b, rl2, x, h0, h1, total, nslot, rs, pre, o, \
                                                rowbuf, rowcnt, maxc)
    if constexpr (MODE == kTiled) {
      if (maxn <= ROWCAP) {
        if (wrap) LJMD_STAGED(true, true); else LJMD_STAGED(false, true);
      } else {
        if (wrap) LJMD_STAGED(true, false); else LJMD_STAGED(false, false);
      }
    } else {
      if (wrap) LJMD_STAGED(true, false); else LJMD_STAGED(false, false);
    }
#undef LJMD_STAGED
  }
  if (!staged) {
    const double L0 = b.L[0], L1 = b.L[1], L2 = b.L[2];
    const double iL0 = b.invL[0], iL1 = b.invL[1], iL2 = b.invL[2];
    for (int32_t i = h0; i < h1; ++i) {
      const double xi = x[3 * (int64_t)i], yi = x[3 * (int64_t)i + 1], zi = x[3 * (int64_t)i + 2];
      int32_t *row = MODE == kTiled
                         ? o.nbr + (int64_t)(i >> 6) * maxn * kWave + (i & (kWave - 1))
                         : nullptr;
      const int64_t off = MODE == kCsr ? o.offsets[i] : 0;
      int32_t base = 0;
      uint32_t mine = 0;  // kCount: the lane's hits by slot
      for (int r = 0; r < nslot; ++r) {
        const int32_t t = r * kWave + lane;
        bool ok = false;
        int32_t j = -1;
        if (t < total) {
          j = locate(t, rs, pre);
          const double dx = min_image(xi - x[3 * (int64_t)j], L0, iL0);
          const double dy = min_image(yi - x[3 * (int64_t)j + 1], L1, iL1);
          const double dz = min_image(zi - x[3 * (int64_t)j + 2], L2, iL2);
          ok = dist2(dx, dy, dz) < rl2 && (HALF ? j > i : j != i);
        }
        const uint64_t m = __ballot(ok);
        if constexpr (MODE == kCount && QUANT) mine |= ok && r < SLOTS ? 1u << r : 0u;
        if (MODE != kCount && ok) {
          const int32_t k = base + (int32_t)__builtin_amdgcn_mbcnt_hi(
                                       (uint32_t)(m >> 32),
                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          if constexpr (MODE == kCsr) {
            if (off + k < o.cap) o.csr[off + k] = j;
          } else if (k < maxn) {
            row[(int64_t)k * kWave] = j;
          }
        }
        base += (int32_t)__popcll(m);
      }
      if constexpr (MODE == kCount && QUANT)
        if (o.hits) o.hits[(int64_t)i * kWave + lane] = (uint16_t)mine;
      if (MODE != kCsr && lane == 0) o.nnbr[i] = MODE == kTiled ? (base < maxn ? base : maxn) : base;
      maxc = base > maxc ? base : maxc;
    }
  }
  // Every wavefront's atomic on the one max_count word is serialised (≈ 11 ns
  // each, 24,389 of them at 500,000 atoms): add only a maximum above the one
  // already there (the value only grows, so a skipped one is never the largest).
  if (lane == 0 && max_count) {
    const int32_t seen = __hip_atomic_load(max_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (maxc > seen) atomicMax(max_count, maxc);
  }
}

// Parts per home cell: grids of fewer than 2,048 cells (two wavefronts per
// SIMD) split each cell's home atoms over up to 8 wavefronts.  Measured (us):
// 32,000 atoms (1,331 cells) 60.9 -> 43.4 with 2 parts (3: 48.5); 256 atoms
// (8 cells) 32.0 -> 11.0 with 8; at 256,000 and 500,000 atoms (12,167 and
// 24,389 cells) 2 parts cost 10-14 %.
constexpr int64_t kSplitCells = 2048;
constexpr int kMaxSplit = 8;

int build_split(int64_t ncells) {
  if (ncells >= kSplitCells) return 1;
  const int64_t s = (kSplitCells + ncells - 1) / ncells;
  return (int)(s < kMaxSplit ? s : kMaxSplit);
}

// Lattice and thresholds of the integer pre-test for this grid and cutoff.
QuantK make_quant(const GridK &g, const BoxK &b, double rl2) {
  const double h = fmax(g.h[0], fmax(g.h[1], g.h[2]));
  QuantK q;
  q.invq = kQuantSpan / (1.5 * h);
  const double R = sqrt(rl2) * q.invq;  // <= kQuantSpan / 1.5: cell edges exceed rlist
  q.t_in = (int32_t)floor((R - 1.75) * (R - 1.75));
  q.t_out = (int32_t)ceil((R + 1.75) * (R + 1.75));
  for (int k = 0; k < 3; ++k) q.home[k] = (0.5 * b.L[k] - sqrt(rl2)) * (1.0 - 1e-12);
  return q;
}

template <bool HALF, int SLOTS, int ROWCAP, int MODE>
void launch_shape(const GridK &g, const BoxK &b, double rl2, const double *x,
                  const int32_t *cell_start, const BuildOut &o, int32_t *max_count, int ns,
                  hipStream_t st) {
  const unsigned nblk = (unsigned)(g.ncells * ns);
  if (g.nc[0] >= 3 && g.nc[1] >= 3 && g.nc[2] >= 3)
    k_build<HALF, SLOTS, ROWCAP, MODE, true><<<nblk, kWave, 0, st>>>(
        g, b, rl2, x, cell_start, o, max_count, ns, make_quant(g, b, rl2));
  else
    k_build<HALF, SLOTS, ROWCAP, MODE, false><<<nblk, kWave, 0, st>>>(
        g, b, rl2, x, cell_start, o, max_count, ns, QuantK{});
}

template <int MODE>
void launch_mode(const GridK &g, const BoxK &b, double rl2, bool half, int64_t n, const double *x,
                 const int32_t *cell_start, const BuildOut &o, int32_t *max_count,
                 hipStream_t st) {
  const int ns = build_split(g.ncells);
  const bool few = mean_stencil_within(g.nc, n, kStandardCandidates);
  if (few && (MODE != kTiled || o.maxn <= kRowCap)) {
    if (half)
      launch_shape<true, kSlots, kRowCap, MODE>(g, b, rl2, x, cell_start, o, max_count, ns, st);
    else
      launch_shape<false, kSlots, kRowCap, MODE>(g, b, rl2, x, cell_start, o, max_count, ns, st);
  } else {
    if (half)
      launch_shape<true, kDenseSlots, kDenseRowCap, MODE>(g, b, rl2, x, cell_start, o, max_count,
                                                          ns, st);
    else
      launch_shape<false, kDenseSlots, kDenseRowCap, MODE>(g, b, rl2, x, cell_start, o, max_count,
                                                           ns, st);
  }
}

}  // namespace

int launch_offsets(int64_t n, const int32_t *counts, int64_t *offsets, void *ws, hipStream_t st);
size_t csr_workspace(int64_t n);

// Compressed rows straight from the cells: a counting pass (true row lengths),
// their exclusive scan into offsets (offsets[n] = total), then a filling pass
// that writes row i at csr[offsets[i] ..] (entries at or beyond cap dropped:
// the caller compares offsets[n] with cap and builds again with more room).
//
// With the full workspace the counting pass also notes every lane's hits (two bytes, so
// 128 per atom) and the filling pass reads them instead of testing again; with less,
// down to build_csr_min_workspace, it tests again.
static_assert(kSlots <= 16 && kDenseSlots <= 16, "one bit per slot");
constexpr size_t align256(size_t b) { return (b + 255) / 256 * 256; }

size_t build_csr_min_workspace(int64_t n) {
  return align256((size_t)(n > 0 ? n : 1) * sizeof(int32_t)) + csr_workspace(n);
}

size_t build_csr_workspace(int64_t n) {
  return align256(build_csr_min_workspace(n)) +
         (size_t)(n > 0 ? n : 1) * kWave * sizeof(uint16_t);
}

int launch_build_csr(const GridK &g, const BoxK &b, double rlist, int kind, int64_t n,
                     const double *x, const int32_t *cell_start, int64_t *offsets, int32_t *csr,
                     int64_t cap, void *ws, size_t ws_bytes, hipStream_t st) {
  int32_t *counts = (int32_t *)ws;
  void *scan_ws = (char *)ws + align256((size_t)(n > 0 ? n : 1) * sizeof(int32_t));
  const double rl2 = rlist * rlist;
  const bool half = kind == LJMD_HALF;
  BuildOut o{};
  o.nnbr = counts;
  o.maxn = 1;
  if (ws_bytes >= build_csr_workspace(n))
    o.hits = (uint16_t *)((char *)ws + align256(build_csr_min_workspace(n)));
  if (n > 0) launch_mode<kCount>(g, b, rl2, half, n, x, cell_start, o, nullptr, st);
  const int rc = launch_offsets(n, counts, offsets, scan_ws, st);
  if (rc != LJMD_OK) return rc;
  if (n > 0) {
    o.offsets = offsets;
    o.csr = csr;
    o.cap = cap;
    launch_mode<kCsr>(g, b, rl2, half, n, x, cell_start, o, nullptr, st);
  }
  return check_launch("ljmd_build_neighbors_csr");
}

int launch_build(const GridK &g, const BoxK &b, double rlist, int kind, int64_t n, const double *x,
                 const int32_t *cell_start, int32_t maxn, int32_t *nbr, int32_t *nnbr,
                 int32_t *max_count, hipStream_t st) {
  k_fill_scalar<<<1, 1, 0, st>>>(max_count, 0);
  if (n > 0) {
    BuildOut o{};
    o.nbr = nbr;
    o.nnbr = nnbr;
    o.maxn = maxn;
    launch_mode<kTiled>(g, b, rlist * rlist, kind == LJMD_HALF, n, x, cell_start, o, max_count, st);
  }
  return check_launch("ljmd_build_neighbors");
}

}  // namespace ljmd
