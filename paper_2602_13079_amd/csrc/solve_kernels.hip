// Solve-phase kernels (gfx950, wave64): everything here is sparse or
// vector work bound by HBM bandwidth, so no matrix cores are used.
//
// A product takes the form of its matrix: diagonal slices, one row per thread
// (k_slices); row blocks whose entries are streamed and whose products are
// summed from LDS, the operand staged there too (k_csr_rows_tiled) or gathered
// (k_csr_rows); a group of lanes per row for what fits neither (k_csr).  Each
// fuses the row's epilogue (residual, Chebyshev update, transfer accumulation),
// so each vector is read and written once per step, and each takes the same
// step of several independent fields in one launch.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "hbgs_internal.h"

namespace hbgs {
namespace solve {

constexpr int BLK = 256;

const char* kind_names[K_COUNT] = {
    "spmv_outer", "spmv_resid", "cheb_pre",  "cheb_post_a", "cheb_post_b", "cheb_other", "resid", "restrict",
    "prolong",    "coarse",     "couple",    "dot1",        "upd_dot2",    "reduce",
    "givens",     "scale",      "xupdate",   "permute",     "cheb_pre_c", "cheb_post_a_c", "cheb_post_b_c",
    "cheb_other_c", "resid_c",  "restrict_c", "prolong_c", "sweep"};

// ---------------------------------------------------------- CSR row engine
template <class T>
__device__ __forceinline__ T lanes_sum(T v, int lpr) {
  for (int off = lpr >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, lpr);
  return v;
}

// column index loaders: plain int32, or packed 16-bit offsets from a base
// per chunk of COL_CHUNK entries (2 bytes per entry instead of 4)
// load4(k, c): the columns of entries k..k+3, k a multiple of 4 (16-byte /
// 8-byte loads; the four share one packed base since 4 divides COL_CHUNK)
struct ColPlain {
  const int* __restrict__ ci;
  __device__ int operator()(int k) const { return ci[k]; }
  __device__ void load4(int k, int* c) const {
    const int4 t = *reinterpret_cast<const int4*>(ci + k);
    c[0] = t.x;
    c[1] = t.y;
    c[2] = t.z;
    c[3] = t.w;
  }
};
struct ColPacked {
  const uint16_t* __restrict__ cd;
  const int* __restrict__ cb;
  __device__ int operator()(int k) const { return cb[k / COL_CHUNK] + (int)cd[k]; }
  __device__ void load4(int k, int* c) const {
    const ushort4 t = *reinterpret_cast<const ushort4*>(cd + k);
    const int b = cb[k / COL_CHUNK];
    c[0] = b + (int)t.x;
    c[1] = b + (int)t.y;
    c[2] = b + (int)t.z;
    c[3] = b + (int)t.w;
  }
};
static_assert(COL_CHUNK % 4 == 0, "a group of four entries shares one packed base");
// values of entries k..k+3 (16-byte loads)
__device__ __forceinline__ void load4(const float* p, float* w) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  w[0] = t.x;
  w[1] = t.y;
  w[2] = t.z;
  w[3] = t.w;
}
__device__ __forceinline__ void load4(const double* p, double* w) {
  const double2 a = *reinterpret_cast<const double2*>(p), b = *reinterpret_cast<const double2*>(p + 2);
  w[0] = a.x;
  w[1] = a.y;
  w[2] = b.x;
  w[3] = b.y;
}

// Up to MAXB jobs (the same operation on several fields' matrices) share one
// launch: job q owns the blocks from first[q] on (UINT_MAX: no such job).
// Independent fields' V-cycles advance together this way, in one stream:
// their small levels fill the chip side by side, and neither events nor a
// second stream's launches stand between a stage and the next.  Against one
// stream per independent chain: the 1M-row mixed solve 5.27 -> 4.57 ms, the
// 4,096-row apply 98 -> 60 us and FP64 solve 1.10 -> 0.67 ms, the 4.2M-row
// solve 11.93 -> 11.82 ms.  Large levels share launches too: fields one after
// the other on levels above 200 MB (so that a pass finds the previous one's
// matrix in the last-level cache) ran 1% slower at 25M rows and for FP64
// applies at 5.3M.
constexpr int MAXB = 4;
template <class D>
struct Batch {
  unsigned rev;  // whole groups of eight blocks to walk backwards (0: forwards)
  unsigned first[MAXB];
  D d[MAXB];
};
// the job of this block (uniform) and the block's index within it
template <class D>
__device__ __forceinline__ const D& batch_job(const Batch<D>& b, int* blk) {
  // A block's first reads are of its arguments, which no cache holds: which
  // job is its own, then that job's fields, one latency after the other.  All
  // lines of the arguments are requested at once instead, with the first (with
  // the row bounds' loads out of their branch: every solve 1.2% faster, of
  // which most are launches of 4-10 us; 4.2M rows mixed 11.53 -> 11.40 ms).
  static_assert(sizeof(Batch<D>) % 4 == 0, "whole words");
  unsigned rev = b.rev;
  const unsigned* words = reinterpret_cast<const unsigned*>(&b);
  unsigned w = 0;
#pragma unroll
  for (int k = 16; k < (int)(sizeof(Batch<D>) / 4); k += 16) w ^= words[k];
  asm("" : "+s"(rev) : "s"(w));  // rev as it is, once the lines are there
  // backwards by groups of eight: the hardware deals consecutive workgroups
  // to the eight XCDs in turn, so a block keeps its XCD (and what the
  // previous pass left in that L2) in either direction
  const unsigned bi = blockIdx.x < 8 * rev ? 8 * (rev - 1 - blockIdx.x / 8) + blockIdx.x % 8 : blockIdx.x;
  int q = 0;
#pragma unroll
  for (int k = 1; k < MAXB; ++k)
    if (bi >= b.first[k]) q = k;
  *blk = (int)(bi - b.first[q]);
  return b.d[q];
}

// a CSR pass of one job: a's rows, the operand x and the rows' epilogue
template <class Col, class TV, class TX, class Epi>
struct CsrJob {
  int n, vec;
  const int* rp;
  Col ci;
  const TV* v;
  const TX* x;
  Epi epi;
};

// acc = sum_k v[k] * x[ci[k]] over row `row`, then epi(row, acc)
template <int LPR, class TV, class TACC, class Col, class TX, class Epi>
__global__ __launch_bounds__(BLK) void k_csr(const Batch<CsrJob<Col, TV, TX, Epi>> batch) {
  int blk;
  const auto& job = batch_job(batch, &blk);
  const int n = job.n;
  const int* __restrict__ rp = job.rp;
  const Col ci = job.ci;
  const TV* __restrict__ v = job.v;
  const TX* __restrict__ x = job.x;
  const Epi epi = job.epi;
  const int lane = threadIdx.x & (LPR - 1);
  const int row = (int)(((int64_t)blk * BLK + threadIdx.x) / LPR);
  if (row >= n) return;
  const int s = rp[row], e = rp[row + 1];
  TACC acc = 0;
  for (int k = s + lane; k < e; k += LPR) acc += (TACC)v[k] * (TACC)x[ci(k)];
  if (LPR > 1) acc = lanes_sum<TACC>(acc, LPR);
  if (lane == 0) epi.store(row, acc, epi.load(row));
}

template <class TACC, class Epi>
__global__ void k_empty(int n, Epi epi) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) epi.store((int)i, TACC(0), epi.load((int)i));
}
// Row-block streaming form for short and medium rows (at most
// ROWS_LDS_BYTES / sizeof(TACC) entries in any block of RB rows).  Block b
// owns rows [RB b, RB (b+1)) and their entries: the
// row epilogues' vector loads and the rows' bounds are issued first, so they
// overlap the entry stream; the threads then stream the entries' values and column indices
// with unit-stride (coalesced) loads, gather the operand and stage the
// products in LDS; finally SBLK/RB lanes per row (or one thread per row when
// RB >= SBLK) sum each row's products from LDS and apply the epilogue.
constexpr int SBLK = 256;
constexpr int ROWS_LDS_BYTES = 16384;
static bool g_vec_entries = true;  // grouped entry loads where the arrays are aligned

// vec: the entry stream in groups of four (16-byte value and 16/8-byte
// column loads) over the block's 4-aligned entries, two groups per step,
// single entries at the two ends; else two single entries per step.  The
// products and their summation order are the same either way.
template <int RB, class TV, class TACC, class Col, class TX, class Epi>
__global__ __launch_bounds__(SBLK) void k_csr_rows(const Batch<CsrJob<Col, TV, TX, Epi>> batch) {
  int blk;
  const auto& job = batch_job(batch, &blk);
  const int n = job.n, vec = job.vec;
  const int* __restrict__ rp = job.rp;
  const Col ci = job.ci;
  const TV* __restrict__ v = job.v;
  const TX* __restrict__ x = job.x;
  const Epi epi = job.epi;
  constexpr int LPR = RB >= SBLK ? 1 : SBLK / RB;  // lanes per row in the row sums
  constexpr int RPT = RB >= SBLK ? RB / SBLK : 1;  // rows per thread
  __shared__ TACC prod[ROWS_LDS_BYTES / sizeof(TACC)];
  const int r0 = blk * RB;
  const int r1 = min(n, r0 + RB);
  const int lane = threadIdx.x & (LPR - 1);
  const int rbase = r0 + (int)threadIdx.x / LPR;
  typename Epi::Pre pre[RPT];
  int rkb[RPT], rke[RPT];  // row bounds for the sums, requested before the barrier
  // (by every lane, rows beyond the block's as its last: a branch around these
  // loads made each of them wait for the one before)
  const int s0 = rp[r0], s1 = rp[r1];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = rbase + q * SBLK;
    pre[q] = epi.load(min(r, r1 - 1));
    rkb[q] = rp[min(r, r1 - 1)];
    rke[q] = rp[min(r, r1 - 1) + 1];
  }
  const int a0 = (s0 + 3) & ~3, a1 = s1 & ~3;  // the 4-aligned middle
  if (vec && a0 < a1) {
    const int t = (int)threadIdx.x;
    // the (at most 3 + 3) entries outside the 4-aligned middle: values and
    // columns requested first, operands gathered after the middle's, so
    // they add no round trip ahead of it (indices clamped into the block)
    const bool hh = s0 + t < a0, ht = a1 + t < s1;
    const int kh = hh ? s0 + t : a0, kt = ht ? a1 + t : a1 - 1;
    const TV vh = v[kh], vt = v[kt];
    const int ch = ci(kh), ct = ci(kt);
    // two groups of four per step, both requested before either is used
    // (a thread without a second group re-reads its first)
    for (int k4 = a0 + 4 * t; k4 < a1; k4 += 8 * SBLK) {
      const int k4b = k4 + 4 * SBLK;
      const bool two = k4b < a1;
      const int kb = two ? k4b : k4;
      TV w0[4], w1[4];
      int c0[4], c1[4];
      load4(v + k4, w0);
      ci.load4(k4, c0);
      load4(v + kb, w1);
      ci.load4(kb, c1);
      TACC x0[4], x1[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x0[q] = (TACC)x[c0[q]];
#pragma unroll
      for (int q = 0; q < 4; ++q) x1[q] = (TACC)x[c1[q]];
#pragma unroll
      for (int q = 0; q < 4; ++q) prod[k4 + q - s0] = (TACC)w0[q] * x0[q];
      if (two)
#pragma unroll
        for (int q = 0; q < 4; ++q) prod[k4b + q - s0] = (TACC)w1[q] * x1[q];
    }
    const TACC xh = (TACC)x[ch], xt = (TACC)x[ct];
    if (hh) prod[kh - s0] = (TACC)vh * xh;
    if (ht) prod[kt - s0] = (TACC)vt * xt;
  } else {
    // two independent entries per step keep more gathers in flight
    int k = s0 + threadIdx.x;
    for (; k + SBLK < s1; k += 2 * SBLK) {
      const int c0 = ci(k), c1 = ci(k + SBLK);
      const TV w0 = v[k], w1 = v[k + SBLK];
      const TACC x0 = (TACC)x[c0], x1 = (TACC)x[c1];
      prod[k - s0] = (TACC)w0 * x0;
      prod[k + SBLK - s0] = (TACC)w1 * x1;
    }
    if (k < s1) prod[k - s0] = (TACC)v[k] * (TACC)x[ci(k)];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = rbase + q * SBLK;
    TACC acc = 0;
    if (r < r1) {
      const int kb = rkb[q] - s0, ke = rke[q] - s0;
      for (int k = kb + lane; k < ke; k += LPR) acc += prod[k];
    }
    if (LPR > 1) acc = lanes_sum<TACC>(acc, LPR);
    if (r < r1 && lane == 0) epi.store(r, acc, pre[q]);
  }
}

// Row-block form with the operand staged in LDS (matrices with operand
// tiles): the block's tiles of TILE_W consecutive operand entries are
// loaded with coalesced loads at the same time as its entries, whose local
// columns (2 bytes each) then index the staged tiles, so no load waits on a
// column index.  The block's entries (at most 4 * SBLK * NG) are held in
// registers across the barrier that publishes the tiles.  Same products,
// LDS positions and row sums as k_csr_rows: bitwise the same result.
template <class TV, class TX, class Epi>
struct TiledJob {
  int n, m, tcnt, prod_bytes;
  const int* rp;
  const uint16_t* lc;
  const int* tiles;
  const TV* v;
  const TX* x;
  Epi epi;
};
template <int RB, class TV, class TACC, class TX, class Epi>
__global__ __launch_bounds__(SBLK) void k_csr_rows_tiled(const Batch<TiledJob<TV, TX, Epi>> batch) {
  int blk;
  const auto& job = batch_job(batch, &blk);
  const int n = job.n, m = job.m, tcnt = job.tcnt, prod_bytes = job.prod_bytes;
  const int* __restrict__ rp = job.rp;
  const uint16_t* __restrict__ lc = job.lc;
  const int* __restrict__ tiles = job.tiles;
  const TV* __restrict__ v = job.v;
  const TX* __restrict__ x = job.x;
  const Epi epi = job.epi;
  constexpr int LPR = RB >= SBLK ? 1 : SBLK / RB;
  constexpr int RPT = RB >= SBLK ? RB / SBLK : 1;
  constexpr int NG = (ROWS_LDS_BYTES / (int)sizeof(TACC)) / (4 * SBLK);  // groups of four per thread
  constexpr int TPP = SBLK / TILE_W;                                      // tiles per pass
  extern __shared__ __align__(16) unsigned char smem[];
  TACC* prod = reinterpret_cast<TACC*>(smem);
  TX* xs = reinterpret_cast<TX*>(smem + prod_bytes);
  const int t = (int)threadIdx.x;
  const int b = blk;
  const int r0 = b * RB, r1 = min(n, r0 + RB);
  const int lane = t & (LPR - 1);
  const int rbase = r0 + t / LPR;
  typename Epi::Pre pre[RPT];
  int rkb[RPT], rke[RPT];
  const int s0 = rp[r0], s1 = rp[r1];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = rbase + q * SBLK;
    pre[q] = epi.load(min(r, r1 - 1));
    rkb[q] = rp[min(r, r1 - 1)];
    rke[q] = rp[min(r, r1 - 1) + 1];
  }
  // the tiles' ids, then their entries (thread t stages element t % TILE_W
  // of tiles t / TILE_W + TPP j)
  const int e = t % TILE_W, j0 = t / TILE_W;
  int id[TILE_MAX / TPP];
#pragma unroll
  for (int j = 0; j < TILE_MAX / TPP; ++j) {
    const int slot = j0 + TPP * j;
    id[j] = slot < tcnt ? tiles[(size_t)b * TILE_MAX + slot] : -1;
  }
  TX xv[TILE_MAX / TPP];
#pragma unroll
  for (int j = 0; j < TILE_MAX / TPP; ++j) {
    const int c = id[j] * TILE_W + e;
    xv[j] = id[j] >= 0 && c < m ? x[c] : TX(0);
  }
  // the entries: the 4-aligned middle [m0, m1) in groups of four, the at
  // most 3 + 3 entries at the ends singly
  const int m0 = min((s0 + 3) & ~3, s1), m1 = max(s1 & ~3, m0);
  const bool hh = s0 + t < m0, ht = m1 + t < s1;
  const int kh = s0 + t, kt = m1 + t;
  const TV vh = hh ? v[kh] : TV(0), vt = ht ? v[kt] : TV(0);
  const int lh = hh ? (int)lc[kh] : 0, lt = ht ? (int)lc[kt] : 0;
  TV w[NG][4];
  int c[NG][4];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int k4 = m0 + 4 * t + 4 * SBLK * g;
    if (k4 < m1) {
      load4(v + k4, w[g]);
      const ushort4 u = *reinterpret_cast<const ushort4*>(lc + k4);
      c[g][0] = u.x;
      c[g][1] = u.y;
      c[g][2] = u.z;
      c[g][3] = u.w;
    }
  }
#pragma unroll
  for (int j = 0; j < TILE_MAX / TPP; ++j)
    if (id[j] >= 0) xs[(j0 + TPP * j) * TILE_W + e] = xv[j];
  __syncthreads();
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int k4 = m0 + 4 * t + 4 * SBLK * g;
    if (k4 < m1)
#pragma unroll
      for (int q = 0; q < 4; ++q) prod[k4 + q - s0] = (TACC)w[g][q] * (TACC)xs[c[g][q]];
  }
  if (hh) prod[kh - s0] = (TACC)vh * (TACC)xs[lh];
  if (ht) prod[kt - s0] = (TACC)vt * (TACC)xs[lt];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = rbase + q * SBLK;
    TACC acc = 0;
    if (r < r1) {
      const int k0 = rkb[q] - s0, k1 = rke[q] - s0;
      for (int k = k0 + lane; k < k1; k += LPR) acc += prod[k];
    }
    if (LPR > 1) acc = lanes_sum<TACC>(acc, LPR);
    if (r < r1 && lane == 0) epi.store(r, acc, pre[q]);
  }
}

// Diagonal slices, one row per thread: the slice's table (wave-uniform,
// scalar loads) gives the columns, so the values and the operand are read
// with unit-stride loads that wait on nothing but the table and the row's
// mask, and neither column indices (2-4 B per entry) nor LDS passes are
// left.  The sums are those of the row-block kernels: products rounded
// before they are added (no contraction), and NACC = lanes per row of the
// row-block form partial sums that take the row's entries in turn; they are
// kept in rotation, which pairs them as that form's shuffles do, since the
// sums of a pair commute.  Absent places are skipped by the mask: their
// operand may be out of range or not finite.
// Bound by memory: at 1,048,576 rows a finest FP32 pass moves 31-48 MB
// against 43-62 MB for the tiled row blocks (no columns, no row pointers) in
// 8.8-10.7 us against 12.7-15.1; the outer product of the 4.2M-row system
// 340 MB against 479 MB in 63 us (5.4 TB/s; a plain copy reaches 6.1)
// against 81; at 262,144 rows 3.6-4.7 us against 4.8-6.4.
template <class TM, class TV, class TX, class Epi>
struct SliceJob {
  int n;
  const int* tab;
  const TM* mask;
  const TV* v;
  const TX* x;
  Epi epi;
};
template <int NACC, class TM, class TV, class TACC, class TX, class Epi>
__global__ __launch_bounds__(BLK) void k_slices(const Batch<SliceJob<TM, TV, TX, Epi>> batch) {
#pragma clang fp contract(off)
  constexpr int CH = 8;  // places whose loads are issued together
  int blk;
  const auto& job = batch_job(batch, &blk);
  const int n = job.n;
  const int* __restrict__ tab = job.tab;
  const TM* __restrict__ mask = job.mask;
  const TV* __restrict__ v = job.v;
  const TX* __restrict__ x = job.x;
  const Epi epi = job.epi;
  const int row = blk * BLK + (int)threadIdx.x;
  if (row >= n) return;
  const int q = __builtin_amdgcn_readfirstlane(row / DIA_ROWS);
  const int* t = tab + (size_t)q * DIA_TS;
  const typename Epi::Pre pre = epi.load(row);
  const uint32_t m = mask[row];
  const int cnt = t[0];
  const TV* vs = v + (size_t)t[DIA_BASE] * DIA_ROWS + (row & (DIA_ROWS - 1));
  TACC acc[NACC];
#pragma unroll
  for (int a = 0; a < NACC; ++a) acc[a] = 0;
  for (int j0 = 0; j0 < cnt; j0 += CH) {
    TV a[CH];
    TX b[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int j = j0 + u;
      if (j < cnt) {
        a[u] = vs[(size_t)j * DIA_ROWS];
        b[u] = x[m >> j & 1u ? row + t[DIA_DIAG + j] : 0];
      } else {
        a[u] = TV(0);
        b[u] = TX(0);
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int j = j0 + u;
      const bool on = j < DIA_MAX && (m >> (j & (DIA_MAX - 1)) & 1u);
      const TACC p = (TACC)a[u] * (TACC)b[u];
      if constexpr (NACC == 1) {
        acc[0] = acc[0] + (on ? p : TACC(0));
      } else {
        const TACC s = acc[0] + p;
#pragma unroll
        for (int c = 0; c + 1 < NACC; ++c) acc[c] = on ? acc[c + 1] : acc[c];
        acc[NACC - 1] = on ? s : acc[NACC - 1];
      }
    }
  }
#pragma unroll
  for (int off = NACC / 2; off > 0; off >>= 1)
#pragma unroll
    for (int c = 0; c < off; ++c) acc[c] = acc[c] + acc[c + off];
  epi.store(row, acc[0], pre);
}

static bool g_tiles_on = true;  // slices, and the LDS-staged operand, where a matrix has them
void set_tiles(bool on) { g_tiles_on = on; }
bool tiles_on() { return g_tiles_on; }

int rows_per_block(const DCsr& a, int cap, bool vec) {
  // the largest RB whose every block's entries fit the LDS staging
  // (blkmax <= cap) and that still gives MIN_BLOCKS blocks, so a coarse
  // level (10^3 - 10^5 rows) spreads over every CU instead of a few hundred
  // blocks; where no RB gives that many, the smallest that fits.  With
  // grouped loads 256-row blocks beat 512-row ones (finest FP32 levels:
  // 13.7 vs 14.3 us at 1M rows); with single loads the larger wins.
  constexpr int64_t MIN_BLOCKS = 1024;  // 4 per CU
  int rb = 0;
  for (int q = vec ? 1 : 0; q < kRowBlocks; ++q) {
    const int r = row_block(q);
    if (a.blkmax[q] <= 0 || a.blkmax[q] > cap) continue;
    rb = r;
    if (((int64_t)a.n + r - 1) / r >= MIN_BLOCKS) break;
  }
  return rb;
}

static unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// one job of a CSR launch: the matrix, the operand, the rows' epilogue
template <class TX, class Epi>
struct Pass {
  const DCsr* a;
  const TX* x;
  Epi epi;
};
// the kernel a matrix takes: passes of one shape can share a launch
struct Shape {
  enum Kind { EMPTY, SLICES, TILED, ROWS, LANES } kind = EMPTY;
  int par = 0;        // rows per block (LANES: lanes per row)
  bool flag = false;  // SLICES: 16-bit masks; ROWS, LANES: packed columns
  int vec = 0;        // ROWS: grouped entry loads
  bool operator==(const Shape& o) const { return kind == o.kind && par == o.par && flag == o.flag && vec == o.vec; }
};
template <class TV>
static const TV* csr_vals(const DCsr& a) {
  if constexpr (sizeof(TV) == sizeof(double))
    return a.v;
  else
    return a.vf;
}
template <class TV>
static const TV* slice_vals(const DCsr& a) {
  if constexpr (sizeof(TV) == sizeof(double))
    return a.dv;
  else
    return a.dvf;
}
static int tile_prod_bytes(const DCsr& a, int rb, int acc_bytes) {
  int q = 0;
  while (row_block(q) != rb) ++q;
  return (a.blkmax[q] * acc_bytes + 15) / 16 * 16;
}
template <class TV, class TACC, class TX>
static Shape shape_of(const DCsr& a) {
  Shape sh;
  if (a.nnz == 0) return sh;  // rows without entries: the epilogue of an empty sum
  constexpr int cap = ROWS_LDS_BYTES / (int)sizeof(TACC);
  if (a.dia_w && g_tiles_on && slice_vals<TV>(a)) {
    const int rb = rows_per_block(a, cap, true);
    if (rb >= 32 && rb <= SBLK) {
      sh.kind = Shape::SLICES;
      sh.par = rb;
      sh.flag = a.dia_m16 != nullptr;
      return sh;
    }
  }
  sh.flag = a.cd != nullptr;
  const bool col_ok = a.cd ? reinterpret_cast<uintptr_t>(a.cd) % 8 == 0 : reinterpret_cast<uintptr_t>(a.ci) % 16 == 0;
  sh.vec = g_vec_entries && reinterpret_cast<uintptr_t>(csr_vals<TV>(a)) % 16 == 0 && col_ok;
  sh.par = rows_per_block(a, cap, sh.vec != 0);
  // the LDS-staged operand where the matrix has tiles for this block size
  // and the staging (products and tiles) takes at most 32 KiB, 5 blocks per
  // CU (at 4.2M DOF the outer SpMV's 21-27 KiB still run faster staged: 95
  // -> 83 us mixed, 102 -> 93 us FP64)
  if (g_tiles_on && sh.vec && a.tile_rb == sh.par && a.lc && (sh.par == 256 || sh.par == 128 || sh.par == 64) &&
      tile_prod_bytes(a, sh.par, (int)sizeof(TACC)) + a.tile_cnt * TILE_W * (int)sizeof(TX) <= 32768) {
    sh.kind = Shape::TILED;
    sh.flag = false;
    return sh;
  }
  if (sh.par) {
    sh.kind = Shape::ROWS;
    return sh;
  }
  sh.kind = Shape::LANES;
  sh.vec = 0;
  const float avg = a.avg_row();
  sh.par = avg <= 1.5f ? 1 : avg <= 3.f ? 2 : avg <= 6.f ? 4 : avg <= 16.f ? 8 : avg <= 64.f ? 16 : avg <= 128.f ? 32 : 64;
  return sh;
}

static Shape shape_for(const DCsr& a, int tv, int tx) {
  if (tv == 4) return shape_of<float, float, float>(a);
  return tx == 4 ? shape_of<double, double, float>(a) : shape_of<double, double, double>(a);
}
void layout_of(const DCsr& a, int tv, int tx, int32_t* out4) {
  const Shape sh = shape_for(a, tv, tx);
  out4[0] = (int32_t)sh.kind;
  out4[1] = sh.par;
  out4[2] = sh.kind == Shape::EMPTY ? 0 : sh.flag || sh.kind == Shape::TILED ? 16 : 32;
  out4[3] = sh.kind == Shape::SLICES ? a.dia_w : 0;
}
double matrix_bytes(const DCsr& a, int tv, int tx) {
  const Shape sh = shape_for(a, tv, tx);
  const double rows = a.n, entries = (double)a.nnz;
  switch (sh.kind) {
    case Shape::EMPTY: return 0.0;
    case Shape::SLICES: {  // values of all places, the rows' masks, the slices' tables
      const double places = (double)a.dia_places, slices = (a.n + DIA_ROWS - 1) / DIA_ROWS;
      return places * tv + rows * (sh.flag ? 2 : 4) + 4.0 * (DIA_DIAG * slices + places / DIA_ROWS);
    }
    case Shape::TILED:
      return entries * (tv + 2) + 4.0 * (rows + 1) + 4.0 * a.tile_cnt * cdiv(a.n, sh.par);
    default:
      return entries * (tv + (sh.flag ? 2 : 4)) + 4.0 * (rows + 1) + (sh.flag ? 4.0 * cdiv(a.nnz, COL_CHUNK) : 0.0);
  }
}

// e0/e1 (optional): events that the dispatch itself stamps with the
// kernel's start and end (no extra packets in the stream), for timing one
// class of launches inside a timed run
template <class K, class B>
static void launch_batch(K kern, unsigned grid, unsigned lds, const B& b, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1) {
  static_assert(BLK == SBLK, "one block size");
  if (e0)
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(BLK), lds, s, e0, e1, 0, b);
  else
    kern<<<grid, BLK, lds, s>>>(b);
  HBGS_HIP(hipGetLastError());
}
// fills a batch's block ranges from `blocks(q)`; returns the grid
template <class B, class F>
static unsigned batch_blocks(B& b, int nj, bool rev, F blocks) {
  unsigned grid = 0;
  for (int q = 0; q < MAXB; ++q) {
    b.first[q] = q < nj ? grid : UINT32_MAX;
    if (q < nj) grid += (unsigned)blocks(q);
  }
  b.rev = rev ? grid / 8 : 0;
  return grid;
}

template <class TM, class TV, class TACC, class TX, class Epi>
static void launch_slices(const Pass<TX, Epi>* const* p, int nj, bool rev, int rb, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1) {
  Batch<SliceJob<TM, TV, TX, Epi>> b;
  for (int q = 0; q < MAXB; ++q) {
    const DCsr& a = *p[q < nj ? q : 0]->a;
    const TM* mask = sizeof(TM) == 2 ? (const TM*)a.dia_m16 : (const TM*)a.dia_m32;
    const Pass<TX, Epi>& j = *p[q < nj ? q : 0];
    b.d[q] = {a.n, a.dia_tab, mask, slice_vals<TV>(a), j.x, j.epi};
  }
  const unsigned grid = batch_blocks(b, nj, rev, [&](int q) { return cdiv(p[q]->a->n, BLK); });
  switch (rb) {
    case 256: launch_batch(k_slices<1, TM, TV, TACC, TX, Epi>, grid, 0, b, s, e0, e1); break;
    case 128: launch_batch(k_slices<2, TM, TV, TACC, TX, Epi>, grid, 0, b, s, e0, e1); break;
    case 64: launch_batch(k_slices<4, TM, TV, TACC, TX, Epi>, grid, 0, b, s, e0, e1); break;
    default: launch_batch(k_slices<8, TM, TV, TACC, TX, Epi>, grid, 0, b, s, e0, e1); break;
  }
}
template <class TV, class TACC, class TX, class Epi>
static void launch_tiled(const Pass<TX, Epi>* const* p, int nj, bool rev, int rb, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1) {
  Batch<TiledJob<TV, TX, Epi>> b;
  unsigned lds = 0;
  for (int q = 0; q < MAXB; ++q) {
    const Pass<TX, Epi>& j = *p[q < nj ? q : 0];
    const DCsr& a = *j.a;
    const int pb = tile_prod_bytes(a, rb, (int)sizeof(TACC));
    lds = std::max(lds, (unsigned)(pb + a.tile_cnt * TILE_W * (int)sizeof(TX)));
    b.d[q] = {a.n, a.m, a.tile_cnt, pb, a.rp, a.lc, a.tiles, csr_vals<TV>(a), j.x, j.epi};
  }
  const unsigned grid = batch_blocks(b, nj, rev, [&](int q) { return cdiv(p[q]->a->n, rb); });
  switch (rb) {
    case 256: launch_batch(k_csr_rows_tiled<256, TV, TACC, TX, Epi>, grid, lds, b, s, e0, e1); break;
    case 128: launch_batch(k_csr_rows_tiled<128, TV, TACC, TX, Epi>, grid, lds, b, s, e0, e1); break;
    default: launch_batch(k_csr_rows_tiled<64, TV, TACC, TX, Epi>, grid, lds, b, s, e0, e1); break;
  }
}
static inline ColPlain col_of(const DCsr& a, ColPlain) { return {a.ci}; }
static inline ColPacked col_of(const DCsr& a, ColPacked) { return {a.cd, a.cb}; }
template <class Col, class TV, class TACC, class TX, class Epi>
static void launch_cols(const Pass<TX, Epi>* const* p, int nj, bool rev, const Shape& sh, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1) {
  Batch<CsrJob<Col, TV, TX, Epi>> b;
  for (int q = 0; q < MAXB; ++q) {
    const Pass<TX, Epi>& j = *p[q < nj ? q : 0];
    b.d[q] = {j.a->n, sh.vec, j.a->rp, col_of(*j.a, Col{}), csr_vals<TV>(*j.a), j.x, j.epi};
  }
  const bool rows = sh.kind == Shape::ROWS;
  const unsigned grid = batch_blocks(b, nj, rev, [&](int q) {
    return rows ? cdiv(p[q]->a->n, sh.par) : cdiv((int64_t)p[q]->a->n * sh.par, BLK);
  });
#define HBGS_KERN(K, N)                                               \
  case N:                                                             \
    launch_batch(K<N, TV, TACC, Col, TX, Epi>, grid, 0, b, s, e0, e1); \
    return;
  if (rows) switch (sh.par) {
      HBGS_KERN(k_csr_rows, 512)
      HBGS_KERN(k_csr_rows, 256)
      HBGS_KERN(k_csr_rows, 128)
      HBGS_KERN(k_csr_rows, 64)
      HBGS_KERN(k_csr_rows, 32)
      HBGS_KERN(k_csr_rows, 16)
      HBGS_KERN(k_csr_rows, 8)
      HBGS_KERN(k_csr_rows, 4)
    }
  else switch (sh.par) {
      HBGS_KERN(k_csr, 1)
      HBGS_KERN(k_csr, 2)
      HBGS_KERN(k_csr, 4)
      HBGS_KERN(k_csr, 8)
      HBGS_KERN(k_csr, 16)
      HBGS_KERN(k_csr, 32)
      HBGS_KERN(k_csr, 64)
    }
#undef HBGS_KERN
}

// the passes of all jobs, as few launches as their shapes allow
template <class TV, class TACC, class TX, class Epi>
static void launch_csr(const Pass<TX, Epi>* jobs, int nj, bool rev, hipStream_t s, hipEvent_t e0 = nullptr,
                       hipEvent_t e1 = nullptr) {
  Shape sh[HBGS_MAX_FIELDS];
  bool done[HBGS_MAX_FIELDS] = {};
  for (int q = 0; q < nj; ++q) {
    done[q] = jobs[q].a->n == 0;
    if (!done[q]) sh[q] = shape_of<TV, TACC, TX>(*jobs[q].a);
  }
  for (int q = 0; q < nj; ++q) {
    if (done[q]) continue;
    if (sh[q].kind == Shape::EMPTY) {
      if (e0) HBGS_HIP(hipEventRecord(e0, s));
      k_empty<TACC, Epi><<<grid_for(jobs[q].a->n, 256), 256, 0, s>>>(jobs[q].a->n, jobs[q].epi);
      HBGS_HIP(hipGetLastError());
      if (e1) HBGS_HIP(hipEventRecord(e1, s));
      continue;
    }
    const Pass<TX, Epi>* p[MAXB];
    int np = 0;
    for (int k = q; k < nj && np < MAXB; ++k)
      if (!done[k] && sh[k] == sh[q]) {
        p[np++] = &jobs[k];
        done[k] = true;
      }
    switch (sh[q].kind) {
      case Shape::SLICES:
        if (sh[q].flag)
          launch_slices<uint16_t, TV, TACC>(p, np, rev, sh[q].par, s, e0, e1);
        else
          launch_slices<uint32_t, TV, TACC>(p, np, rev, sh[q].par, s, e0, e1);
        break;
      case Shape::TILED: launch_tiled<TV, TACC>(p, np, rev, sh[q].par, s, e0, e1); break;
      default:
        if (sh[q].flag)
          launch_cols<ColPacked, TV, TACC>(p, np, rev, sh[q], s, e0, e1);
        else
          launch_cols<ColPlain, TV, TACC>(p, np, rev, sh[q], s, e0, e1);
    }
  }
}
template <class TV, class TACC, class TX, class Epi>
static void launch_csr(const DCsr& a, const TX* x, const Epi& epi, bool rev, hipStream_t s, hipEvent_t e0 = nullptr,
                       hipEvent_t e1 = nullptr) {
  const Pass<TX, Epi> j{&a, x, epi};
  launch_csr<TV, TACC>(&j, 1, rev, s, e0, e1);
}

// Epilogues: load(i) issues the row's vector loads (before the row sum, so
// they overlap it); store(i, acc, pre) finishes the row.
template <class T, class TACC>
struct EpiStore {
  T* __restrict__ y;
  struct Pre {};
  __device__ Pre load(int) const { return {}; }
  __device__ void store(int i, TACC acc, Pre) const { y[i] = (T)acc; }
};
template <class T, class TACC>
struct EpiAdd {
  T* __restrict__ y;
  struct Pre {
    T y;
  };
  __device__ Pre load(int i) const { return {y[i]}; }
  __device__ void store(int i, TACC acc, Pre p) const { y[i] = p.y + (T)acc; }
};
// right-hand side of the next level: y = acc and, when the consumer level
// smooths with degree 2, its first Chebyshev direction d0 = (D^-1 y) / theta
template <class T>
struct EpiRhs {
  T* __restrict__ y;
  const T* __restrict__ dinv;
  T* __restrict__ d0;
  T c0;
  struct Pre {
    T dinv;
  };
  __device__ Pre load(int i) const { return {d0 ? dinv[i] : T(0)}; }
  __device__ void store(int i, T acc, Pre p) const {
    y[i] = acc;
    if (d0) d0[i] = p.dinv * acc * c0;
  }
};
template <class T>
struct EpiResid {
  const T* __restrict__ b;
  T* __restrict__ r;
  struct Pre {
    T b;
  };
  __device__ Pre load(int i) const { return {b[i]}; }
  __device__ void store(int i, T acc, Pre p) const { r[i] = p.b - acc; }
};
// degree-2 pre-smoothing from zero, d0 = (D^-1 b) / theta given:
// x = d0 + c1 d0 + c2 D^-1 (b - A d0)
template <class T>
struct EpiChebPre2 {
  const T* __restrict__ dinv;
  const T* __restrict__ b;
  const T* __restrict__ d0;
  T* __restrict__ x;
  T c1, c2;
  struct Pre {
    T dinv, b, d0;
  };
  __device__ Pre load(int i) const { return {dinv[i], b[i], d0[i]}; }
  __device__ void store(int i, T ad, Pre p) const {
    T r1 = p.b - ad;
    T d1 = c1 * p.d0 + c2 * (p.dinv * r1);
    x[i] = p.d0 + d1;
  }
};
// post-smoothing start from x: r = b - A x, d = D^-1 r / theta
template <class T>
struct EpiChebPostA {
  const T* __restrict__ dinv;
  const T* __restrict__ b;
  T* __restrict__ r;
  T* __restrict__ d;
  T c0;
  struct Pre {
    T dinv, b;
  };
  __device__ Pre load(int i) const { return {dinv[i], b[i]}; }
  __device__ void store(int i, T ax, Pre p) const {
    T ri = p.b - ax;
    r[i] = ri;
    d[i] = p.dinv * ri * c0;
  }
};
// Chebyshev step: r -= A d; dn = c1 d + c2 D^-1 r; x (+ d if pending) += dn
template <class T, bool ADD_D, bool KEEP>
struct EpiChebStep {
  const T* __restrict__ dinv;
  const T* __restrict__ d;
  T* __restrict__ r;
  T* __restrict__ dn;
  T* __restrict__ x;
  T c1, c2;
  struct Pre {
    T dinv, d, r, x;
  };
  __device__ Pre load(int i) const { return {dinv[i], d[i], r[i], x[i]}; }
  __device__ void store(int i, T ad, Pre p) const {
    T ri = p.r - ad;
    T di = c1 * p.d + c2 * (p.dinv * ri);
    T xi = ADD_D ? p.x + p.d : p.x;
    x[i] = xi + di;
    if (KEEP) {
      r[i] = ri;
      dn[i] = di;
    }
  }
};
// coupling: t = (T)v - sum a z, plus the fine level's d0 = (D^-1 t) / theta
template <class T>
struct EpiCouple {
  const double* __restrict__ v;
  T* __restrict__ t;
  const T* __restrict__ dinv;
  T* __restrict__ d0;
  T c0;
  const double* __restrict__ vs;  // divisor of v (null: none)
  struct Pre {
    double v;
    T dinv;
  };
  __device__ Pre load(int i) const { return {vs ? v[i] / *vs : v[i], d0 ? dinv[i] : T(0)}; }
  __device__ void store(int i, T acc, Pre p) const {
    T ti = (T)p.v - acc;
    t[i] = ti;
    if (d0) d0[i] = p.dinv * ti * c0;
  }
};

// rows of the interleaved [A P; P] operator: even row 2i gives
// r_i = r_i - (A P xc)_i and d_i = D^-1 r_i / theta, odd row 2i+1 gives
// x_i = x_i + (P xc)_i
template <class T>
struct EpiPostQ {
  const T* __restrict__ dinv;
  T* __restrict__ r;
  T* __restrict__ x;
  T* __restrict__ d;
  T c0;
  struct Pre {
    T a, b;
  };
  __device__ Pre load(int k) const {
    const int i = k >> 1;
    if (k & 1) return {x[i], T(0)};
    return {r[i], dinv[i]};
  }
  __device__ void store(int k, T acc, Pre p) const {
    const int i = k >> 1;
    if (k & 1) {
      x[i] = p.a + acc;
    } else {
      const T ri = p.a - acc;
      r[i] = ri;
      d[i] = p.b * ri * c0;
    }
  }
};

// group right-hand side of the nested form: t = v / vs - sum a z (FP64 out)
struct EpiSubFrom {
  const double* __restrict__ v;
  double* __restrict__ t;
  const double* __restrict__ vs;  // divisor of v (null: none)
  struct Pre {
    double v;
  };
  __device__ Pre load(int i) const { return {vs ? v[i] / *vs : v[i]}; }
  __device__ void store(int i, double acc, Pre p) const { t[i] = p.v - acc; }
};

// ---------------------------------------------------------- outer SpMV
void spmv_outer_f64(const DCsr& a, const double* x, double* y, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  launch_csr<double, double>(a, x, EpiStore<double, double>{y}, true, s, e0, e1);
}
void spmv_outer_mixed(const DCsr& a, const float* x, double* y, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  launch_csr<double, double>(a, x, EpiStore<double, double>{y}, true, s, e0, e1);
}
template <class TZ>
void couple_f64(const DCsr& a, const double* v, const TZ* z, double* t, const double* vs, hipStream_t s) {
  launch_csr<double, double>(a, z, EpiSubFrom{v, t, vs}, false, s);
}
template void couple_f64<float>(const DCsr&, const double*, const float*, double*, const double*, hipStream_t);
template void couple_f64<double>(const DCsr&, const double*, const double*, double*, const double*, hipStream_t);
void spmv_resid_f64(const DCsr& a, const double* x, const double* b, double* r, hipStream_t s) {
  launch_csr<double, double>(a, x, EpiResid<double>{b, r}, false, s);
}

// ------------------------------------------------------- V-cycle pieces
// Element-wise passes over several jobs' vectors: block blk of a job takes
// its elements [BLK blk, BLK (blk + 1)).
template <class T>
struct InitJob {
  int n;
  const T *dinv, *b;
  T c0;
  T *r, *d, *x;
};
template <class T>
__global__ __launch_bounds__(BLK) void k_cheb_init0(const Batch<InitJob<T>> batch) {
  int blk;
  const auto& j = batch_job(batch, &blk);
  const int64_t i = (int64_t)blk * BLK + threadIdx.x;
  if (i >= j.n) return;
  const T bi = j.b[i];
  const T di = j.dinv[i] * bi * j.c0;
  j.r[i] = bi;
  j.d[i] = di;
  j.x[i] = di;
}
template <class T>
__global__ void k_add(int n, const T* __restrict__ d, T* __restrict__ x) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) x[i] = x[i] + d[i];
}

// jobs -> passes through `make(job)`, then the launches
template <class T, class F>
static void level_pass(const LevelJob<T>* j, int nj, bool rev, hipStream_t s, F make) {
  using P = decltype(make(j[0]));
  P p[HBGS_MAX_FIELDS];
  for (int q = 0; q < nj; ++q) p[q] = make(j[q]);
  launch_csr<T, T>(p, nj, rev, s);
}
template <class T>
void VcOps<T>::pre2(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) {
    return Pass<T, EpiChebPre2<T>>{J.A, J.d, {J.dinv, J.b, J.d, J.x, (T)J.cc->c1[1], (T)J.cc->c2[1]}};
  });
}
template <class T>
void VcOps<T>::init0(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  for (int q0 = 0; q0 < nj; q0 += MAXB) {
    const int m = std::min(MAXB, nj - q0);
    Batch<InitJob<T>> b;
    for (int q = 0; q < MAXB; ++q) {
      const LevelJob<T>& J = j[q0 + (q < m ? q : 0)];
      b.d[q] = {J.A->n, J.dinv, J.b, (T)J.cc->c0, J.r, J.d, J.x};
    }
    const unsigned grid = batch_blocks(b, m, rev, [&](int q) { return cdiv(j[q0 + q].A->n, BLK); });
    launch_batch(k_cheb_init0<T>, grid, 0, b, s, nullptr, nullptr);
  }
}
template <class T>
void VcOps<T>::post_start(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) {
    return Pass<T, EpiChebPostA<T>>{J.A, J.x, {J.dinv, J.b, J.r, J.d, (T)J.cc->c0}};
  });
}
template <class T, bool ADD_D, bool KEEP>
static void cheb_step(const LevelJob<T>* j, int nj, int k, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [k](const LevelJob<T>& J) {
    return Pass<T, EpiChebStep<T, ADD_D, KEEP>>{
        J.A, J.d, {J.dinv, J.d, J.r, J.dn, J.x, (T)J.cc->c1[k], (T)J.cc->c2[k]}};
  });
}
template <class T>
void VcOps<T>::step(const LevelJob<T>* j, int nj, int k, bool add_d, bool keep, bool rev, hipStream_t s) {
  if (add_d && keep)
    cheb_step<T, true, true>(j, nj, k, rev, s);
  else if (add_d)
    cheb_step<T, true, false>(j, nj, k, rev, s);
  else if (keep)
    cheb_step<T, false, true>(j, nj, k, rev, s);
  else
    cheb_step<T, false, false>(j, nj, k, rev, s);
}
template <class T>
void VcOps<T>::add(int n, const T* d, T* x, hipStream_t s) {
  k_add<T><<<grid_for(n, BLK), BLK, 0, s>>>(n, d, x);
  HBGS_HIP(hipGetLastError());
}
template <class T>
void VcOps<T>::resid(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) { return Pass<T, EpiResid<T>>{J.A, J.x, {J.b, J.r}}; });
}
template <class T>
void VcOps<T>::restrict_(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) {
    return Pass<T, EpiRhs<T>>{J.R, J.r, {J.bc, J.dinv_c, J.d0_c, (T)J.c0_c}};
  });
}
template <class T>
void VcOps<T>::prolong(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) { return Pass<T, EpiAdd<T, T>>{J.P, J.xc, {J.x}}; });
}
template <class T>
void VcOps<T>::post_q(const LevelJob<T>* j, int nj, bool rev, hipStream_t s) {
  level_pass<T>(j, nj, rev, s, [](const LevelJob<T>& J) {
    return Pass<T, EpiPostQ<T>>{J.Q, J.xc, {J.dinv, J.r, J.x, J.d, (T)J.cc->c0}};
  });
}
template <class T>
void VcOps<T>::couple(const RhsJob<T>* j, int nj, const T* z, const double* vs, bool rev, hipStream_t s) {
  Pass<T, EpiCouple<T>> p[HBGS_MAX_FIELDS];
  for (int q = 0; q < nj; ++q) p[q] = {j[q].cpl, z, {j[q].v, j[q].t, j[q].dinv, j[q].d0, (T)j[q].c0, vs}};
  launch_csr<T, T>(p, nj, rev, s);
}

template <class T>
struct CastJob {
  int n;
  const double* v;
  T* t;  // null: not wanted
  const T* dinv;
  T c0;
  T* d0;  // null: not wanted
};
template <class T>
__global__ __launch_bounds__(BLK) void k_cast_in(const Batch<CastJob<T>> batch, const double* __restrict__ vs) {
  int blk;
  const auto& j = batch_job(batch, &blk);
  const int64_t i = (int64_t)blk * BLK + threadIdx.x;
  if (i >= j.n) return;
  const double v = j.v[i];
  const T ti = (T)(vs ? v / *vs : v);
  if (j.t) j.t[i] = ti;
  if (j.d0) j.d0[i] = j.dinv[i] * ti * j.c0;
}
template <class T>
void VcOps<T>::cast_in(const RhsJob<T>* j, int nj, const double* vs, bool rev, hipStream_t s) {
  for (int q0 = 0; q0 < nj; q0 += MAXB) {
    const int m = std::min(MAXB, nj - q0);
    Batch<CastJob<T>> b;
    for (int q = 0; q < MAXB; ++q) {
      const RhsJob<T>& J = j[q0 + (q < m ? q : 0)];
      b.d[q] = {J.n, J.v, J.t, J.dinv, (T)J.c0, J.d0};
    }
    const unsigned grid = batch_blocks(b, m, rev, [&](int q) { return cdiv(j[q0 + q].n, BLK); });
    k_cast_in<T><<<grid, BLK, 0, s>>>(b, vs);
    HBGS_HIP(hipGetLastError());
  }
}

// coarsest level: x = A^-1 b with the dense FP64 inverse (row-major; the
// transposed solve passes the stored transpose).  One block per row: the
// row's 8 n bytes are streamed by 256 threads and reduced in fixed order.
template <class T>
__global__ __launch_bounds__(BLK) void k_gemv_block(const Batch<DenseJob<T>> batch) {
  __shared__ double sh[BLK / 64];
  int row;
  const auto& j = batch_job(batch, &row);
  const int n = j.n;
  const double* __restrict__ m = j.inv + (int64_t)row * n;
  const T* __restrict__ b = j.b;
  double acc = 0.0;
  for (int k = threadIdx.x; k < n; k += BLK) acc += m[k] * (double)b[k];
  acc = lanes_sum<double>(acc, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < BLK / 64; ++q) t += sh[q];
    j.x[row] = (T)t;
  }
}
template <class T>
void VcOps<T>::coarse(const DenseJob<T>* j, int nj, hipStream_t s) {
  for (int q0 = 0; q0 < nj; q0 += MAXB) {
    const int m = std::min(MAXB, nj - q0);
    Batch<DenseJob<T>> b;
    for (int q = 0; q < MAXB; ++q) b.d[q] = j[q0 + (q < m ? q : 0)];
    const unsigned grid = batch_blocks(b, m, false, [&](int q) { return j[q0 + q].n; });
    launch_batch(k_gemv_block<T>, grid, 0, b, s, nullptr, nullptr);
  }
}

// DD(0)-ILU(0) sweeps: one block per subdomain, level by level, one thread
// per row (each sum in ascending column)
template <class T>
struct SweepJob {
  const int *ord, *lev, *sub, *rp, *ci;
  const T* v;
  const int* dpos;
  const T* t;
  T* y;
};
template <class T, bool DIAG>
__global__ __launch_bounds__(BLK) void k_ilu_lower(const Batch<SweepJob<T>> batch) {
  int b;
  const SweepJob<T>& j = batch_job(batch, &b);
  const int *__restrict__ ord = j.ord, *__restrict__ lev = j.lev, *__restrict__ sub = j.sub, *__restrict__ rp = j.rp,
            *__restrict__ ci = j.ci, *__restrict__ dpos = j.dpos;
  const T *__restrict__ v = j.v, *__restrict__ t = j.t;
  T* y = j.y;
  for (int l = sub[b]; l + 1 < sub[b + 1]; ++l) {
    for (int q = lev[l] + threadIdx.x; q < lev[l + 1]; q += BLK) {
      const int i = ord[q];
      T s = t[i];
      for (int k = rp[i]; k < dpos[i]; ++k) s -= v[k] * y[ci[k]];
      y[i] = DIAG ? s / v[dpos[i]] : s;
    }
    __syncthreads();
  }
}
template <class T, bool DIAG>
__global__ __launch_bounds__(BLK) void k_ilu_upper(const Batch<SweepJob<T>> batch) {
  int b;
  const SweepJob<T>& j = batch_job(batch, &b);
  const int *__restrict__ ord = j.ord, *__restrict__ lev = j.lev, *__restrict__ sub = j.sub, *__restrict__ rp = j.rp,
            *__restrict__ ci = j.ci, *__restrict__ dpos = j.dpos;
  const T *__restrict__ v = j.v, *__restrict__ t = j.t;
  T* y = j.y;
  for (int l = sub[b]; l + 1 < sub[b + 1]; ++l) {
    for (int q = lev[l] + threadIdx.x; q < lev[l + 1]; q += BLK) {
      const int i = ord[q];
      T s = t[i];
      for (int k = dpos[i] + 1; k < rp[i + 1]; ++k) s -= v[k] * y[ci[k]];
      y[i] = DIAG ? s / v[dpos[i]] : s;
    }
    __syncthreads();
  }
}
template <class T>
static const T* ilu_vals(const IluLeaf& f, int transpose);
template <>
const double* ilu_vals<double>(const IluLeaf& f, int transpose) {
  return transpose ? f.vT : f.F.v;
}
template <>
const float* ilu_vals<float>(const IluLeaf& f, int transpose) {
  return transpose ? f.vTf : f.F.vf;
}
// z = U^-1 L^-1 t, or z = L^-T U^-T t (lower sweep on the transposed
// factors dividing by the diagonal, then the unit upper sweep)
template <class T>
void VcOps<T>::ilu(const IluJob<T>* j, int nj, int transpose, hipStream_t s) {
  for (int q0 = 0; q0 < nj; q0 += MAXB) {
    const int m = std::min(MAXB, nj - q0);
    Batch<SweepJob<T>> lo, up;
    for (int q = 0; q < MAXB; ++q) {
      const IluJob<T>& J = j[q0 + (q < m ? q : 0)];
      const IluLeaf& f = *J.f;
      const T* v = ilu_vals<T>(f, transpose);
      T* y = sizeof(T) == sizeof(double) ? reinterpret_cast<T*>(f.yd) : reinterpret_cast<T*>(f.yf);
      lo.d[q] = {f.ford, f.flev, f.fsub, f.F.rp, f.F.ci, v, f.dpos, J.t, y};
      up.d[q] = {f.bord, f.blev, f.bsub, f.F.rp, f.F.ci, v, f.dpos, y, J.z};
    }
    const unsigned grid = batch_blocks(lo, m, false, [&](int q) { return j[q0 + q].f->nsub; });
    batch_blocks(up, m, false, [&](int q) { return j[q0 + q].f->nsub; });
    if (!transpose) {
      launch_batch(k_ilu_lower<T, false>, grid, 0, lo, s, nullptr, nullptr);
      launch_batch(k_ilu_upper<T, true>, grid, 0, up, s, nullptr, nullptr);
    } else {
      launch_batch(k_ilu_lower<T, true>, grid, 0, lo, s, nullptr, nullptr);
      launch_batch(k_ilu_upper<T, false>, grid, 0, up, s, nullptr, nullptr);
    }
  }
}

template struct VcOps<float>;
template struct VcOps<double>;

// --------------------------------------------------------------- GMRES
__global__ void k_permute_in(int n, const int* __restrict__ perm, const double* __restrict__ x,
                             double* __restrict__ xp) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) xp[perm[i]] = x[i];
}
__global__ void k_permute_out(int n, const int* __restrict__ perm, const double* __restrict__ xp,
                              double* __restrict__ x) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) x[i] = xp[perm[i]];
}
void permute_in(int n, const int* perm, const double* x, double* xp, hipStream_t s) {
  k_permute_in<<<grid_for(n, BLK), BLK, 0, s>>>(n, perm, x, xp);
  HBGS_HIP(hipGetLastError());
}
void permute_out(int n, const int* perm, const double* xp, double* x, hipStream_t s) {
  k_permute_out<<<grid_for(n, BLK), BLK, 0, s>>>(n, perm, xp, x);
  HBGS_HIP(hipGetLastError());
}
__global__ void k_permute_out_f32(int n, const int* __restrict__ perm, const float* __restrict__ xp,
                                  double* __restrict__ x) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
    x[i] = (double)xp[perm[i]];
}
void permute_out_f32(int n, const int* perm, const float* xp, double* x, hipStream_t s) {
  k_permute_out_f32<<<grid_for(n, BLK), BLK, 0, s>>>(n, perm, xp, x);
  HBGS_HIP(hipGetLastError());
}

constexpr int DOT_BLOCKS_MAX = 1024;
int dot_blocks(int n) {
  int64_t b = ((int64_t)n + BLK * 8 - 1) / (BLK * 8);
  if (b < 1) b = 1;
  if (b > DOT_BLOCKS_MAX) b = DOT_BLOCKS_MAX;
  return (int)b;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = lanes_sum<double>(v, 64);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < BLK / 64; ++q) t += sh[q];
  return t;
}

// Givens rotation update of Hessenberg column j (H is (m+1) x m, row-major
// with leading dimension m) by one thread, on a copy of the column in LDS:
// col[k] = h1[k] + h2[k] (k <= j) on entry; the earlier rotations' cosines
// and sines in cs/sn (LDS).  h1/h2: first and second Gram-Schmidt
// coefficients; h2[j+1] = ||w||^2 after the first pass; ga.h1[j+1] = ||w||^2
// before orthogonalisation.  On exit col[0..j+1] is the rotated column;
// scal (device) and host_scal (pinned host memory) receive |g_{j+1}|,
// h_{j+1,j} and ||w||.
__device__ void givens_update(const GivensArgs& ga, const double* h2, double* col, const double* cs,
                              const double* sn) {
  const int j = ga.j;
  // ||w - V h2||^2 = ||w||^2 - ||h2||^2 for orthonormal V
  double ss = h2[j + 1];
  for (int k = 0; k <= j; ++k) ss -= h2[k] * h2[k];
  const double hn = ss > 0.0 ? sqrt(ss) : 0.0;
  col[j + 1] = hn;
  // the rotated entry k+1 is carried in a register to the next rotation
  double a = col[0];
  for (int k = 0; k < j; ++k) {
    const double b = col[k + 1];
    col[k] = cs[k] * a + sn[k] * b;
    a = -sn[k] * a + cs[k] * b;
  }
  const double b = hn;
  const double den = sqrt(a * a + b * b);
  const double c = a / den, sj = b / den;
  ga.cs[j] = c;
  ga.sn[j] = sj;
  col[j] = den;
  col[j + 1] = 0.0;
  const double gj = ga.g[j];
  ga.g[j + 1] = -sj * gj;
  ga.g[j] = c * gj;
  const double est = fabs(-sj * gj), w0 = sqrt(ga.h1[j + 1]);
  ga.scal[0] = est;
  ga.scal[1] = hn;
  ga.scal[2] = w0;
  if (ga.host_scal) {  // the estimate last: the host polls it
    ga.host_scal[1] = hn;
    ga.host_scal[2] = w0;
    __threadfence_system();  // orders the two values before the estimate
    ga.host_scal[0] = est;   // no wait for its arrival: the thread has nothing left to do
  }
}

// Last-level (Infinity) cache of the MI355X, 256 MB.
constexpr double kLastLevelCache = 256e6;

// Classical Gram-Schmidt pass over rows: w holds column j+1 of V.
//   UPD:  w -= sum_k h_k V_k           (k <= j)
//   DOTS: part_k = sum V_k . w          (k <= j), after the update
//   FIN:  (with DOTS, not UPD) column j still holds the previous step's
//         once-orthogonalised vector u; it is finished first, in place, as
//         V_j = (u - sum_{k<j} hp_k V_k) / scal[1] (the previous step's
//         second-pass coefficients hp and h_{j,j-1}), then used in the dots
//   always: part_{j+1} = w . w
// (per-block partial sums; the reduction over blocks is a separate launch,
// since a grid-wide completion fence costs more than the launch)
template <int MAXV, bool UPD, bool DOTS, bool FIN>
__global__ __launch_bounds__(BLK) void k_cgs(int n, int nv, double* __restrict__ V, size_t ldv,
                                             double* __restrict__ w, const double* __restrict__ h,
                                             double* __restrict__ part, const double* __restrict__ hp,
                                             const double* __restrict__ scal, bool rev) {
  static_assert(!(FIN && UPD) && (!FIN || DOTS), "FIN finishes a basis vector ahead of a dots-only pass");
  __shared__ double sh[BLK / 64][MAXV + 1];
  double acc[DOTS ? MAXV : 1];
  double hh[UPD ? MAXV : 1];
#pragma unroll
  for (int k = 0; k < (DOTS ? MAXV : 1); ++k) acc[k] = 0.0;
  if (UPD) {
#pragma unroll
    for (int k = 0; k < MAXV; ++k) hh[k] = k < nv ? h[k < nv ? k : 0] : 0.0;
  }
  const int nrd = FIN ? nv - 1 : nv;  // columns read as they stand
  const double hn = FIN ? scal[1] : 1.0;
  double hq[FIN ? MAXV : 1];  // in registers: zero beyond nrd, where vk is zero too
  if (FIN) {
#pragma unroll
    for (int k = 0; k < MAXV; ++k) hq[k] = k < nrd ? hp[k < nrd ? k : 0] : 0.0;
  }
  double ww = 0.0, accf = 0.0;
  // U rows per step (i, i + stride, ...), all their loads issued before any
  // use; the rows are accumulated in the order of a one-row loop
  constexpr int U = MAXV <= 16 ? 2 : 1;
  const int64_t stride = (int64_t)gridDim.x * BLK;
  const int64_t steps = ((int64_t)n + U * stride - 1) / (U * stride);
  for (int64_t st = 0; st < steps; ++st) {
    const int64_t i0 = (int64_t)blockIdx.x * BLK + threadIdx.x + (rev ? steps - 1 - st : st) * U * stride;
    double vk[U][MAXV], uu[U], wv[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = i0 + r * stride;
      const bool in = i < n;
#pragma unroll
      for (int k = 0; k < MAXV; ++k) vk[r][k] = in && k < nrd ? V[(size_t)(k < nrd ? k : 0) * ldv + i] : 0.0;
      uu[r] = FIN && in ? V[(size_t)nrd * ldv + i] : 0.0;
      wv[r] = in ? w[i] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = i0 + r * stride;
      if (i >= n) break;
      double vf = 0.0;
      if (FIN) {
        double u = uu[r];
#pragma unroll
        for (int k = 0; k < MAXV; ++k) u -= hq[k] * vk[r][k];
        vf = u / hn;
        V[(size_t)nrd * ldv + i] = vf;
      }
      double wi = wv[r];
      if (UPD) {
#pragma unroll
        for (int k = 0; k < MAXV; ++k) wi -= hh[k] * vk[r][k];
        w[i] = wi;
      }
      if (DOTS) {
#pragma unroll
        for (int k = 0; k < MAXV; ++k) acc[k] += vk[r][k] * wi;
        if (FIN) accf += vf * wi;  // the finished column's dot: acc[nrd] only saw zeros
      }
      ww += wi * wi;
    }
  }
  // the block's sums, each over lanes, then over wavefronts in order; all of
  // them pass through LDS at once (against a barrier pair per sum: the 1.4M-row
  // 2D FP64 adjoint solve, 26 steps, 13.53 -> 13.41 ms)
  const int nb = gridDim.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (DOTS) {
#pragma unroll
    for (int k = 0; k < MAXV; ++k) {
      if (k < nv) {
        const double t = lanes_sum<double>(FIN && k == nrd ? accf : acc[k], 64);
        if (lane == 0) sh[wave][k] = t;
      }
    }
  }
  const double t = lanes_sum<double>(ww, 64);
  if (lane == 0) sh[wave][nv] = t;
  __syncthreads();
  if ((int)threadIdx.x <= nv && (DOTS || (int)threadIdx.x == nv)) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < BLK / 64; ++q) v += sh[q][threadIdx.x];
    part[(size_t)threadIdx.x * nb + blockIdx.x] = v;
  }
}

template <bool UPD, bool DOTS, bool FIN = false>
static void launch_cgs(int n, int nv, double* V, size_t ldv, double* w, const double* h, double* part,
                       const double* hp, const double* scal, bool rev, hipStream_t s) {
  int nb = dot_blocks(n);
  if (nv <= 8)
    k_cgs<8, UPD, DOTS, FIN><<<nb, BLK, 0, s>>>(n, nv, V, ldv, w, h, part, hp, scal, rev);
  else if (nv <= 16)
    k_cgs<16, UPD, DOTS, FIN><<<nb, BLK, 0, s>>>(n, nv, V, ldv, w, h, part, hp, scal, rev);
  else if (nv <= 32)
    k_cgs<32, UPD, DOTS, FIN><<<nb, BLK, 0, s>>>(n, nv, V, ldv, w, h, part, hp, scal, rev);
  else if (nv <= 48)  // 16-25% faster than the 64-vector form (one wave per SIMD) at 33-48 vectors
    k_cgs<48, UPD, DOTS, FIN><<<nb, BLK, 0, s>>>(n, nv, V, ldv, w, h, part, hp, scal, rev);
  else
    k_cgs<64, UPD, DOTS, FIN><<<nb, BLK, 0, s>>>(n, nv, V, ldv, w, h, part, hp, scal, rev);
  HBGS_HIP(hipGetLastError());
}

// out[k] = sum over blocks of part[k*nb + b] (fixed order per k)
__global__ __launch_bounds__(BLK) void k_reduce(int nb, const double* __restrict__ part, double* __restrict__ out) {
  __shared__ double sh[BLK / 64];
  const double* p = part + (size_t)blockIdx.x * nb;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += BLK) acc += p[b];
  double t = block_sum(acc, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}
void mdot_reduce(int nvec, int nblocks, const double* part, double* out, hipStream_t s) {
  k_reduce<<<nvec, BLK, 0, s>>>(nblocks, part, out);
  HBGS_HIP(hipGetLastError());
}

// one block: out[k] = sum over blocks of part[k*nb + b] for k < nvec (one
// wave per vector, fixed order), then the Givens update from out.  The
// column's first-pass coefficients and the earlier rotations are read by
// many threads at once into LDS, so the one thread's sequential update
// waits on no global loads.
constexpr int RG_BLK = 1024;
constexpr int RG_MAXV = 66;
__global__ __launch_bounds__(RG_BLK) void k_reduce_givens(int nvec, int nb, const double* __restrict__ part,
                                                          double* __restrict__ out, GivensArgs ga) {
  __shared__ double red[RG_MAXV], col[RG_MAXV], scs[RG_MAXV], ssn[RG_MAXV];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int j = ga.j;
  const double h1 = tid <= j ? ga.h1[tid] : 0.0;
  if (tid < j) {
    scs[tid] = ga.cs[tid];
    ssn[tid] = ga.sn[tid];
  }
  for (int k = wave; k < nvec; k += RG_BLK / 64) {
    const double* p = part + (size_t)k * nb;
    double a = 0.0;
    for (int b = lane; b < nb; b += 64) a += p[b];
    a = lanes_sum<double>(a, 64);
    if (lane == 0) red[k] = a;
  }
  __syncthreads();
  if (tid < nvec) out[tid] = red[tid];
  if (tid <= j) col[tid] = h1 + red[tid];
  __syncthreads();
  if (tid == 0) givens_update(ga, red, col, scs, ssn);
  __syncthreads();
  if (tid <= j + 1) ga.H[(size_t)tid * ga.m + j] = col[tid];
}

void cgs_dots(int n, int j, const double* V, size_t ldv, const double* w, double* part, hipStream_t s) {
  launch_cgs<false, true>(n, j + 1, const_cast<double*>(V), ldv, const_cast<double*>(w), nullptr, part, nullptr,
                          nullptr, false, s);
}
void cgs_finish_dots(int n, int j, double* V, size_t ldv, const double* w, const double* hp, const double* scal,
                     double* part, hipStream_t s) {
  launch_cgs<false, true, true>(n, j + 1, V, ldv, const_cast<double*>(w), nullptr, part, hp, scal, false, s);
}
void cgs_update_dots(int n, int j, const double* V, size_t ldv, double* w, const double* h1, double* part,
                     hipStream_t s) {
  // where the basis exceeds the last-level cache this pass walks the rows
  // backwards: it meets the rows that the first pass read last
  const bool rev = (double)n * (j + 2) * sizeof(double) > kLastLevelCache;
  launch_cgs<true, true>(n, j + 1, const_cast<double*>(V), ldv, w, h1, part, nullptr, nullptr, rev, s);
}
void reduce_givens(int n, int j, const double* part, double* h2, const GivensArgs& ga, hipStream_t s) {
  if (j + 2 > RG_MAXV) HBGS_FAIL(HBGS_EINVAL, "Gram-Schmidt basis too large");
  k_reduce_givens<<<1, RG_BLK, 0, s>>>(j + 2, dot_blocks(n), part, h2, ga);
  HBGS_HIP(hipGetLastError());
}
// y = R^-1 g with R the leading jend x jend upper triangle of H: the block
// stages R and g in LDS, then one thread substitutes backwards (no global
// loads inside the dependent chain)
constexpr int BS_MAX = 64;
__global__ __launch_bounds__(BLK) void k_backsolve(int jend, int m, const double* __restrict__ H,
                                                   const double* __restrict__ g, double* __restrict__ y) {
  __shared__ double sr[BS_MAX][BS_MAX + 1];
  __shared__ double sy[BS_MAX], sg[BS_MAX];
  for (int e = threadIdx.x; e < jend * jend; e += BLK) {
    const int i = e / jend, k = e % jend;
    if (k >= i) sr[i][k] = H[(size_t)i * m + k];
  }
  if ((int)threadIdx.x < jend) sg[threadIdx.x] = g[threadIdx.x];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int i = jend - 1; i >= 0; --i) {
      double t = sg[i];
      for (int k = i + 1; k < jend; ++k) t -= sr[i][k] * sy[k];
      sy[i] = t / sr[i][i];
    }
  __syncthreads();
  if ((int)threadIdx.x < jend) y[threadIdx.x] = sy[threadIdx.x];
}
void backsolve(int jend, int m, const double* H, const double* g, double* y, hipStream_t s) {
  if (jend > BS_MAX) HBGS_FAIL(HBGS_EINVAL, "least-squares system too large");
  k_backsolve<<<1, BLK, 0, s>>>(jend, m, H, g, y);
  HBGS_HIP(hipGetLastError());
}

template <class TZ>
__global__ void k_xupdate(int n, int jend, const TZ* __restrict__ Z, size_t ldz, const double* __restrict__ y,
                          bool zero, double* __restrict__ x) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
    double xi = zero ? 0.0 : x[i];
    for (int k = 0; k < jend; ++k) xi += y[k] * (double)Z[(size_t)k * ldz + i];
    x[i] = xi;
  }
}
template <class TZ>
void xupdate(int n, int jend, const TZ* Z, size_t ldz, const double* y, bool zero, double* x, hipStream_t s) {
  k_xupdate<TZ><<<grid_for(n, BLK), BLK, 0, s>>>(n, jend, Z, ldz, y, zero, x);
  HBGS_HIP(hipGetLastError());
}
template void xupdate<float>(int, int, const float*, size_t, const double*, bool, double*, hipStream_t);
template void xupdate<double>(int, int, const double*, size_t, const double*, bool, double*, hipStream_t);

__global__ __launch_bounds__(BLK) void k_norm2_part(int n, const double* __restrict__ x, double* __restrict__ part) {
  __shared__ double sh[BLK / 64];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
    acc += x[i] * x[i];
  double t = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}
void norm2_partial(int n, const double* x, double* part, hipStream_t s) {
  k_norm2_part<<<dot_blocks(n), BLK, 0, s>>>(n, x, part);
  HBGS_HIP(hipGetLastError());
}

// the sums k_reduce forms, of one vector, to the device and (last, the host
// polls it) to pinned host memory
__global__ __launch_bounds__(BLK) void k_sum_to_host(int nb, const double* __restrict__ part, double* __restrict__ out,
                                                     double* __restrict__ host) {
  __shared__ double sh[BLK / 64];
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += BLK) acc += part[b];
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    *out = t;
    *host = t;
  }
}
void sum_to_host(int nblocks, const double* part, double* out, double* host, hipStream_t s) {
  k_sum_to_host<<<1, BLK, 0, s>>>(nblocks, part, out, host);
  HBGS_HIP(hipGetLastError());
}

__global__ void k_start_cycle(int n, const double* __restrict__ r, const double* __restrict__ ss,
                              double* __restrict__ v, int m, double* __restrict__ g) {
  const double nr = sqrt(*ss);
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= m; i += BLK) g[i] = i == 0 ? nr : 0.0;
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) v[i] = r[i] / nr;
}
void start_cycle(int n, const double* r, const double* sum, double* v, int m, double* g, hipStream_t s) {
  k_start_cycle<<<grid_for(n, BLK), BLK, 0, s>>>(n, r, sum, v, m, g);
  HBGS_HIP(hipGetLastError());
}

__global__ void k_grad(int n, const int* __restrict__ rp, const int* __restrict__ ci, const double* __restrict__ lam,
                       const double* __restrict__ x, double* __restrict__ g) {
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
    double li = lam[i];
    for (int k = rp[i]; k < rp[i + 1]; ++k) g[k] = -li * x[ci[k]];
  }
}
void grad_values(int n, const int* rp, const int* ci, const double* lam, const double* x, double* g,
                 hipStream_t s) {
  k_grad<<<grid_for(n, BLK), BLK, 0, s>>>(n, rp, ci, lam, x, g);
  HBGS_HIP(hipGetLastError());
}

struct FieldRanges {
  int nf;
  int lo[HBGS_MAX_FIELDS], hi[HBGS_MAX_FIELDS];
};
__global__ void k_column_fields(int64_t nnz, const int* __restrict__ ci, FieldRanges fr, int* mask) {
  int m = 0;
  for (int64_t k = (int64_t)blockIdx.x * BLK + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * BLK) {
    int c = ci[k];
    for (int f = 0; f < fr.nf; ++f)
      if (c >= fr.lo[f] && c < fr.hi[f]) m |= 1 << f;
  }
  if (m) atomicOr(mask, m);
}
void column_fields(const DCsr& c, int nf, const int* lo, const int* hi, int* mask, hipStream_t s) {
  if (c.nnz == 0) return;
  FieldRanges fr;
  fr.nf = nf;
  for (int f = 0; f < nf; ++f) {
    fr.lo[f] = lo[f];
    fr.hi[f] = hi[f];
  }
  k_column_fields<<<grid_for(c.nnz, BLK, 4096), BLK, 0, s>>>(c.nnz, c.ci, fr, mask);
  HBGS_HIP(hipGetLastError());
}

}  // namespace solve
}  // namespace hbgs
