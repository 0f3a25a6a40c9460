// Device setup of the block Gauss-Seidel / SA-AMG preconditioner (gfx950).
//
// Built with -ffp-contract=off: every floating-point value below is produced
// by the sequential, rounded-product-then-add evaluation that the method's
// definitions state (ascending column order within a row), so aggregates,
// sparsity patterns and hierarchy values are reproducible bit for bit.
// Parallelism comes from rows: a row has one thread, or a group of lanes
// that read its entries with coalesced loads and combine them with
// cross-lane shuffles, adding order-dependent sums in entry order.  Only
// integer decisions and order-independent max reductions use atomics.
#include <atomic>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "hbgs_internal.h"

namespace hbgs {
namespace setup {

constexpr int BLK = 256;
constexpr int SCAN_PER_THREAD = 4;
constexpr int SCAN_TILE = BLK * SCAN_PER_THREAD;

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// aggregation priority: hash32(i ^ salt) << 32 | i (distinct per row)
__device__ __forceinline__ uint64_t agg_key(int i, uint64_t salt) {
  uint64_t h = splitmix64((uint64_t)(uint32_t)i ^ salt) >> 32;
  return (h << 32) | (uint64_t)(uint32_t)i;
}

#define GRID_STRIDE(i, n) \
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// ------------------------------------------------------------- row groups
// Rows of n handled by groups of L lanes (grid-stride over row groups); gl
// is the lane's index in its group.  Every lane of a group runs the same
// iterations, so the group's shuffles below always see their whole group.
#define ROW_GROUPS(L, i, gl, n)                                                       \
  const int gl = (int)(threadIdx.x % (L));                                             \
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / (L); i < (n); \
       i += (int64_t)gridDim.x * blockDim.x / (L))

template <int L, class T>
__device__ __forceinline__ T grp_max(T x) {
  for (int off = L >> 1; off > 0; off >>= 1) {
    const T o = __shfl_xor(x, off, L);
    x = o > x ? o : x;
  }
  return x;
}
template <int L, class T>
__device__ __forceinline__ T grp_min(T x) {
  for (int off = L >> 1; off > 0; off >>= 1) {
    const T o = __shfl_xor(x, off, L);
    x = o < x ? o : x;
  }
  return x;
}
template <int L>
__device__ __forceinline__ int grp_sum(int x) {
  for (int off = L >> 1; off > 0; off >>= 1) x += __shfl_xor(x, off, L);
  return x;
}
// s + (the x of the group's lanes with take set, added one by one in lane
// order): the sequential sum over a row's entries, L entries at a time
template <int L>
__device__ __forceinline__ double grp_ordered_add(double s, double x, bool take) {
  if constexpr (L == 1) return take ? s + x : s;
  const uint64_t b = __ballot(take);
  const int lane = (int)(threadIdx.x & 63), base = lane & ~(L - 1);
  uint64_t g = L == 64 ? b : (b >> base) & ((1ull << (L & 63)) - 1);
  while (g) {  // the group's takers, lowest lane first
    const int j = __builtin_ctzll(g);
    s += __shfl(x, j, L);
    g &= g - 1;
  }
  return s;
}
// number of lanes below this one in the group with pred set; *total: in the group
template <int L>
__device__ __forceinline__ int grp_rank(bool pred, int* total) {
  if constexpr (L == 1) {
    *total = pred;
    return 0;
  }
  const uint64_t b = __ballot(pred);
  const int lane = (int)(threadIdx.x & 63), base = lane & ~(L - 1);
  const uint64_t g = L == 64 ? b : (b >> base) & ((1ull << (L & 63)) - 1);
  *total = __popcll(g);
  return __popcll(g & ((1ull << (lane - base)) - 1));
}

// lanes per row from the mean row length
static int row_lanes(int64_t n, int64_t nnz) {
  const double avg = n ? (double)nnz / (double)n : 0.0;
  return avg <= 7.5 ? 8 : avg <= 15.0 ? 16 : 32;
}
// For passes that look at a row's entries once or twice: one thread per row
// where rows are short.  It requests the row's first entries (row_regs)
// together, and no cross-lane steps are left; eight lanes per row are eight
// times the waves, each with the same chain of dependent loads (an aggregation
// pass over 1M rows of 7 entries, four fields side by side: 130-190 us, one
// thread per row 36-63; the strengths 172 -> 50, the filtered matrix 459 ->
// 141, the prolongator 712 -> 162).
// Where a few rows are long, one thread would hold up the rest (the
// prolongator walks a row once per aggregate it meets): 262k rows of 5 entries
// with 20 rows of 29 / 45 / 85 among them, aggregation and prolongator of the
// whole hierarchy 2.47 / 3.60 / 5.94 ms with one thread, 2.45 / 3.42 / 5.22
// with eight; with longest rows of 21, 1.90 against 1.91; with none, 1.27
// against 1.37.
constexpr int SCAN_LONG = 24;
static int scan_lanes(const DCsr& a) {
  const int L = row_lanes(a.n, a.nnz);
  return L == 8 && a.maxlen <= SCAN_LONG ? 1 : L;
}
// entries per lane requested together
constexpr int row_regs(int L) { return L == 1 ? 8 : 1; }
#define LAUNCH_ROW_GROUPS(kern, L, nrows, s, ...) LAUNCH_ROW_GROUPS_CAP(kern, L, nrows, 1 << 20, s, __VA_ARGS__)
// cap: most blocks (kernels that end in one atomic per block use a small cap)
#define LAUNCH_ROW_GROUPS_CAP(kern, L, nrows, cap, s, ...)            \
  do {                                                                 \
    const unsigned g_ = grid_for((int64_t)(nrows) * (L), BLK, cap);    \
    switch (L) {                                                       \
      case 1: kern<1><<<g_, BLK, 0, s>>>(__VA_ARGS__); break;          \
      case 8: kern<8><<<g_, BLK, 0, s>>>(__VA_ARGS__); break;          \
      case 16: kern<16><<<g_, BLK, 0, s>>>(__VA_ARGS__); break;        \
      default: kern<32><<<g_, BLK, 0, s>>>(__VA_ARGS__); break;        \
    }                                                                  \
    HBGS_HIP(hipGetLastError());                                       \
  } while (0)

// ------------------------------------------------------- results on the host
// one block: the message's words, then (every thread's stores fenced) its flag
__device__ __forceinline__ void mail_flag(MailArg m) {
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(m.slot, m.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ __launch_bounds__(BLK) void k_mail(const uint32_t* __restrict__ src, int words, MailArg m) {
  uint32_t* dst = reinterpret_cast<uint32_t*>(m.slot + 8);
  for (int t = threadIdx.x; t < words; t += BLK) dst[t] = src[t];
  mail_flag(m);
}
// most matrices whose layouts are built together: A, P, R and [A P; P] of
// every level of a field
constexpr int MATRICES = 4 * HBGS_MAX_LEVELS;
void read_back(void* dst, const void* src, size_t bytes, hipStream_t s) {
  Scratch* sc = tmp_scratch();
  if (!sc) {
    HBGS_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
    HBGS_HIP(hipStreamSynchronize(s));
    return;
  }
  const MailArg m = sc->mail.next();
  k_mail<<<1, BLK, 0, s>>>(static_cast<const uint32_t*>(src), (int)(bytes / 4), m);
  HBGS_HIP(hipGetLastError());
  std::memcpy(dst, sc->mail.wait(s), bytes);
}

// ------------------------------------------------------------------ scans
// Exclusive scan in tiles of 1024: tile sums, one block scans the tile sums
// (and posts the total to the host, which goes on while the last kernel
// runs), then a block-local scan with the tile offset.  Integers only.
// Three launches and one wait; scanning the tile sums by recursion with the
// totals copied back took eight launches and three waits.
template <class TI>
__global__ void k_tile_sums(const TI* in, int64_t n, int64_t* tsum) {
  __shared__ int64_t sh[BLK / 64];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER_THREAD;
  int64_t acc = 0;
  for (int q = 0; q < SCAN_PER_THREAD; ++q)
    if (base + q < n) acc += (int64_t)in[base + q];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) tsum[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}
static_assert(BLK == 256, "four waves per tile");

// exclusive scan of one value per thread of the block; *total: their sum
template <int NT>
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t* sh, int64_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t inc = v;
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  __syncthreads();
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  int64_t before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    before += k < w ? sh[k] : 0;
    all += sh[k];
  }
  *total = all;
  return before + inc - v;
}
// toff[t] = sum of tsum[0 .. t-1], toff[nt] = total (mailed when m.slot is set)
// (a block of 1,024 threads waited up to 330 us for a compute unit with room
// for it beside the other fields' work)
constexpr int SCAN_TOP = 256;
__global__ __launch_bounds__(SCAN_TOP) void k_scan_tiles(const int64_t* __restrict__ tsum, int64_t nt,
                                                         int64_t* __restrict__ toff, MailArg m) {
  __shared__ int64_t sh[SCAN_TOP / 64];
  int64_t run = 0;
  for (int64_t b = 0; b < nt; b += SCAN_TOP) {
    const int64_t i = b + threadIdx.x;
    int64_t all;
    const int64_t x = block_scan<SCAN_TOP>(i < nt ? tsum[i] : 0, sh, &all);
    if (i < nt) toff[i] = run + x;
    run += all;
  }
  if (threadIdx.x == 0) {
    toff[nt] = run;
    if (m.slot) m.slot[8] = (uint64_t)run;
  }
  if (m.slot) mail_flag(m);
}

// toff null: one tile, whose total goes to *total and (m.slot set) the host
template <class TI, class TO>
__global__ __launch_bounds__(BLK) void k_tile_scan(const TI* in, int64_t n, const int64_t* toff, TO* out,
                                                   int64_t* total, MailArg m) {
  __shared__ int64_t sh[BLK / 64];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER_THREAD;
  int64_t v[SCAN_PER_THREAD];
  int64_t acc = 0;
  for (int q = 0; q < SCAN_PER_THREAD; ++q) {
    v[q] = base + q < n ? (int64_t)in[base + q] : 0;
    acc += v[q];
  }
  int64_t all;
  int64_t run = block_scan<BLK>(acc, sh, &all);
  if (toff) run += toff[blockIdx.x];
  for (int q = 0; q < SCAN_PER_THREAD; ++q) {
    if (base + q < n) out[base + q] = (TO)run;
    run += v[q];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int64_t t = toff ? toff[gridDim.x] : all;
    out[n] = (TO)t;
    if (!toff) {
      *total = t;
      if (m.slot) m.slot[8] = (uint64_t)t;
    }
  }
  if (!toff && m.slot) mail_flag(m);
}

// out[0..n] exclusive prefix of in[0..n-1] (out[n] = total)
template <class TI, class TO>
static int64_t scan_impl(const TI* in, TO* out, int64_t n, hipStream_t s) {
  const int64_t nt = std::max<int64_t>(1, (n + SCAN_TILE - 1) / SCAN_TILE);
  Tmp<int64_t> tsum(nt), toff(nt + 1);
  Scratch* sc = tmp_scratch();
  const MailArg m = sc ? sc->mail.next() : MailArg{nullptr, 0};
  if (nt == 1) {
    k_tile_scan<TI, TO><<<1, BLK, 0, s>>>(in, n, nullptr, out, toff.p + nt, m);
  } else {
    k_tile_sums<TI><<<(unsigned)nt, BLK, 0, s>>>(in, n, tsum.p);
    k_scan_tiles<<<1, SCAN_TOP, 0, s>>>(tsum.p, nt, toff.p, m);
    k_tile_scan<TI, TO><<<(unsigned)nt, BLK, 0, s>>>(in, n, toff.p, out, nullptr, MailArg{nullptr, 0});
  }
  HBGS_HIP(hipGetLastError());
  int64_t total = 0;
  if (sc)
    std::memcpy(&total, sc->mail.wait(s), sizeof(total));
  else
    read_back(&total, toff.p + nt, sizeof(total), s);
  return total;
}

int64_t scan_i32_to_i64(const int* in, int64_t* out, int64_t n, hipStream_t s) {
  return scan_impl<int, int64_t>(in, out, n, s);
}
int64_t scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
  return scan_impl<int64_t, int64_t>(in, out, n, s);
}
int64_t counts_to_rowptr(const int* counts, int* rp, int n, hipStream_t s) {
  return scan_impl<int, int>(counts, rp, n, s);
}

// --------------------------------------------------------------- validate
// flags bit 0: bad row pointers, 1: column out of range, 2: unsorted or
// duplicate columns, 3: missing or zero diagonal, 4: field id out of range,
// 5: non-finite value
__global__ void k_validate(int n, int64_t nnz, const int* rp, const int* ci, const double* v, int nf,
                           const int* field, int* flags) {
  GRID_STRIDE(i, n) {
    int f = 0;
    int s = rp[i], e = rp[i + 1];
    if (s < 0 || e < s || (int64_t)e > nnz) {
      atomicOr(flags, 1);
      continue;
    }
    bool diag = false;
    for (int k = s; k < e; ++k) {
      int c = ci[k];
      if (c < 0 || c >= n) f |= 2;
      if (k > s && c <= ci[k - 1]) f |= 4;
      if (c == i && v[k] != 0.0) diag = true;
      if (!isfinite(v[k])) f |= 32;
    }
    if (!diag) f |= 8;
    if (field[i] < 0 || field[i] >= nf) f |= 16;
    if (f) atomicOr(flags, f);
  }
}

void validate(int n, int64_t nnz, const int* rp, const int* ci, const double* v, int nf, const int* field,
              int* flags, hipStream_t s) {
  k_validate<<<grid_for(n, BLK, 65536), BLK, 0, s>>>(n, nnz, rp, ci, v, nf, field, flags);
  HBGS_HIP(hipGetLastError());
}

// ------------------------------------------------------------ permutation
__global__ void k_field_hist(int n, const int* field, int nf, int* counts) {
  __shared__ int sh[HBGS_MAX_FIELDS];
  if (threadIdx.x < HBGS_MAX_FIELDS) sh[threadIdx.x] = 0;
  __syncthreads();
  GRID_STRIDE(i, n) atomicAdd(&sh[field[i]], 1);
  __syncthreads();
  if ((int)threadIdx.x < nf) atomicAdd(&counts[threadIdx.x], sh[threadIdx.x]);
}

void field_histogram(int n, const int* field, int nf, int* counts, hipStream_t s) {
  HBGS_HIP(hipMemsetAsync(counts, 0, nf * sizeof(int), s));
  k_field_hist<<<grid_for(n, BLK, 4096), BLK, 0, s>>>(n, field, nf, counts);
  HBGS_HIP(hipGetLastError());
}

__global__ void k_flag_field(int n, const int* field, int f, int* flag) {
  GRID_STRIDE(i, n) flag[i] = field[i] == f ? 1 : 0;
}

__global__ void k_perm_from_rank(int n, const int* field, int f, int lo, const int64_t* rank, int* perm) {
  GRID_STRIDE(i, n) if (field[i] == f) perm[i] = lo + (int)rank[i];
}

void field_ranks_all(int n, const int* field, int nf, const int* f_lo_host, int* perm, hipStream_t s) {
  Tmp<int> flag(n);
  Tmp<int64_t> rank(n + 1);
  for (int f = 0; f < nf; ++f) {
    k_flag_field<<<grid_for(n, BLK), BLK, 0, s>>>(n, field, f, flag.p);
    HBGS_HIP(hipGetLastError());
    scan_i32_to_i64(flag.p, rank.p, n, s);
    k_perm_from_rank<<<grid_for(n, BLK), BLK, 0, s>>>(n, field, f, f_lo_host[f], rank.p, perm);
    HBGS_HIP(hipGetLastError());
  }
}

__global__ void k_invert_perm(int n, const int* perm, int* iperm) {
  GRID_STRIDE(i, n) iperm[perm[i]] = (int)i;
}
void invert_perm(int n, const int* perm, int* iperm, hipStream_t s) {
  k_invert_perm<<<grid_for(n, BLK), BLK, 0, s>>>(n, perm, iperm);
  HBGS_HIP(hipGetLastError());
}

__global__ void k_perm_len(int n, const int* rp, const int* perm, int* len) {
  GRID_STRIDE(i, n) len[perm[i]] = rp[i + 1] - rp[i];
}
void permuted_lengths(int n, const int* rp, const int* perm, int* len, hipStream_t s) {
  k_perm_len<<<grid_for(n, BLK), BLK, 0, s>>>(n, rp, perm, len);
  HBGS_HIP(hipGetLastError());
}

// the pattern of row p of P A P^T: old row iperm[p] with columns mapped and
// re-sorted (insertion sort), and each entry's position in A
__global__ void k_permute_pattern(int n, const int* rp, const int* ci, const int* perm, const int* iperm,
                                  const int* rp_p, int* ci_p, int* pos_p) {
  GRID_STRIDE(p, n) {
    int i = iperm[p];
    int s = rp[i], e = rp[i + 1], o = rp_p[p];
    for (int k = s; k < e; ++k) {
      int c = perm[ci[k]];
      int q = o + (k - s) - 1;
      while (q >= o && ci_p[q] > c) {
        ci_p[q + 1] = ci_p[q];
        pos_p[q + 1] = pos_p[q];
        --q;
      }
      ci_p[q + 1] = c;
      pos_p[q + 1] = k;
    }
  }
}
void permute_pattern(int n, const int* rp, const int* ci, const int* perm, const int* iperm, const int* rp_p,
                     int* ci_p, int* pos_p, hipStream_t s) {
  k_permute_pattern<<<grid_for(n, BLK), BLK, 0, s>>>(n, rp, ci, perm, iperm, rp_p, ci_p, pos_p);
  HBGS_HIP(hipGetLastError());
}

// --------------------------------------------------------------- transpose
__global__ void k_col_count(int64_t nnz, const int* ci, int* cnt) {
  GRID_STRIDE(k, nnz) atomicAdd(&cnt[ci[k]], 1);
}
template <int L>
__global__ void k_transpose_scatter(int n, const int* rp, const int* ci, const double* v, int* cursor,
                                    int* tci, double* tv) {
  ROW_GROUPS(L, i, gl, n) {
    for (int k = rp[i] + gl; k < rp[i + 1]; k += L) {
      const int q = atomicAdd(&cursor[ci[k]], 1);
      tci[q] = (int)i;
      if (v) tv[q] = v[k];
    }
  }
}
// Sort each row by column (entries are distinct, so the result is unique):
// an entry's place is its rank, the number of smaller columns in the row.
// One wavefront per row of up to SORT_WAVE entries, whose columns it reads
// from LDS four at a time (broadcast); longer rows are listed and sorted one
// block per row.  The transposed prolongators have 30 to 400 entries per row:
// one thread per row up to 32 entries and a block for each longer one took
// 730 us for the 95,000 rows of a 1M-row field's (four fields side by side),
// this 140.
constexpr int SORT_WAVE = 256;
constexpr int LONG_LDS = 2048;
__global__ __launch_bounds__(BLK) void k_sort_rows_wave(int n, const int* rp, int* ci, double* v, int* n_long,
                                                        int* long_rows) {
  constexpr int E = SORT_WAVE / 64;  // entries per lane
  __shared__ __align__(16) int sc[BLK / 64][SORT_WAVE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int64_t i = (int64_t)blockIdx.x * (BLK / 64) + wave; i < n; i += (int64_t)gridDim.x * (BLK / 64)) {
    const int s = rp[i], len = rp[i + 1] - s;
    if (len < 2) continue;
    if (len > SORT_WAVE) {
      if (lane == 0) long_rows[atomicAdd(n_long, 1)] = (int)i;
      continue;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the previous row's columns have been read
    __builtin_amdgcn_wave_barrier();
    int c[E];
    double x[E];
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int k = lane + 64 * q;
      c[q] = k < len ? ci[s + k] : INT32_MAX;
      x[q] = v && k < len ? v[s + k] : 0.0;
      if (64 * q < len) sc[wave][k] = c[q];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int rank[E] = {};
    for (int p = 0; p < len; p += 4) {  // beyond len: INT32_MAX, below no column
      const int4 d = *reinterpret_cast<const int4*>(&sc[wave][p]);
#pragma unroll
      for (int q = 0; q < E; ++q)
        if (64 * q < len) rank[q] += (d.x < c[q]) + (d.y < c[q]) + (d.z < c[q]) + (d.w < c[q]);
    }
#pragma unroll
    for (int q = 0; q < E; ++q)
      if (lane + 64 * q < len) {
        ci[s + rank[q]] = c[q];
        if (v) v[s + rank[q]] = x[q];
      }
  }
}

// the *count listed rows of up to LONG_LDS entries, one block per row:
// every entry's destination is its rank (the number of smaller columns in
// the row)
__global__ __launch_bounds__(BLK) void k_sort_long_rows(const int* count, const int* rows, const int* rp, int* ci,
                                                        double* v) {
  __shared__ int sc[LONG_LDS];
  __shared__ double sv[LONG_LDS];
  const int cnt = *count;
  for (int b = blockIdx.x; b < cnt; b += gridDim.x) {
    const int row = rows[b];
    const int s = rp[row], len = rp[row + 1] - s;
    if (len > LONG_LDS) continue;
    __syncthreads();  // the previous row's entries are no longer read
    for (int k = threadIdx.x; k < len; k += BLK) {
      sc[k] = ci[s + k];
      sv[k] = v ? v[s + k] : 0.0;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < len; k += BLK) {
      const int c = sc[k];
      int rank = 0;
      for (int q = 0; q < len; ++q) rank += sc[q] < c;
      ci[s + rank] = c;
      if (v) v[s + rank] = sv[k];
    }
  }
}

// rows longer than LONG_LDS: insertion sort by one thread per listed row
__global__ void k_sort_huge_rows(const int* count, const int* rows, const int* rp, int* ci, double* v) {
  const int cnt = *count;
  GRID_STRIDE(t, cnt) {
    const int i = rows[t];
    int s = rp[i], e = rp[i + 1];
    if (e - s <= LONG_LDS) continue;
    for (int k = s + 1; k < e; ++k) {
      int c = ci[k];
      double x = v ? v[k] : 0.0;
      int q = k - 1;
      while (q >= s && ci[q] > c) {
        ci[q + 1] = ci[q];
        if (v) v[q + 1] = v[q];
        --q;
      }
      ci[q + 1] = c;
      if (v) v[q + 1] = x;
    }
  }
}

void sort_rows(const DCsr& a, hipStream_t s) {
  if (a.n == 0) return;
  Tmp<int> n_long(1), long_rows(a.n);
  HBGS_HIP(hipMemsetAsync(n_long.p, 0, sizeof(int), s));
  // (a wavefront for every row would pass a launch's 2^32 threads from 2^26 rows on)
  k_sort_rows_wave<<<grid_for(a.n, BLK / 64, 1 << 22), BLK, 0, s>>>(a.n, a.rp, a.ci, a.v, n_long.p, long_rows.p);
  static_assert(BLK == 256, "four rows per block");
  HBGS_HIP(hipGetLastError());
  k_sort_long_rows<<<grid_for(a.n, 1, 2048), BLK, 0, s>>>(n_long.p, long_rows.p, a.rp, a.ci, a.v);
  HBGS_HIP(hipGetLastError());
  if (a.m > LONG_LDS) {  // a row can be that long
    k_sort_huge_rows<<<grid_for(a.n, BLK, 256), BLK, 0, s>>>(n_long.p, long_rows.p, a.rp, a.ci, a.v);
    HBGS_HIP(hipGetLastError());
  }
}

void transpose(const DCsr& a, DCsr& t, hipStream_t s) {
  t.n = a.m;
  t.m = a.n;
  t.nnz = a.nnz;
  Tmp<int> cnt(a.m);
  HBGS_HIP(hipMemsetAsync(cnt.p, 0, sizeof(int) * a.m, s));
  k_col_count<<<grid_for(a.nnz, BLK), BLK, 0, s>>>(a.nnz, a.ci, cnt.p);
  HBGS_HIP(hipGetLastError());
  counts_to_rowptr(cnt.p, t.rp, a.m, s);
  HBGS_HIP(hipMemcpyAsync(cnt.p, t.rp, sizeof(int) * a.m, hipMemcpyDeviceToDevice, s));
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_transpose_scatter, L, a.n, s, a.n, a.rp, a.ci, a.v, cnt.p, t.ci, t.v);
  sort_rows(t, s);
}

// ----------------------------------------------------------- block extract
template <int L>
__global__ void k_block_count(int r0, int r1, const int* rp, const int* ci, int c0, int c1, int* cnt) {
  const int64_t m = r1 - r0;
  ROW_GROUPS(L, t, gl, m) {
    const int i = r0 + (int)t;
    int c = 0;
    for (int k = rp[i] + gl; k < rp[i + 1]; k += L) c += (ci[k] >= c0 && ci[k] < c1) ? 1 : 0;
    c = grp_sum<L>(c);
    if (gl == 0) cnt[t] = c;
  }
}
// the block's pattern, and for each entry pos[k] (null: k) of its entry k of a
template <int L>
__global__ void k_block_fill(int r0, int r1, const int* rp, const int* ci, const int* pos, int c0, int c1, int coff,
                             const int* rpo, int* cio, int* src) {
  const int64_t m = r1 - r0;
  ROW_GROUPS(L, t, gl, m) {
    const int i = r0 + (int)t, e = rp[i + 1];
    int q = rpo[t];
    for (int b = rp[i]; b < e; b += L) {
      const int k = b + gl;
      const int c = k < e ? ci[k] : -1;
      const bool keep = k < e && c >= c0 && c < c1;
      int tot;
      const int r = grp_rank<L>(keep, &tot);
      if (keep) {
        cio[q + r] = c - coff;
        src[q + r] = pos ? pos[k] : k;
      }
      q += tot;
    }
  }
}
void block_count(const DCsr& a, int r0, int r1, int c0, int c1, int* cnt, hipStream_t s) {
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_block_count, L, r1 - r0, s, r0, r1, a.rp, a.ci, c0, c1, cnt);
}
void block_pattern(const DCsr& a, const int* pos, int r0, int r1, int c0, int c1, int coff, const int* rp_out,
                   int* ci_out, int* src, hipStream_t s) {
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_block_fill, L, r1 - r0, s, r0, r1, a.rp, a.ci, pos, c0, c1, coff, rp_out, ci_out, src);
}

// ---------------------------------------------------------------- strength
template <int L>
__global__ void k_diagonal(int n, const int* rp, const int* ci, const double* v, double* d, int* missing) {
  ROW_GROUPS(L, i, gl, n) {
    int pos = -1;
    for (int k = rp[i] + gl; k < rp[i + 1]; k += L)
      if (ci[k] == (int)i) pos = k;
    pos = grp_max<L>(pos);
    if (gl == 0) {
      const double x = pos >= 0 ? v[pos] : 0.0;
      d[i] = x;
      if (pos < 0 || x == 0.0) atomicOr(missing, 1);
    }
  }
}
void diagonal(const DCsr& a, double* d, int* missing, hipStream_t s) {
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_diagonal, L, a.n, s, a.n, a.rp, a.ci, a.v, d, missing);
}

// (i,j) strong: a_ij*a_ij >= (theta^2 |a_ii|) |a_jj|, or the same test on the
// transposed entry (j,i); rows with no off-diagonal entry are excluded
template <int L>
__global__ void k_strength(int n, const int* rp, const int* ci, const double* v, const double* d, double th2,
                           char* strong, char* excluded) {
  constexpr int U = row_regs(L);
  ROW_GROUPS(L, i, gl, n) {
    int offd = 0;
    const int e = rp[i + 1];
    const double di = fabs(d[i]);
    for (int b = rp[i] + gl; b < e; b += L * U) {
      int c[U];
      double x[U], dj[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = b + u * L;
        c[u] = k < e ? ci[k] : (int)i;
        x[u] = k < e ? v[k] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) dj[u] = fabs(d[c[u]]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = b + u * L, j = c[u];
        if (k >= e) continue;
        if (j == (int)i) {
          strong[k] = 0;
          continue;
        }
        offd = 1;
        bool st = x[u] * x[u] >= (th2 * di) * dj[u];
        if (!st) {
          int lo = rp[j], hi = rp[j + 1] - 1;
          while (lo <= hi) {
            const int mid = (lo + hi) >> 1;
            const int cm = ci[mid];
            if (cm == (int)i) {
              st = v[mid] * v[mid] >= (th2 * dj[u]) * di;
              break;
            }
            if (cm < (int)i)
              lo = mid + 1;
            else
              hi = mid - 1;
          }
        }
        strong[k] = st ? 1 : 0;
      }
    }
    offd = grp_max<L>(offd);
    if (gl == 0) excluded[i] = offd ? 0 : 1;
  }
}
void strength(const DCsr& a, const double* d, double theta, char* strong, char* excluded, hipStream_t s) {
  const int L = scan_lanes(a);
  LAUNCH_ROW_GROUPS(k_strength, L, a.n, s, a.n, a.rp, a.ci, a.v, d, theta * theta, strong, excluded);
}

// ---------------------------------------------------------------- MIS-2
// Synchronous rounds: an undecided row becomes a root when its key is the
// largest among the undecided rows within strength distance 2 (the maxima
// propagate through all rows, decided or not); rows within distance 2 of a
// root leave.  This yields the greedy maximal distance-2 independent set
// taken in decreasing key order.
// A row without undecided rows among itself and its neighbours (m1 = 0) never
// has one again, and what a round leaves in its r1 only decided rows would
// read, so every round after the first passes over such rows: a round's four
// passes then read 8-12 bytes per row instead of its entries (four fields of
// 1M rows side by side: rounds 5 to 7 of 7 took 200-300 us each, now 90-180).
__global__ void k_mis2_init(int n, const char* excluded, char* state) {
  GRID_STRIDE(i, n) state[i] = excluded[i] ? 3 : 0;
}
// f(j) for every strong neighbour j that lane gl of row i's group holds
template <int L, class F>
__device__ __forceinline__ void strong_neighbours(int s, int e, int gl, const int* ci, const char* strong, F f) {
  constexpr int U = row_regs(L);
  for (int b = s + gl; b < e; b += L * U) {
    int c[U];
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = b + u * L;
      on[u] = k < e && strong[k];
      c[u] = k < e ? ci[k] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (on[u]) f(c[u]);
  }
}
template <int L>
__global__ void k_mis2_max1(int n, const int* rp, const int* ci, const char* strong, uint64_t salt,
                            const char* state, uint64_t* m1, bool first, int* undecided) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *undecided = 0;  // counted by the round's last pass
  ROW_GROUPS(L, i, gl, n) {
    if (!first && m1[i] == 0) continue;
    uint64_t m = (gl == 0 && state[i] == 0) ? agg_key((int)i, salt) : 0;
    strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int j) {
      const uint64_t kj = state[j] == 0 ? agg_key(j, salt) : 0;
      m = kj > m ? kj : m;
    });
    m = grp_max<L>(m);
    if (gl == 0) m1[i] = m;
  }
}
template <int L>
__global__ void k_mis2_max2(int n, const int* rp, const int* ci, const char* strong, uint64_t salt,
                            const uint64_t* m1, char* state) {
  ROW_GROUPS(L, i, gl, n) {
    if (state[i] != 0) continue;
    uint64_t m = m1[i];
    strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int j) {
      const uint64_t mj = m1[j];
      m = mj > m ? mj : m;
    });
    m = grp_max<L>(m);
    if (gl == 0 && m == agg_key((int)i, salt)) state[i] = 1;
  }
}
template <int L>
__global__ void k_mis2_near1(int n, const int* rp, const int* ci, const char* strong, const char* state,
                             const uint64_t* m1, char* r1, bool first) {
  ROW_GROUPS(L, i, gl, n) {
    if (!first && (m1[i] == 0 || r1[i])) continue;  // once next to a root, always
    int r = state[i] == 1;
    strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int j) { r |= state[j] == 1; });
    r = grp_max<L>(r);
    if (gl == 0) r1[i] = (char)r;
  }
}
template <int L>
__global__ void k_mis2_near2(int n, const int* rp, const int* ci, const char* strong, const char* r1,
                             char* state, int* undecided) {
  int local = 0;
  ROW_GROUPS(L, i, gl, n) {
    if (state[i] != 0) continue;
    int out = r1[i];
    if (!out) strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int j) { out |= r1[j]; });
    out = grp_max<L>(out);
    if (gl == 0) {
      if (out)
        state[i] = 2;
      else
        ++local;
    }
  }
  // one atomic per block (the grid is capped, so there are few)
  __shared__ int red[BLK / 64];
  for (int off = 32; off > 0; off >>= 1) local += __shfl_xor(local, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = local;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < BLK / 64; ++w) local += red[w];
    if (local) atomicAdd(undecided, local);
  }
}

void mis2_init(int n, const char* excluded, char* state, hipStream_t s) {
  k_mis2_init<<<grid_for(n, BLK), BLK, 0, s>>>(n, excluded, state);
  HBGS_HIP(hipGetLastError());
}

void mis2_round(const DCsr& a, const char* strong, uint64_t salt, char* state, uint64_t* m1, char* r1,
                bool first, int* undecided, hipStream_t s) {
  const int L = scan_lanes(a);
  LAUNCH_ROW_GROUPS(k_mis2_max1, L, a.n, s, a.n, a.rp, a.ci, strong, salt, state, m1, first, undecided);
  LAUNCH_ROW_GROUPS(k_mis2_max2, L, a.n, s, a.n, a.rp, a.ci, strong, salt, m1, state);
  LAUNCH_ROW_GROUPS(k_mis2_near1, L, a.n, s, a.n, a.rp, a.ci, strong, state, m1, r1, first);
  LAUNCH_ROW_GROUPS_CAP(k_mis2_near2, L, a.n, 2048, s, a.n, a.rp, a.ci, strong, r1, state, undecided);
}

__global__ void k_agg_roots(int n, const char* state, int* flag) {
  GRID_STRIDE(i, n) flag[i] = state[i] == 1 ? 1 : 0;
}
void agg_roots(int n, const char* state, int* flag, hipStream_t s) {
  k_agg_roots<<<grid_for(n, BLK), BLK, 0, s>>>(n, state, flag);
  HBGS_HIP(hipGetLastError());
}

// phase 1: a row next to a root joins it (the root is unique: roots are at
// least 3 apart); phase 2: other rows join the phase-1 neighbour of largest
// key; rows left over are flagged for phase 3
template <int L>
__global__ void k_agg_phase1(int n, const int* rp, const int* ci, const char* strong, const char* state,
                             const int64_t* root_rank, int* p1) {
  ROW_GROUPS(L, i, gl, n) {
    int a = -1;
    if (state[i] == 1) {
      a = (int)root_rank[i];
    } else if (state[i] != 3) {
      int root = -1;
      strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int j) { root = state[j] == 1 ? j : root; });
      a = root >= 0 ? (int)root_rank[root] : -1;
      a = grp_max<L>(a);
    }
    if (gl == 0) p1[i] = a;
  }
}
// the phase-1 neighbour of largest key (keys are distinct, so the maximum
// is the row's unique choice)
template <int L>
__global__ void k_agg_phase2(int n, const int* rp, const int* ci, const char* strong, uint64_t salt,
                             const char* state, const int* p1, int* agg, int* single_flag) {
  ROW_GROUPS(L, i, gl, n) {
    int a = p1[i];
    int single = 0;
    if (state[i] != 3 && a < 0) {
      uint64_t best = 0;
      int bestu = -1;
      strong_neighbours<L>(rp[i], rp[i + 1], gl, ci, strong, [&](int u) {
        if (p1[u] >= 0 && state[u] != 1) {
          const uint64_t ku = agg_key(u, salt);
          if (bestu < 0 || ku > best) {
            best = ku;
            bestu = u;
          }
        }
      });
      const uint64_t top = grp_max<L>(bestu < 0 ? 0ull : best + 1);  // 0: no candidate
      a = top ? p1[(int)(uint32_t)((top - 1) & 0xffffffffull)] : -1;
      single = top ? 0 : 1;
    }
    if (gl == 0) {
      agg[i] = a;
      single_flag[i] = single;
    }
  }
}
__global__ void k_agg_phase3(int n, const int* single_flag, const int64_t* single_rank, int nroot, int* agg) {
  GRID_STRIDE(i, n) if (single_flag[i]) agg[i] = nroot + (int)single_rank[i];
}

void agg_phase12(const DCsr& a, const char* strong, uint64_t salt, const char* state, const int64_t* root_rank,
                 int* agg, int* single_flag, hipStream_t s) {
  Tmp<int> p1(a.n);
  const int L = scan_lanes(a);
  LAUNCH_ROW_GROUPS(k_agg_phase1, L, a.n, s, a.n, a.rp, a.ci, strong, state, root_rank, p1.p);
  LAUNCH_ROW_GROUPS(k_agg_phase2, L, a.n, s, a.n, a.rp, a.ci, strong, salt, state, p1.p, agg, single_flag);
}
void agg_phase3(int n, const int* single_flag, const int64_t* single_rank, int nroot, int* agg, hipStream_t s) {
  k_agg_phase3<<<grid_for(n, BLK), BLK, 0, s>>>(n, single_flag, single_rank, nroot, agg);
  HBGS_HIP(hipGetLastError());
}

// ------------------------------------------------------------------ filter
// A_F: strong off-diagonal entries kept, dropped entries added to the
// diagonal in ascending column order; D_abs = sum |A_F| along the row
template <int L>
__global__ void k_filter_count(int n, const int* rp, const int* ci, const char* strong, int* cnt) {
  constexpr int U = row_regs(L);
  ROW_GROUPS(L, i, gl, n) {
    int c = 0;
    const int e = rp[i + 1];
    for (int b = rp[i] + gl; b < e; b += L * U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = b + u * L;
        const int j = k < e ? ci[k] : -1;
        const bool st = k < e && strong[k];
        c += j == (int)i || st;
      }
    }
    c = grp_sum<L>(c);
    if (gl == 0) cnt[i] = c;
  }
}
// the group's first L * row_regs(L) entries stay in registers; only longer
// rows read the rest again
template <int L>
__global__ void k_filter_fill(int n, const int* rp, const int* ci, const double* v, const char* strong,
                              const int* rpf, int* cif, double* vf, double* dabs) {
  constexpr int U = row_regs(L);
  ROW_GROUPS(L, i, gl, n) {
    const int s = rp[i], e = rp[i + 1], more = s + L * U;
    int c[U];
    double x[U];
    bool st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = s + u * L + gl;
      c[u] = k < e ? ci[k] : -1;
      x[u] = k < e ? v[k] : 0.0;
      st[u] = k < e && strong[k];
    }
    int pos = -1;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] == (int)i) pos = s + u * L + gl;
    for (int k = more + gl; k < e; k += L)
      if (ci[k] == (int)i) pos = k;
    pos = grp_max<L>(pos);
    // diagonal of A_F: a_ii, then the dropped entries in column order
    double d = pos >= 0 ? v[pos] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool drop = c[u] >= 0 && c[u] != (int)i && !st[u];
      d = grp_ordered_add<L>(d, drop ? x[u] : 0.0, drop);
    }
    for (int b = more; b < e; b += L) {
      const int k = b + gl;
      const bool drop = k < e && ci[k] != (int)i && !strong[k];
      d = grp_ordered_add<L>(d, drop ? v[k] : 0.0, drop);
    }
    int q = rpf[i];
    double sa = 0.0;
    auto put = [&](int col, double val, bool on) {
      const bool diag = col == (int)i;
      const bool keep = diag || on;
      const double w = keep ? (diag ? d : val) : 0.0;
      int tot;
      const int r = grp_rank<L>(keep, &tot);
      if (keep) {
        cif[q + r] = col;
        vf[q + r] = w;
      }
      q += tot;
      sa = grp_ordered_add<L>(sa, fabs(w), keep);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) put(c[u], x[u], st[u]);
    for (int b = more; b < e; b += L) {
      const int k = b + gl;
      put(k < e ? ci[k] : -1, k < e ? v[k] : 0.0, k < e && strong[k]);
    }
    if (gl == 0) dabs[i] = sa;
  }
}
void filter_count(const DCsr& a, const char* strong, int* cnt, hipStream_t s) {
  const int L = scan_lanes(a);
  LAUNCH_ROW_GROUPS(k_filter_count, L, a.n, s, a.n, a.rp, a.ci, strong, cnt);
}
void filter_fill(const DCsr& a, const char* strong, const int* rp_f, int* ci_f, double* v_f, double* dabs,
                 hipStream_t s) {
  const int L = scan_lanes(a);
  LAUNCH_ROW_GROUPS(k_filter_fill, L, a.n, s, a.n, a.rp, a.ci, a.v, strong, rp_f, ci_f, v_f, dabs);
}

// ------------------------------------------------------------ power method
__global__ void k_pw_init(int n, uint64_t salt, double* w) {
  GRID_STRIDE(i, n) {
    uint64_t h = splitmix64((uint64_t)(uint32_t)i ^ salt);
    w[i] = 2.0 * ((double)(h >> 11) * 0x1.0p-53) - 1.0;
  }
}
// y = D^-1 B w with every row summed in ascending column order; tracks max |y|.
// w is win, or (amax_in set) win scaled by 2^-e with max|win| = f * 2^e,
// f in [0.5, 1), as the power method normalises its iterate (zero if
// max|win| = 0); the scaling is exact, so folding it into the gather gives
// bitwise the products of the scaled vector.  A block of PW_BLK threads
// takes RB rows: its threads stage the products of PW_CH consecutive
// entries at a time in LDS with coalesced loads, then each row's thread
// (the first RB threads) adds its products in order.  Coarse levels (few
// rows of hundreds of entries) take small RB, so they spread over many
// blocks instead of walking many chunks in a few.
constexpr int PW_BLK = 256;
constexpr int PW_CH = 2048;
template <int RB>
__global__ __launch_bounds__(PW_BLK) void k_pw_apply(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                     const double* __restrict__ v, const double* __restrict__ d,
                                                     const double* __restrict__ win,
                                                     const unsigned long long* amax_in, double* __restrict__ y,
                                                     unsigned long long* amax) {
  static_assert(RB <= PW_BLK, "one thread per row in the sums");
  __shared__ double prod[PW_CH];
  __shared__ unsigned long long sh[PW_BLK / 64];
  bool scaled = amax_in != nullptr, zero = false;
  int e = 0;
  if (scaled) {
    const double mx = __longlong_as_double((long long)*amax_in);
    if (mx > 0.0)
      frexp(mx, &e);
    else
      zero = true;
  }
  unsigned long long m = 0;
  const int64_t nblk = ((int64_t)n + RB - 1) / RB;
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int r0 = (int)(b * RB), r1 = min(r0 + RB, n);
    const int i = r0 + (int)threadIdx.x;
    const bool own = (int)threadIdx.x < RB && i < r1;
    const int e0 = rp[r0], e1 = rp[r1];
    const int my0 = own ? rp[i] : 0, my1 = own ? rp[i + 1] : 0;
    double s = 0.0;
    for (int c0 = e0; c0 < e1; c0 += PW_CH) {
      const int c1 = min(c0 + PW_CH, e1);
      for (int k = c0 + (int)threadIdx.x; k < c1; k += PW_BLK) {
        double w = win[ci[k]];
        if (scaled) w = zero ? 0.0 : ldexp(w, -e);
        prod[k - c0] = v[k] * w;
      }
      __syncthreads();
      const int a = max(my0, c0), z = min(my1, c1);
      for (int k = a; k < z; ++k) s += prod[k - c0];
      __syncthreads();
    }
    if (own) {
      const double yi = d[i] != 0.0 ? s / d[i] : 0.0;  // a zero weight only where the row is zero
      y[i] = yi;
      const unsigned long long bits = (unsigned long long)__double_as_longlong(fabs(yi));
      m = bits > m ? bits : m;
    }
  }
  if (!amax) return;
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < PW_BLK / 64; ++q) m = sh[q] > m ? sh[q] : m;
    atomicMax(amax, m);
  }
}
// rows per block: the largest of 256 ... 4 that still gives 1024 blocks
// (4 per CU), else 4; the grid is capped at 2048 blocks (8 per CU, one
// atomicMax each on a single address) that stride over the row blocks
static void pw_apply(const DCsr& b, const double* d, const double* win, const unsigned long long* amax_in,
                     double* y, unsigned long long* amax, hipStream_t s) {
  const int n = b.n;
  int rb = 4;
  for (int r = 256; r >= 4; r >>= 1)
    if (((int64_t)n + r - 1) / r >= 1024) {
      rb = r;
      break;
    }
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)n + rb - 1) / rb, 2048));
#define HBGS_PW(R)                                                                                   \
  case R:                                                                                            \
    k_pw_apply<R><<<g, PW_BLK, 0, s>>>(n, b.rp, b.ci, b.v, d, win, amax_in, y, amax);                \
    break;
  switch (rb) {
    HBGS_PW(256)
    HBGS_PW(128)
    HBGS_PW(64)
    HBGS_PW(32)
    HBGS_PW(16)
    HBGS_PW(8)
    HBGS_PW(4)
  }
#undef HBGS_PW
  HBGS_HIP(hipGetLastError());
}
// w = y * 2^-e with max|y| = f * 2^e, f in [0.5, 1); *mx_out = max|y|
__global__ void k_pw_scale(int n, const double* y, const unsigned long long* amax, double* w, double* mx_out) {
  double mx = __longlong_as_double((long long)*amax);
  int e = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *mx_out = mx;
  if (mx > 0.0) frexp(mx, &e);
  GRID_STRIDE(i, n) w[i] = mx > 0.0 ? ldexp(y[i], -e) : 0.0;
}
// fixed-association sum: consecutive runs of 256 terms summed in order ...
// A block of 256 threads takes 16 runs: it stages their 4096 products in
// LDS with coalesced loads (every load in flight at once), then 16 threads
// add one run each, in index order.  Terms beyond n are staged as +0.0,
// which leaves a sum that starts at +0.0 unchanged.
constexpr int DOT_RUNS = 16;
// blockIdx.y = 0: x . y, 1: x . x (part: m run sums each)
__global__ __launch_bounds__(256) void k_chunk_dot(int64_t n, const double* x, const double* y, double* part) {
  __shared__ double tile[DOT_RUNS][257];
  const int64_t m = (n + 255) / 256;
  const int t = (int)threadIdx.x;
  if (blockIdx.y) {
    y = x;
    part += m;
  }
  for (int64_t c0 = (int64_t)blockIdx.x * DOT_RUNS; c0 < m; c0 += (int64_t)gridDim.x * DOT_RUNS) {
#pragma unroll
    for (int r = 0; r < DOT_RUNS; ++r) {
      const int64_t i = (c0 + r) * 256 + t;
      tile[r][t] = i < n ? x[i] * y[i] : 0.0;
    }
    __syncthreads();
    if (t < DOT_RUNS && c0 + t < m) {
      double s = 0.0;
      for (int j = 0; j < 256; ++j) s += tile[t][j];
      part[c0 + t] = s;
    }
    __syncthreads();
  }
}
// ... then the m run sums added in order: block q stages 4096 of sum q's in
// LDS at a time, one thread adds them
constexpr int RUN_STAGE = 4096;
__global__ void __launch_bounds__(256) k_chunk_total(int64_t m, const double* part, double* out) {
  __shared__ double sh[RUN_STAGE];
  part += (int64_t)blockIdx.x * m;
  double s = 0.0;
  for (int64_t c0 = 0; c0 < m; c0 += RUN_STAGE) {
    const int e = (int)(m - c0 < RUN_STAGE ? m - c0 : RUN_STAGE);
    for (int t = threadIdx.x; t < e; t += blockDim.x) sh[t] = part[c0 + t];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll 16
      for (int t = 0; t < e; ++t) s += sh[t];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// out[0] = x . y, out[1] = x . x
static void chunked_dots(int64_t n, const double* x, const double* y, double* part, double* out, hipStream_t s) {
  const int64_t m = (n + 255) / 256;
  k_chunk_dot<<<dim3(grid_for(m, DOT_RUNS, 2048), 2), 256, 0, s>>>(n, x, y, part);
  k_chunk_total<<<2, 256, 0, s>>>(m, part, out);
  HBGS_HIP(hipGetLastError());
}

double power_estimate(const DCsr& b, const double* d, int iters, uint64_t salt, hipStream_t s) {
  const int n = b.n;
  if (n == 0) return 0.0;
  Tmp<double> w(n), y(n), pa(2 * (((int64_t)n + 255) / 256));
  Tmp<double> res(3);  // the two dots and the last iterate's largest entry
  Tmp<unsigned long long> amax(iters > 0 ? iters : 1);
  const unsigned g = grid_for(n, BLK);
  k_pw_init<<<g, BLK, 0, s>>>(n, salt, w.p);
  HBGS_HIP(hipGetLastError());
  if (iters > 0) HBGS_HIP(hipMemsetAsync(amax.p, 0, sizeof(unsigned long long) * iters, s));
  // iterate it reads the previous one scaled on the fly: w -> y -> w -> ...
  double* buf[2] = {y.p, w.p};
  for (int it = 0; it < iters; ++it) {
    pw_apply(b, d, buf[(it + 1) & 1], it ? amax.p + it - 1 : nullptr, buf[it & 1], amax.p + it, s);
  }
  double h[3] = {0.0, 0.0, 0.0};
  if (iters > 0) {
    // the normalised last iterate and its image (all zero when it vanished)
    double* last = buf[(iters - 1) & 1];
    double* other = buf[iters & 1];
    k_pw_scale<<<g, BLK, 0, s>>>(n, last, amax.p + iters - 1, other, res.p + 2);
    HBGS_HIP(hipGetLastError());
    pw_apply(b, d, other, nullptr, last, nullptr, s);
    chunked_dots(n, other, last, pa.p, res.p, s);
    read_back(h, res.p, sizeof(h), s);
    return h[2] == 0.0 ? 0.0 : h[0] / h[1];
  }
  pw_apply(b, d, w.p, nullptr, y.p, nullptr, s);
  chunked_dots(n, w.p, y.p, pa.p, res.p, s);
  read_back(h, res.p, 2 * sizeof(double), s);
  return h[0] / h[1];
}

// ------------------------------------------------------ smoothed prolongator
// Row i of P = P_tent - omega D_abs^-1 A_F P_tent: its columns are the
// aggregates met along row i of A_F (ascending); entry c is
// [agg(i)==c] - (omega / D_abs_i) * sum_{k: agg(k)==c} a_F(i,k).
// A group's first L * row_regs(L) entries stay in registers over the passes
// below, one per aggregate met; only longer rows read the rest again.
template <int L>
__global__ void k_psmooth_count(int n, const int* rp, const int* ci, const int* agg, int* cnt) {
  constexpr int U = row_regs(L);
  ROW_GROUPS(L, i, gl, n) {
    int c = 0;
    if (agg[i] >= 0) {
      const int s = rp[i], e = rp[i + 1];
      int a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = s + u * L + gl < e ? ci[s + u * L + gl] : -1;
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = a[u] >= 0 ? agg[a[u]] : -1;
      int prev = -1;
      for (;;) {
        int next = INT32_MAX;
#pragma unroll
        for (int u = 0; u < U; ++u) next = a[u] > prev && a[u] < next ? a[u] : next;
        for (int k = s + L * U + gl; k < e; k += L) {
          const int b = agg[ci[k]];
          if (b > prev && b < next) next = b;
        }
        next = grp_min<L>(next);
        if (next == INT32_MAX) break;
        ++c;
        prev = next;
      }
    }
    if (gl == 0) cnt[i] = c;
  }
}
template <int L>
__global__ void k_psmooth_fill(int n, const int* rp, const int* ci, const double* v, const int* agg,
                               const double* dabs, double omega, const int* rpp, int* cip, double* vp) {
  constexpr int U = row_regs(L);
  ROW_GROUPS(L, i, gl, n) {
    const int ai = agg[i];
    if (ai < 0) continue;
    const double q = dabs[i] != 0.0 ? omega / dabs[i] : 0.0;  // a zero row of A_F: no smoothing term
    const int s = rp[i], e = rp[i + 1];
    int a[U];
    double x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = s + u * L + gl;
      a[u] = k < e ? ci[k] : -1;
      x[u] = k < e ? v[k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = a[u] >= 0 ? agg[a[u]] : -1;
    int o = rpp[i];
    int cur = -1;
    // one pass per aggregate met: its entries summed in column order, and
    // the next larger aggregate (the first pass looks for the smallest only)
    for (;;) {
      double sum = 0.0;
      int next = INT32_MAX;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool hit = cur >= 0 && a[u] == cur;
        sum = grp_ordered_add<L>(sum, hit ? x[u] : 0.0, hit);
        next = a[u] > cur && a[u] < next ? a[u] : next;
      }
      for (int b = s + L * U; b < e; b += L) {
        const int k = b + gl;
        const int ak = k < e ? agg[ci[k]] : -1;
        const bool hit = cur >= 0 && ak == cur;
        sum = grp_ordered_add<L>(sum, hit ? v[k] : 0.0, hit);
        if (ak > cur && ak < next) next = ak;
      }
      next = grp_min<L>(next);
      if (cur >= 0) {
        if (gl == 0) {
          const double tent = ai == cur ? 1.0 : 0.0;
          cip[o] = cur;
          vp[o] = tent - q * sum;
        }
        ++o;
      }
      if (next == INT32_MAX) break;
      cur = next;
    }
  }
}
void psmooth_count(const DCsr& af, const int* agg, int* cnt, hipStream_t s) {
  const int L = scan_lanes(af);
  LAUNCH_ROW_GROUPS(k_psmooth_count, L, af.n, s, af.n, af.rp, af.ci, agg, cnt);
}
void psmooth_fill(const DCsr& af, const int* agg, const double* dabs, double omega, const int* rp_p, int* ci_p,
                  double* v_p, hipStream_t s) {
  const int L = scan_lanes(af);
  LAUNCH_ROW_GROUPS(k_psmooth_fill, L, af.n, s, af.n, af.rp, af.ci, af.v, agg, dabs, omega, rp_p, ci_p, v_p);
}

// ------------------------------------------------------------------ SpGEMM
// C = A B, Gustavson row by row.  Each row of C owns an open-addressing
// table whose slots accumulate the products a_ik b_kj in the order they are
// generated, i.e. ascending k, starting from 0.0; the occupied slots are
// then written out in column order.  The pattern is structural (entries
// that cancel to zero are kept).
//
// Rows whose tables fit in LDS are done by one wavefront each: the wave
// walks the row of A in order and its lanes take the entries of one row of
// B at a time.  The columns of one B row are distinct, so no two lanes
// update the same slot in one step, and a wave's LDS operations complete in
// program order, so each slot still sums its products in ascending k.  The
// remaining rows use one thread each and a table in global scratch memory.
// (one thread per row took 240-310 us on the long rows of R)
template <int L>
__global__ void k_spgemm_ub(int n, const int* arp, const int* aci, const int* brp, int64_t* ub) {
  ROW_GROUPS(L, i, gl, n) {
    int64_t u = 0;
    for (int k = arp[i] + gl; k < arp[i + 1]; k += L) {
      const int c = aci[k];
      u += brp[c + 1] - brp[c];
    }
    for (int off = L >> 1; off > 0; off >>= 1) u += __shfl_xor(u, off, L);
    if (gl == 0) ub[i] = u;
  }
}
__host__ __device__ __forceinline__ int64_t table_size(int64_t ub) {
  if (ub == 0) return 0;
  int64_t t = 16;
  while (t < 2 * ub) t <<= 1;
  return t;
}
__device__ __forceinline__ uint32_t hslot(int c, uint32_t mask) { return ((uint32_t)c * 2654435761u) & mask; }

constexpr int SPG_WAVES = 4;          // rows (waves) per block
constexpr int SPG_SYM_SLOTS = 1024;   // symbolic: keys per wave (4 KB: 8 blocks of 4 waves per CU)
constexpr int SPG_NUM_SLOTS = 512;    // numeric: keys and values per wave (6 KB: 6 blocks per CU)
constexpr int SPG_BLK_SLOTS = 4096;  // numeric, one block per row: keys and values (48 KB)
// distinct columns of a product row are at most min(ub, columns of B)
__device__ __forceinline__ int64_t sym_need(int64_t ub, int m) { return ub < m ? ub : (int64_t)m; }

// slot holding key c (claimed if absent); -1 if the table is full, which
// the table sizes rule out (the caller reports it instead of looping);
// lds_claim_bounded gives up after max_probes slots
__device__ __forceinline__ int lds_claim_bounded(int* keys, uint32_t mask, int c, uint32_t max_probes, bool* fresh) {
  uint32_t h = hslot(c, mask);
  for (uint32_t probe = 0; probe < max_probes && probe <= mask; ++probe) {
    int prev = atomicCAS(&keys[h], -1, c);
    if (prev == -1 || prev == c) {
      *fresh = prev == -1;
      return (int)h;
    }
    h = (h + 1) & mask;
  }
  *fresh = false;
  return -1;
}
__device__ __forceinline__ int lds_claim(int* keys, uint32_t mask, int c, bool* fresh) {
  uint32_t h = hslot(c, mask);
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    int prev = atomicCAS(&keys[h], -1, c);
    if (prev == -1 || prev == c) {
      *fresh = prev == -1;
      return (int)h;
    }
    h = (h + 1) & mask;
  }
  *fresh = false;
  return -1;
}

// Groups of LPR lanes (64 / LPR rows per wavefront): a group walks its row
// of A in order and its lanes take the entries of one row of B at a time.
// Each row owns SLOTS / (64 / LPR) table slots.  The narrow kernels
// (LPR < 64) take the rows whose size measure is at most hi and append the
// others to a list for the one-row-per-wavefront kernels, which stride over
// that list (or over every row) with a device-side count (lanes of one
// wavefront stay in lockstep, so the per-slot order argument above holds
// group by group).
__device__ __forceinline__ int group_table(int64_t need) {  // power of two >= 2 need, at least 16
  int t = 16;
  while (t < 2 * need) t <<= 1;
  return t;
}
template <int LPR>
__global__ __launch_bounds__(64 * SPG_WAVES) void k_spgemm_sym_grp(int n, int bm, const int* arp, const int* aci,
                                                                  const int* brp, const int* bci, const int64_t* ub,
                                                                  int64_t hi, int* cnt, int* overflow) {
  constexpr int G = 64 / LPR, SLOTS = SPG_SYM_SLOTS / G;
  static_assert(LPR < 64, "the wide rows use k_spgemm_sym_wave");
  __shared__ int tab[SPG_WAVES][SPG_SYM_SLOTS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane / LPR, gl = lane % LPR;
  const int64_t i = ((int64_t)blockIdx.x * SPG_WAVES + wave) * G + grp;
  const int64_t need = i < n ? sym_need(ub[i], bm) : 0;
  const bool active = i < n && need <= hi && 2 * need <= SLOTS;
  int u = 0;
  if (active) {
    const int T = group_table(need);
    int* keys = tab[wave] + grp * SLOTS;
    for (int q = gl; q < T; q += LPR) keys[q] = -1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t mask = (uint32_t)(T - 1);
    const int a0 = arp[i], a1 = arp[i + 1], gbase = grp * LPR;
    // A's row LPR entries at a time: the lanes load the entries' B row
    // bounds together, then take the B rows one after another (the distinct
    // count does not depend on the order)
    for (int c0 = a0; c0 < a1; c0 += LPR) {
      const int kl = c0 + gl;
      int bl0 = 0, bl1 = 0;
      if (kl < a1) {
        const int kk = aci[kl];
        bl0 = brp[kk];
        bl1 = brp[kk + 1];
      }
      const int nt = min(LPR, a1 - c0);
      if constexpr (LPR <= 16) {
        int pk[LPR];
#pragma unroll
        for (int t = 0; t < LPR; ++t) {
          const int q = __shfl(bl0, gbase + t) + gl;
          pk[t] = t < nt && q < __shfl(bl1, gbase + t) ? bci[q] : -1;
        }
#pragma unroll
        for (int t = 0; t < LPR; ++t) {
          if (pk[t] >= 0) {
            bool fresh;
            if (lds_claim(keys, mask, pk[t], &fresh) < 0) atomicOr(overflow, 1);
            u += fresh;
          }
        }
        // rows of B longer than LPR
        for (int t = 0; t < nt; ++t) {
          const int b1 = __shfl(bl1, gbase + t);
          for (int q = __shfl(bl0, gbase + t) + gl + LPR; q < b1; q += LPR) {
            bool fresh;
            if (lds_claim(keys, mask, bci[q], &fresh) < 0) atomicOr(overflow, 1);
            u += fresh;
          }
        }
      } else {
        for (int t = 0; t < nt; ++t) {
          const int b1 = __shfl(bl1, gbase + t);
          for (int q = __shfl(bl0, gbase + t) + gl; q < b1; q += LPR) {
            bool fresh;
            if (lds_claim(keys, mask, bci[q], &fresh) < 0) atomicOr(overflow, 1);
            u += fresh;
          }
        }
      }
    }
  }
  for (int off = LPR >> 1; off > 0; off >>= 1) u += __shfl_xor(u, off, LPR);
  if (active && gl == 0) cnt[i] = u;
}

// Symbolic product of one row per wavefront.  The distinct count does not
// depend on the order of insertion, so the row's products are flattened:
// 64 entries of A at a time are loaded together, a prefix sum of their B row
// lengths maps every lane to one product, and each step claims 64 products.
// Rows too large for a table of 2 * need slots (big) get the whole table
// with probing bounded by SPG_BIG_PROBES: the distinct count is usually far
// below the bound need, and a row whose claims fail is marked (cnt = -1) for
// the global-table pass.
constexpr uint32_t SPG_BIG_PROBES = 64;
__global__ __launch_bounds__(64 * SPG_WAVES) void k_spgemm_sym_wave(int n, int bm, const int* arp, const int* aci,
                                                                   const int* brp, const int* bci,
                                                                   const int64_t* ub, const int* rows,
                                                                   const int* nrows, int* cnt) {
  __shared__ int tab[SPG_WAVES][SPG_SYM_SLOTS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t count = rows ? *nrows : n;
  int* keys = tab[wave];
  for (int64_t w = (int64_t)blockIdx.x * SPG_WAVES + wave; w < count; w += (int64_t)gridDim.x * SPG_WAVES) {
    const int i = rows ? rows[w] : (int)w;
    const int64_t need = sym_need(ub[i], bm);
    const bool big = 2 * need > SPG_SYM_SLOTS;
    const int T = big ? SPG_SYM_SLOTS : group_table(need);
    const uint32_t mask = (uint32_t)(T - 1);
    for (int q = lane; q < T; q += 64) keys[q] = -1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int u = 0, failed = 0;
    const int ae = arp[i + 1];
    for (int kb = arp[i]; kb < ae; kb += 64) {
      const int k = kb + lane;
      int beg = 0, len = 0;
      if (k < ae) {
        const int kk = aci[k];
        beg = brp[kk];
        len = brp[kk + 1] - beg;
      }
      int incl = len;
      for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
      }
      const int total = __shfl(incl, 63, 64);
      const int excl = incl - len;
      for (int t0 = 0; t0 < total; t0 += 64) {
        const int tp = t0 + lane;
        int j = 0;  // lanes whose products all come before tp
        for (int step = 32; step > 0; step >>= 1)
          if (__shfl(incl, j + step - 1, 64) <= tp) j += step;
        const int bj = __shfl(beg, j & 63, 64), ej = __shfl(excl, j & 63, 64);
        if (tp < total) {
          bool fresh;
          if (lds_claim_bounded(keys, mask, bci[bj + (tp - ej)], big ? SPG_BIG_PROBES : mask + 1, &fresh) < 0)
            failed = 1;
          u += fresh;
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      u += __shfl_xor(u, off, 64);
      failed |= __shfl_xor(failed, off, 64);
    }
    if (lane == 0) cnt[i] = failed ? -1 : u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// rows whose size measure lies in (lo, hi]: min(ub, bm) with ub given, else
// the row length of crp; one atomic per block reserves the block's places
__global__ __launch_bounds__(BLK) void k_spgemm_list(int n, const int64_t* ub, int bm, const int* crp, int64_t lo,
                                                     int64_t hi, int* list, int* count) {
  __shared__ int nb, base;
  for (int64_t r0 = (int64_t)blockIdx.x * BLK; r0 < n; r0 += (int64_t)gridDim.x * BLK) {
    if (threadIdx.x == 0) nb = 0;
    __syncthreads();
    const int64_t i = r0 + threadIdx.x;
    bool in = false;
    if (i < n) {
      const int64_t m = ub ? sym_need(ub[i], bm) : (int64_t)(crp[i + 1] - crp[i]);
      in = m > lo && m <= hi;
    }
    const int slot = in ? atomicAdd(&nb, 1) : 0;
    __syncthreads();
    if (threadIdx.x == 0 && nb) base = atomicAdd(count, nb);
    __syncthreads();
    if (in) list[base + slot] = (int)i;
    __syncthreads();
  }
}

// numeric: rows is null for every row, else the listed rows (count *nrows)
template <int LPR>
__global__ __launch_bounds__(64 * SPG_WAVES) void k_spgemm_num_grp(int n, const int* arp, const int* aci,
                                                                  const double* av, const int* brp, const int* bci,
                                                                  const double* bv, const int* crp, int64_t hi,
                                                                  const int* rows, const int* nrows, int* cci,
                                                                  double* cv, int* overflow) {
  constexpr int G = 64 / LPR, SLOTS = SPG_NUM_SLOTS / G;
  __shared__ int tk[SPG_WAVES][SPG_NUM_SLOTS];
  __shared__ double tv[SPG_WAVES][SPG_NUM_SLOTS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane / LPR, gl = lane % LPR;
  const int64_t count = rows ? *nrows : n;
  for (int64_t w = ((int64_t)blockIdx.x * SPG_WAVES + wave) * G + grp; w < count;
       w += (int64_t)gridDim.x * SPG_WAVES * G) {
  const int i = rows ? rows[w] : (int)w;
  const int o = crp[i], cnt = crp[i + 1] - o;
  if (cnt > hi || 2 * cnt > SLOTS) continue;  // a wider kernel's row
  const int T = group_table(cnt);
  int* keys = tk[wave] + grp * SLOTS;
  double* vals = tv[wave] + grp * SLOTS;
  for (int q = gl; q < T; q += LPR) {
    keys[q] = -1;
    vals[q] = 0.0;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint32_t mask = (uint32_t)(T - 1);
  const int a0 = arp[i], a1 = arp[i + 1], gbase = grp * LPR;
  // A's row LPR entries at a time: the group's lanes load the entries and
  // the bounds of their rows of B together, then the steps take the entries
  // in order (ascending k), each broadcast from its lane
  for (int c0 = a0; c0 < a1; c0 += LPR) {
    const int kl = c0 + gl;
    double al = 0.0;
    int bl0 = 0, bl1 = 0;
    if (kl < a1) {
      const int kk = aci[kl];
      al = av[kl];
      bl0 = brp[kk];
      bl1 = brp[kk + 1];
    }
    const int nt = min(LPR, a1 - c0);
    if constexpr (LPR <= 16) {
      // every step's first LPR entries of B, requested before the first step
      int pk[LPR];
      double pv[LPR];
#pragma unroll
      for (int t = 0; t < LPR; ++t) {
        const int q = __shfl(bl0, gbase + t) + gl;
        const bool ok = t < nt && q < __shfl(bl1, gbase + t);
        pk[t] = ok ? bci[q] : -1;
        pv[t] = ok ? bv[q] : 0.0;
      }
#pragma unroll
      for (int t = 0; t < LPR; ++t) {
        if (t < nt) {
          const double a = __shfl(al, gbase + t);
          const int b1 = __shfl(bl1, gbase + t);
          int q = __shfl(bl0, gbase + t) + gl;
          if (q < b1) {
            bool fresh;
            const int h = lds_claim(keys, mask, pk[t], &fresh);
            if (h >= 0)
              vals[h] += a * pv[t];
            else
              atomicOr(overflow, 1);
          }
          for (q += LPR; q < b1; q += LPR) {
            bool fresh;
            const int h = lds_claim(keys, mask, bci[q], &fresh);
            if (h >= 0)
              vals[h] += a * bv[q];
            else
              atomicOr(overflow, 1);
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
    } else {
      for (int t = 0; t < nt; ++t) {
        const double a = __shfl(al, gbase + t);
        const int b0 = __shfl(bl0, gbase + t), b1 = __shfl(bl1, gbase + t);
        for (int q = b0 + gl; q < b1; q += LPR) {
          bool fresh;
          const int h = lds_claim(keys, mask, bci[q], &fresh);
          if (h >= 0)
            vals[h] += a * bv[q];
          else
            atomicOr(overflow, 1);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  }
  // Compact the occupied slots to the front of the table, LPR slots at a
  // time (a round's slots are read before its writes, which land at or
  // before them), then each entry goes to its rank among the row's columns.
  int m = 0;
  for (int q0 = 0; q0 < T; q0 += LPR) {
    const bool in = q0 + gl < T;  // T < LPR for short rows of the wide groups
    const int c = in ? keys[q0 + gl] : -1;
    const double x = in ? vals[q0 + gl] : 0.0;
    int tot;
    const int r = grp_rank<LPR>(c >= 0, &tot);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (c >= 0) {
      keys[m + r] = c;
      vals[m + r] = x;
    }
    m += tot;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int q = gl; q < m; q += LPR) {
    const int c = keys[q];
    int rank = 0;
    for (int p = 0; p < m; ++p) rank += keys[p] < c;
    cci[o + rank] = c;
    cv[o + rank] = vals[q];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// one thread per row with its table in global scratch (rows with ts == 0
// are done by the wave kernels)
__global__ void k_spgemm_symbolic(int r0, int r1, const int* arp, const int* aci, const int* brp, const int* bci,
                                  const int64_t* toff, int64_t tbase, int* keys, int* cnt) {
  GRID_STRIDE(t, r1 - r0) {
    int i = r0 + (int)t;
    int64_t ts = toff[i + 1] - toff[i];
    if (ts == 0) continue;
    int* tk = keys + (toff[i] - tbase);
    for (int64_t q = 0; q < ts; ++q) tk[q] = -1;
    int u = 0;
    uint32_t mask = (uint32_t)(ts - 1);
    for (int k = arp[i]; k < arp[i + 1]; ++k) {
      int kk = aci[k];
      for (int q = brp[kk]; q < brp[kk + 1]; ++q) {
        int c = bci[q];
        uint32_t h = hslot(c, mask);
        while (tk[h] != -1 && tk[h] != c) h = (h + 1) & mask;
        if (tk[h] == -1) {
          tk[h] = c;
          ++u;
        }
      }
    }
    cnt[i] = u;
  }
}
__global__ void k_spgemm_numeric(int r0, int r1, const int* arp, const int* aci, const double* av, const int* brp,
                                 const int* bci, const double* bv, const int64_t* toff, int64_t tbase, int* keys,
                                 double* vals, const int* crp, int* cci, double* cv) {
  GRID_STRIDE(t, r1 - r0) {
    int i = r0 + (int)t;
    int64_t ts = toff[i + 1] - toff[i];
    if (ts == 0) continue;
    int* tk = keys + (toff[i] - tbase);
    double* tv = vals + (toff[i] - tbase);
    for (int64_t q = 0; q < ts; ++q) {
      tk[q] = -1;
      tv[q] = 0.0;
    }
    uint32_t mask = (uint32_t)(ts - 1);
    for (int k = arp[i]; k < arp[i + 1]; ++k) {
      int kk = aci[k];
      double a = av[k];
      for (int q = brp[kk]; q < brp[kk + 1]; ++q) {
        int c = bci[q];
        uint32_t h = hslot(c, mask);
        while (tk[h] != -1 && tk[h] != c) h = (h + 1) & mask;
        tk[h] = c;
        tv[h] += a * bv[q];
      }
    }
    int o = crp[i], e = crp[i + 1];
    for (int64_t q = 0; q < ts; ++q)
      if (tk[q] != -1) {
        cci[o] = tk[q];
        cv[o] = tv[q];
        ++o;
      }
    int s = crp[i];
    for (int k = s + 1; k < e; ++k) {
      int c = cci[k];
      double x = cv[k];
      int q = k - 1;
      while (q >= s && cci[q] > c) {
        cci[q + 1] = cci[q];
        cv[q + 1] = cv[q];
        --q;
      }
      cci[q + 1] = c;
      cv[q + 1] = x;
    }
  }
}
// every row with products goes to the global-table pass (route 3)
__global__ void k_spgemm_mark_all(int n, const int64_t* ub, int* cnt) {
  GRID_STRIDE(i, n) cnt[i] = ub[i] > 0 ? -1 : 0;
}
// global table sizes of the rows the group kernels marked (cnt < 0); *any:
// some row has one
__global__ void k_spgemm_tsize_sym(int n, int bm, const int64_t* ub, const int* cnt, int64_t* ts, int* any) {
  int some = 0;
  GRID_STRIDE(i, n) {
    const int64_t t = cnt[i] < 0 ? table_size(sym_need(ub[i], bm)) : 0;
    ts[i] = t;
    some |= t > 0;
  }
  if (some) atomicOr(any, 1);
}
// rows beyond the wave kernels (more than wave_max entries) are listed for
// the one-block-per-row kernel; rows beyond it (block_max) get a global table
// (*any: some row does).  *longest (where given): the longest row, mostly
// found by the first blocks, so that the others only look
__global__ void k_spgemm_tsize_num(int n, const int* crp, int64_t wave_max, int64_t block_max, int64_t* ts,
                                   int* nmid, int* mid, int* any, int* longest) {
  GRID_STRIDE(i, n) {
    const int64_t cnt = crp[i + 1] - crp[i];
    if (longest && (int)cnt > *(volatile int*)longest) atomicMax(longest, (int)cnt);
    ts[i] = 0;
    if (cnt <= wave_max) continue;
    if (cnt <= block_max)
      mid[atomicAdd(nmid, 1)] = (int)i;
    else {
      ts[i] = table_size(cnt);
      atomicOr(any, 1);
    }
  }
}

// numeric product of the *count listed rows, one per block (rows of up to
// SPG_BLK_SLOTS / 2 entries): the threads take the entries of one B row at a
// time and the block synchronises between rows of B, so every slot sums its
// products in ascending k
__global__ __launch_bounds__(BLK) void k_spgemm_num_block(const int* count, const int* rows, const int* arp,
                                                          const int* aci, const double* av, const int* brp, const int* bci,
                                                          const double* bv, const int* crp, int* cci, double* cv,
                                                          int* overflow) {
  __shared__ int keys[SPG_BLK_SLOTS];
  __shared__ double vals[SPG_BLK_SLOTS];
  const int nrows = *count;
  for (int r = blockIdx.x; r < nrows; r += gridDim.x) {
    const int i = rows[r];
    const int o = crp[i], cnt = crp[i + 1] - o;
    int T = 64;
    while (T < 2 * cnt) T <<= 1;
    for (int q = threadIdx.x; q < T; q += BLK) {
      keys[q] = -1;
      vals[q] = 0.0;
    }
    __syncthreads();
    const uint32_t mask = (uint32_t)(T - 1);
    for (int k = arp[i]; k < arp[i + 1]; ++k) {
      const int kk = aci[k];
      const double a = av[k];
      for (int q = brp[kk] + threadIdx.x; q < brp[kk + 1]; q += BLK) {
        bool fresh;
        const int h = lds_claim(keys, mask, bci[q], &fresh);
        if (h >= 0)
          vals[h] += a * bv[q];
        else
          atomicOr(overflow, 1);
      }
      __syncthreads();
    }
    for (int q = threadIdx.x; q < T; q += BLK) {
      const int c = keys[q];
      if (c < 0) continue;
      int rank = 0;
      for (int p = 0; p < T; ++p) {
        const int d = keys[p];
        rank += (d >= 0) & (d < c);
      }
      cci[o + rank] = c;
      cv[o + rank] = vals[q];
    }
    __syncthreads();  // the tables are cleared for the next row
  }
}

// row batches whose global tables fit the scratch budget; returns the largest batch
static int64_t batch_rows(const std::vector<int64_t>& off, int n, std::vector<int>& cuts) {
  const int64_t budget = int64_t(64) << 20;  // table slots
  cuts.assign(1, 0);
  int64_t maxbatch = 0;
  while (cuts.back() < n) {
    int r0 = cuts.back();
    int r1 = (int)(std::upper_bound(off.begin() + r0 + 1, off.end(), off[r0] + budget) - off.begin()) - 1;
    if (r1 <= r0) r1 = r0 + 1;
    if (r1 > n) r1 = n;
    maxbatch = std::max(maxbatch, off[r1] - off[r0]);
    cuts.push_back(r1);
  }
  return maxbatch;
}

static std::atomic<int> g_spgemm_route{0};
void set_spgemm_route(int route) { g_spgemm_route.store(route); }

void spgemm(const DCsr& a, const DCsr& b, DCsr& c, Pool& pool, hipStream_t s, bool longest) {
  const int n = a.n;
  // route: 0 by row size; 1 every row to the one-row-per-wavefront kernels;
  // 2 numeric rows to the one-block-per-row kernel; 3 every row to the
  // global-memory tables (the paths give bitwise the same product)
  const int route = g_spgemm_route.load();
  c.n = n;
  c.m = b.m;
  Tmp<int64_t> ub(n), ts(n), toff(n + 1);
  // counters: accumulator overflow, rows with global tables (symbolic,
  // numeric), wide rows (symbolic, numeric), one-block rows, longest row
  enum { OVF, ANY_SYM, ANY_NUM, WIDE_SYM, WIDE_NUM, MID, LONGEST, NFLAGS };
  Tmp<int> cnt(n), flags(NFLAGS);
  int* overflow = flags.p + OVF;
  HBGS_HIP(hipMemsetAsync(flags.p, 0, NFLAGS * sizeof(int), s));
  LAUNCH_ROW_GROUPS(k_spgemm_ub, row_lanes(n, a.nnz), n, s, n, a.rp, a.ci, b.rp, ub.p);
  // lanes per row from the mean length of B's rows; rows too long for the
  // group tables go to the one-row-per-wavefront kernels
  const double bavg = b.n ? (double)b.nnz / b.n : 0.0;
  const int lpr = bavg <= 8.0 ? 8 : bavg <= 16.0 ? 16 : bavg <= 32.0 ? 32 : 64;
  const int64_t sym_g = route ? 0 : SPG_SYM_SLOTS / (64 / lpr) / 2;
  const int64_t num_g = route ? 0 : SPG_NUM_SLOTS / (64 / lpr) / 2;
  const int64_t num_w = route >= 2 ? 0 : SPG_NUM_SLOTS / 2;              // wave kernel's rows
  const int64_t num_b = route == 3 ? 0 : SPG_BLK_SLOTS / 2;              // block kernel's rows
  auto groups = [&](int l) { return (unsigned)(((int64_t)n + (int64_t)SPG_WAVES * (64 / l) - 1) / (SPG_WAVES * (64 / l))); };
  // the wide kernels stride over the listed rows (every row when lpr = 64)
  Tmp<int> wide(lpr < 64 ? n : 1);
  int* wl = lpr < 64 ? wide.p : nullptr;
  int* wn = lpr < 64 ? flags.p + WIDE_SYM : nullptr;
  const unsigned wgrid = lpr < 64 ? grid_for(n, SPG_WAVES, 8192) : grid_for(n, SPG_WAVES);
  // symbolic: distinct columns per row
#define HBGS_SYM(L)                                                                                            \
  k_spgemm_sym_grp<L><<<groups(L), 64 * SPG_WAVES, 0, s>>>(n, b.m, a.rp, a.ci, b.rp, b.ci, ub.p, sym_g, cnt.p, \
                                                           overflow)
  if (route == 3) {
    k_spgemm_mark_all<<<grid_for(n, BLK), BLK, 0, s>>>(n, ub.p, cnt.p);
  } else {
    switch (lpr) {
      case 8: HBGS_SYM(8); break;
      case 16: HBGS_SYM(16); break;
      case 32: HBGS_SYM(32); break;
      default: break;
    }
    if (lpr < 64)
      k_spgemm_list<<<grid_for(n, BLK, 8192), BLK, 0, s>>>(n, ub.p, b.m, nullptr, sym_g, INT64_MAX, wide.p,
                                                           flags.p + WIDE_SYM);
    k_spgemm_sym_wave<<<wgrid, 64 * SPG_WAVES, 0, s>>>(n, b.m, a.rp, a.ci, b.rp, b.ci, ub.p, wl, wn, cnt.p);
  }
#undef HBGS_SYM
  HBGS_HIP(hipGetLastError());
  k_spgemm_tsize_sym<<<grid_for(n, BLK, 4096), BLK, 0, s>>>(n, b.m, ub.p, cnt.p, ts.p, flags.p + ANY_SYM);
  HBGS_HIP(hipGetLastError());
  std::vector<int64_t> h_off;  // row offsets of the global tables, only when some row needs one
  std::vector<int> cuts;
  if (read_one(flags.p + ANY_SYM, s)) {
    scan_i64(ts.p, toff.p, n, s);
    h_off.resize(n + 1);
    HBGS_HIP(hipMemcpyAsync(h_off.data(), toff.p, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToHost, s));
    HBGS_HIP(hipStreamSynchronize(s));
    Tmp<int> keys(batch_rows(h_off, n, cuts));
    for (size_t q = 0; q + 1 < cuts.size(); ++q) {
      int r0 = cuts[q], r1 = cuts[q + 1];
      if (h_off[r1] == h_off[r0]) continue;
      k_spgemm_symbolic<<<grid_for(r1 - r0, 64), 64, 0, s>>>(r0, r1, a.rp, a.ci, b.rp, b.ci, toff.p, h_off[r0],
                                                             keys.p, cnt.p);
      HBGS_HIP(hipGetLastError());
    }
  }
  c.rp = pool.make<int>(n + 1);
  c.nnz = counts_to_rowptr(cnt.p, c.rp, n, s);
  c.ci = pool.make<int>(c.nnz);
  c.v = pool.make<double>(c.nnz);
  // numeric
#define HBGS_NUM(L)                                                                                            \
  k_spgemm_num_grp<L><<<groups(L), 64 * SPG_WAVES, 0, s>>>(n, a.rp, a.ci, a.v, b.rp, b.ci, b.v, c.rp, num_g,     \
                                                           nullptr, nullptr, c.ci, c.v, overflow)
  switch (lpr) {
    case 8: HBGS_NUM(8); break;
    case 16: HBGS_NUM(16); break;
    case 32: HBGS_NUM(32); break;
    default: break;
  }
#undef HBGS_NUM
  if (lpr < 64)
    k_spgemm_list<<<grid_for(n, BLK, 8192), BLK, 0, s>>>(n, nullptr, 0, c.rp, num_g, num_w, wide.p,
                                                         flags.p + WIDE_NUM);
  wn = lpr < 64 ? flags.p + WIDE_NUM : nullptr;
  k_spgemm_num_grp<64><<<wgrid, 64 * SPG_WAVES, 0, s>>>(n, a.rp, a.ci, a.v, b.rp, b.ci, b.v, c.rp, num_w, wl, wn,
                                                         c.ci, c.v, overflow);
  HBGS_HIP(hipGetLastError());
  Tmp<int> mid(n);
  k_spgemm_tsize_num<<<grid_for(n, BLK), BLK, 0, s>>>(n, c.rp, num_w, num_b, ts.p, flags.p + MID, mid.p,
                                                      flags.p + ANY_NUM, longest ? flags.p + LONGEST : nullptr);
  HBGS_HIP(hipGetLastError());
  if (b.m > num_w) {  // a row can have more entries than the wave kernel takes
    k_spgemm_num_block<<<grid_for(n, 1, 1024), BLK, 0, s>>>(flags.p + MID, mid.p, a.rp, a.ci, a.v, b.rp, b.ci, b.v,
                                                            c.rp, c.ci, c.v, overflow);
    HBGS_HIP(hipGetLastError());
  }
  int h_flags[NFLAGS];
  read_back(h_flags, flags.p, sizeof(h_flags), s);
  c.maxlen = h_flags[LONGEST];
  if (h_flags[ANY_NUM]) {
    scan_i64(ts.p, toff.p, n, s);
    h_off.resize(n + 1);
    HBGS_HIP(hipMemcpyAsync(h_off.data(), toff.p, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToHost, s));
    HBGS_HIP(hipStreamSynchronize(s));
    const int64_t maxbatch = batch_rows(h_off, n, cuts);
    Tmp<int> keys(maxbatch);
    Tmp<double> vals(maxbatch);
    for (size_t q = 0; q + 1 < cuts.size(); ++q) {
      int r0 = cuts[q], r1 = cuts[q + 1];
      if (h_off[r1] == h_off[r0]) continue;
      k_spgemm_numeric<<<grid_for(r1 - r0, 64), 64, 0, s>>>(r0, r1, a.rp, a.ci, a.v, b.rp, b.ci, b.v, toff.p,
                                                            h_off[r0], keys.p, vals.p, c.rp, c.ci, c.v);
      HBGS_HIP(hipGetLastError());
    }
  }
  if (h_flags[OVF]) HBGS_FAIL(HBGS_ESETUP, "sparse product: accumulator table overflow");
}

// ------------------------------------------------------- dense coarsest LU
__global__ void k_dense_fill(int n, const int* rp, const int* ci, const double* v, double* m) {
  GRID_STRIDE(i, n) {
    for (int j = 0; j < n; ++j) m[i * (int64_t)n + j] = 0.0;
    for (int k = rp[i]; k < rp[i + 1]; ++k) m[i * (int64_t)n + ci[k]] = v[k];
  }
}
// step k: pivot = first row with maximal |a_ik| (i >= k); swap rows; multipliers
__global__ void k_lu_pivot(int n, int k, double* m, int* piv, int* singular) {
  __shared__ double sv[BLK];
  __shared__ int si[BLK];
  double best = -1.0;
  int bi = n;
  for (int i = k + threadIdx.x; i < n; i += BLK) {
    double a = fabs(m[(int64_t)i * n + k]);
    if (a > best) {
      best = a;
      bi = i;
    }
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int st = BLK / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      double a = sv[threadIdx.x + st];
      int ai = si[threadIdx.x + st];
      if (a > sv[threadIdx.x] || (a == sv[threadIdx.x] && ai < si[threadIdx.x])) {
        sv[threadIdx.x] = a;
        si[threadIdx.x] = ai;
      }
    }
    __syncthreads();
  }
  int p = si[0];
  if (threadIdx.x == 0) {
    piv[k] = p;
    if (!(sv[0] > 0.0)) *singular = 1;
  }
  if (!(sv[0] > 0.0)) return;
  if (p != k)
    for (int j = threadIdx.x; j < n; j += BLK) {
      double t = m[(int64_t)k * n + j];
      m[(int64_t)k * n + j] = m[(int64_t)p * n + j];
      m[(int64_t)p * n + j] = t;
    }
  __syncthreads();
  double akk = m[(int64_t)k * n + k];
  for (int i = k + 1 + threadIdx.x; i < n; i += BLK) m[(int64_t)i * n + k] = m[(int64_t)i * n + k] / akk;
}
__global__ void k_lu_update(int n, int k, double* m) {
  int64_t w = (int64_t)(n - k - 1);
  GRID_STRIDE(t, w * w) {
    int i = k + 1 + (int)(t / w), j = k + 1 + (int)(t % w);
    m[(int64_t)i * n + j] -= m[(int64_t)i * n + k] * m[(int64_t)k * n + j];
  }
}
// Inverse of up to LU_MAXN rows: LU factorisation with partial pivoting (the
// first row of maximal |a_ik|), then X = U^-1 (L^-1 P).  Forward, by panels of
// NB columns, one launch per panel: with K a panel's rows and columns, after
// its row interchanges, and B the K rows,
//   K rows      <- L11^-1 B                (substitution),
//   rows below  <- A - L21 (L11^-1 B)
// in every column: right of K that is the factorisation, left of K it turns
// what earlier panels left there into rows of L^-1 (in K itself B is the
// identity; U11 stays in its upper triangle).  Launch k applies step k to the
// rows from its panel on (tiles, from one buffer to another, so the
// interchanged rows are read where they lie) while its block 0 forms the next
// panel: it applies step k to those NB columns only, the remaining rows in
// registers, and factors them.  Then each row lies, final, in the buffer its
// panel's step wrote; k_lu_turn parts U from L^-1, and k_lu_back finishes
// X block row by block row, one launch each.
// Every column of X is a forward and a backward substitution, so A X is as
// near I as the factorisation allows, rows of any scale.  (In-place
// Gauss-Jordan elimination, which needs no second pass, is not: on 400-row
// diffusion matrices with rows scaled over 1e4 its ||b - A X b|| is some 500
// times that of LU, over 1e8 some 1e4 times.)
// Bound by the serial chain of n pivot searches in one block: a launch takes
// 29 us with one row per thread, 41 with two and 55 with three, its tiles
// alone 6-16; the backward pass 14.5 us per 32 rows.  484 / 900 / 1,444 /
// 1,936 rows 1.2 / 2.4 / 4.6 / 6.9 ms, where three launches per panel of the
// factorisation, then four per 32 rows of two substitutions, took 2.4 / 4.2 /
// 7.5 / 10.8 (and Gauss-Jordan 0.9 / 2.2 / 4.7 / 7.2).
constexpr int LU_T = 512;             // threads; two waves per SIMD leave a thread 256 registers
constexpr int LU_R = 4;               // panel rows per thread at most
constexpr int LU_MAXN = LU_T * LU_R;
// columns of a panel: 8 while a thread holds four rows, whose 16 columns
// would not stay in registers
constexpr int lu_nb(int rows_per_thread) { return rows_per_thread < 4 ? 16 : 8; }
constexpr int LU_NB = 16;             // at most
constexpr int LU_TR = 64, LU_TC = 128;  // rows and columns of a tile
constexpr int LU_BACK = 32;           // rows of a block of the backward pass
constexpr int LU_MOVED = 32;          // rows that one panel's interchanges move at most
// interchanges of a panel: count, then the rows that change, then where each
// takes its values from; the panel's own rows come first
constexpr int LU_LIST = 1 + 2 * LU_MOVED;

// Register-only (DPP) maximum within rows of 16 lanes; all 64 lanes must be
// active.  Every lane of a 16-lane row ends with the row's result: pairs
// within quads (quad_perm [1,0,3,2] and [2,3,0,1]), then quads (rotate right
// by 4 and by 8 lanes).
__device__ __forceinline__ unsigned max_row16(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x124, 0xF, 0xF, false));
  return max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xF, 0xF, false));
}
__device__ __forceinline__ unsigned readlane_u32(unsigned v, int lane) {
  return (unsigned)__builtin_amdgcn_readlane((int)v, lane);
}
// the wavefront's maximum (uniform)
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  v = max_row16(v);
  return max(max(readlane_u32(v, 0), readlane_u32(v, 16)), max(readlane_u32(v, 32), readlane_u32(v, 48)));
}

struct LuStep {
  int n, ld;   // rows; ld: at least n + LU_T
  int k0, nb;  // the step's panel (nb = 0: no step, the first launch)
  int p0, pb;  // the panel that block 0 forms (pb = 0: none, and no such block)
  int q0, qb;  // the panel after it: its columns are written to Tn as well
  const double* src;
  double* dst;
  const double* M;  // the step's panel, factored, by columns: M[t * ld + r], rows from k0 on
  double* Mn;       // the next step's
  const int* list;  // the interchanges (LU_LIST)
  int* listn;
  const double* T;  // columns of panel p0 before the step: T[t * ld + r]
  double* Tn;
  int* orig;  // orig[r]: the original index of the row now at r
  int* singular;
};
// x / d from dinv = 1 / d (both ordinary numbers), corrected by the remainder:
// the division's result but for a rare last bit, in 3 dependent operations
__device__ __forceinline__ double lu_quotient(double x, double d, double dinv) {
  const double q = x * dinv;
  return fma(fma(-d, q, x), dinv, q);
}
// v <- L11^-1 v for one column; L: L11 (unit lower, the rest not read)
template <int NB>
__device__ __forceinline__ void lu_unit_lower(double (&v)[NB], const double (&L)[NB][NB]) {
#pragma unroll
  for (int w = 0; w + 1 < NB; ++w)
#pragma unroll
    for (int u = w + 1; u < NB; ++u) v[u] = fma(-L[u][w], v[w], v[u]);
}
// R rows per thread, from p0 on; NB: columns of the panel; NBS: of the step's
template <int R, int NB, int NBS>
__device__ void lu_panel(const LuStep& g) {
  constexpr int NW = LU_T / 64;
  static_assert(NW <= 16, "the wavefronts' candidates are combined within one 16-lane row");
  // per column: each wavefront's pivot candidate (magnitude's high and low
  // word, the row inverted, its values) and row j before the interchange; two
  // sets, used by alternate columns, so one barrier per column suffices
  __shared__ uint4 ckey[2][NW];
  __shared__ __align__(16) double crow[2][NW][NB];
  __shared__ __align__(16) double xrow[2][NB];
  __shared__ double Lp[NBS][NBS];
  __shared__ __align__(16) double Bp[NBS][NB];
  __shared__ uint16_t at[LU_T * R];  // where row p0 + i takes its values from
  __shared__ int spiv[NB];
  const int n = g.n, p0 = g.p0, pb = g.pb;
  const unsigned LD = (unsigned)g.ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < NB) spiv[tid] = p0 + tid;  // no interchange unless a pivot is found
  double a[R][NB];
  if (g.nb > 0) {
#pragma unroll
    for (int q = 0; q < R; ++q) at[tid + q * LU_T] = (uint16_t)min(p0 + tid + q * LU_T, n - 1);
    for (int e = tid; e < NBS * NB; e += LU_T) {
      const int u = e / NB, t = e % NB;
      Bp[u][t] = u < g.nb && t < pb ? g.T[t * LD + g.list[1 + LU_MOVED + u]] : 0.0;
    }
    for (int e = tid; e < NBS * NBS; e += LU_T) {
      const int u = e / NBS, w = e % NBS;
      Lp[u][w] = u < g.nb && w < u ? g.M[w * LD + g.k0 + u] : 0.0;
    }
    __syncthreads();
    if (tid < g.list[0] && g.list[1 + tid] >= p0) at[g.list[1 + tid] - p0] = (uint16_t)g.list[1 + LU_MOVED + tid];
    if (tid < NB) {
      double v[NBS];
#pragma unroll
      for (int u = 0; u < NBS; ++u) v[u] = Bp[u][tid];
      lu_unit_lower<NBS>(v, Lp);
#pragma unroll
      for (int u = 0; u < NBS; ++u) Bp[u][tid] = v[u];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = p0 + tid + q * LU_T;
      const unsigned from = at[tid + q * LU_T];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const double x = g.T[t * LD + from];
        a[q][t] = r < n && t < pb ? x : 0.0;
      }
    }
#pragma unroll 4
    for (int u = 0; u < NBS; ++u) {
      double m[R];
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int r = p0 + tid + q * LU_T;
        m[q] = r < n ? -g.M[u * LD + (unsigned)r] : 0.0;
      }
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const double b = Bp[u][t];
#pragma unroll
        for (int q = 0; q < R; ++q) a[q][t] = fma(m[q], b, a[q][t]);
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int r = p0 + tid + q * LU_T;
        const double x = g.T[t * LD + (unsigned)r];
        a[q][t] = r < n && t < pb ? x : 0.0;
      }
  }
  // The columns rotate through the registers: the current one is always the
  // first and leaves as the last, so the loop stays rolled, but for a copy of
  // its body per four columns: columns that left before them only move on.
  // i = r - p0.
#pragma unroll
  for (int j0 = 0; j0 < NB; j0 += 4) {
#pragma unroll 1
    for (int j = j0; j < min(j0 + 4, pb); ++j) {
      const int b = j & 1;
      // this wavefront's candidate among its rows i >= j: the first of the
      // largest magnitude, by the bits of |a_rj| (0: none, and never NaN).
      // One lane mostly has the largest high word, and the rest is its own
      uint64_t top = 0;
      int tq = 0;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        uint64_t mag = (uint64_t)__double_as_longlong(a[q][0]) & 0x7fffffffffffffffull;
        mag = tid + q * LU_T >= j && mag <= 0x7ff0000000000000ull ? mag : 0;
        if (q > 0 && mag > top) tq = q;
        top = mag > top ? mag : top;
      }
      unsigned hi = wave_max((unsigned)(top >> 32)), lo;
      uint64_t tie = __ballot((unsigned)(top >> 32) == hi);
      int bq, bl = __builtin_ctzll(tie);
      if ((tie & (tie - 1)) == 0) {
        lo = readlane_u32((unsigned)top, bl);
        bq = (int)readlane_u32((unsigned)tq, bl);
      } else {
        lo = wave_max((unsigned)(top >> 32) == hi ? (unsigned)top : 0u);
        tie = __ballot(top == ((uint64_t)hi << 32 | lo));
        bq = 0;
#pragma unroll
        for (int q = R; q-- > 0;) {
          const uint64_t m = __ballot(tq == q) & tie;
          if (m) {
            bl = __builtin_ctzll(m);
            bq = q;
          }
        }
      }
      if (lane == 0) ckey[b][wave] = make_uint4(hi, lo, ~(unsigned)(bq * LU_T + wave * 64 + bl), 0);
#pragma unroll
      for (int q = 0; q < R; ++q) {
        if (q == bq && lane == bl)
#pragma unroll
          for (int t = 0; t < NB; ++t) crow[b][wave][t] = a[q][t];
        if (tid + q * LU_T == j)
#pragma unroll
          for (int t = 0; t < NB; ++t) xrow[b][t] = a[q][t];
      }
      __syncthreads();
      // lanes 0..NW-1 of every wavefront hold the wavefronts' candidates: the
      // largest magnitude, then the first row
      const uint4 cand = lane < NW ? ckey[b][lane] : make_uint4(0, 0, 0, 0);
      hi = readlane_u32(max_row16(cand.x), 0);
      uint64_t best = __ballot(lane < NW && cand.x == hi);
      int pw = __builtin_ctzll(best);
      if (best & (best - 1)) {
        lo = readlane_u32(max_row16(cand.x == hi ? cand.y : 0u), 0);
        const unsigned first = readlane_u32(max_row16(cand.x == hi && cand.y == lo ? cand.z : 0u), 0);
        pw = __builtin_ctzll(__ballot(lane < NW && cand.x == hi && cand.z == first));
        if ((hi | lo) == 0 && tid == 0) *g.singular = 1;  // (what follows is not used)
      }
      const int p = (int)~readlane_u32(cand.z, pw);
      const double* prow = crow[b][pw];  // the pivot row (LDS)
      if (tid == 0) spiv[j] = p0 + p;
      // row j is final: column t of the rotated panel is column t + j of it
      if (tid < NB) g.Mn[(unsigned)((tid + j) % NB) * LD + (unsigned)(p0 + j)] = prow[tid];
      const double d = prow[0];
      double pv[NB - 1];  // of the columns still to come
#pragma unroll
      for (int t = 0; t + 1 < NB - j0; ++t) {
        const double x = prow[t + 1];
        pv[t] = t + 1 < NB - j0 - 3 || t + 1 < NB - j ? x : 0.0;
      }
#pragma unroll
      for (int q = 0; q < R; ++q) {  // (rows up to j are done with: their registers hold anything)
        if (tid + q * LU_T == p)  // the interchange
#pragma unroll
          for (int t = 0; t < NB; ++t) a[q][t] = xrow[b][t];
        const double l = a[q][0] / d;
#pragma unroll
        for (int t = 0; t + 1 < NB; ++t) a[q][t] = t + 1 < NB - j0 ? fma(-l, pv[t], a[q][t + 1]) : a[q][t + 1];
        a[q][NB - 1] = l;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (tid + q * LU_T >= pb)
#pragma unroll
      for (int t = 0; t < NB; ++t) g.Mn[(unsigned)((t + pb) % NB) * LD + (unsigned)(p0 + tid + q * LU_T)] = a[q][t];
  __syncthreads();
  // The interchanges, applied in order, move values among at most LU_MOVED
  // rows: wavefront 0 works out where each of them takes its value from, in
  // registers (all 64 lanes active): lane e holds slot e's (row, source),
  // the panel rows first, then each other row as it is met; a row's slot is
  // found by a ballot and two slots' sources are swapped through lane reads.
  static_assert(2 * NB <= LU_MOVED && LU_MOVED <= 64, "one slot per lane");
  if (tid < 64) {
    const int e = tid;
    const int mp = e < pb ? spiv[e < NB ? e : 0] : 0;
    int d = e < pb ? p0 + e : -1, sr = d;
    int cnt = pb;
    for (int t = 0; t < pb; ++t) {
      const int p = __builtin_amdgcn_readlane(mp, t);
      if (p > p0 + t && p < n) {
        const unsigned long long hit = __ballot(d == p);  // at most one slot holds row p
        int q;
        if (hit) {
          q = __builtin_ctzll(hit);
        } else {
          q = cnt++;
          if (e == q) d = sr = p;
        }
        const int st = __builtin_amdgcn_readlane(sr, t), sq = __builtin_amdgcn_readlane(sr, q);
        if (e == t) sr = sq;
        if (e == q) sr = st;
      }
    }
    if (e < LU_MOVED) {
      g.listn[1 + e] = d;
      g.listn[1 + LU_MOVED + e] = e < cnt ? sr : 0;
    }
    if (e == 0) g.listn[0] = cnt;
    const int o = e < cnt ? g.orig[sr] : 0;  // all read before any is written
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (e < cnt) g.orig[d] = o;
  }
}
// A tile's update on the matrix cores: wavefront w takes 16 rows and 64
// columns of it, four 16 x 16 blocks whose entries a lane holds in column
// l % 16 and rows l / 16 + 4 v.  (On the vector units, eight rows and two
// columns per thread, reading sM and sB from LDS, a backward launch took 18.7
// us instead of 14.5.)  The substitution is repeated by every tile of a column
// range (an eighth of its multiply-adds).
typedef double lu_acc __attribute__((ext_vector_type(4)));
constexpr int LU_PADM = LU_TR + 16, LU_PADB = LU_TC + 16;  // rows of 4 k's on different banks
static_assert(LU_TR == 64 && LU_TC == 128 && LU_T == 512, "eight wavefronts of 16 x 64 entries");
struct LuLane {
  int row, col, k;  // of its first entry in the tile; l / 16
  __device__ __forceinline__ LuLane() {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    k = l / 16;
    row = w % 4 * 16 + k;
    col = w / 4 * 64 + l % 16;
  }
};
// z -= sM^T sB for the wavefront's entries
template <int NB>
__device__ __forceinline__ void lu_tile_update(lu_acc (&z)[4], const double (&sM)[NB][LU_PADM],
                                               const double (&sB)[NB][LU_PADB], const LuLane& at) {
  static_assert(NB % 4 == 0, "four k's per matrix instruction");
  const int l16 = threadIdx.x & 15;
  lu_acc y[4] = {};
#pragma unroll
  for (int u = 0; u < NB; u += 4) {
    const double m = sM[u + at.k][at.row - at.k + l16];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      y[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, sB[u + at.k][at.col + 16 * q], y[q], 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) z[q] -= y[q];
}
template <int NB>
__device__ void lu_tile(const LuStep& g, int tile) {
  __shared__ double sM[NB][LU_PADM];
  __shared__ double sB[NB][LU_PADB];
  __shared__ double sL[NB][NB];
  __shared__ int srow[LU_TR];
  const int n = g.n, k0 = g.k0, nb = g.nb, p0 = k0 + nb;
  const int tcols = (n + LU_TC - 1) / LU_TC;
  const int r0 = k0 + tile / tcols * LU_TR, c0 = tile % tcols * LU_TC;
  const int tid = threadIdx.x;
  const LuLane at;
  if (tid < LU_TR) {
    const int r = r0 + tid, cnt = g.list[0];
    int from = min(r, n - 1);
    for (int e = 0; e < cnt; ++e)
      if (g.list[1 + e] == r) from = g.list[1 + LU_MOVED + e];
    srow[tid] = from;
  }
#pragma unroll
  for (int e = tid; e < NB * LU_TR; e += LU_T) {
    const int u = e / LU_TR, r = r0 + e % LU_TR;
    sM[u][e % LU_TR] = u < nb && r >= p0 && r < n ? g.M[(size_t)u * g.ld + r] : 0.0;
  }
#pragma unroll
  for (int e = tid; e < NB * LU_TC; e += LU_T) {
    const int u = e / LU_TC, c = c0 + e % LU_TC;
    const bool own = c >= k0 && c < p0;  // a column of the panel
    sB[u][e % LU_TC] = own ? (c - k0 == u ? 1.0 : 0.0)
                           : u < nb && c < n ? g.src[(size_t)g.list[1 + LU_MOVED + u] * n + c] : 0.0;
  }
  if (tid < NB * NB) {
    const int u = tid / NB, w = tid % NB;
    sL[u][w] = u < nb && w < nb ? g.M[(size_t)w * g.ld + k0 + u] : 0.0;
  }
  static_assert(NB * NB <= LU_T && LU_TC <= LU_T, "one pass each");
  __syncthreads();
  lu_acc z[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = c0 + at.col + 16 * q;
    const bool col = c < n && !(c >= k0 && c < p0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = at.row + 4 * v, r = r0 + i;
      const double x = g.src[(size_t)srow[i] * n + min(c, n - 1)];
      z[q][v] = col && r >= p0 && r < n ? x : 0.0;
    }
  }
  if (tid < LU_TC) {
    double v[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) v[u] = sB[u][tid];
    lu_unit_lower<NB>(v, sL);
#pragma unroll
    for (int u = 0; u < NB; ++u) sB[u][tid] = v[u];
  }
  __syncthreads();
  lu_tile_update(z, sM, sB, at);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int cl = at.col + 16 * q, c = c0 + cl;
    if (c >= n) continue;
    const bool own = c >= k0 && c < p0, ahead = c >= g.q0 && c < g.q0 + g.qb;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + at.row + 4 * v;
      if (r >= n) break;
      double x = z[q][v];
      if (r < p0)  // a row of the panel, final; in its own columns U11 above L11^-1
        x = own && c >= r ? sL[r - k0][c - k0] : sB[r - k0][cl];
      g.dst[(size_t)r * n + c] = x;
      if (ahead) g.Tn[(size_t)(c - g.q0) * g.ld + r] = x;
    }
  }
}
template <int R, int NB, int NBS>
__global__ __launch_bounds__(LU_T) void k_lu_step(const LuStep g) {
  const int panel = g.pb > 0;
  if (panel && blockIdx.x == 0)
    lu_panel<R, NB, NBS>(g);
  else
    lu_tile<NBS>(g, (int)blockIdx.x - panel);
}
// the dense matrix, one block per row; the first two panels (nb0, nb1
// columns) by columns
__global__ __launch_bounds__(BLK) void k_lu_fill(int n, int ld, int nb0, int nb1, const int* __restrict__ rp,
                                                 const int* __restrict__ ci, const double* __restrict__ v,
                                                 double* __restrict__ m, double* __restrict__ t0,
                                                 double* __restrict__ t1, int* __restrict__ orig) {
  __shared__ double row[LU_MAXN];
  const int i = blockIdx.x;
  for (int j = threadIdx.x; j < n; j += BLK) row[j] = 0.0;
  __syncthreads();
  for (int k = rp[i] + (int)threadIdx.x; k < rp[i + 1]; k += BLK) row[ci[k]] = v[k];
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += BLK) {
    m[(size_t)i * n + j] = row[j];
    if (j < nb0)
      t0[(size_t)j * ld + i] = row[j];
    else if (j < nb0 + nb1)
      t1[(size_t)(j - nb0) * ld + i] = row[j];
  }
  if (threadIdx.x == 0) orig[i] = i;
}
// Between the passes, one block per row: the row's final form (in buffer a or
// b: panels of 8 columns up to row e8, of 16 after it, alternate) parts into
// L^-1 (to y) and U (to u; y and u are a and b in some order), U's diagonal
// blocks of LU_BACK rows to diag
__global__ __launch_bounds__(BLK) void k_lu_turn(int n, int e8, const double* a, const double* b, double* y, double* u,
                                                 double* __restrict__ diag) {
  __shared__ double row[LU_MAXN];
  const int r = blockIdx.x;
  const int k = r < e8 ? r / 8 : e8 / 8 + (r - e8) / 16;
  const double* f = (k & 1 ? a : b) + (size_t)r * n;  // step k wrote buffer (k + 1) % 2
  for (int c = threadIdx.x; c < n; c += BLK) row[c] = f[c];
  __syncthreads();
  for (int c = threadIdx.x; c < n; c += BLK) {
    y[(size_t)r * n + c] = c < r ? row[c] : c == r ? 1.0 : 0.0;
    u[(size_t)r * n + c] = row[c];
  }
  const int b0 = r / LU_BACK * LU_BACK;
  for (int w = threadIdx.x; w < LU_BACK; w += BLK) diag[(size_t)r * LU_BACK + w] = b0 + w >= r && b0 + w < n ? row[b0 + w] : 0.0;
}
// The backward pass at rows k0 .. k0+nb: X_K = U_KK^-1 Y_K by substitution (in
// every tile), Y_r -= U_rK X_K for the rows above; X_K replaces U's rows K,
// whose part right of K the launches before this have used
// rows o .. o + LU_BACK/2 of one column of sB against the upper triangle of sD
// (by columns) there
__device__ __forceinline__ void lu_upper_half(double (&sB)[LU_BACK][LU_PADB], const double (&sD)[LU_BACK][LU_BACK],
                                              const double (&sInv)[LU_BACK], int o, int c) {
  constexpr int H = LU_BACK / 2;
  double v[H];
#pragma unroll
  for (int t = 0; t < H; ++t) v[t] = sB[o + t][c];
#pragma unroll
  for (int w = H; w-- > 0;) {
    v[w] = lu_quotient(v[w], sD[o + w][o + w], sInv[o + w]);
#pragma unroll
    for (int t = 0; t < w; ++t) v[t] = fma(-sD[o + w][o + t], v[w], v[t]);
  }
#pragma unroll
  for (int t = 0; t < H; ++t) sB[o + t][c] = v[t];
}
__global__ __launch_bounds__(LU_T) void k_lu_back(int n, int k0, int nb, const double* __restrict__ diag, double* u,
                                                  double* y) {
  __shared__ double sM[LU_BACK][LU_PADM];
  __shared__ double sB[LU_BACK][LU_PADB];
  __shared__ __align__(16) double sD[LU_BACK][LU_BACK];  // by columns
  __shared__ double sInv[LU_BACK];
  constexpr int H = LU_BACK / 2;
  const int tcols = (n + LU_TC - 1) / LU_TC;
  const int r0 = (int)blockIdx.x / tcols * LU_TR, c0 = (int)blockIdx.x % tcols * LU_TC;
  const int tid = threadIdx.x, lane = tid & 63;
  const LuLane at;
#pragma unroll
  for (int e = tid; e < LU_BACK * LU_TC; e += LU_T) {
    const int t = e / LU_TC, c = c0 + e % LU_TC;
    sB[t][e % LU_TC] = t < nb && c < n ? y[(size_t)(k0 + t) * n + c] : 0.0;
  }
#pragma unroll
  for (int e = tid; e < LU_BACK * LU_BACK; e += LU_T) {
    const int t = e / LU_BACK, w = e % LU_BACK;
    const double d = t < nb && w < nb ? diag[(size_t)(k0 + t) * LU_BACK + w] : t == w ? 1.0 : 0.0;
    sD[w][t] = d;
    if (t == w) sInv[w] = 1.0 / d;
  }
#pragma unroll
  for (int e = tid; e < LU_BACK * LU_TR; e += LU_T) {
    const int r = r0 + e / LU_BACK, t = e % LU_BACK;
    sM[t][e / LU_BACK] = t < nb && r < k0 ? u[(size_t)r * n + k0 + t] : 0.0;
  }
  __syncthreads();
  lu_acc z[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v)  // (entries outside are not stored)
      z[q][v] = y[(size_t)min(r0 + at.row + 4 * v, n - 1) * n + min(c0 + at.col + 16 * q, n - 1)];
  // U_KK^-1: quotients by way of 1 / d unless a d is near the ends of the
  // range; half of the rows at a time, in registers
  const double dd = fabs(sD[lane % LU_BACK][lane % LU_BACK]);
  if (__all(dd > 1e-290 && dd < 1e290)) {
    if (tid < LU_TC) lu_upper_half(sB, sD, sInv, H, tid);
    __syncthreads();
    for (int e = tid; e < H * LU_TC; e += LU_T) {
      const int t = e / LU_TC, c = e % LU_TC;
      double x = sB[t][c];
#pragma unroll
      for (int w = H; w < LU_BACK; ++w) x = fma(-sD[w][t], sB[w][c], x);
      sB[t][c] = x;
    }
    __syncthreads();
    if (tid < LU_TC) lu_upper_half(sB, sD, sInv, 0, tid);
  } else if (tid < LU_TC) {
    for (int w = LU_BACK; w-- > 0;) {
      const double x = sB[w][tid] = sB[w][tid] / sD[w][w];
      for (int t = 0; t < w; ++t) sB[t][tid] = fma(-sD[w][t], x, sB[t][tid]);
    }
  }
  __syncthreads();
  if (r0 == 0)
    for (int e = tid; e < nb * LU_TC; e += LU_T) {
      const int c = c0 + e % LU_TC;
      if (c < n) u[(size_t)(k0 + e / LU_TC) * n + c] = sB[e / LU_TC][e % LU_TC];
    }
  if (k0 == 0) return;
  lu_tile_update(z, sM, sB, at);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + at.row + 4 * v, c = c0 + at.col + 16 * q;
      if (r < k0 && c < n) y[(size_t)r * n + c] = z[q][v];
    }
}
// x is the inverse of the interchanged matrix: its columns go back in order
__global__ __launch_bounds__(BLK) void k_lu_finish(int n, const double* __restrict__ x, const int* __restrict__ orig,
                                                   double* __restrict__ inv) {
  const int64_t i = blockIdx.x;
  for (int c = threadIdx.x; c < n; c += BLK) inv[i * n + orig[c]] = x[i * n + c];
}
static int lu_inverse(const DCsr& a, double* inv, hipStream_t s) {
  const int n = a.n, ld = n + LU_T;
  struct Panel {
    int k0, nb, per;  // per: rows per thread when it is formed
  };
  std::vector<Panel> panels;
  int e8 = 0;  // columns in panels of 8
  for (int k0 = 0; k0 < n;) {
    const int per = (n - k0 + LU_T - 1) / LU_T, nb = std::min(lu_nb(per), n - k0);
    panels.push_back({k0, nb, per});
    k0 += nb;
    if (per == LU_R) e8 = k0;
  }
  const int np = (int)panels.size();
  Tmp<double> work((size_t)n * n), m((size_t)2 * LU_NB * ld), t((size_t)2 * LU_NB * ld), diag((size_t)n * LU_BACK);
  Tmp<int> list(2 * LU_LIST), orig(n), sing(1);
  double* x[2] = {inv, work.p};
  auto at = [&](Tmp<double>& w, int q) { return w.p + (size_t)(q & 1) * LU_NB * ld; };
  HBGS_HIP(hipMemsetAsync(sing.p, 0, sizeof(int), s));
  k_lu_fill<<<n, BLK, 0, s>>>(n, ld, panels[0].nb, np > 1 ? panels[1].nb : 0, a.rp, a.ci, a.v, x[0], at(t, 0), at(t, 1),
                              orig.p);
  const int tcols = (n + LU_TC - 1) / LU_TC;
  for (int k = -1; k < np; ++k) {
    const Panel none{n, 0, 1};
    const Panel step = k < 0 ? Panel{0, 0, panels[0].per} : panels[k];
    const Panel next = k + 1 < np ? panels[k + 1] : none, after = k + 2 < np ? panels[k + 2] : none;
    LuStep g{};
    g.n = n;
    g.ld = ld;
    g.k0 = step.k0;
    g.nb = step.nb;
    g.p0 = next.k0;
    g.pb = next.nb;
    g.q0 = after.k0;
    g.qb = after.nb;
    g.src = x[k & 1];
    g.dst = x[(k + 1) & 1];
    g.M = at(m, k);
    g.Mn = at(m, k + 1);
    g.list = list.p + (k & 1) * LU_LIST;
    g.listn = list.p + ((k + 1) & 1) * LU_LIST;
    g.T = at(t, k + 1);
    g.Tn = at(t, k);
    g.orig = orig.p;
    g.singular = sing.p;
    const int tiles = k < 0 ? 0 : (n - step.k0 + LU_TR - 1) / LU_TR * tcols;
    const unsigned grid = (unsigned)(tiles + (g.pb > 0));
    switch (next.per) {
      case 4: k_lu_step<4, lu_nb(4), lu_nb(4)><<<grid, LU_T, 0, s>>>(g); break;
      case 3:
        if (step.per == 4)
          k_lu_step<3, lu_nb(3), lu_nb(4)><<<grid, LU_T, 0, s>>>(g);
        else
          k_lu_step<3, lu_nb(3), lu_nb(3)><<<grid, LU_T, 0, s>>>(g);
        break;
      case 2: k_lu_step<2, lu_nb(2), lu_nb(2)><<<grid, LU_T, 0, s>>>(g); break;
      default: k_lu_step<1, lu_nb(1), lu_nb(1)><<<grid, LU_T, 0, s>>>(g); break;
    }
    HBGS_HIP(hipGetLastError());
  }
  k_lu_turn<<<n, BLK, 0, s>>>(n, e8, x[0], x[1], inv, work.p, diag.p);
  for (int k0 = (n - 1) / LU_BACK * LU_BACK; k0 >= 0; k0 -= LU_BACK)
    k_lu_back<<<(unsigned)(std::max(1, (k0 + LU_TR - 1) / LU_TR) * tcols), LU_T, 0, s>>>(
        n, k0, std::min(LU_BACK, n - k0), diag.p, work.p, inv);
  k_lu_finish<<<n, BLK, 0, s>>>(n, work.p, orig.p, inv);
  HBGS_HIP(hipGetLastError());
  return read_one(sing.p, s) ? -4 : 0;
}

// Explicit inverse from the factors, X = U^-1 (L^-1 P), by blocks of
// INV_NB rows: each block row of X is finished by a small triangular solve
// (one thread per column) and then removed from the other block rows by a
// tiled update (forward: the rows below; backward: the rows above).
constexpr int INV_NB = 32;
// X = P: column c holds a 1 in row pinv[c]
__global__ void k_inv_init(int n, const int* pinv, double* x) {
  GRID_STRIDE(e, (int64_t)n * n) {
    const int i = (int)(e / n), c = (int)(e % n);
    x[e] = pinv[c] == i ? 1.0 : 0.0;
  }
}
// rows kb..kb+nb of X: unit lower (forward) or upper (backward) block solve,
// one thread per column with the block's rows in registers and the diagonal
// block of the factors in LDS (rows beyond nb: zero, with a unit diagonal)
template <bool UPPER>
__global__ __launch_bounds__(BLK) void k_inv_trsm(int n, int kb, int nb, const double* f, double* x) {
  // The unit lower solve is run as an upper solve on reversed indices
  // (position i holds row INV_NB-1-i, with unit diagonal), so both use the
  // one loop below.
  __shared__ double sf[INV_NB][INV_NB + 1];
  for (int e = threadIdx.x; e < INV_NB * INV_NB; e += BLK) {
    const int i = e / INV_NB, w = e % INV_NB;
    const int r = UPPER ? i : INV_NB - 1 - i, u = UPPER ? w : INV_NB - 1 - w;
    double val = r == u ? 1.0 : 0.0;
    if (r < nb && u < nb && (UPPER || r != u)) val = f[(int64_t)(kb + r) * n + kb + u];
    sf[i][w] = val;
  }
  __syncthreads();
  // one column per thread.  The terms are fused multiply-adds, so each row
  // is one dependent chain that stays in registers; the explicit inverse is
  // checked through the coarse solve's result, not bit for bit.
  const int64_t c = (int64_t)blockIdx.x * BLK + threadIdx.x;
  if (c >= n) return;
  double v[INV_NB];
#pragma unroll
  for (int i = 0; i < INV_NB; ++i) {
    const int r = UPPER ? i : INV_NB - 1 - i;
    v[i] = r < nb ? x[(int64_t)(kb + r) * n + c] : 0.0;
  }
#pragma unroll
  for (int i = INV_NB - 1; i >= 0; --i) {
    double s = v[i];
#pragma unroll
    for (int w = i + 1; w < INV_NB; ++w) s = fma(-sf[i][w], v[w], s);
    v[i] = s / sf[i][i];
  }
#pragma unroll
  for (int i = 0; i < INV_NB; ++i) {
    const int r = UPPER ? i : INV_NB - 1 - i;
    if (r < nb) x[(int64_t)(kb + r) * n + c] = v[i];
  }
}
// X[i, :] -= F[i, kb..kb+nb) X[kb..kb+nb, :] for rows i in [r_lo, r_hi), in
// tiles of 32 rows x 64 columns (fused multiply-adds, like the block solves)
__global__ __launch_bounds__(BLK) void k_inv_update(int n, int kb, int nb, int r_lo, int r_hi, const double* f,
                                                    double* x) {
  __shared__ double sF[32][INV_NB];
  __shared__ double sX[INV_NB][64];
  const int r0 = r_lo + blockIdx.y * 32, c0 = blockIdx.x * 64;
  for (int e = threadIdx.x; e < 32 * INV_NB; e += BLK) {
    const int i = e / INV_NB, t = e % INV_NB;
    sF[i][t] = (r0 + i < r_hi && t < nb) ? f[(int64_t)(r0 + i) * n + kb + t] : 0.0;
  }
  for (int e = threadIdx.x; e < INV_NB * 64; e += BLK) {
    const int t = e / 64, jj = e % 64;
    sX[t][jj] = (c0 + jj < n && t < nb) ? x[(int64_t)(kb + t) * n + c0 + jj] : 0.0;
  }
  __syncthreads();
  const int jj = threadIdx.x & 63, ib = (threadIdx.x >> 6) * 8;
  if (c0 + jj >= n) return;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int i = r0 + ib + u;
    if (i >= r_hi) break;
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < INV_NB; ++t) acc = fma(sF[ib + u][t], sX[t][jj], acc);
    x[(int64_t)i * n + c0 + jj] -= acc;
  }
}

int dense_inverse(const DCsr& a, double* inv, hipStream_t s) {
  const int n = a.n;
  if (n <= LU_MAXN) return lu_inverse(a, inv, s);
  Tmp<double> m((size_t)n * n);
  Tmp<int> piv(n), sing(1), pinv(n);
  HBGS_HIP(hipMemsetAsync(sing.p, 0, sizeof(int), s));
  k_dense_fill<<<grid_for(n, 64), 64, 0, s>>>(n, a.rp, a.ci, a.v, m.p);
  HBGS_HIP(hipGetLastError());
  for (int k = 0; k < n; ++k) {
    k_lu_pivot<<<1, BLK, 0, s>>>(n, k, m.p, piv.p, sing.p);
    if (k + 1 < n)
      k_lu_update<<<grid_for((int64_t)(n - k - 1) * (n - k - 1), BLK, 8192), BLK, 0, s>>>(n, k, m.p);
  }
  HBGS_HIP(hipGetLastError());
  int singular = 0;
  std::vector<int> hp(n);
  HBGS_HIP(hipMemcpyAsync(&singular, sing.p, sizeof(int), hipMemcpyDeviceToHost, s));
  HBGS_HIP(hipMemcpyAsync(hp.data(), piv.p, sizeof(int) * n, hipMemcpyDeviceToHost, s));
  HBGS_HIP(hipStreamSynchronize(s));
  if (singular) return -4;
  // P e_c: apply the interchanges k <-> piv[k] in order to the identity row ids
  std::vector<int> rowof(n), where(n);
  for (int i = 0; i < n; ++i) rowof[i] = i;  // rowof[r] = original index now at position r
  for (int k = 0; k < n; ++k) std::swap(rowof[k], rowof[hp[k]]);
  for (int r = 0; r < n; ++r) where[rowof[r]] = r;
  HBGS_HIP(hipMemcpyAsync(pinv.p, where.data(), sizeof(int) * n, hipMemcpyHostToDevice, s));
  k_inv_init<<<grid_for((int64_t)n * n, BLK), BLK, 0, s>>>(n, pinv.p, inv);
  HBGS_HIP(hipGetLastError());
  const unsigned cgrid = (unsigned)((n + 63) / 64);
  for (int kb = 0; kb < n; kb += INV_NB) {  // L Y = P
    const int nb = std::min(INV_NB, n - kb);
    k_inv_trsm<false><<<(n + BLK - 1) / BLK, BLK, 0, s>>>(n, kb, nb, m.p, inv);
    const int below = n - kb - nb;
    if (below > 0)
      k_inv_update<<<dim3(cgrid, (below + 31) / 32), BLK, 0, s>>>(n, kb, nb, kb + nb, n, m.p, inv);
  }
  for (int kb = (n - 1) / INV_NB * INV_NB; kb >= 0; kb -= INV_NB) {  // U X = Y
    const int nb = std::min(INV_NB, n - kb);
    k_inv_trsm<true><<<(n + BLK - 1) / BLK, BLK, 0, s>>>(n, kb, nb, m.p, inv);
    if (kb > 0) k_inv_update<<<dim3(cgrid, (kb + 31) / 32), BLK, 0, s>>>(n, kb, nb, 0, kb, m.p, inv);
  }
  HBGS_HIP(hipGetLastError());
  HBGS_HIP(hipStreamSynchronize(s));
  return 0;
}

// --------------------------------------------- transposes for the solve phase
// (A^T)_{ji} = A_{ij}: for a structurally symmetric A the pattern is A's own;
// each entry's value is found in the mirrored row by binary search
template <int L>
__global__ void k_transpose_sym(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                const double* __restrict__ v, double* __restrict__ vt) {
  ROW_GROUPS(L, j, gl, n) {
    for (int q = rp[j] + gl; q < rp[j + 1]; q += L) {
      const int i = ci[q];
      int lo = rp[i], hi = rp[i + 1] - 1;
      double x = 0.0;
      while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        if (ci[mid] == (int)j) {
          x = v[mid];
          break;
        }
        if (ci[mid] < (int)j)
          lo = mid + 1;
        else
          hi = mid - 1;
      }
      vt[q] = x;
    }
  }
}
// dst[q] = src[position of (j, i)] for entry q = (i, j); *missing: some entry
// has no mirror image (the pattern is not symmetric)
template <int L>
__global__ void k_mirror(int n, const int* __restrict__ rp, const int* __restrict__ ci, const int* __restrict__ src,
                         int* __restrict__ dst, int* missing) {
  int bad = 0;
  ROW_GROUPS(L, j, gl, n) {
    for (int q = rp[j] + gl; q < rp[j + 1]; q += L) {
      const int i = ci[q];
      int lo = rp[i], hi = rp[i + 1] - 1, at = -1;
      while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int c = ci[mid];
        if (c == (int)j) {
          at = mid;
          break;
        }
        if (c < (int)j)
          lo = mid + 1;
        else
          hi = mid - 1;
      }
      bad |= at < 0;
      dst[q] = at < 0 ? 0 : src[at];
    }
  }
  if (bad) atomicOr(missing, 1);
}
bool mirror_positions(const DCsr& a, const int* src, int* dst, hipStream_t s) {
  if (a.n == 0) return true;
  Tmp<int> missing(1);
  HBGS_HIP(hipMemsetAsync(missing.p, 0, sizeof(int), s));
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_mirror, L, a.n, s, a.n, a.rp, a.ci, src, dst, missing.p);
  return read_one(missing.p, s) == 0;
}

// Q with rows 2i = row i of a and 2i+1 = row i of b (same column count):
// one row-block pass over Q then forms both products with one operand
template <int L>
__global__ void k_interleave(int n, const int* arp, const int* aci, const double* av, const int* brp,
                             const int* bci, const double* bv, const int* qrp, int* qci, double* qv) {
  ROW_GROUPS(L, i, gl, n) {
    const int qa = qrp[2 * i], qb = qrp[2 * i + 1];
    for (int k = arp[i] + gl; k < arp[i + 1]; k += L) {
      qci[qa + k - arp[i]] = aci[k];
      qv[qa + k - arp[i]] = av[k];
    }
    for (int k = brp[i] + gl; k < brp[i + 1]; k += L) {
      qci[qb + k - brp[i]] = bci[k];
      qv[qb + k - brp[i]] = bv[k];
    }
  }
}
__global__ void k_interleave_rp(int n, const int* arp, const int* brp, int* qrp) {
  GRID_STRIDE(i, n + 1) {
    qrp[2 * i] = arp[i] + brp[i];
    if (i < n) qrp[2 * i + 1] = arp[i + 1] + brp[i];
  }
}
void interleave_rows(Pool& pool, const DCsr& a, const DCsr& b, DCsr& q, hipStream_t s) {
  q = DCsr{};
  q.n = 2 * a.n;
  q.m = a.m;
  q.nnz = a.nnz + b.nnz;
  q.rp = pool.make<int>(q.n + 1);
  q.ci = pool.make<int>(q.nnz);
  q.v = pool.make<double>(q.nnz);
  k_interleave_rp<<<grid_for(a.n + 1, BLK), BLK, 0, s>>>(a.n, a.rp, b.rp, q.rp);
  HBGS_HIP(hipGetLastError());
  const int L = row_lanes(a.n, a.nnz + b.nnz);
  LAUNCH_ROW_GROUPS(k_interleave, L, a.n, s, a.n, a.rp, a.ci, a.v, b.rp, b.ci, b.v, q.rp, q.ci, q.v);
}

void transpose_symmetric(const DCsr& a, double* vt, hipStream_t s) {
  const int L = row_lanes(a.n, a.nnz);
  LAUNCH_ROW_GROUPS(k_transpose_sym, L, a.n, s, a.n, a.rp, a.ci, a.v, vt);
}

// Per-block row statistics: part[9 b] = longest row, part[9 b + 1 + q] =
// entries of the fullest block of row_block(q) consecutive rows, over the
// units block b visits.  Unit u covers rows [4u, 4u + 4); the unit that
// starts a row block of each size also reads that block's end.  Wave maxima
// through shuffles, block maxima through LDS, then one atomic per block and
// figure (at most 256 blocks: same-address atomics from every wave cost more
// than the kernel's loads).
__global__ __launch_bounds__(BLK) void k_row_stats(int n, const int* __restrict__ rp, int* __restrict__ part) {
  __shared__ int red[BLK / 64][1 + kRowBlocks];
  int m[1 + kRowBlocks] = {};
  const int64_t nu = ((int64_t)n + 3) / 4;
  GRID_STRIDE(u, nu) {
    const int r0 = (int)(4 * u), r1 = min(n, r0 + 4);
    const int base = rp[r0];
    int prev = base;
    for (int r = r0 + 1; r <= r1; ++r) {
      const int x = rp[r];
      m[0] = max(m[0], x - prev);
      prev = x;
    }
#pragma unroll
    for (int q = 0; q < kRowBlocks; ++q) {
      const int rb = row_block(q);
      if (r0 % rb == 0) m[1 + q] = max(m[1 + q], rp[min(n, r0 + rb)] - base);
    }
  }
  const int w = (int)threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q <= kRowBlocks; ++q) {
    int x = m[q];
    for (int o = 32; o > 0; o >>= 1) x = max(x, __shfl_xor(x, o));
    if ((threadIdx.x & 63) == 0) red[w][q] = x;
  }
  __syncthreads();
  if (threadIdx.x <= kRowBlocks) {
    int x = 0;
    for (int k = 0; k < BLK / 64; ++k) x = max(x, red[k][threadIdx.x]);
    if (x) atomicMax(&part[threadIdx.x], x);
  }
}
constexpr int STATS = 1 + kRowBlocks;  // k_row_stats' results
static void set_stats(DCsr& a, const int* h) {
  a.maxlen = h[0];
  for (int q = 0; q < kRowBlocks; ++q) a.blkmax[q] = h[1 + q];
}
static void launch_row_stats(const DCsr& a, int* part, hipStream_t s) {
  if (a.n <= 0) return;
  k_row_stats<<<grid_for(((int64_t)a.n + 3) / 4, BLK, 256), BLK, 0, s>>>(a.n, a.rp, part);
  HBGS_HIP(hipGetLastError());
}
void row_stats(DCsr& a, hipStream_t s) {
  int h[STATS] = {};
  if (a.n > 0) {
    Tmp<int> part(STATS);
    HBGS_HIP(hipMemsetAsync(part.p, 0, sizeof(h), s));
    launch_row_stats(a, part.p, s);
    read_back(h, part.p, sizeof(h), s);
  }
  set_stats(a, h);
}

// Operand tiles of one row block per workgroup: the tile ids (col /
// TILE_W) of the block's entries go into an LDS hash set; each distinct id's
// slot is its rank among them (ascending), and each entry's slot is found by
// binary search in the ranked list.  A block with more than TILE_MAX tiles
// sets *too_many and writes nothing.
constexpr int TILE_ENTRIES = 4096;  // entries of one row block at most (the FP32 staging limit)
constexpr int TILE_HASH = 128;   // hash slots (> 2 TILE_MAX)
__global__ __launch_bounds__(256) void k_tiles(int n, int rb, const int* __restrict__ rp, const int* __restrict__ ci,
                                               int* __restrict__ tiles, uint16_t* __restrict__ lc,
                                               int* __restrict__ too_many, int* __restrict__ cnt_max) {
  __shared__ int tab[TILE_HASH];
  __shared__ int uniq[TILE_MAX];
  __shared__ int cnt, full;
  const int b = (int)blockIdx.x, t = (int)threadIdx.x;
  const int r0 = b * rb, r1 = min(n, r0 + rb);
  const int s0 = rp[r0], s1 = rp[r1];
  if (t < TILE_HASH) tab[t] = -1;
  if (t == 0) {
    cnt = 0;
    full = 0;
  }
  __syncthreads();
  for (int k = s0 + t; k < s1; k += 256) {
    const int id = ci[k] / TILE_W;
    uint32_t h = ((uint32_t)id * 2654435761u) & (TILE_HASH - 1);
    for (int probe = 0;; ++probe) {
      if (probe == TILE_HASH) {
        full = 1;
        break;
      }
      const int prev = atomicCAS(&tab[h], -1, id);
      if (prev == -1) {
        atomicAdd(&cnt, 1);
        break;
      }
      if (prev == id) break;
      h = (h + 1) & (TILE_HASH - 1);
    }
  }
  __syncthreads();
  const int nt = cnt;
  if (full || nt > TILE_MAX) {
    if (t == 0) atomicOr(too_many, 1);
    return;
  }
  if (t == 0 && nt) atomicMax(cnt_max, nt);
  if (t < TILE_HASH) {
    const int id = tab[t];
    if (id >= 0) {
      int rank = 0;
      for (int q = 0; q < TILE_HASH; ++q) rank += tab[q] >= 0 && tab[q] < id;
      uniq[rank] = id;
    }
  }
  __syncthreads();
  if (t < TILE_MAX) tiles[(size_t)b * TILE_MAX + t] = t < nt ? uniq[t] : -1;
  for (int k = s0 + t; k < s1; k += 256) {
    const int col = ci[k], id = col / TILE_W;
    int lo = 0, hi = nt - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (uniq[mid] < id)
        lo = mid + 1;
      else
        hi = mid;
    }
    lc[k] = (uint16_t)(lo * TILE_W + col % TILE_W);
  }
}
void build_tiles(Pool& pool, DCsr* const* a, const int* rb, int count, hipStream_t s) {
  Tmp<int> flags(2 * (size_t)count);
  bool any = false;
  for (int k = 0; k < count; ++k) {
    DCsr& m = *a[k];
    m.tile_rb = 0;
    m.tile_cnt = 0;
    m.tiles = nullptr;
    m.lc = nullptr;
    if (m.n <= 0 || m.nnz <= 0 || rb[k] <= 0) continue;
    int q = 0;
    while (q < kRowBlocks && row_block(q) != rb[k]) ++q;
    if (q == kRowBlocks || m.blkmax[q] > TILE_ENTRIES) continue;
    if (!any) HBGS_HIP(hipMemsetAsync(flags.p, 0, 2 * (size_t)count * sizeof(int), s));
    any = true;
    const int64_t nblk = ((int64_t)m.n + rb[k] - 1) / rb[k];
    m.tiles = pool.make<int>((size_t)nblk * TILE_MAX);
    m.lc = pool.make<uint16_t>(m.nnz);
    k_tiles<<<(unsigned)nblk, 256, 0, s>>>(m.n, rb[k], m.rp, m.ci, m.tiles, m.lc, flags.p + 2 * k,
                                           flags.p + 2 * k + 1);
    HBGS_HIP(hipGetLastError());
  }
  if (!any) return;
  static_assert(2 * MATRICES * sizeof(int) <= Mail::kBytes, "one message");
  std::vector<int> h(2 * (size_t)count);
  read_back(h.data(), flags.p, h.size() * sizeof(int), s);
  for (int k = 0; k < count; ++k) {
    DCsr& m = *a[k];
    if (!m.tiles) continue;
    if (h[2 * k] || h[2 * k + 1] <= 0) {
      pool.release(m.lc);
      pool.release(m.tiles);
      m.lc = nullptr;
      m.tiles = nullptr;
      continue;
    }
    m.tile_rb = rb[k];
    m.tile_cnt = h[2 * k + 1];
  }
}

// --------------------------------------------------------- diagonal slices
// One wavefront per slice of 64 rows, one row per lane: the lanes walk their
// rows' ascending entries together, each step taking the smallest pending
// column - row of the slice as its next diagonal.  stat[0]: largest count,
// stat[1]: a slice with more than DIA_MAX diagonals.
__global__ __launch_bounds__(256) void k_slice_diags(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                     int* __restrict__ tab, int* __restrict__ count,
                                                     uint16_t* __restrict__ m16, uint32_t* __restrict__ m32,
                                                     int* stat) {
  const int nsl = (n + DIA_ROWS - 1) / DIA_ROWS;
  const int lane = threadIdx.x & 63;
  int most = 0, bad = 0;
  for (int q = (int)blockIdx.x * 4 + (threadIdx.x >> 6); q < nsl; q += (int)gridDim.x * 4) {
    const int row = q * DIA_ROWS + lane;
    int k = row < n ? rp[row] : 0;
    const int e = row < n ? rp[row + 1] : 0;
    uint32_t mask = 0;
    int cnt = 0;
    int* t = tab + (size_t)q * DIA_TS;
    for (;;) {
      const int d = k < e ? ci[k] - row : INT_MAX;
      const int lo = grp_min<64>(d);
      if (lo == INT_MAX) break;
      if (cnt == DIA_MAX) {
        bad = 1;
        break;
      }
      if (d == lo) {
        mask |= 1u << cnt;
        ++k;
      }
      if (lane == 0) t[DIA_DIAG + cnt] = lo;
      ++cnt;
    }
    if (bad) break;
    if (lane == 0) t[0] = count[q] = cnt;
    if (row < n) {
      m16[row] = (uint16_t)mask;
      m32[row] = mask;
    }
    most = max(most, cnt);
  }
  if (lane == 0) {
    if (bad) atomicOr(&stat[1], 1);
    if (most) atomicMax(&stat[0], most);
  }
}
__global__ void k_slice_base(int nsl, const int* __restrict__ base, int* __restrict__ tab) {
  GRID_STRIDE(q, nsl) tab[(size_t)q * DIA_TS + DIA_BASE] = base[q];
}
void build_slices(Pool& pool, DCsr& a, hipStream_t s) {
  a.dia_w = 0;
  a.dia_tab = nullptr;
  a.dia_m16 = nullptr;
  a.dia_m32 = nullptr;
  a.dv = nullptr;
  a.dvf = nullptr;
  if (a.n <= 0 || a.nnz <= 0) return;
  const int nsl = (a.n + DIA_ROWS - 1) / DIA_ROWS;
  Tmp<int> tab((size_t)nsl * DIA_TS), stat(2), count(nsl), base(nsl + 1);
  Tmp<uint16_t> m16(a.n);
  Tmp<uint32_t> m32(a.n);
  HBGS_HIP(hipMemsetAsync(stat.p, 0, 2 * sizeof(int), s));
  k_slice_diags<<<grid_for((nsl + 3) / 4, 1, 2048), 256, 0, s>>>(a.n, a.rp, a.ci, tab.p, count.p, m16.p, m32.p,
                                                                 stat.p);
  HBGS_HIP(hipGetLastError());
  int h[2] = {0, 0};
  read_back(h, stat.p, sizeof(h), s);
  if (h[1] || h[0] <= 0) return;
  a.dia_places = counts_to_rowptr(count.p, base.p, nsl, s) * DIA_ROWS;
  if ((double)a.dia_places > 1.25 * (double)a.nnz || a.dia_places > INT_MAX) return;
  k_slice_base<<<grid_for(nsl, 256), 256, 0, s>>>(nsl, base.p, tab.p);
  HBGS_HIP(hipGetLastError());
  auto keep = [&](void* dst, const void* from, size_t bytes) {
    HBGS_HIP(hipMemcpyAsync(dst, from, bytes, hipMemcpyDeviceToDevice, s));
  };
  a.dia_w = h[0];
  a.dia_tab = pool.make<int>(tab.count);
  keep(a.dia_tab, tab.p, tab.count * sizeof(int));
  if (h[0] <= 16)
    keep(a.dia_m16 = pool.make<uint16_t>(a.n), m16.p, sizeof(uint16_t) * a.n);
  else
    keep(a.dia_m32 = pool.make<uint32_t>(a.n), m32.p, sizeof(uint32_t) * a.n);
}

void alloc_slice_values(Pool& pool, DCsr& a, bool f32) {
  if (!a.dia_w) return;
  a.dv = pool.make<double>(a.dia_places);
  a.dvf = f32 ? pool.make<float>(a.dia_places) : nullptr;
}
// A matrix's values from an array they are read from by position: in row
// order (v, FP32 copy vf) and in the slices' places (dv, dvf), each where
// the matrix has the array.  A block takes the
// entries of 256 rows with consecutive threads and leaves them in LDS, from
// which each thread then takes its row's; blocks with more than LOAD_LDS
// entries (the fullest blocks of a few long rows) read the source again.
constexpr int LOAD_LDS = 4096;
template <class TM>
__global__ __launch_bounds__(256) void k_load_values(int n, const int* __restrict__ rp, const double* __restrict__ from,
                                                     const int* __restrict__ src, double* __restrict__ v,
                                                     float* __restrict__ vf, const int* __restrict__ tab,
                                                     const TM* __restrict__ mask, double* __restrict__ dv,
                                                     float* __restrict__ dvf) {
  __shared__ double sh[LOAD_LDS];
  const int r0 = (int)((int64_t)blockIdx.x * 256), r1 = min(n, r0 + 256);
  const int row = r0 + (int)threadIdx.x;
  const int e0 = rp[r0], e1 = rp[r1];
  const bool staged = e1 - e0 <= LOAD_LDS;
  for (int k = e0 + (int)threadIdx.x; k < e1; k += 256) {
    const double x = from[src[k]];
    if (v) v[k] = x;
    if (vf) vf[k] = (float)x;
    if (staged) sh[k - e0] = x;
  }
  const int q = row / DIA_ROWS;
  if (!dv) return;
  __syncthreads();
  if (q * DIA_ROWS >= n) return;  // the last slice's absent rows get zeros
  const int* t = tab + (size_t)q * DIA_TS;
  const int cnt = t[0];
  const uint32_t m = row < n ? (uint32_t)mask[row] : 0u;
  int k = row < n ? rp[row] : 0;
  const size_t base = (size_t)t[DIA_BASE] * DIA_ROWS + row % DIA_ROWS;
  for (int j = 0; j < cnt; ++j) {
    double x = 0.0;
    if (m >> j & 1u) {
      x = staged ? sh[k - e0] : from[src[k]];
      ++k;
    }
    dv[base + (size_t)j * DIA_ROWS] = x;
    if (dvf) dvf[base + (size_t)j * DIA_ROWS] = (float)x;
  }
}
void load_values(const DCsr& a, const double* from, const int* src, hipStream_t s) {
  if (a.n == 0) return;
  const unsigned g = (unsigned)(((int64_t)a.n + 255) / 256);
  if (a.dia_m32)
    k_load_values<uint32_t><<<g, 256, 0, s>>>(a.n, a.rp, from, src, a.v, a.vf, a.dia_tab, a.dia_m32, a.dv, a.dvf);
  else
    k_load_values<uint16_t><<<g, 256, 0, s>>>(a.n, a.rp, from, src, a.v, a.vf, a.dia_tab, a.dia_m16, a.dv, a.dvf);
  HBGS_HIP(hipGetLastError());
}
// each entry's place in the slices' values (where), or the values in row
// order (v, vf) from the slices'; null arrays are skipped
template <class TM>
__global__ __launch_bounds__(256) void k_unslice(int n, const int* __restrict__ rp, const int* __restrict__ tab,
                                                 const TM* __restrict__ mask, const double* __restrict__ dv,
                                                 const float* __restrict__ dvf, int* __restrict__ where,
                                                 double* __restrict__ v, float* __restrict__ vf) {
  const int row = (int)((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (row >= n) return;
  const int* t = tab + (size_t)(row / DIA_ROWS) * DIA_TS;
  const int64_t base = (int64_t)t[DIA_BASE] * DIA_ROWS + row % DIA_ROWS;
  const uint32_t m = mask[row];
  int k = rp[row];
  for (int j = 0; j < t[0]; ++j)
    if (m >> j & 1u) {
      const int64_t p = base + (int64_t)j * DIA_ROWS;
      if (where) where[k] = (int)p;
      if (v) v[k] = dv[p];
      if (vf) vf[k] = dvf[p];
      ++k;
    }
}
void unslice(const DCsr& a, int* where, double* v, float* vf, hipStream_t s) {
  const unsigned g = (unsigned)(((int64_t)a.n + 255) / 256);
  if (a.dia_m32)
    k_unslice<uint32_t><<<g, 256, 0, s>>>(a.n, a.rp, a.dia_tab, a.dia_m32, a.dv, a.dvf, where, v, vf);
  else
    k_unslice<uint16_t><<<g, 256, 0, s>>>(a.n, a.rp, a.dia_tab, a.dia_m16, a.dv, a.dvf, where, v, vf);
  HBGS_HIP(hipGetLastError());
}
__global__ void k_gather_i32(int64_t n, const int* __restrict__ from, int* __restrict__ idx) {
  GRID_STRIDE(i, n) idx[i] = from[idx[i]];
}
void remap(int64_t n, const int* from, int* idx, hipStream_t s) {
  if (n == 0) return;
  k_gather_i32<<<grid_for(n, BLK, 65536), BLK, 0, s>>>(n, from, idx);
  HBGS_HIP(hipGetLastError());
}

// ------------------------------------------------------- DD(0)-ILU(0) leaf
__global__ void k_sub_count(int n, const int* rp, const int* ci, int sub, int* cnt) {
  GRID_STRIDE(i, n) {
    const int b = (int)(i / sub);
    int c = 0;
    for (int k = rp[i]; k < rp[i + 1]; ++k) c += ci[k] / sub == b;
    cnt[i] = c;
  }
}
__global__ void k_sub_fill(int n, const int* rp, const int* ci, const double* v, int sub, const int* orp, int* oci,
                           double* ov, int* dpos, int* missing) {
  GRID_STRIDE(i, n) {
    const int b = (int)(i / sub);
    int o = orp[i], d = -1;
    for (int k = rp[i]; k < rp[i + 1]; ++k)
      if (ci[k] / sub == b) {
        if (ci[k] == (int)i) d = o;
        oci[o] = ci[k];
        ov[o] = v[k];
        ++o;
      }
    dpos[i] = d;
    if (d < 0) atomicOr(missing, 1);
  }
}
// one block per subdomain, level by level, one thread per row: the IKJ
// row update (each l_ik, then a_ij -= l_ik u_kj in ascending j), the rows it
// reads being final
__global__ __launch_bounds__(BLK) void k_ilu_factor(const int* ford, const int* flev, const int* fsub, const int* rp,
                                                    const int* ci, double* v, const int* dpos, int* zero_pivot) {
  const int b = blockIdx.x;
  for (int l = fsub[b]; l + 1 < fsub[b + 1]; ++l) {
    for (int t = flev[l] + threadIdx.x; t < flev[l + 1]; t += BLK) {
      const int i = ford[t];
      for (int p = rp[i]; p < dpos[i]; ++p) {
        const int k = ci[p];
        const double lik = v[p] / v[dpos[k]];
        v[p] = lik;
        int q = dpos[k] + 1;
        for (int r = p + 1; r < rp[i + 1]; ++r) {
          while (q < rp[k + 1] && ci[q] < ci[r]) ++q;
          if (q < rp[k + 1] && ci[q] == ci[r]) v[r] = v[r] - lik * v[q];
        }
      }
      if (v[dpos[i]] == 0.0) atomicOr(zero_pivot, 1);
    }
    __syncthreads();
  }
}

// level schedule of one direction on the host: level(i) = 1 + max level of
// the rows it reads (lower part for fwd, upper part for bwd), per subdomain
static void ilu_schedule(int n, int sub, const std::vector<int>& rp, const std::vector<int>& ci,
                         const std::vector<int>& dpos, bool fwd, std::vector<int>& order, std::vector<int>& lev,
                         std::vector<int>& subp) {
  std::vector<int> level(n, 0);
  if (fwd) {
    for (int i = 0; i < n; ++i)
      for (int k = rp[i]; k < dpos[i]; ++k) level[i] = std::max(level[i], level[ci[k]] + 1);
  } else {
    for (int i = n - 1; i >= 0; --i)
      for (int k = dpos[i] + 1; k < rp[i + 1]; ++k) level[i] = std::max(level[i], level[ci[k]] + 1);
  }
  const int nsub = (n + sub - 1) / sub;
  order.resize(n);
  lev.clear();
  subp.assign(nsub + 1, 0);
  for (int b = 0; b < nsub; ++b) {
    const int r0 = b * sub, r1 = std::min(n, r0 + sub);
    int nl = 0;
    for (int i = r0; i < r1; ++i) nl = std::max(nl, level[i] + 1);
    std::vector<int> cnt(nl + 1, 0);
    for (int i = r0; i < r1; ++i) cnt[level[i] + 1]++;
    for (int q = 0; q < nl; ++q) cnt[q + 1] += cnt[q];
    subp[b] = (int)lev.size();
    for (int q = 0; q <= nl; ++q) lev.push_back(r0 + cnt[q]);
    std::vector<int> fill(cnt.begin(), cnt.end() - 1);
    for (int i = r0; i < r1; ++i) order[r0 + fill[level[i]]++] = i;
  }
  subp[nsub] = (int)lev.size();
}

int ilu_setup(Pool& pool, const DCsr& a, int sub, IluLeaf& out, hipStream_t s) {
  const int n = a.n;
  DCsr& F = out.F;
  F.n = F.m = n;
  {
    Tmp<int> cnt(n), missing(1);
    F.rp = pool.make<int>(n + 1);
    k_sub_count<<<grid_for(n, BLK), BLK, 0, s>>>(n, a.rp, a.ci, sub, cnt.p);
    HBGS_HIP(hipGetLastError());
    F.nnz = counts_to_rowptr(cnt.p, F.rp, n, s);
    F.ci = pool.make<int>(F.nnz);
    F.v = pool.make<double>(F.nnz);
    out.dpos = pool.make<int>(n);
    HBGS_HIP(hipMemsetAsync(missing.p, 0, sizeof(int), s));
    k_sub_fill<<<grid_for(n, BLK), BLK, 0, s>>>(n, a.rp, a.ci, a.v, sub, F.rp, F.ci, F.v, out.dpos, missing.p);
    HBGS_HIP(hipGetLastError());
    int h_missing = 0;
    read_back(&h_missing, missing.p, sizeof(int), s);
    if (h_missing) return -4;
  }
  // schedules (host)
  std::vector<int> rp(n + 1), ci(F.nnz), dp(n);
  HBGS_HIP(hipMemcpyAsync(rp.data(), F.rp, sizeof(int) * (n + 1), hipMemcpyDeviceToHost, s));
  HBGS_HIP(hipMemcpyAsync(ci.data(), F.ci, sizeof(int) * F.nnz, hipMemcpyDeviceToHost, s));
  HBGS_HIP(hipMemcpyAsync(dp.data(), out.dpos, sizeof(int) * n, hipMemcpyDeviceToHost, s));
  HBGS_HIP(hipStreamSynchronize(s));
  out.nsub = (n + sub - 1) / sub;
  for (int pass = 0; pass < 2; ++pass) {
    std::vector<int> order, lev, subp;
    ilu_schedule(n, sub, rp, ci, dp, pass == 0, order, lev, subp);
    int* o = pool.make<int>(n);
    int* l = pool.make<int>(lev.size());
    int* sp = pool.make<int>(subp.size());
    HBGS_HIP(hipMemcpyAsync(o, order.data(), sizeof(int) * n, hipMemcpyHostToDevice, s));
    HBGS_HIP(hipMemcpyAsync(l, lev.data(), sizeof(int) * lev.size(), hipMemcpyHostToDevice, s));
    HBGS_HIP(hipMemcpyAsync(sp, subp.data(), sizeof(int) * subp.size(), hipMemcpyHostToDevice, s));
    HBGS_HIP(hipStreamSynchronize(s));  // the host vectors go out of scope
    if (pass == 0) {
      out.ford = o;
      out.flev = l;
      out.fsub = sp;
    } else {
      out.bord = o;
      out.blev = l;
      out.bsub = sp;
    }
  }
  // factorisation, transposed factors, FP32 copies, work vector
  Tmp<int> zp(1);
  HBGS_HIP(hipMemsetAsync(zp.p, 0, sizeof(int), s));
  k_ilu_factor<<<out.nsub, BLK, 0, s>>>(out.ford, out.flev, out.fsub, F.rp, F.ci, F.v, out.dpos, zp.p);
  HBGS_HIP(hipGetLastError());
  int h_zero = 0;
  read_back(&h_zero, zp.p, sizeof(int), s);
  if (h_zero) return -4;
  F.vf = pool.make<float>(F.nnz);
  cast_f32(F.nnz, F.v, F.vf, s);
  out.yd = pool.make<double>(n);
  out.yf = pool.make<float>(n);
  HBGS_HIP(hipStreamSynchronize(s));
  return 0;
}

// the factors transposed (same pattern), for the adjoint sweep
void ilu_transpose(Pool& pool, IluLeaf& leaf, hipStream_t s) {
  const DCsr& F = leaf.F;
  leaf.vT = pool.make<double>(F.nnz);
  transpose_symmetric(F, leaf.vT, s);
  leaf.vTf = pool.make<float>(F.nnz);
  cast_f32(F.nnz, leaf.vT, leaf.vTf, s);
}

// One wavefront per chunk of COL_CHUNK entries.  k_col_base: the chunk's
// smallest column goes to cb; a chunk whose columns span 65536 or more sets
// bad.  k_col_pack: every entry's offset from its chunk's base.
static_assert(COL_CHUNK % 64 == 0, "chunks are whole wavefronts");
constexpr int COL_PER_LANE = COL_CHUNK / 64;
__global__ __launch_bounds__(256) void k_col_base(int64_t nnz, const int* __restrict__ ci, int* __restrict__ cb,
                                                  int* bad) {
  const int lane = threadIdx.x & 63;
  const int64_t nch = (nnz + COL_CHUNK - 1) / COL_CHUNK;
  int wide = 0;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); ch < nch; ch += (int64_t)gridDim.x * 4) {
    if (*(volatile int*)bad) break;  // another wave already found a wide chunk
    const int64_t k0 = ch * COL_CHUNK + lane;
    int lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
    for (int q = 0; q < COL_PER_LANE; ++q) {
      const int64_t k = k0 + q * 64;
      if (k < nnz) {
        const int c = ci[k];
        lo = min(lo, c);
        hi = max(hi, c);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      lo = min(lo, __shfl_xor(lo, off, 64));
      hi = max(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) cb[ch] = lo;
    if ((int64_t)hi - (int64_t)lo > 65535) {
      wide = 1;
      break;
    }
  }
  if (lane == 0 && wide) atomicOr(bad, 1);
}
__global__ __launch_bounds__(256) void k_col_pack(int64_t nnz, const int* __restrict__ ci,
                                                  const int* __restrict__ cb, uint16_t* __restrict__ cd) {
  const int lane = threadIdx.x & 63;
  const int64_t nch = (nnz + COL_CHUNK - 1) / COL_CHUNK;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); ch < nch; ch += (int64_t)gridDim.x * 4) {
    const int base = cb[ch];
    const int64_t k0 = ch * COL_CHUNK + lane;
#pragma unroll
    for (int q = 0; q < COL_PER_LANE; ++q) {
      const int64_t k = k0 + q * 64;
      if (k < nnz) cd[k] = (uint16_t)(ci[k] - base);
    }
  }
}
// a's packed columns, whose validity *bad tells (zeroed by the caller)
static void launch_pack(Pool& pool, DCsr& a, int* bad, hipStream_t s) {
  a.cd = nullptr;
  a.cb = nullptr;
  if (a.nnz == 0) return;
  const int64_t nch = (a.nnz + COL_CHUNK - 1) / COL_CHUNK;
  a.cb = pool.make<int>(nch);
  a.cd = pool.make<uint16_t>(a.nnz);
  k_col_base<<<grid_for((nch + 3) / 4, 1, 8192), 256, 0, s>>>(a.nnz, a.ci, a.cb, bad);
  HBGS_HIP(hipGetLastError());
  k_col_pack<<<grid_for((nch + 3) / 4, 1), 256, 0, s>>>(a.nnz, a.ci, a.cb, a.cd);
  HBGS_HIP(hipGetLastError());
}
static void drop_packed(Pool& pool, DCsr& a) {
  pool.release(a.cd);
  pool.release(a.cb);
  a.cd = nullptr;
  a.cb = nullptr;
}
void pack_columns(Pool& pool, DCsr& a, hipStream_t s) {
  Tmp<int> bad(1);
  HBGS_HIP(hipMemsetAsync(bad.p, 0, sizeof(int), s));
  launch_pack(pool, a, bad.p, s);
  if (a.cd && read_one(bad.p, s)) drop_packed(pool, a);
}
void stats_and_columns(Pool& pool, DCsr* const* a, int count, hipStream_t s) {
  if (count <= 0) return;
  constexpr int W = STATS + 1;
  static_assert(W * MATRICES * sizeof(int) <= Mail::kBytes, "one message");
  Tmp<int> part(W * (size_t)count);
  HBGS_HIP(hipMemsetAsync(part.p, 0, W * (size_t)count * sizeof(int), s));
  for (int k = 0; k < count; ++k) {
    launch_row_stats(*a[k], part.p + W * k, s);
    launch_pack(pool, *a[k], part.p + W * k + STATS, s);
  }
  std::vector<int> h(W * (size_t)count);
  read_back(h.data(), part.p, h.size() * sizeof(int), s);
  for (int k = 0; k < count; ++k) {
    set_stats(*a[k], &h[W * k]);
    if (h[W * k + STATS] && a[k]->cd) drop_packed(pool, *a[k]);
  }
}

__global__ void k_dense_transpose(int n, const double* __restrict__ in, double* __restrict__ out) {
  GRID_STRIDE(t, (int64_t)n * n) {
    int i = (int)(t / n), j = (int)(t % n);
    out[(int64_t)j * n + i] = in[t];
  }
}
void dense_transpose(int n, const double* in, double* out, hipStream_t s) {
  k_dense_transpose<<<grid_for((int64_t)n * n, BLK), BLK, 0, s>>>(n, in, out);
  HBGS_HIP(hipGetLastError());
}

// ------------------------------------------------------------------ casts
__global__ void k_cast_f32(int64_t n, const double* in, float* out) {
  GRID_STRIDE(i, n) out[i] = (float)in[i];
}
void cast_f32(int64_t n, const double* in, float* out, hipStream_t s) {
  if (n == 0) return;
  k_cast_f32<<<grid_for(n, BLK), BLK, 0, s>>>(n, in, out);
  HBGS_HIP(hipGetLastError());
}
__global__ void k_reciprocal(int n, const double* d, double* dinv, float* dinvf) {
  GRID_STRIDE(i, n) {
    double r = 1.0 / d[i];
    dinv[i] = r;
    dinvf[i] = (float)r;
  }
}
void reciprocal(int n, const double* d, double* dinv, float* dinvf, hipStream_t s) {
  k_reciprocal<<<grid_for(n, BLK), BLK, 0, s>>>(n, d, dinv, dinvf);
  HBGS_HIP(hipGetLastError());
}

}  // namespace setup
}  // namespace hbgs
