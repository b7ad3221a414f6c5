// A_hat = D^-1/2 (A + I) D^-1/2 from an undirected edge list, as canonical
// CSR (rows ascending, columns ascending and unique), plus the heavy-row
// schedule used by the sparse aggregation.
//
// Steps (all integer, so the CSR is bit-identical from run to run):
//  * both directions of every pair, and (i, i) for every vertex, become keys
//    row << b | column, b the bits of a vertex id; a pair (v, v) and a repeat
//    become repeats of a key that is there anyway;
//  * a radix sort of the keys (radix.h): 32-bit keys up to n = 65536, else
//    64-bit ones.  Its time does not depend on how the entries are spread
//    over the rows: sorting row segments instead left the hubs of a power-law
//    graph to one workgroup each, and counting them took atomics on few
//    addresses (R-MAT scale 18, 8.7 M keys: 6.3 ms in all before, the
//    numbers now are at normalize_run);
//  * the distinct keys of every tile are counted and scanned, then written
//    out in order: columns, row pointers (where a row begins; no row is
//    empty) and the entry's row, which the values need;
//  * from 2^31 keys on all of this range by range of the keys (RangedKeys), so
//    that the workspace stays below 5 bytes per key;
//  * degrees and dinv = fp32(1 / sqrt(fp64(deg))); values dinv[row] *
//    dinv[col] in the value precision, one thread per entry; optional dense.
#include "radix.h"

#include <algorithm>

namespace gcn {

namespace {

constexpr int SCAN_BLOCK = 1024;   // elements per scan block (256 threads x 4)

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int64_t scan_scratch_elems(int64_t count) {
  int64_t total = 0;
  while (count > SCAN_BLOCK) {
    count = (count + SCAN_BLOCK - 1) / SCAN_BLOCK;
    total += count;
  }
  return total + 1;
}

// ------------------------------------------------------------------ scan ----
// Four row counts scanned together: two int64 of two 32-bit halves each
// (every total stays below 2^31, so no half carries into the other).
struct Counts4 {
  int64_t a, b;
  __device__ __forceinline__ Counts4 operator+(const Counts4& o) const { return {a + o.a, b + o.b}; }
  __device__ __forceinline__ Counts4 operator-(const Counts4& o) const { return {a - o.a, b - o.b}; }
  __host__ __device__ static int64_t pack(int64_t hi, int64_t lo) { return hi << 32 | lo; }
  __host__ __device__ static int64_t hi(int64_t x) { return x >> 32; }
  __host__ __device__ static int64_t lo(int64_t x) { return x & 0xffffffffll; }
};

template <typename V>
__global__ __launch_bounds__(256) void scan_block_kernel(V* __restrict__ data, int64_t count,
                                                         V* __restrict__ block_sums) {
  __shared__ V s[256];
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x * 4;
  V v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = base + i < count ? data[base + i] : V{};
  const V tsum = v[0] + v[1] + v[2] + v[3];
  s[threadIdx.x] = tsum;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const V add = threadIdx.x >= off ? s[threadIdx.x - off] : V{};
    __syncthreads();
    s[threadIdx.x] = s[threadIdx.x] + add;
    __syncthreads();
  }
  V run = s[threadIdx.x] - tsum;   // exclusive prefix of this thread
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (base + i < count) data[base + i] = run;
    run = run + v[i];
  }
  if (threadIdx.x == 255 && block_sums) block_sums[blockIdx.x] = s[255];
}

template <typename V>
__global__ __launch_bounds__(256) void scan_add_kernel(V* __restrict__ data, int64_t count,
                                                       const V* __restrict__ block_off) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x * 4;
  const V add = block_off[blockIdx.x];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (base + i < count) data[base + i] = data[base + i] + add;
}

// In-place exclusive scan of data[0..count); scratch holds scan_scratch_elems(count).
template <typename V>
hipError_t scan_exclusive(V* data, int64_t count, V* scratch, hipStream_t s) {
  const int64_t nb = (count + SCAN_BLOCK - 1) / SCAN_BLOCK;
  hipLaunchKernelGGL(scan_block_kernel<V>, dim3((unsigned)nb), dim3(256), 0, s, data, count, nb > 1 ? scratch : nullptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nb <= 1) return e;
  e = scan_exclusive(scratch, nb, scratch + nb, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(scan_add_kernel<V>, dim3((unsigned)nb), dim3(256), 0, s, data, count, scratch);
  return hipGetLastError();
}

// ---------------------------------------------------------------- helpers ----
__global__ void fill_zero_kernel(uint32_t* p, int64_t words) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

unsigned grid_for(int64_t items, int per_block = 256, int64_t cap = 65536) {
  int64_t g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

// ---------------------------------------------------------------- kernels ----
// Item i of the sort: pair i forwards, pair i - E backwards, then the
// self-loops.  A pair with a vertex id outside [0, n) raises *bad and stands
// for the self-loop of vertex 0.
template <typename I>
struct EdgeItems {
  typedef I Item;
  static constexpr bool FILTERED = false;
  int64_t n, E;
  const int32_t* src;
  const int32_t* dst;
  int b;
  int32_t* bad;
  __device__ __forceinline__ I load(int64_t i) const {
    typedef decltype(I::k) K;
    I x;
    if (i >= 2 * E) {
      const K r = (K)(i - 2 * E);
      x.k = (K)(r << b) | r;
      return x;
    }
    const int64_t k = i < E ? i : i - E;
    const int32_t u = src[k], v = dst[k];
    const bool ok = u >= 0 && v >= 0 && u < n && v < n;
    if (!ok) *reinterpret_cast<volatile int32_t*>(bad) = 1;
    const K r = ok ? (K)(i < E ? u : v) : (K)0, c = ok ? (K)(i < E ? v : u) : (K)0;
    x.k = (K)(r << b) | c;
    return x;
  }
};

// The items with keys in [lo, hi].
template <typename I>
struct RangeItems : EdgeItems<I> {
  static constexpr bool FILTERED = true;
  uint64_t lo, hi;
  __device__ __forceinline__ bool keep(const I& x) const { return x.key() >= lo && x.key() <= hi; }
};

// cnt[(key - lo) >> shift] += 1 for the keys in [lo, hi]; at most RANGE_BINS
// bins, cleared beforehand.
constexpr int RANGE_BITS = 10, RANGE_BINS = 1 << RANGE_BITS;

template <typename I>
__global__ __launch_bounds__(256) void range_hist_kernel(RangeItems<I> src, int64_t total, int shift,
                                                         unsigned long long* __restrict__ cnt) {
  constexpr int U = 8;
  __shared__ uint32_t h[RANGE_BINS];                 // a workgroup's share: below 2^32
  for (int b = threadIdx.x; b < RANGE_BINS; b += 256) h[b] = 0;
  __syncthreads();
  for (int64_t base = (int64_t)blockIdx.x * (256 * U); base < total; base += (int64_t)gridDim.x * (256 * U)) {
    I x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = base + u * 256 + threadIdx.x;
      x[u] = src.load(i < total ? i : total - 1);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + u * 256 + threadIdx.x < total && src.keep(x[u])) atomicAdd(&h[(x[u].key() - src.lo) >> shift], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < RANGE_BINS; b += 256)
    if (h[b]) atomicAdd(&cnt[b], (unsigned long long)h[b]);
}

template <typename I>
__global__ void one_key_kernel(I* p, uint64_t key) {
  p->k = (decltype(I::k))key;
}

constexpr int UNIQ_IPT = 8;
constexpr int UNIQ_TILE = 256 * UNIQ_IPT;

// A wave's 64 * UNIQ_IPT sorted keys and, per round, the lanes whose key
// differs from the one before it.
template <typename I>
struct UniqWave {
  typedef decltype(I::k) K;
  K k[UNIQ_IPT], prev[UNIQ_IPT];
  uint64_t first[UNIQ_IPT];
  __device__ __forceinline__ void load(const I* __restrict__ keys, int64_t w0, int64_t total) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < UNIQ_IPT; ++r) {
      const int64_t i = w0 + r * 64 + lane;
      k[r] = keys[i < total ? i : total - 1].k;
      prev[r] = keys[i < total ? (i > 0 ? i - 1 : 0) : total - 1].k;
    }
#pragma unroll
    for (int r = 0; r < UNIQ_IPT; ++r) {
      const int64_t i = w0 + r * 64 + lane;
      first[r] = __ballot(i < total && (i == 0 || k[r] != prev[r]));
    }
  }
};

// cnt[tile] = distinct keys that begin in the tile; cnt[tiles] = 0.
template <typename I>
__global__ __launch_bounds__(256) void uniq_count_kernel(const I* __restrict__ keys, int64_t total,
                                                         int64_t* __restrict__ cnt) {
  __shared__ int wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  UniqWave<I> x;
  x.load(keys, (int64_t)blockIdx.x * UNIQ_TILE + wave * (64 * UNIQ_IPT), total);
  int a = 0;
#pragma unroll
  for (int r = 0; r < UNIQ_IPT; ++r) a += __popcll(x.first[r]);
  if (lane == 0) wsum[wave] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    cnt[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (blockIdx.x == 0) cnt[gridDim.x] = 0;
  }
}

// Distinct keys in order, from entry `first` on: colidx, the row of every entry
// (if rows is not NULL), and rowptr where a row begins (each row holds its
// self-loop, so each begins somewhere); the keys' first row began before if it
// is prev_row.
template <typename I, typename IdxT>
__global__ __launch_bounds__(256) void uniq_write_kernel(const I* __restrict__ keys, int64_t total, int b, int64_t n,
                                                         const int64_t* __restrict__ off, int64_t first,
                                                         int64_t prev_row, int32_t* __restrict__ colidx,
                                                         int32_t* __restrict__ rows, IdxT* __restrict__ rowptr) {
  typedef decltype(I::k) K;
  __shared__ int wsum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t w0 = (int64_t)blockIdx.x * UNIQ_TILE + wave * (64 * UNIQ_IPT);
  UniqWave<I> x;
  x.load(keys, w0, total);
  int a = 0;
#pragma unroll
  for (int r = 0; r < UNIQ_IPT; ++r) a += __popcll(x.first[r]);
  if (lane == 0) wsum[wave] = a;
  __syncthreads();
  int64_t run = first + off[blockIdx.x];
  for (int w = 0; w < wave; ++w) run += wsum[w];
  const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  const K cmask = (K)(((K)1 << b) - 1);
#pragma unroll
  for (int r = 0; r < UNIQ_IPT; ++r) {
    if (x.first[r] >> lane & 1) {
      const int64_t pos = run + __popcll(x.first[r] & lt);
      const K row = x.k[r] >> b;
      colidx[pos] = (int32_t)(x.k[r] & cmask);
      if (rows) rows[pos] = (int32_t)row;
      if (w0 + r * 64 + lane == 0 ? (int64_t)row != prev_row : row != x.prev[r] >> b) rowptr[row] = (IdxT)pos;
    }
    run += __popcll(x.first[r]);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) rowptr[n] = (IdxT)(first + off[gridDim.x]);
}

template <typename IdxT>
__global__ void degree_kernel(int64_t n, const IdxT* __restrict__ rowptr, int32_t* __restrict__ deg,
                              float* __restrict__ dinv) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int32_t d = (int32_t)((int64_t)rowptr[r + 1] - (int64_t)rowptr[r]);
    if (deg) deg[r] = d;
    dinv[r] = (float)(1.0 / sqrt((double)d));
  }
}

// One thread per entry (four in flight each); *nnz entries.
template <typename T>
__global__ __launch_bounds__(256) void values_kernel(const int64_t* __restrict__ nnz, const int32_t* __restrict__ rows,
                                                     const int32_t* __restrict__ colidx, const float* __restrict__ dinv,
                                                     T* __restrict__ values, T* __restrict__ dense, int64_t ld_dense) {
  constexpr int U = 4;
  const int64_t total = *nnz;
  for (int64_t base = (int64_t)blockIdx.x * (256 * U); base < total; base += (int64_t)gridDim.x * (256 * U)) {
    int32_t r[U], c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = base + u * 256 + threadIdx.x;
      r[u] = rows[k < total ? k : total - 1];
      c[u] = colidx[k < total ? k : total - 1];
    }
    float a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { a[u] = dinv[r[u]]; b[u] = dinv[c[u]]; }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = base + u * 256 + threadIdx.x;
      if (k >= total) break;
      const T v = from_f32<T>(a[u] * b[u]);
      if (values) values[k] = v;
      if (dense) dense[(int64_t)r[u] * ld_dense + c[u]] = v;
    }
  }
}

// The same without the rows of the entries: a workgroup finds the rows of its
// first and last entry in rowptr, a thread the row of its own between them.
constexpr int VALUES_TILE = 2048;

template <typename T, typename IdxT>
__global__ __launch_bounds__(256) void values_search_kernel(int64_t nnz, int64_t n, const IdxT* __restrict__ rowptr,
                                                            const int32_t* __restrict__ colidx,
                                                            const float* __restrict__ dinv, T* __restrict__ values,
                                                            T* __restrict__ dense, int64_t ld_dense) {
  auto row_of = [&](int64_t k, int64_t lo, int64_t hi) {   // the last r in [lo, hi] with rowptr[r] <= k
    while (lo < hi) {
      const int64_t m = hi - ((hi - lo) >> 1);
      if ((int64_t)rowptr[m] <= k) lo = m;
      else hi = m - 1;
    }
    return lo;
  };
  for (int64_t base = (int64_t)blockIdx.x * VALUES_TILE; base < nnz; base += (int64_t)gridDim.x * VALUES_TILE) {
    const int64_t end = base + VALUES_TILE < nnz ? base + VALUES_TILE : nnz;
    const int64_t ra = row_of(base, 0, n - 1), rb = row_of(end - 1, ra, n - 1);
    for (int64_t k = base + threadIdx.x; k < end; k += 256) {
      const int64_t r = row_of(k, ra, rb);
      const int32_t c = colidx[k];
      const T v = from_f32<T>(dinv[r] * dinv[c]);
      if (values) values[k] = v;
      if (dense) dense[r * ld_dense + c] = v;
    }
  }
}

// ---------------------------------------------------------------- schedule ----
// Heavy rows are cut into pieces: at the boundaries of the P column ranges
// (column c lies in range floor(c P / n)) and then every `seg` entries.
// Range q ends at the first entry of the (sorted) row whose column c has
// c P >= (q + 1) n, i.e. c >= ceil((q + 1) n / P).
// First column of range q: ceil(q n / P).
__device__ __forceinline__ int64_t range_first(int64_t q, int64_t n, int64_t parts) {
  return (q * n + parts - 1) / parts;
}

__device__ __forceinline__ int64_t range_end(const int32_t* __restrict__ colidx, int64_t lo, int64_t hi, int64_t bound) {
  while (lo < hi) {                       // first k in [lo, hi) with colidx[k] >= bound
    const int64_t mid = lo + ((hi - lo) >> 1);
    if ((int64_t)colidx[mid] < bound) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// A heavy row's share of the scan: itself and its pieces; whether the fix-up
// adds its partials with a whole workgroup or with a lane group.
__device__ __forceinline__ Counts4 row_counts(int64_t pieces) {
  const int64_t big = pieces > GCN_FIX_BIG_PIECES, small = pieces >= 2 && pieces <= GCN_FIX_BIG_PIECES;
  return {Counts4::pack(1, pieces), Counts4::pack(big, small)};
}

// The scan of the rows' counts (heavy rows, their pieces; rows of many and of
// a few pieces) says where everything of a row goes: its slot in heavy_rows,
// its pieces, its place in fix_rows (rows of many pieces first).
template <typename IdxT>
__global__ void piece_fill_kernel(int64_t n, int64_t nnz, const IdxT* __restrict__ rowptr,
                                  const int32_t* __restrict__ colidx, int64_t thr, int64_t seg, int64_t parts,
                                  const Counts4* __restrict__ off, int32_t* __restrict__ heavy_rows,
                                  int32_t* __restrict__ heavy_chunk_off, int32_t* __restrict__ chunk_heavy,
                                  int64_t* __restrict__ chunk_beg, int32_t* __restrict__ fix_rows) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= n; r += (int64_t)gridDim.x * blockDim.x) {
    if (r == n) {
      const int64_t t = off[n].a;
      heavy_chunk_off[Counts4::hi(t)] = (int32_t)Counts4::lo(t);
      chunk_beg[Counts4::lo(t)] = nnz;
      continue;
    }
    const int64_t beg = (int64_t)rowptr[r], end = (int64_t)rowptr[r + 1];
    if (end - beg <= thr) continue;
    const Counts4 o = off[r], o1 = off[r + 1];
    const int64_t h = Counts4::hi(o.a);
    heavy_rows[h] = (int32_t)r;
    heavy_chunk_off[h] = (int32_t)Counts4::lo(o.a);
    if (Counts4::hi(o1.b) != Counts4::hi(o.b)) fix_rows[Counts4::hi(o.b)] = (int32_t)h;
    else if (Counts4::lo(o1.b) != Counts4::lo(o.b)) fix_rows[Counts4::hi(off[n].b) + Counts4::lo(o.b)] = (int32_t)h;
    int64_t c = Counts4::lo(o.a), a = beg;
    for (int64_t q = 0; q < parts; ++q) {
      const int64_t b = q + 1 == parts ? end : range_end(colidx, a, end, range_first(q + 1, n, parts));
      for (int64_t k = a; k < b; k += seg) {
        chunk_heavy[c] = (int32_t)h;
        chunk_beg[c] = k;
        ++c;
      }
      a = b;
    }
  }
}

// Light rows, block by block of `blk` consecutive row ids, by decreasing
// degree inside a block: a counting sort over the buckets
// (r / blk) (thr + 1) + thr - deg (deg <= thr), except the rows of exactly
// one entry, which all go to one last bucket so that the product can take
// them in bundles (on R-MAT scale 21 they are 42 % of the light rows).  Rows of similar length
// share a wave, and on large graphs rows whose ids are close -- whose
// neighbours overlap more in an R-MAT graph -- run together (R-MAT scale 21:
// 5 % faster than one global degree order).  Below 2^20 rows one block (a
// global decreasing-degree order) is kept: there the longest rows must
// start first or they form the tail (R-MAT scale 17, F = 256: 23 % slower
// with blocks of 4096).  A workgroup owns a contiguous range of rows and
// first counts them per bucket in LDS, so the global atomics are one per
// bucket and workgroup; buckets beyond LIGHT_LDS_BINS of the workgroup's
// first bucket use global atomics.
constexpr int LIGHT_LDS_BINS = 1024;

int64_t light_block(int64_t n) { return n >= ((int64_t)1 << 20) ? 4096 : (n > 0 ? n : 1); }
int64_t light_buckets(int64_t n, int64_t thr) {
  const int64_t blk = light_block(n);
  return (n + blk - 1) / blk * (thr + 1) + 1;
}

// Bucket of a light row r of degree d (nb buckets, the last for one-entry
// rows) and its LDS slot in a workgroup whose first block bucket is base
// (LIGHT_LDS_BINS for the last bucket; -1: no slot, global atomics).
__device__ __forceinline__ int64_t light_bucket(int64_t r, int64_t d, int64_t thr, int64_t blk, int64_t nb) {
  return d == 1 ? nb - 1 : (r / blk) * (thr + 1) + thr - d;
}
__device__ __forceinline__ int light_slot(int64_t b, int64_t base, int64_t nb) {
  if (b == nb - 1) return LIGHT_LDS_BINS;
  return b - base < LIGHT_LDS_BINS ? (int)(b - base) : -1;
}
// Bucket of LDS slot k (or -1 when the slot maps to no bucket of the block range).
__device__ __forceinline__ int64_t slot_bucket(int k, int64_t base, int64_t nb) {
  if (k == LIGHT_LDS_BINS) return nb - 1;
  return base + k < nb - 1 ? base + k : -1;
}

__device__ __forceinline__ void row_range(int64_t n, int64_t* r0, int64_t* r1) {
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  *r0 = (int64_t)blockIdx.x * per;
  *r1 = *r0 + per < n ? *r0 + per : n;
}

// Workgroups of the two kernels over the light rows: 1024 rows each, so that the
// global atomics, one per bucket and workgroup, stay few (a workgroup per 256
// rows spent 20 us on them at 262144 rows), and 4096 workgroups, until each has
// 8192 rows, two blocks of light rows: at most 258 buckets with the default
// threshold, where LDS holds 1024.  n = 2^27 (whole gcn_schedule): 5.24 ms with 4096
// workgroups of eight blocks, 4.45 so, 4.63 with 65536.
unsigned light_grid(int64_t n) { return grid_for(n, 1024, std::max<int64_t>(4096, (n + 8191) / 8192)); }

// Per row: its counts for the scan (counts[n] = 0), and, for a light row, its
// bucket's histogram.
template <typename IdxT>
__global__ __launch_bounds__(256) void row_count_kernel(int64_t n, const IdxT* __restrict__ rowptr,
                                                        const int32_t* __restrict__ colidx, int64_t thr, int64_t seg,
                                                        int64_t parts, int64_t blk, int64_t nb,
                                                        Counts4* __restrict__ counts, int32_t* __restrict__ hist) {
  __shared__ int32_t lh[LIGHT_LDS_BINS + 1];
  for (int b = threadIdx.x; b <= LIGHT_LDS_BINS; b += 256) lh[b] = 0;
  __syncthreads();
  int64_t r0, r1;
  row_range(n, &r0, &r1);
  const int64_t base = (r0 / blk) * (thr + 1);
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const int64_t beg = (int64_t)rowptr[r], end = (int64_t)rowptr[r + 1], d = end - beg;
    if (d > thr) {
      int64_t cnt = 0, a = beg;
      for (int64_t q = 0; q < parts; ++q) {
        const int64_t b = q + 1 == parts ? end : range_end(colidx, a, end, range_first(q + 1, n, parts));
        cnt += (b - a + seg - 1) / seg;
        a = b;
      }
      counts[r] = row_counts(cnt);
      continue;
    }
    counts[r] = Counts4{};
    const int64_t b = light_bucket(r, d, thr, blk, nb);
    const int k = light_slot(b, base, nb);
    if (k >= 0) atomicAdd(&lh[k], 1);
    else atomicAdd(&hist[b], 1);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) counts[n] = Counts4{};
  __syncthreads();
  for (int k = threadIdx.x; k <= LIGHT_LDS_BINS; k += 256) {
    const int64_t b = slot_bucket(k, base, nb);
    if (b >= 0 && lh[k]) atomicAdd(&hist[b], lh[k]);
  }
}

// Places the light rows: row_perm and, so that a lane group learns where a row
// lies with one load, their 16-byte descriptors {first entry, row, length}.
template <typename IdxT>
__global__ __launch_bounds__(256) void light_scatter_kernel(int64_t n, const IdxT* __restrict__ rowptr, int64_t thr,
                                                            int64_t blk, int64_t nb, const int64_t* __restrict__ boff,
                                                            int32_t* __restrict__ cur, int32_t* __restrict__ perm,
                                                            RowDesc* __restrict__ desc) {
  __shared__ int32_t lh[LIGHT_LDS_BINS + 1];     // count, then this workgroup's base within the bucket
  __shared__ int32_t lc[LIGHT_LDS_BINS + 1];     // local cursor
  for (int b = threadIdx.x; b <= LIGHT_LDS_BINS; b += 256) { lh[b] = 0; lc[b] = 0; }
  __syncthreads();
  int64_t r0, r1;
  row_range(n, &r0, &r1);
  const int64_t base = (r0 / blk) * (thr + 1);
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const int64_t d = (int64_t)rowptr[r + 1] - (int64_t)rowptr[r];
    if (d > thr) continue;
    const int k = light_slot(light_bucket(r, d, thr, blk, nb), base, nb);
    if (k >= 0) atomicAdd(&lh[k], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= LIGHT_LDS_BINS; k += 256) {
    const int64_t b = slot_bucket(k, base, nb);
    if (b >= 0 && lh[k]) lh[k] = atomicAdd(&cur[b], lh[k]);
  }
  __syncthreads();
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const int64_t beg = (int64_t)rowptr[r], d = (int64_t)rowptr[r + 1] - beg;
    if (d > thr) continue;
    const int64_t b = light_bucket(r, d, thr, blk, nb);
    const int k = light_slot(b, base, nb);
    const int64_t pos = boff[b] + (k >= 0 ? (int64_t)lh[k] + atomicAdd(&lc[k], 1) : (int64_t)atomicAdd(&cur[b], 1));
    perm[pos] = (int32_t)r;
    desc[pos] = RowDesc{beg, (int32_t)r, (int32_t)d};
  }
}

// Piece launch order: counting sort of the pieces by the column bucket of
// their first entry (CHUNK_BUCKETS buckets over [0, n)).  The bucket of a
// column, c * 4096 / n, nests in its column range c * P / n for every P
// that divides 4096, so the sorted pieces of range p are one run, starting
// at the offset of bucket p * 4096 / P.  The first pieces of the hubs crowd
// into the lowest buckets, so a workgroup counts its pieces in LDS first (one
// global atomic per piece took 33 us for 27,000 pieces, twice).
constexpr int64_t CHUNK_BUCKETS = 4096;

// Pieces [c0, c1) of this workgroup; *total = all of them.
__device__ __forceinline__ void piece_range(const Counts4* __restrict__ total, int64_t* c0, int64_t* c1) {
  const int64_t m = Counts4::lo(total->a), per = (m + gridDim.x - 1) / gridDim.x;
  *c0 = (int64_t)blockIdx.x * per;
  *c1 = *c0 + per < m ? *c0 + per : m;
}

__device__ __forceinline__ int chunk_bucket(int64_t n, int32_t col) { return (int)((int64_t)col * CHUNK_BUCKETS / n); }

__global__ __launch_bounds__(256) void chunk_hist_kernel(int64_t n, const Counts4* __restrict__ total,
                                                         const int32_t* __restrict__ colidx,
                                                         const int64_t* __restrict__ chunk_beg,
                                                         int32_t* __restrict__ hist) {
  __shared__ int32_t lh[CHUNK_BUCKETS];
  int64_t c0, c1;
  piece_range(total, &c0, &c1);
  if (c0 >= c1) return;
  for (int b = threadIdx.x; b < CHUNK_BUCKETS; b += 256) lh[b] = 0;
  __syncthreads();
  for (int64_t c = c0 + threadIdx.x; c < c1; c += 256) atomicAdd(&lh[chunk_bucket(n, colidx[chunk_beg[c]])], 1);
  __syncthreads();
  for (int b = threadIdx.x; b < CHUNK_BUCKETS; b += 256)
    if (lh[b]) atomicAdd(&hist[b], lh[b]);
}

// Results of a schedule, read back by the host in one copy.
struct SchedTotals {
  int64_t rows_a, rows_b;      // Counts4 totals
  int64_t n_light, n_multi;    // light rows; of them, rows of several entries
  int64_t slots;               // most pieces on one XCD
};

// The light rows' bucket counts as the operand of a grid-wide scan: off[b] =
// hist[b], off[nb] = 0.
__global__ void light_widen_kernel(int64_t nb, const int32_t* __restrict__ hist, int64_t* __restrict__ off) {
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b <= nb; b += (int64_t)gridDim.x * blockDim.x)
    off[b] = b < nb ? hist[b] : 0;
}

// Light-row buckets up to which one workgroup scans them, beside the one that
// scans the pieces' buckets: each of its threads walks nb / 1024 buckets alone.
// Above, the grid does, in four launches more: whole gcn_schedule at n = 2^20
// with 4097 buckets 177 us by one workgroup, 183 by the grid, with 16385 162 /
// 152, with 65537 252 / 151; n = 2^24, 528,385 buckets 2296 / 738.
constexpr int64_t LIGHT_SCAN_ONE_WG = 1 << 14;

// Bucket offsets from the histograms (workgroup 0: light rows, nb buckets,
// unless loff holds their offsets already; workgroup 1: pieces), the column
// ranges' piece offsets and the totals.
__global__ __launch_bounds__(1024) void bucket_scan_kernel(int64_t nb, const int32_t* __restrict__ lhist,
                                                           int64_t* __restrict__ loff, bool scanned,
                                                           const int32_t* __restrict__ chist,
                                                           int64_t* __restrict__ coff, int64_t parts,
                                                           int64_t* __restrict__ part_off,
                                                           const Counts4* __restrict__ rows, SchedTotals* __restrict__ out) {
  __shared__ int64_t red[16];
  const int32_t* hist = blockIdx.x ? chist : lhist;
  int64_t* off = blockIdx.x ? coff : loff;
  const int64_t m = blockIdx.x ? CHUNK_BUCKETS : nb;
  if (blockIdx.x || !scanned) {
    const int64_t per = (m + 1023) / 1024;
    const int64_t b0 = threadIdx.x * per < m ? threadIdx.x * per : m, b1 = b0 + per < m ? b0 + per : m;
    int64_t sum = 0;
    for (int64_t b = b0; b < b1; ++b) sum += hist[b];
    int64_t run = radix_block_scan<1024, int64_t>(sum, red);
    for (int64_t b = b0; b < b1; ++b) {
      off[b] = run;
      run += hist[b];
    }
    if (threadIdx.x == 1023) off[m] = run;            // past the last bucket: the total
    __syncthreads();                                  // the offsets are visible to the workgroup
  }
  if (!blockIdx.x) {
    if (threadIdx.x == 0) {
      out->n_light = loff[nb];
      out->n_multi = loff[nb - 1];
      out->rows_a = rows->a;
      out->rows_b = rows->b;
    }
    return;
  }
  for (int64_t q = threadIdx.x; q <= parts; q += 1024) part_off[q] = coff[q * (CHUNK_BUCKETS / parts)];
  if (threadIdx.x == 0) {                             // ranges x, x + 8, ... run on XCD x
    int64_t most = coff[CHUNK_BUCKETS];
    if (parts > 1) {
      most = 0;
      for (int64_t x = 0; x < XCDS; ++x) {
        int64_t t = 0;
        for (int64_t q = x; q < parts; q += XCDS)
          t += coff[(q + 1) * (CHUNK_BUCKETS / parts)] - coff[q * (CHUNK_BUCKETS / parts)];
        if (t > most) most = t;
      }
    }
    out->slots = most;
  }
}

// Places the pieces: chunk_order, their launch positions and their 16-byte
// descriptors {first entry, row, length | 2^31 if the row has no other piece}.
template <typename IdxT>
__global__ __launch_bounds__(256) void chunk_scatter_kernel(
    int64_t n, const Counts4* __restrict__ total, const IdxT* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const int64_t* __restrict__ boff, int32_t* __restrict__ cur, const int32_t* __restrict__ chunk_heavy,
    const int32_t* __restrict__ heavy_rows, const int32_t* __restrict__ heavy_chunk_off,
    const int64_t* __restrict__ chunk_beg, int32_t* __restrict__ order, RowDesc* __restrict__ desc,
    int32_t* __restrict__ pos_of) {
  __shared__ int32_t lh[CHUNK_BUCKETS];              // count, then the next position within the bucket
  int64_t c0, c1;
  piece_range(total, &c0, &c1);
  if (c0 >= c1) return;
  for (int b = threadIdx.x; b < CHUNK_BUCKETS; b += 256) lh[b] = 0;
  __syncthreads();
  for (int64_t c = c0 + threadIdx.x; c < c1; c += 256) atomicAdd(&lh[chunk_bucket(n, colidx[chunk_beg[c]])], 1);
  __syncthreads();
  for (int b = threadIdx.x; b < CHUNK_BUCKETS; b += 256)
    if (lh[b]) lh[b] = atomicAdd(&cur[b], lh[b]);
  __syncthreads();
  for (int64_t c = c0 + threadIdx.x; c < c1; c += 256) {
    const int64_t b = chunk_beg[c];
    const int k = chunk_bucket(n, colidx[b]);
    const int64_t pos = boff[k] + atomicAdd(&lh[k], 1);
    const int32_t h = chunk_heavy[c];
    const int32_t r = heavy_rows[h];
    const int64_t rend = (int64_t)rowptr[r + 1];
    const int64_t e = chunk_beg[c + 1] < rend ? chunk_beg[c + 1] : rend;
    const bool single = heavy_chunk_off[h + 1] - heavy_chunk_off[h] == 1;
    order[pos] = (int32_t)c;
    desc[pos] = RowDesc{b, r, (int32_t)((uint32_t)(e - b) | (single ? 0x80000000u : 0u))};
    pos_of[c] = (int32_t)pos;
  }
}

}  // namespace

int64_t segment_scan_scratch_elems(int64_t count) { return scan_scratch_elems(count); }

hipError_t segment_scan_exclusive(int64_t* data, int64_t count, int64_t* scratch, hipStream_t s) {
  return scan_exclusive(data, count, scratch, s);
}

hipError_t fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  // callers pass 4-byte multiples
  const int64_t words = (int64_t)(bytes / 4);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(words, 256, 16384)), dim3(256), 0, s, (uint32_t*)p, words);
  return hipGetLastError();
}

namespace {
int id_bits(int64_t n) {
  int b = 1;
  while (((int64_t)1 << b) < n) ++b;
  return b;
}

// Keys from which they are sorted in ranges of a quarter of them each (and some
// more, so that even rows make four), the ranges in turn in the same two buffers:
// 4.6 bytes of workspace per key of 8 bytes instead of 16.5, which would be more
// than an eighth of the memory here.  The price is that every range reads the
// edge list twice: R-MAT scale 26, 2.2 G keys, all in one sort 172 ms and 36.0 GB,
// in ranges 235 ms and 9.7 GB; scale 27 389 ms, 73.1 GB and 545 ms, 20.5 GB.
constexpr int64_t NORM_RANGES_FROM = (int64_t)1 << 31;

// Workspace of normalize_run: two key buffers, the sort's scratch, the
// distinct keys per tile with their scan, the bad-id flag, the ranges' bins.
struct NormLayout {
  char *kA, *kB;
  void* radix;
  int64_t *off, *scr;
  int32_t* bad;
  unsigned long long* bins;
  bool ranges;
  int64_t most;              // keys a buffer holds
  size_t bytes;
};
NormLayout norm_layout(int64_t n, int64_t E, void* ws) {
  const int64_t total = 2 * E + n;
  NormLayout L;
  L.ranges = total >= NORM_RANGES_FROM;
  L.most = L.ranges ? total / 4 + total / 128 : total;
  const int64_t nu = (L.most + UNIQ_TILE - 1) / UNIQ_TILE;
  const bool k32 = 2 * id_bits(n) <= 32;
  const size_t kb = (k32 ? sizeof(Key32) : sizeof(Key64)) * (size_t)L.most;
  char* base = static_cast<char*>(ws);
  size_t o = 0;
  auto take = [&](size_t bytes) { char* p = base ? base + o : nullptr; o += align256(bytes); return p; };
  L.kA = take(kb);
  L.kB = take(kb);
  L.radix = take(k32 ? radix_scratch_bytes<Key32>(total) : radix_scratch_bytes<Key64>(total));
  L.off = (int64_t*)take(sizeof(int64_t) * (nu + 2));   // the scan's total (nnz), then the flag: read back together
  L.scr = (int64_t*)take(sizeof(int64_t) * scan_scratch_elems(nu + 1));
  L.bad = base ? (int32_t*)(L.off + nu + 1) : nullptr;
  L.bins = L.ranges ? (unsigned long long*)take(sizeof(unsigned long long) * RANGE_BINS) : nullptr;
  L.bytes = o;
  return L;
}

struct NormOut {
  void* rowptr;
  bool idx64;
  int32_t *colidx, *deg;
  float* dinv;
  int value_prec;
  void *values, *dense;
  int64_t ld_dense;
};

#define GCN_TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)

// Sorts the `kept` keys that src keeps of its `total` items.
template <typename I, typename Src>
hipError_t sort_keys(const Src& src, int64_t total, int64_t kept, int bits, const NormLayout& L, const I** keys,
                     I** spare, hipStream_t s) {
  hipError_t e;
  int passes = 0, width = 0;
  radix_plan(bits, &passes, &width);
  ItemArray<I> in{(I*)L.kB}, out{(I*)L.kA};
  for (int ps = 0; ps < passes; ++ps) {
    const int shift = ps * width, w = std::min(width, bits - shift);
    if (ps == 0) GCN_TRY(radix_pass(src, out, total, shift, w, L.radix, s));
    else GCN_TRY(radix_pass(in, out, kept, shift, w, L.radix, s));
    std::swap(in, out);
  }
  *keys = in.p;
  *spare = out.p;
  return hipSuccess;
}

// Distinct ones of `count` sorted keys to the CSR arrays, from entry `first` on.
template <typename I>
hipError_t write_distinct(const I* keys, int64_t count, int64_t n, int64_t first, int64_t prev_row, int32_t* rows,
                          const NormOut& o, const NormLayout& L, hipStream_t s) {
  hipError_t e;
  const int b = id_bits(n);
  const int64_t nu = (count + UNIQ_TILE - 1) / UNIQ_TILE;
  const dim3 ug((unsigned)nu);
  hipLaunchKernelGGL(uniq_count_kernel<I>, ug, dim3(256), 0, s, keys, count, L.off);
  GCN_TRY(hipGetLastError());
  GCN_TRY(scan_exclusive(L.off, nu + 1, L.scr, s));
  if (o.idx64)
    hipLaunchKernelGGL((uniq_write_kernel<I, int64_t>), ug, dim3(256), 0, s, keys, count, b, n, L.off, first, prev_row,
                       o.colidx, rows, (int64_t*)o.rowptr);
  else
    hipLaunchKernelGGL((uniq_write_kernel<I, int32_t>), ug, dim3(256), 0, s, keys, count, b, n, L.off, first, prev_row,
                       o.colidx, rows, (int32_t*)o.rowptr);
  return hipGetLastError();
}

hipError_t degrees(int64_t n, const NormOut& o, hipStream_t s) {
  if (o.idx64)
    hipLaunchKernelGGL(degree_kernel<int64_t>, dim3(grid_for(n)), dim3(256), 0, s, n, (const int64_t*)o.rowptr, o.deg,
                       o.dinv);
  else
    hipLaunchKernelGGL(degree_kernel<int32_t>, dim3(grid_for(n)), dim3(256), 0, s, n, (const int32_t*)o.rowptr, o.deg,
                       o.dinv);
  return hipGetLastError();
}

// All keys in one sort; the values from the entries' rows, which go to the
// other key buffer.
template <typename I>
hipError_t normalize_keys(const EdgeItems<I>& edges, const NormOut& o, const NormLayout& L, int64_t* nnz_out,
                          int32_t* bad_ids, hipStream_t s) {
  const int64_t n = edges.n, total = 2 * edges.E + n;
  const I* keys;
  I* spare;
  hipError_t e;
  GCN_TRY(sort_keys(edges, total, total, 2 * edges.b, L, &keys, &spare, s));
  int32_t* rows = (int32_t*)spare;
  GCN_TRY(write_distinct(keys, total, n, 0, -1, rows, o, L, s));
  GCN_TRY(degrees(n, o, s));
  const int64_t* nnz = L.off + (total + UNIQ_TILE - 1) / UNIQ_TILE;
  if (o.dense) GCN_TRY(fill_zero(o.dense, (size_t)n * (size_t)o.ld_dense * (o.value_prec == 0 ? 4 : 2), s));
  if (o.values || o.dense) {
    const dim3 g(grid_for(total, 1024, 8192));
    switch (o.value_prec) {
      case 0: hipLaunchKernelGGL(values_kernel<float>, g, dim3(256), 0, s, nnz, rows, o.colidx, o.dinv, (float*)o.values, (float*)o.dense, o.ld_dense); break;
      case 1: hipLaunchKernelGGL(values_kernel<f16>, g, dim3(256), 0, s, nnz, rows, o.colidx, o.dinv, (f16*)o.values, (f16*)o.dense, o.ld_dense); break;
      case 2: hipLaunchKernelGGL(values_kernel<bf16>, g, dim3(256), 0, s, nnz, rows, o.colidx, o.dinv, (bf16*)o.values, (bf16*)o.dense, o.ld_dense); break;
      default: return hipErrorInvalidValue;
    }
    GCN_TRY(hipGetLastError());
  }
  // the one synchronisation: nnz and the bad-id flag back to the host
  int64_t host[2] = {0, 0};
  GCN_TRY(hipMemcpyAsync(host, nnz, sizeof(host), hipMemcpyDeviceToHost, s));
  GCN_TRY(hipStreamSynchronize(s));
  *nnz_out = host[0];
  *bad_ids = (int32_t)host[1];
  return hipSuccess;
}

// The keys range by range in ascending order.
template <typename I>
struct RangedKeys {
  const EdgeItems<I>& edges;
  const NormOut& o;
  const NormLayout& L;
  hipStream_t s;
  int64_t nnz = 0, prev_row = -1;           // entries written, the row of the last
  int32_t bad = 0;

  RangeItems<I> items(uint64_t lo, uint64_t hi) const {
    RangeItems<I> r;
    static_cast<EdgeItems<I>&>(r) = edges;
    r.lo = lo;
    r.hi = hi;
    return r;
  }

  // The `count` > 0 keys in [lo, hi], sorted in the buffers unless they are all one.
  hipError_t write(uint64_t lo, uint64_t hi, int64_t count) {
    const int64_t total = 2 * edges.E + edges.n;
    hipError_t e;
    const I* keys = (const I*)L.kA;
    I* spare;
    if (lo == hi) {
      count = 1;
      hipLaunchKernelGGL(one_key_kernel<I>, dim3(1), dim3(1), 0, s, (I*)L.kA, lo);
      GCN_TRY(hipGetLastError());
    } else {
      GCN_TRY(sort_keys(items(lo, hi), total, count, 2 * edges.b, L, &keys, &spare, s));
    }
    GCN_TRY(write_distinct(keys, count, edges.n, nnz, prev_row, (int32_t*)nullptr, o, L, s));
    int64_t added = 0;
    I last{};
    GCN_TRY(hipMemcpyAsync(&added, L.off + (count + UNIQ_TILE - 1) / UNIQ_TILE, sizeof(added), hipMemcpyDeviceToHost, s));
    GCN_TRY(hipMemcpyAsync(&last, keys + count - 1, sizeof(last), hipMemcpyDeviceToHost, s));
    GCN_TRY(hipStreamSynchronize(s));
    nnz += added;
    prev_row = (int64_t)(last.k >> edges.b);
    return hipSuccess;
  }

  // The keys in [lo, lo + 2^bits): counted in up to RANGE_BINS bins, neighbouring
  // bins together as long as they fit a buffer, larger bins split again.
  hipError_t run(uint64_t lo, int bits) {
    const int64_t total = 2 * edges.E + edges.n;
    const int shift = bits > RANGE_BITS ? bits - RANGE_BITS : 0;
    unsigned long long cnt[RANGE_BINS];
    hipError_t e;
    GCN_TRY(fill_zero(L.bins, sizeof(cnt), s));
    hipLaunchKernelGGL(range_hist_kernel<I>, dim3(grid_for(total, 2048, 4096)), dim3(256), 0, s,
                       items(lo, lo + (((uint64_t)1 << bits) - 1)), total, shift, L.bins);
    GCN_TRY(hipGetLastError());
    GCN_TRY(hipMemcpyAsync(cnt, L.bins, sizeof(cnt), hipMemcpyDeviceToHost, s));
    GCN_TRY(hipMemcpyAsync(&bad, L.bad, sizeof(bad), hipMemcpyDeviceToHost, s));
    GCN_TRY(hipStreamSynchronize(s));
    if (bad) return hipSuccess;
    uint64_t from = lo;                     // keys of the open range, which ends before bin d
    int64_t held = 0;
    for (int d = 0; d < 1 << (bits - shift); ++d) {
      const uint64_t at = lo + ((uint64_t)d << shift);
      const int64_t c = (int64_t)cnt[d];
      if (held + c <= L.most) {
        held += c;
        continue;
      }
      if (held) GCN_TRY(write(from, at - 1, held));
      from = at;
      held = c;
      if (c <= L.most) continue;
      if (shift) GCN_TRY(run(at, shift));
      else GCN_TRY(write(at, at, c));
      from = at + ((uint64_t)1 << shift);
      held = 0;
    }
    if (held) GCN_TRY(write(from, lo + (((uint64_t)1 << bits) - 1), held));
    return hipSuccess;
  }
};

template <typename T, typename IdxT>
hipError_t values_by_search(int64_t nnz, int64_t n, const NormOut& o, hipStream_t s) {
  hipLaunchKernelGGL((values_search_kernel<T, IdxT>), dim3(grid_for(nnz, VALUES_TILE)), dim3(256), 0, s, nnz, n,
                     (const IdxT*)o.rowptr, o.colidx, o.dinv, (T*)o.values, (T*)o.dense, o.ld_dense);
  return hipGetLastError();
}

template <typename I>
hipError_t normalize_ranges(const EdgeItems<I>& edges, const NormOut& o, const NormLayout& L, int64_t* nnz_out,
                            int32_t* bad_ids, hipStream_t s) {
  const int64_t n = edges.n;
  RangedKeys<I> r{edges, o, L, s};
  hipError_t e;
  GCN_TRY(r.run(0, 2 * edges.b));
  *nnz_out = r.nnz;
  *bad_ids = r.bad;
  if (r.bad) return hipSuccess;
  GCN_TRY(degrees(n, o, s));
  if (o.dense) GCN_TRY(fill_zero(o.dense, (size_t)n * (size_t)o.ld_dense * (o.value_prec == 0 ? 4 : 2), s));
  if (!o.values && !o.dense) return hipSuccess;
  if (!o.idx64) return hipErrorInvalidValue;        // 32-bit row pointers end before the ranges begin
  switch (o.value_prec) {
    case 0: return values_by_search<float, int64_t>(r.nnz, n, o, s);
    case 1: return values_by_search<f16, int64_t>(r.nnz, n, o, s);
    case 2: return values_by_search<bf16, int64_t>(r.nnz, n, o, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename I>
hipError_t normalize_t(const EdgeItems<I>& edges, const NormOut& o, const NormLayout& L, int64_t* nnz_out,
                       int32_t* bad_ids, hipStream_t s) {
  return L.ranges ? normalize_ranges(edges, o, L, nnz_out, bad_ids, s)
                  : normalize_keys(edges, o, L, nnz_out, bad_ids, s);
}
}  // namespace

// Measured (MI355X, R-MAT scale 18, 8.65 M keys of 36 bits, four passes of 9
// bits): gcn_normalize + gcn_schedule 6.33 -> 0.50 ms; a pass 64 us (counts
// 14, scan 12, scatter 38: 3.5 TB/s of keys read and written), distinct keys
// 32 us, values 36 us.
size_t normalize_workspace_bytes(int64_t n, int64_t E) { return norm_layout(n, E, nullptr).bytes; }

hipError_t normalize_run(int64_t n, int64_t E, const int32_t* src, const int32_t* dst, bool idx64,
                         void* rowptr, int32_t* colidx, int32_t* deg, float* dinv, int value_prec,
                         void* values, void* dense, int64_t ld_dense, int64_t* nnz_out, int32_t* bad_ids,
                         void* ws, size_t ws_bytes, hipStream_t s) {
  const NormLayout L = norm_layout(n, E, ws);
  if (L.bytes > ws_bytes) return hipErrorInvalidValue;
  const NormOut o{rowptr, idx64, colidx, deg, dinv, value_prec, values, dense, ld_dense};
  const int b = id_bits(n);
  hipError_t e;
  GCN_TRY(fill_zero(L.bad, sizeof(int64_t), s));
  if (2 * b <= 32) return normalize_t(EdgeItems<Key32>{n, E, src, dst, b, L.bad}, o, L, nnz_out, bad_ids, s);
  return normalize_t(EdgeItems<Key64>{n, E, src, dst, b, L.bad}, o, L, nnz_out, bad_ids, s);
}
#undef GCN_TRY

// Most pieces a schedule can hold: every heavy row (more than thr entries,
// so at most nnz / (thr + 1) of them) has at most one piece per column range
// plus one per chunk_nnz entries.
int64_t max_pieces(int64_t n, int64_t nnz, int64_t thr, int64_t chunk_nnz, int64_t parts) {
  const int64_t rows = std::min<int64_t>(n, nnz / (thr + 1));
  return nnz / chunk_nnz + rows * parts + 1;
}

namespace {
// The schedule buffer: what the product reads, then what only the
// construction needs.
struct SchedLayout {
  int32_t *order, *heavy_rows, *heavy_chunk_off, *chunk_heavy, *piece_pos, *fix_rows, *perm;
  int64_t *chunk_beg, *part_off;
  RowDesc *piece_desc, *row_desc;
  Counts4 *counts, *scr;
  int32_t *chist, *ccur, *hist, *cur;      // contiguous: cleared together
  size_t zero_bytes;
  int64_t *cboff, *boff, *bscr;
  SchedTotals* totals;
  size_t bytes;
};
SchedLayout sched_layout(int64_t n, int64_t nnz, int64_t thr, int64_t chunk, int64_t parts, void* sched) {
  const int64_t mc = max_pieces(n, nnz, thr, chunk, parts), nb = light_buckets(n, thr);
  SchedLayout L;
  char* base = static_cast<char*>(sched);
  size_t o = 0;
  auto take = [&](size_t bytes) { char* p = base ? base + o : nullptr; o += align256(bytes); return p; };
  L.order = (int32_t*)take(sizeof(int32_t) * mc);
  L.heavy_rows = (int32_t*)take(sizeof(int32_t) * n);
  L.heavy_chunk_off = (int32_t*)take(sizeof(int32_t) * (n + 1));
  L.chunk_heavy = (int32_t*)take(sizeof(int32_t) * mc);
  L.chunk_beg = (int64_t*)take(sizeof(int64_t) * (mc + 1));
  L.part_off = (int64_t*)take(sizeof(int64_t) * (parts + 1));
  L.piece_desc = (RowDesc*)take(sizeof(RowDesc) * mc);
  L.piece_pos = (int32_t*)take(sizeof(int32_t) * mc);
  L.fix_rows = (int32_t*)take(sizeof(int32_t) * n);
  L.row_desc = (RowDesc*)take(sizeof(RowDesc) * n);
  L.perm = (int32_t*)take(sizeof(int32_t) * n);
  L.counts = (Counts4*)take(sizeof(Counts4) * (n + 1));
  L.scr = (Counts4*)take(sizeof(Counts4) * scan_scratch_elems(n + 1));
  const size_t z0 = o;
  L.chist = (int32_t*)take(sizeof(int32_t) * CHUNK_BUCKETS);
  L.ccur = (int32_t*)take(sizeof(int32_t) * CHUNK_BUCKETS);
  L.hist = (int32_t*)take(sizeof(int32_t) * nb);
  L.cur = (int32_t*)take(sizeof(int32_t) * nb);
  L.zero_bytes = o - z0;
  L.cboff = (int64_t*)take(sizeof(int64_t) * (CHUNK_BUCKETS + 1));
  L.boff = (int64_t*)take(sizeof(int64_t) * (nb + 1));
  L.bscr = (int64_t*)take(sizeof(int64_t) * scan_scratch_elems(nb + 1));
  L.totals = (SchedTotals*)take(sizeof(SchedTotals));
  L.bytes = o;
  return L;
}

// Ten launches (more for long scans) and one synchronisation: nothing on the way needs a count on
// the host (the kernels over the pieces read their number on the device).
template <typename IdxT>
hipError_t schedule_t(int64_t n, int64_t nnz, const IdxT* rowptr, const int32_t* colidx, int64_t thr, int64_t chunk,
                      int64_t parts, const SchedLayout& L, SchedTotals* host, hipStream_t s) {
  const int64_t nb = light_buckets(n, thr), blk = light_block(n);
  const dim3 rg(light_grid(n));
  const dim3 cg(grid_for(max_pieces(n, nnz, thr, chunk, parts), 2048, 512));
  hipError_t e;
#define GCN_TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
  GCN_TRY(fill_zero(L.chist, L.zero_bytes, s));
  hipLaunchKernelGGL(row_count_kernel<IdxT>, rg, dim3(256), 0, s, n, rowptr, colidx, thr, chunk, parts, blk, nb,
                     L.counts, L.hist);
  GCN_TRY(hipGetLastError());
  GCN_TRY(scan_exclusive(L.counts, n + 1, L.scr, s));
  const Counts4* total = L.counts + n;
  hipLaunchKernelGGL(piece_fill_kernel<IdxT>, dim3(grid_for(n + 1)), dim3(256), 0, s, n, nnz, rowptr, colidx, thr, chunk,
                     parts, L.counts, L.heavy_rows, L.heavy_chunk_off, L.chunk_heavy, L.chunk_beg, L.fix_rows);
  GCN_TRY(hipGetLastError());
  hipLaunchKernelGGL(chunk_hist_kernel, cg, dim3(256), 0, s, n, total, colidx, L.chunk_beg, L.chist);
  GCN_TRY(hipGetLastError());
  const bool wide = nb > LIGHT_SCAN_ONE_WG;
  if (wide) {
    hipLaunchKernelGGL(light_widen_kernel, dim3(grid_for(nb + 1)), dim3(256), 0, s, nb, L.hist, L.boff);
    GCN_TRY(hipGetLastError());
    GCN_TRY(scan_exclusive(L.boff, nb + 1, L.bscr, s));
  }
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(2), dim3(1024), 0, s, nb, L.hist, L.boff, wide, L.chist, L.cboff, parts,
                     L.part_off, total, L.totals);
  GCN_TRY(hipGetLastError());
  hipLaunchKernelGGL(light_scatter_kernel<IdxT>, rg, dim3(256), 0, s, n, rowptr, thr, blk, nb, L.boff, L.cur, L.perm,
                     L.row_desc);
  GCN_TRY(hipGetLastError());
  hipLaunchKernelGGL(chunk_scatter_kernel<IdxT>, cg, dim3(256), 0, s, n, total, rowptr, colidx, L.cboff, L.ccur,
                     L.chunk_heavy, L.heavy_rows, L.heavy_chunk_off, L.chunk_beg, L.order, L.piece_desc, L.piece_pos);
  GCN_TRY(hipGetLastError());
  GCN_TRY(hipMemcpyAsync(host, L.totals, sizeof(SchedTotals), hipMemcpyDeviceToHost, s));
  GCN_TRY(hipStreamSynchronize(s));
#undef GCN_TRY
  return hipSuccess;
}
}  // namespace

size_t schedule_bytes(int64_t n, int64_t nnz, int64_t thr, int64_t chunk_nnz, int64_t parts) {
  return sched_layout(n, nnz, thr, chunk_nnz, parts, nullptr).bytes;
}

hipError_t schedule_run(int64_t n, int64_t nnz, bool idx64, const void* rowptr, const int32_t* colidx, int64_t thr,
                        int64_t chunk, int64_t parts, void* sched, size_t sched_bytes, SchedOut* out, hipStream_t s) {
  const SchedLayout L = sched_layout(n, nnz, thr, chunk, parts, sched);
  if (L.bytes > sched_bytes) return hipErrorInvalidValue;
  SchedTotals t{};
  const hipError_t e = idx64 ? schedule_t(n, nnz, (const int64_t*)rowptr, colidx, thr, chunk, parts, L, &t, s)
                             : schedule_t(n, nnz, (const int32_t*)rowptr, colidx, thr, chunk, parts, L, &t, s);
  if (e != hipSuccess) return e;
  const int64_t n_chunks = Counts4::lo(t.rows_a);
  if (n_chunks > max_pieces(n, nnz, thr, chunk, parts)) return hipErrorInvalidValue;
  out->heavy_rows = L.heavy_rows; out->heavy_chunk_off = L.heavy_chunk_off; out->chunk_heavy = L.chunk_heavy;
  out->row_perm = L.perm;
  out->chunk_order = n_chunks > 0 ? L.order : nullptr;
  out->chunk_beg = L.chunk_beg; out->part_off = L.part_off; out->part_slots = n_chunks > 0 ? t.slots : 0;
  out->piece_desc = L.piece_desc; out->piece_pos = L.piece_pos; out->row_desc = L.row_desc;
  out->fix_rows = L.fix_rows;
  out->n_fix_big = Counts4::hi(t.rows_b);
  out->n_fix = Counts4::hi(t.rows_b) + Counts4::lo(t.rows_b);
  out->n_heavy = Counts4::hi(t.rows_a); out->n_chunks = n_chunks;
  out->n_light = t.n_light; out->n_light_single = t.n_light - t.n_multi;
  return hipSuccess;
}

}  // namespace gcn
