// Link prediction with the graph auto-encoder of Section "Graph
// Auto-Encoders", Eq. (2): A' = sigmoid(Z Z^T), evaluated on sampled vertex
// pairs rather than on all n^2 entries.
//
//  * sample_pairs_kernel: one Philox-4x64-10 block per pair (key (seed,
//    PAIR_STREAM), counter (k, epoch, 0, 0)); positives are training edges,
//    negatives uniform pairs of distinct vertices.
//  * pair_loss_kernel: a group of LPR lanes per pair gathers the two rows of
//    Z as 16-byte slices, reduces their inner product with shuffles, and
//    takes the logistic loss and its gradient g_k in fp32.  Per-pair losses
//    are summed per workgroup in a fixed order, then across workgroups.
//  * pair backward: the pair endpoints are sorted by vertex with a stable
//    radix sort (so each row's entries stay in increasing k), then cut into
//    equal segments of entries; a lane group per segment sums the rows
//    inside it and a fix-up pass adds the partial sums of rows that cross
//    segment ends, in segment order: dZ is run-to-run identical without
//    floating-point atomics, and hub rows no longer serialise on one group.
//  * pair metrics: exact AUC and AP of held-out pairs.  The scores are
//    sorted once (the same stable radix sort, on order-preserving 32-bit
//    keys), the negatives before every position are counted by a scan, and
//    every positive finds the ends of its run of equal scores by binary
//    search: negatives below / equal and all scores >= it follow from the
//    counts at those ends, O((P + N) log(P + N)) in all.  Fixed-order sums.
#include "radix.h"

#include <algorithm>

namespace gcn {

namespace {

constexpr uint64_t PAIR_STREAM = 0x50414952ull;   // second key word of the pair sampler

__global__ __launch_bounds__(256) void sample_pairs_kernel(int64_t n, const int32_t* __restrict__ edge_u,
                                                           const int32_t* __restrict__ edge_v, int64_t n_edges,
                                                           int64_t n_pos, int64_t total, uint64_t seed, uint64_t epoch,
                                                           int32_t* __restrict__ pu, int32_t* __restrict__ pv) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const Philox8 o = philox4x64_10((uint64_t)k, epoch, 0, 0, seed, PAIR_STREAM);
    if (k < n_pos) {
      const int64_t e = (int64_t)(o.w[0] % (uint64_t)n_edges);
      pu[k] = edge_u[e];
      pv[k] = edge_v[e];
    } else {
      const uint64_t u = o.w[0] % (uint64_t)n;
      const uint64_t v = (u + 1 + o.w[1] % (uint64_t)(n - 1)) % (uint64_t)n;
      pu[k] = (int32_t)u;
      pv[k] = (int32_t)v;
    }
  }
}

__device__ __forceinline__ float softplus_f(float x) { return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x))); }
__device__ __forceinline__ float sigmoid_f(float x) {
  if (x >= 0.f) return 1.f / (1.f + expf(-x));
  const float e = expf(x);
  return e / (1.f + e);
}

struct PairLossParams {
  int64_t n, F, ld;
  const void* Z;
  const int32_t* pu;
  const int32_t* pv;
  int64_t n_pos, total;
  float inv_total;
  const float* loss_scale;
  float* scores;
  float* g;
  float* part;          // [gridDim.x]
  int32_t* flag;
};

// A lane group takes R consecutive pairs per iteration: lane k of the group
// loads the ids of the k-th, the group gathers the rows of B pairs at a time
// and reduces their inner products, and lane k then takes the logistic loss of
// the k-th.  With R = 1 every wave ran the exponentials and the logarithm for
// its 64 / LPR pairs alone, which bound the kernel: 2^21 pairs, F = 64, fp16
// 88.8 us, with R = 8 56.1 us (9.6 TB/s of gathered rows), same bits of every pair.
template <typename T, int LPR, int R>
__global__ __launch_bounds__(256) void pair_loss_kernel(PairLossParams p) {
  constexpr int VE = Vec<T>::N;
  constexpr int G = 64 / LPR;
  constexpr int B = R < 4 ? R : 4;
  static_assert(R <= LPR, "a lane per pair");
  __shared__ float s_loss[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane / LPR, li = lane % LPR;
  const int64_t col0 = (int64_t)li * VE;
  const int64_t nf = p.F - col0;
  const int vc = nf <= 0 ? 0 : nf >= VE ? VE : (int)nf;   // live elements of this lane's slice
  const float scale = (p.loss_scale ? *p.loss_scale : 1.f) * p.inv_total;
  const T* __restrict__ Z = reinterpret_cast<const T*>(p.Z) + (vc > 0 ? col0 : 0);
  const int slot = (wave * G + g) * R + (li < R ? li : 0);
  float acc_loss = 0.f;
  for (int64_t base = (int64_t)blockIdx.x * (4 * G * R); base < p.total; base += (int64_t)gridDim.x * (4 * G * R)) {
    const int64_t k = base + slot;
    const bool live = li < R && k < p.total;
    const int64_t kc = k < p.total ? k : p.total - 1;
    const int32_t u = p.pu[kc], v = p.pv[kc];
    const bool ok = live && u >= 0 && v >= 0 && u < p.n && v < p.n;
    const int32_t us = ok ? u : 0, vs = ok ? v : 0;        // in bounds; the product is not used otherwise
    float mine = 0.f;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += B) {
      uint4 a[B], b[B];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        const int from = g * LPR + r0 + r;
        a[r] = ldg16(Z + (int64_t)__shfl(us, from) * p.ld);
        b[r] = ldg16(Z + (int64_t)__shfl(vs, from) * p.ld);
      }
#pragma unroll
      for (int r = 0; r < B; ++r) {
        float x[VE], y[VE];
        unpack<T>(a[r], x);
        unpack<T>(b[r], y);
        float dot = 0.f;
#pragma unroll
        for (int i = 0; i < VE; ++i) dot = i < vc ? fmaf(x[i], y[i], dot) : dot;
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
        mine = li == r0 + r ? dot : mine;
      }
    }
    if (live) {
      const float y = k < p.n_pos ? 1.f : 0.f;
      if (ok) {
        const float gk = (sigmoid_f(mine) - y) * scale;
        acc_loss += softplus_f(mine) - y * mine;
        if (p.scores) p.scores[k] = mine;
        p.g[k] = gk;
        if (!finite_f32(gk) || !finite_f32(mine)) raise_flag(p.flag);
      } else {   // vertex id outside [0, n): the pair is skipped
        if (p.scores) p.scores[k] = __int_as_float(0x7fc00000);
        p.g[k] = 0.f;
        raise_flag(p.flag);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc_loss += __shfl_xor(acc_loss, o);
  if (lane == 0) s_loss[wave] = acc_loss;
  __syncthreads();
  if (threadIdx.x == 0) p.part[blockIdx.x] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
}

__global__ __launch_bounds__(256) void pair_loss_final_kernel(const float* __restrict__ part, int64_t nb, float inv_total,
                                                              float* loss, int32_t* flag) {
  __shared__ float sl[256];
  float a = 0.f;
  for (int64_t i = threadIdx.x; i < nb; i += 256) a += part[i];
  sl[threadIdx.x] = a;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sl[threadIdx.x] += sl[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float l = sl[0] * inv_total;
    *loss = l;
    if (!finite_f32(l)) raise_flag(flag);
  }
}

int lpr_for(int prec, int64_t F) {
  const int VE = prec == 0 ? 4 : 8;
  const int64_t nvec = (F + VE - 1) / VE;
  int l = 1;
  while (l < nvec && l < 64) l <<= 1;
  return l;
}

int64_t capped_blocks(int64_t items, int64_t per_block) {
  const int64_t b = (items + per_block - 1) / per_block;
  return b < 1 ? 1 : b < 65536 ? b : 65536;
}

// Workgroups that several pairs per lane group and iteration must leave: with
// fewer the chip is not full and one pair at a time is the shorter chain.
// Whole call at the line and above: 2^17 pairs, F = 64, fp16 13.9 -> 10.3 us,
// 2^16, F = 130 19.8 -> 12.5, 2^14, F = 500 14.2 -> 10.5, 2^15, F = 128, fp32 13.6
// -> 10.4; below it the launches bound both (9.6 to 10.9 us).
constexpr int64_t PAIR_LOSS_MIN_WG = 512;

template <typename T, int LPR>
hipError_t pair_loss_lpr(const PairLossParams& p, hipStream_t s, int64_t* nb_out) {
  constexpr int R = LPR < 8 ? LPR : 8;
  const bool several = R > 1 && p.total >= PAIR_LOSS_MIN_WG * 4 * (64 / LPR) * R;
  // at most 4096 workgroups (each loops over pairs), so that the final
  // fixed-order sum over their partials is short
  int64_t nb = capped_blocks(p.total, 4 * (64 / LPR) * (several ? R : 1));
  if (nb > 4096) nb = 4096;
  *nb_out = nb;
  if (several) hipLaunchKernelGGL((pair_loss_kernel<T, LPR, R>), dim3((unsigned)nb), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((pair_loss_kernel<T, LPR, 1>), dim3((unsigned)nb), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <typename T>
hipError_t pair_loss_t(const PairLossParams& p, int lpr, hipStream_t s, int64_t* nb_out) {
  switch (lpr) {
    case 1: return pair_loss_lpr<T, 1>(p, s, nb_out);
    case 2: return pair_loss_lpr<T, 2>(p, s, nb_out);
    case 4: return pair_loss_lpr<T, 4>(p, s, nb_out);
    case 8: return pair_loss_lpr<T, 8>(p, s, nb_out);
    case 16: return pair_loss_lpr<T, 16>(p, s, nb_out);
    case 32: return pair_loss_lpr<T, 32>(p, s, nb_out);
    default: return pair_loss_lpr<T, 64>(p, s, nb_out);
  }
}

// ---- backward: pair entries sorted by endpoint, then a balanced gather
//
// Entry i of the 2K entries is endpoint (i even ? u : v) of pair k = i / 2;
// its key is that endpoint (n for a pair with an id outside [0, n)).  A
// stable radix sort by key (radix.h) puts each row's entries together in
// increasing k without atomics.  2^21 pairs, n = 2^17: two passes of 9 bits
// instead of three of 8, no workgroup barrier between the rounds of a tile:
// 215 -> 97 us.  The
// sorted entries are cut into segments of SEG entries; a lane group per
// segment sums the rows that lie inside it and leaves partial sums for the
// rows that cross its ends, which a fix-up pass adds in segment order.
constexpr int SEG = 64;                             // sorted entries per gather segment

// A pair endpoint: its vertex (the key), the gradient g_k of its pair (as
// bits) and the other endpoint, so that the segment sums read g_k with the
// entry instead of gathering it by pair index.
struct PairEnd {
  int32_t k, g, other;
  __device__ __forceinline__ uint64_t key() const { return (uint32_t)k; }
};

// The unsorted endpoints, in pair order.
struct PairEnds {
  typedef PairEnd Item;
  static constexpr bool FILTERED = false;
  int64_t n;
  const int32_t* pu;
  const int32_t* pv;
  const float* g;
  __device__ __forceinline__ PairEnd load(int64_t i) const {
    const int32_t u = pu[i >> 1], v = pv[i >> 1];
    const bool ok = u >= 0 && v >= 0 && u < n && v < n;
    return PairEnd{ok ? ((i & 1) ? v : u) : (int32_t)n, __float_as_int(g[i >> 1]), (i & 1) ? u : v};
  }
};

// Row offsets from sorted keys: off[r] = first position with key >= r,
// r = 0 .. n (keys equal to n, the skipped pairs, lie past off[n]).
__global__ void rs_bounds_kernel(int64_t n, const PairEnd* __restrict__ ends, int64_t total,
                                 int64_t* __restrict__ off) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j <= total; j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t lo = j == 0 ? -1 : ends[j - 1].k;
    const int64_t hi = j == total ? n : min<int64_t>(ends[j].k, n);
    for (int64_t r = lo + 1; r <= hi; ++r) off[r] = j;
  }
}

struct SegParams {
  int64_t n, F, ld;
  const void* Z;
  const int64_t* off;                               // [n + 1]
  const PairEnd* ends;                              // sorted
  int64_t nseg;
  float* head;                                      // [nseg][ldp]
  float* tail;                                      // [nseg][ldp]
  int32_t* tail_row;                                // [nseg]
  int64_t ldp;
  Epilogue ep;
};

// The (g, other endpoint) of a segment's entries from the sorted list itself, or
// from the segment's copy in LDS, whose entry 0 is entry `first` of the list.
struct EndsGlobal {
  const PairEnd* ends;
  __device__ __forceinline__ int2 operator()(int64_t e) const {
    const PairEnd x = ends[e];
    return make_int2(x.g, x.other);
  }
};
struct EndsLds {
  const int2* ends;
  int64_t first;
  __device__ __forceinline__ int2 operator()(int64_t e) const { return ends[(int)(e - first)]; }
};

// Sum of g_k Z[other endpoint] over sorted entries [e0, e1) into acc.
template <typename T, typename Ends>
__device__ __forceinline__ void seg_sum(const SegParams& p, const Ends& ends, int64_t e0, int64_t e1, int64_t col0,
                                        float* acc) {
  constexpr int VE = Vec<T>::N, U = 8;
  const T* __restrict__ Z = reinterpret_cast<const T*>(p.Z);
  for (int64_t e = e0; e < e1; e += U) {
    int32_t other[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ee = e + u < e1 ? e + u : e1 - 1;
      const int2 x = ends(ee);
      w[u] = __int_as_float(x.x);
      other[u] = x.y;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = e + u < e1 ? w[u] : 0.f;
    uint4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = ldg16(Z + (int64_t)other[u] * p.ld + col0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xv[VE];
      unpack<T>(x[u], xv);
#pragma unroll
      for (int q = 0; q < VE; ++q) acc[q] = fmaf(w[u], xv[q], acc[q]);
    }
  }
}

// What bounds it is the chain of dependent loads of a lane group (row ends,
// entries, gathered rows) per eight entries, so from 4 lanes per group on the
// group first copies its segment's entries to LDS, all loads at once, and a
// row's end is loaded while the row before it is summed.  2^21 pairs, n = 2^17,
// F = 64, fp16: 117.6 us with the entries read as they are used, 89.3 us so.
// (Groups of 1 or 2 lanes would need 64 KB of LDS per workgroup or more.)
template <typename T, int LPR>
__global__ __launch_bounds__(256, 4) void pair_segment_kernel(SegParams p) {
  constexpr int VE = Vec<T>::N;
  constexpr int G = 64 / LPR;
  constexpr bool STAGED = LPR >= 4;
  __shared__ int2 s_ends[STAGED ? 4 * G * SEG : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gi = lane / LPR, li = lane % LPR;
  const int64_t col0 = (int64_t)li * VE;
  if (col0 >= p.ep.ldo) return;
  const bool live = col0 < p.F;                     // padding slices only write zeros
  const int lanes = (int)min((int64_t)LPR, (p.ep.ldo + VE - 1) / VE);   // of the group, still running
  int2* mine = s_ends + (STAGED ? (wave * G + gi) * SEG : 0);
  const int64_t total = p.off[p.n];                 // entries of valid pairs
  const int64_t nuse = total > 0 ? (total + SEG - 1) / SEG : 1;
  for (int64_t sgi = ((int64_t)blockIdx.x * 4 + wave) * G + gi; sgi < p.nseg; sgi += (int64_t)gridDim.x * 4 * G) {
    if (sgi >= nuse) {                              // past the valid entries
      if (li == 0) p.tail_row[sgi] = -1;
      continue;
    }
    // rows starting in [a, b) belong to this segment; the last one also
    // takes the empty rows that start at the end.  The first row with
    // off[r] >= x is the one after the row of entry x - 1 (a binary search
    // in off took 17 dependent loads per end).
    const int64_t a = sgi * SEG, b = min(a + SEG, total);
    const int64_t r0 = a > 0 ? (int64_t)p.ends[a - 1].k + 1 : 0;
    const int64_t r1 = sgi == nuse - 1 ? p.n : (int64_t)p.ends[b - 1].k + 1;
    if constexpr (STAGED) {
      // a group's lanes share a wave, whose LDS operations complete in order:
      // the fences only keep the compiler from moving them
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll 8
      for (int j = li; j < (int)(b - a); j += lanes) mine[j] = EndsGlobal{p.ends}(a + j);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    const auto ends = [&] {
      if constexpr (STAGED) return EndsLds{mine, a};
      else return EndsGlobal{p.ends};
    }();
    float acc[VE];
    // head: the row that started before this segment
    if (r0 > 0 && p.off[r0] > a && a < b) {
#pragma unroll
      for (int q = 0; q < VE; ++q) acc[q] = 0.f;
      if (live) seg_sum<T>(p, ends, a, min(p.off[r0], b), col0, acc);
      if (col0 < p.ldp) {
#pragma unroll
        for (int q = 0; q < VE; ++q) p.head[sgi * p.ldp + col0 + q] = acc[q];
      }
    }
    int32_t trow = -1;
    int64_t rs = 0, re = 0;
    if (r0 < r1) {
      rs = p.off[r0];
      re = p.off[r0 + 1];
    }
    for (int64_t r = r0; r < r1; ++r) {
      const int64_t re_next = p.off[r + 2 <= r1 ? r + 2 : r1];
#pragma unroll
      for (int q = 0; q < VE; ++q) acc[q] = 0.f;
      if (re <= b) {
        if (live) seg_sum<T>(p, ends, rs, re, col0, acc);
        epi_store_vec<T>(p.ep, r, col0, acc);
      } else {                                      // crosses the end: partial, fixed up later
        if (live) seg_sum<T>(p, ends, rs, b, col0, acc);
        if (col0 < p.ldp) {
#pragma unroll
          for (int q = 0; q < VE; ++q) p.tail[sgi * p.ldp + col0 + q] = acc[q];
        }
        trow = (int32_t)r;
      }
      rs = re;
      re = re_next;
    }
    if (li == 0) p.tail_row[sgi] = trow;
  }
}

// VE floats of a partial row.
template <int VE>
__device__ __forceinline__ void add_row(float* acc, const float4 (&v)[VE / 4], bool live) {
#pragma unroll
  for (int i = 0; i < VE / 4; ++i) {
    acc[4 * i] = live ? acc[4 * i] + v[i].x : acc[4 * i];
    acc[4 * i + 1] = live ? acc[4 * i + 1] + v[i].y : acc[4 * i + 1];
    acc[4 * i + 2] = live ? acc[4 * i + 2] + v[i].z : acc[4 * i + 2];
    acc[4 * i + 3] = live ? acc[4 * i + 3] + v[i].w : acc[4 * i + 3];
  }
}

// Head partials of segments [t0, t1) added in order, eight in flight.
template <int VE>
__device__ __forceinline__ void add_heads(const SegParams& p, int64_t t0, int64_t t1, int64_t col0, float* acc) {
  constexpr int U = 8;
#pragma unroll 1
  for (int64_t t = t0; t < t1; t += U) {
    float4 v[U][VE / 4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < VE / 4; ++i)
        v[u][i] = reinterpret_cast<const float4*>(p.head + (t + u < t1 ? t + u : t1 - 1) * p.ldp + col0)[i];
#pragma unroll
    for (int u = 0; u < U; ++u) add_row<VE>(acc, v[u], t + u < t1);
  }
}

// Rows that cross segment ends: the tail partial of the segment where the
// row starts plus the head partials of the following segments, in order.  A
// row of more than FIX_BIG segments is left to the whole workgroup: its lane
// groups add contiguous runs of segments, then the runs are added in order
// (one lane group alone walked the 650 segments of a hub for 174 us while the
// rest of the chip idled; 19 us now, 2^21 pairs, n = 2^17, F = 64).
constexpr int FIX_BIG = 32;

template <typename T, int LPR>
__global__ __launch_bounds__(256) void pair_fixup_kernel(SegParams p) {
  constexpr int VE = Vec<T>::N;
  constexpr int G = 64 / LPR, NG = 4 * G;
  __shared__ int big[NG];
  __shared__ float red[NG][LPR * VE];
  const int gi = threadIdx.x / LPR, li = threadIdx.x % LPR;
  const int64_t col0 = (int64_t)li * VE;
  const bool live = col0 < p.F, out = col0 < p.ep.ldo;
  for (int64_t s0 = (int64_t)blockIdx.x * NG; s0 < p.nseg; s0 += (int64_t)gridDim.x * NG) {
    const int64_t sgi = s0 + gi;
    const int32_t r = sgi < p.nseg ? p.tail_row[sgi] : -1;
    const int64_t last = r >= 0 ? (p.off[r + 1] - 1) / SEG : 0;
    const bool is_big = r >= 0 && last - sgi > FIX_BIG;
    if (li == 0) big[gi] = is_big;
    if (r >= 0 && !is_big && out) {
      float acc[VE];
#pragma unroll
      for (int q = 0; q < VE; ++q) acc[q] = live ? p.tail[sgi * p.ldp + col0 + q] : 0.f;
      if (live) add_heads<VE>(p, sgi + 1, last + 1, col0, acc);
      epi_store_vec<T>(p.ep, r, col0, acc);
    }
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < NG; ++k) {
      if (!big[k]) continue;
      const int64_t sk = s0 + k;
      const int32_t rk = p.tail_row[sk];
      const int64_t t0 = sk + 1, t1 = (p.off[rk + 1] - 1) / SEG + 1, per = (t1 - t0 + NG - 1) / NG;
      const int64_t a0 = t0 + gi * per < t1 ? t0 + gi * per : t1, a1 = a0 + per < t1 ? a0 + per : t1;
      float acc[VE];
#pragma unroll
      for (int q = 0; q < VE; ++q) acc[q] = 0.f;
      if (live) add_heads<VE>(p, a0, a1, col0, acc);
#pragma unroll
      for (int q = 0; q < VE; ++q) red[gi][li * VE + q] = acc[q];
      __syncthreads();
      if (gi == 0 && out) {
#pragma unroll
        for (int q = 0; q < VE; ++q) acc[q] = live ? p.tail[sk * p.ldp + col0 + q] : 0.f;
#pragma unroll 4
        for (int j = 0; j < NG; ++j)
#pragma unroll
          for (int q = 0; q < VE; ++q) acc[q] += red[j][li * VE + q];
        epi_store_vec<T>(p.ep, rk, col0, acc);
      }
      __syncthreads();
    }
    __syncthreads();                                 // big is free for the next round
  }
}

template <typename T>
hipError_t pair_segments_t(SegParams p, int lpr, hipStream_t s) {
  const int64_t per_block = 4 * (64 / lpr);
  const unsigned blocks = (unsigned)capped_blocks(p.nseg, per_block);
#define PG(L)                                                                                   \
  hipLaunchKernelGGL((pair_segment_kernel<T, L>), dim3(blocks), dim3(256), 0, s, p);            \
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;                            \
  hipLaunchKernelGGL((pair_fixup_kernel<T, L>), dim3(blocks), dim3(256), 0, s, p);              \
  break;
  switch (lpr) {
    case 1: PG(1)
    case 2: PG(2)
    case 4: PG(4)
    case 8: PG(8)
    case 16: PG(16)
    case 32: PG(32)
    default: PG(64)
  }
#undef PG
  return hipGetLastError();
}

// ---- metrics

// Order-preserving key of a finite score: unsigned comparison of the keys
// agrees with < on the floats; -0 is taken as +0 (the two compare equal).
__device__ __forceinline__ uint32_t score_key(float x) {
  uint32_t b = __float_as_uint(x);
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// A score to sort: its key and whether it is a positive's.
struct ScoreItem {
  uint32_t k;
  int32_t pos;
  __device__ __forceinline__ uint64_t key() const { return k; }
};
struct ScoreItems {
  typedef ScoreItem Item;
  static constexpr bool FILTERED = false;
  const float* scores;
  int64_t P;
  __device__ __forceinline__ ScoreItem load(int64_t i) const { return ScoreItem{score_key(scores[i]), i < P ? 1 : 0}; }
};

// cnt[j] = 1 for a negative at sorted position j, cnt[total] = 0; an
// exclusive scan then gives the negatives before every position.
__global__ __launch_bounds__(256) void metrics_negflag_kernel(const ScoreItem* __restrict__ items, int64_t total,
                                                              int64_t* __restrict__ cnt) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j <= total; j += (int64_t)gridDim.x * blockDim.x)
    cnt[j] = j < total ? 1 - items[j].pos : 0;
}

// For the positive at sorted position j with key k: lo = first position
// with key k, hi = first position past them (binary searches).  Negatives
// below: neg[lo]; equal: neg[hi] - neg[lo]; scores >= s: total - lo, of
// which positives: P - (lo - neg[lo]).  Sums per workgroup in position order.
__global__ __launch_bounds__(256) void metrics_count_kernel(const ScoreItem* __restrict__ items,
                                                            const int64_t* __restrict__ neg, int64_t P, int64_t total,
                                                            unsigned long long* __restrict__ auc_part,
                                                            double* __restrict__ ap_part) {
  __shared__ double sd[256];
  __shared__ unsigned long long su[256];
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double ap = 0.0;
  unsigned long long auc2 = 0;
  if (j < total && items[j].pos) {
    const uint32_t k = items[j].k;
    int64_t a = 0, b = j;                           // first position in [0, j] with key >= k
    while (a < b) {
      const int64_t m = a + (b - a) / 2;
      if (items[m].k < k) a = m + 1; else b = m;
    }
    const int64_t lo = a;
    a = j + 1; b = total;                           // first position in [j + 1, total) with key > k
    while (a < b) {
      const int64_t m = a + (b - a) / 2;
      if (items[m].k <= k) a = m + 1; else b = m;
    }
    const int64_t hi = a;
    const int64_t nlo = neg[lo], nhi = neg[hi];
    auc2 = 2ull * (unsigned long long)nlo + (unsigned long long)(nhi - nlo);
    ap = (double)(P - (lo - nlo)) / (double)(total - lo);
  }
  sd[threadIdx.x] = ap;
  su[threadIdx.x] = auc2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sd[threadIdx.x] += sd[threadIdx.x + s];
      su[threadIdx.x] += su[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    ap_part[blockIdx.x] = sd[0];
    auc_part[blockIdx.x] = su[0];
  }
}

__global__ __launch_bounds__(256) void pair_metrics_final_kernel(const unsigned long long* __restrict__ auc_part,
                                                                 const double* __restrict__ ap_part, int64_t nb,
                                                                 int64_t P, int64_t N, double* out) {
  __shared__ double sd[256];
  __shared__ unsigned long long su[256];
  double a = 0.0;
  unsigned long long c = 0;
  for (int64_t b = threadIdx.x; b < nb; b += 256) { a += ap_part[b]; c += auc_part[b]; }
  sd[threadIdx.x] = a;
  su[threadIdx.x] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sd[threadIdx.x] += sd[threadIdx.x + s];
      su[threadIdx.x] += su[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = (double)su[0] / (2.0 * (double)P * (double)N);
    out[1] = sd[0] / (double)P;
  }
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

hipError_t sample_pairs_launch(int64_t n, const int32_t* edge_u, const int32_t* edge_v, int64_t n_edges, int64_t n_pos,
                               int64_t n_neg, uint64_t seed, uint64_t epoch, int32_t* pair_u, int32_t* pair_v,
                               hipStream_t s) {
  const int64_t total = n_pos + n_neg;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(sample_pairs_kernel, dim3((unsigned)capped_blocks(total, 256)), dim3(256), 0, s, n, edge_u, edge_v,
                     n_edges, n_pos, total, seed, epoch, pair_u, pair_v);
  return hipGetLastError();
}

size_t pair_loss_workspace_bytes(int64_t n_pairs) {
  (void)n_pairs;
  return 65536 * sizeof(float) + 256;
}

hipError_t pair_loss_launch(int prec, int64_t n, int64_t F, int64_t ld, const void* Z, const int32_t* pair_u,
                            const int32_t* pair_v, int64_t n_pos, int64_t n_neg, const float* loss_scale, float* loss,
                            float* scores, float* g, int32_t* flag, void* ws, hipStream_t s) {
  PairLossParams p;
  p.n = n; p.F = F; p.ld = ld; p.Z = Z; p.pu = pair_u; p.pv = pair_v;
  p.n_pos = n_pos; p.total = n_pos + n_neg; p.inv_total = 1.f / (float)p.total;
  p.loss_scale = loss_scale; p.scores = scores; p.g = g;
  p.part = reinterpret_cast<float*>(ws);
  p.flag = flag;
  const int lpr = lpr_for(prec, F);
  int64_t nb = 0;
  hipError_t e;
  switch (prec) {
    case 0: e = pair_loss_t<float>(p, lpr, s, &nb); break;
    case 1: e = pair_loss_t<f16>(p, lpr, s, &nb); break;
    case 2: e = pair_loss_t<bf16>(p, lpr, s, &nb); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pair_loss_final_kernel, dim3(1), dim3(256), 0, s, p.part, nb, p.inv_total, loss, flag);
  return hipGetLastError();
}

// Bits of the keys 0 .. n.
int pair_key_bits(int64_t n) {
  int bits = 1;
  while (((int64_t)1 << bits) <= n) ++bits;
  return bits;
}

int64_t pair_seg_count(int64_t n_pairs) {
  const int64_t t = (2 * n_pairs + SEG - 1) / SEG;
  return t < 1 ? 1 : t;
}

int64_t pair_partial_ld(int prec, int64_t F) {
  const int64_t ve = prec == 0 ? 4 : 8;
  return (F + ve - 1) / ve * ve;
}

namespace {
struct PairLayout {
  PairEnd *eA, *eB;
  void* radix;
  int64_t* off;
  float *head, *tail;
  int32_t* tail_row;
  size_t bytes;
};
// Carves the workspace (ws may be NULL to size it, for every precision).
PairLayout pair_layout(int64_t n, int64_t n_pairs, int64_t F, void* ws) {
  const int64_t total = 2 * n_pairs, nseg = pair_seg_count(n_pairs);
  const int64_t ldp = std::max(pair_partial_ld(1, F), pair_partial_ld(0, F));
  PairLayout L;
  char* base = static_cast<char*>(ws);
  size_t o = 0;
  auto take = [&](size_t bytes) { char* q = base ? base + o : nullptr; o += align256(bytes); return q; };
  L.eA = (PairEnd*)take(sizeof(PairEnd) * (total > 0 ? total : 1));
  L.eB = (PairEnd*)take(sizeof(PairEnd) * (total > 0 ? total : 1));
  L.radix = take(radix_scratch_bytes<PairEnd>(total));
  L.off = (int64_t*)take(sizeof(int64_t) * (n + 1));
  L.head = (float*)take(sizeof(float) * nseg * ldp);
  L.tail = (float*)take(sizeof(float) * nseg * ldp);
  L.tail_row = (int32_t*)take(sizeof(int32_t) * nseg);
  L.bytes = o;
  return L;
}
}  // namespace

size_t pair_backward_workspace_bytes(int64_t n, int64_t n_pairs, int64_t F) {
  return pair_layout(n, n_pairs, F, nullptr).bytes;
}

hipError_t pair_backward_launch(int prec, int64_t n, int64_t F, int64_t ld, const void* Z, const int32_t* pair_u,
                                const int32_t* pair_v, int64_t n_pairs, const float* g, void* dZ, int64_t ldz,
                                int32_t* flag, void* ws, hipStream_t s) {
  const int64_t total = 2 * n_pairs;
  const PairLayout L = pair_layout(n, n_pairs, F, ws);
  hipError_t e;
#define GCN_TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
  ItemArray<PairEnd> in{L.eB}, out{L.eA};
  if (total > 0) {
    const int bits = pair_key_bits(n);
    int passes = 0, width = 0;
    radix_plan(bits, &passes, &width);
    for (int ps = 0; ps < passes; ++ps) {
      const int shift = ps * width, w = std::min(width, bits - shift);
      if (ps == 0) GCN_TRY(radix_pass(PairEnds{n, pair_u, pair_v, g}, out, total, shift, w, L.radix, s));
      else GCN_TRY(radix_pass(in, out, total, shift, w, L.radix, s));
      std::swap(in, out);
    }
  }
  const unsigned bb = (unsigned)capped_blocks(total + 1, 256);
  hipLaunchKernelGGL(rs_bounds_kernel, dim3(bb), dim3(256), 0, s, n, in.p, total, L.off);
  GCN_TRY(hipGetLastError());
  SegParams p;
  p.n = n; p.F = F; p.ld = ld; p.Z = Z; p.off = L.off;
  p.ends = in.p;
  p.nseg = pair_seg_count(n_pairs); p.head = L.head; p.tail = L.tail; p.tail_row = L.tail_row;
  p.ldp = pair_partial_ld(prec, F);
  Epilogue ep{};
  ep.out = dZ; ep.ldo = ldz; ep.rows = n; ep.cols = F; ep.mode = EPI_STORE; ep.flag = flag; ep.keep_scale = 1.f;
  p.ep = ep;
  const int lpr = lpr_for(prec, F);
  switch (prec) {
    case 0: GCN_TRY(pair_segments_t<float>(p, lpr, s)); break;
    case 1: GCN_TRY(pair_segments_t<f16>(p, lpr, s)); break;
    case 2: GCN_TRY(pair_segments_t<bf16>(p, lpr, s)); break;
    default: return hipErrorInvalidValue;
  }
#undef GCN_TRY
  return hipSuccess;
}

namespace {
struct MetricsLayout {
  ScoreItem *iA, *iB;
  void* radix;
  int64_t *scr, *neg;
  double* ap_part;
  unsigned long long* auc_part;
  size_t bytes;
};
// Carves the workspace (ws may be NULL to size it).
MetricsLayout metrics_layout(int64_t total, void* ws) {
  const int64_t nb = (total + 255) / 256;
  MetricsLayout L;
  char* base = static_cast<char*>(ws);
  size_t o = 0;
  auto take = [&](size_t bytes) { char* q = base ? base + o : nullptr; o += align256(bytes); return q; };
  L.iA = (ScoreItem*)take(sizeof(ScoreItem) * total);
  L.iB = (ScoreItem*)take(sizeof(ScoreItem) * total);
  L.radix = take(radix_scratch_bytes<ScoreItem>(total));
  L.scr = (int64_t*)take(sizeof(int64_t) * segment_scan_scratch_elems(total + 1));
  L.neg = (int64_t*)take(sizeof(int64_t) * (total + 1));
  L.ap_part = (double*)take(sizeof(double) * nb);
  L.auc_part = (unsigned long long*)take(sizeof(unsigned long long) * nb);
  L.bytes = o;
  return L;
}
}  // namespace

size_t pair_metrics_workspace_bytes(int64_t n_pos, int64_t n_neg) {
  return metrics_layout(n_pos + n_neg, nullptr).bytes;
}

hipError_t pair_metrics_launch(const float* scores, int64_t n_pos, int64_t n_neg, double* auc_ap, void* ws,
                               hipStream_t s) {
  const int64_t total = n_pos + n_neg;
  const MetricsLayout L = metrics_layout(total, ws);
  const int64_t nb = (total + 255) / 256;
  const unsigned gb = (unsigned)capped_blocks(total + 1, 256);
  hipError_t e;
#define GCN_TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
  // four stable 8-bit passes over the 32-bit keys
  ItemArray<ScoreItem> in{L.iB}, out{L.iA};
  for (int shift = 0; shift < 32; shift += 8) {
    if (shift == 0) GCN_TRY(radix_pass(ScoreItems{scores, n_pos}, out, total, shift, 8, L.radix, s));
    else GCN_TRY(radix_pass(in, out, total, shift, 8, L.radix, s));
    std::swap(in, out);
  }
  hipLaunchKernelGGL(metrics_negflag_kernel, dim3(gb), dim3(256), 0, s, in.p, total, L.neg);
  GCN_TRY(hipGetLastError());
  GCN_TRY(segment_scan_exclusive(L.neg, total + 1, L.scr, s));
  hipLaunchKernelGGL(metrics_count_kernel, dim3((unsigned)nb), dim3(256), 0, s, in.p, L.neg, n_pos, total,
                     L.auc_part, L.ap_part);
  GCN_TRY(hipGetLastError());
  hipLaunchKernelGGL(pair_metrics_final_kernel, dim3(1), dim3(256), 0, s, L.auc_part, L.ap_part, nb, n_pos, n_neg,
                     auc_ap);
#undef GCN_TRY
  return hipGetLastError();
}

}  // namespace gcn
