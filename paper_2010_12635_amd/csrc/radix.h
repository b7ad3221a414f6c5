// Stable LSD radix sort of short keys (with or without a payload), the
// building block of the CSR construction.
//
// One pass = three launches: per-tile digit histograms, one exclusive scan
// of every digit's counts along the tiles, and a stable scatter.  What
// bounds a pass is memory (two reads and one write of every item) and the
// ranking arithmetic, so:
//  * a tile is 512 * IPT consecutive items, a wave owning 64 * IPT
//    consecutive ones, all requested before the first is ranked;
//  * equal digits of the 64 items of a round are found with one ballot per
//    digit bit; the items of earlier rounds are counted in LDS counters
//    private to the wave, so the rounds need no workgroup barrier (the
//    wave's own LDS operations complete in order);
//  * the ranked tile is placed in LDS in digit order and written out digit
//    run by digit run, so that neighbouring lanes store to neighbouring
//    addresses;
//  * counts are stored tile by tile (coalesced) and scanned by one workgroup
//    per 16 digits.
#pragma once
#include "internal.h"

namespace gcn {

// Items are sorted by key() >> shift & (digits - 1).
struct Key32 {
  uint32_t k;
  __device__ __forceinline__ uint64_t key() const { return k; }
};
struct Key64 {
  uint64_t k;
  __device__ __forceinline__ uint64_t key() const { return k; }
};

// Plain array of items, source or destination of a pass.  (A source with
// FILTERED set has a keep(item): the pass leaves the other items out.)
template <typename I>
struct ItemArray {
  typedef I Item;
  static constexpr bool FILTERED = false;
  I* p;
  __device__ __forceinline__ I load(int64_t i) const { return p[i]; }
  __device__ __forceinline__ void store(int64_t i, const I& x) const { p[i] = x; }
};

constexpr int RADIX_NT = 512;                        // threads per tile
constexpr int RADIX_MAX_BITS = 9;                    // widest digit

// Items per thread: 8, or 16 from 2^25 items of up to 8 bytes and 2^27 larger ones
// on.  Longer digit runs write fuller lines, which count once the items leave the
// caches (138 M 8-byte keys sorted and compacted in 10.4 ms with 8, 8.8 ms with
// 16), but a short list then fills fewer compute units (20,000 keys 95 -> 114
// us, 8.7 M 387 -> 400), and a tile of 12-byte items with 16 takes 104 KB of LDS,
// one workgroup per compute unit: gcn_pair_backward, F = 8, with 8 / 16 at 2^25
// items 1246 / 1326 us, 2^26 3.51 / 3.67 ms, 2^27 8.25 / 7.97.
template <typename Item>
int radix_ipt(int64_t total) { return total < ((int64_t)1 << (sizeof(Item) <= 8 ? 25 : 27)) ? 8 : 16; }
template <typename Item>
int64_t radix_tiles(int64_t total) {
  const int64_t t = RADIX_NT * radix_ipt<Item>(total);
  return (total + t - 1) / t;
}

// Passes and digit width for keys of `bits` bits: as few passes as 9-bit
// digits allow, of equal width.
inline void radix_plan(int bits, int* passes, int* width) {
  *passes = (bits + RADIX_MAX_BITS - 1) / RADIX_MAX_BITS;
  if (*passes < 1) *passes = 1;
  *width = (bits + *passes - 1) / *passes;
  if (*width < 1) *width = 1;
}

// Scratch of a pass over `total` items: the tiles' counts and the digit
// totals, 32-bit while every position fits.
template <typename Item>
size_t radix_scratch_bytes(int64_t total) {
  const size_t w = total < ((int64_t)1 << 32) ? sizeof(uint32_t) : sizeof(uint64_t);
  const int64_t t = radix_tiles<Item>(total);
  return ((size_t)(t > 0 ? t : 1) + 1) * ((size_t)1 << RADIX_MAX_BITS) * w;
}

namespace {

template <typename Src, typename Item>
__device__ __forceinline__ bool radix_keeps(const Src& src, const Item& x) {
  if constexpr (Src::FILTERED) return src.keep(x);
  else return true;
}

// cnt[tile][d] = items of the tile with digit d.
template <int LOGD, int RADIX_IPT, typename Src, typename OffT>
__global__ __launch_bounds__(RADIX_NT) void radix_hist_kernel(Src src, int64_t total, int shift, uint32_t mask,
                                                              OffT* __restrict__ cnt) {
  constexpr int D = 1 << LOGD, NW = RADIX_NT / 64, RADIX_TILE = RADIX_NT * RADIX_IPT;
  __shared__ uint32_t h[NW][D];
  for (int i = threadIdx.x; i < NW * D; i += RADIX_NT) (&h[0][0])[i] = 0;
  __syncthreads();
  const int wave = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * RADIX_TILE;
  uint32_t d[RADIX_IPT];
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r) {              // every load before the first count
    const int64_t i = base + r * RADIX_NT + threadIdx.x;
    const auto x = src.load(i < total ? i : total - 1);
    d[r] = radix_keeps(src, x) ? (uint32_t)(x.key() >> shift) & mask : ~0u;
  }
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r)
    if (base + r * RADIX_NT + threadIdx.x < total && (!Src::FILTERED || d[r] != ~0u)) atomicAdd(&h[wave][d[r]], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < D; i += RADIX_NT) {
    uint32_t a = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) a += h[w][i];
    cnt[(int64_t)blockIdx.x * D + i] = a;
  }
}

// In place: cnt[t][d] -> items with digit d in the tiles before t; tot[d] =
// all of them.  A workgroup takes DW digits, its 1024 / DW groups of DW threads
// a contiguous range of tiles each.  16 digits are a whole 64-byte piece of a
// count row; with 4 (four times as many workgroups, which then share lines they
// write) sorting 8.7 M keys took 425 instead of 390 us.
template <int LOGD, typename OffT>
__global__ __launch_bounds__(1024) void radix_scan_kernel(OffT* __restrict__ cnt, int64_t ntiles, OffT* __restrict__ tot) {
  constexpr int D = 1 << LOGD, U = 8, DW = 16, GR = 1024 / DW;
  __shared__ OffT part[DW][GR + 1];
  const int dl = threadIdx.x % DW, grp = threadIdx.x / DW;
  const int d = blockIdx.x * DW + dl;
  const int64_t per = (ntiles + GR - 1) / GR;
  const int64_t t0 = grp * per < ntiles ? grp * per : ntiles, t1 = t0 + per < ntiles ? t0 + per : ntiles;
  OffT a = 0;
  for (int64_t t = t0; t < t1; t += U) {
    OffT x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = cnt[(t + u < t1 ? t + u : t1 - 1) * D + d];
#pragma unroll
    for (int u = 0; u < U; ++u) a += t + u < t1 ? x[u] : (OffT)0;
  }
  part[dl][grp] = a;
  __syncthreads();
  {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;   // wave w: digit w's 64 group sums
    const OffT v = part[w][lane];
    OffT x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const OffT y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    part[w][lane] = x - v;
    if (lane == 63) tot[blockIdx.x * DW + w] = x;
  }
  __syncthreads();
  OffT run = part[dl][grp];
  for (int64_t t = t0; t < t1; t += U) {
    OffT x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = cnt[(t + u < t1 ? t + u : t1 - 1) * D + d];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + u < t1) {
        cnt[(t + u) * D + d] = run;
        run += x[u];
      }
  }
}

// Exclusive scan over the workgroup's NT values, one per thread; red holds
// NT / 64 values.  Every thread must call it.
template <int NT, typename V>
__device__ __forceinline__ V radix_block_scan(V v, V* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  V x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) red[wave] = x;
  __syncthreads();
  V before = 0;
  for (int w = 0; w < wave; ++w) before += red[w];
  __syncthreads();
  return before + x - v;
}

template <int LOGD, int RADIX_IPT, typename Src, typename Dst, typename OffT>
__global__ __launch_bounds__(RADIX_NT) void radix_scatter_kernel(Src src, Dst dst, int64_t total, int shift,
                                                                 uint32_t mask, const OffT* __restrict__ cnt,
                                                                 const OffT* __restrict__ tot) {
  typedef typename Src::Item Item;
  constexpr int D = 1 << LOGD, NW = RADIX_NT / 64, W = sizeof(Item) / 4;
  constexpr int RADIX_TILE = RADIX_NT * RADIX_IPT;
  static_assert(D <= RADIX_NT, "at most one digit per thread");
  __shared__ uint32_t stage[W][RADIX_TILE];
  __shared__ uint16_t wc[NW][D];                     // items of the digit in the wave's earlier rounds; then its slot base
  __shared__ OffT gb[D];                             // global position of the digit's first item minus its tile slot
  __shared__ OffT red[NW];
  __shared__ int kept;                               // FILTERED: items of the tile
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * RADIX_TILE;
  const int64_t wbase = base + wave * (64 * RADIX_IPT);
  Item it[RADIX_IPT];
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r) {
    const int64_t i = wbase + r * 64 + lane;
    it[r] = src.load(i < total ? i : total - 1);
  }
  const int dt = threadIdx.x;
  const OffT dtot = dt < D ? tot[dt] : (OffT)0;
  const OffT dbefore = dt < D ? cnt[(int64_t)blockIdx.x * D + dt] : (OffT)0;
  for (int i = threadIdx.x; i < NW * D; i += RADIX_NT) (&wc[0][0])[i] = 0;
  const OffT dstart = radix_block_scan<RADIX_NT, OffT>(dtot, red);   // its barriers also cover wc

  const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  uint32_t rank[RADIX_IPT];
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r) {
    const bool valid = wbase + r * 64 + lane < total && radix_keeps(src, it[r]);
    const uint32_t d = (uint32_t)(it[r].key() >> shift) & mask;
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < LOGD; ++bit) {
      const uint64_t bb = __ballot((d >> bit) & 1u);
      const uint64_t mine = (d >> bit) & 1u ? ~0ull : 0ull;
      m &= ~(bb ^ mine);
    }
    const uint32_t pre = (uint32_t)__popcll(m & lt);
    const uint32_t prev = wc[wave][d];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && pre == 0) wc[wave][d] = (uint16_t)(prev + (uint32_t)__popcll(m));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    rank[r] = prev + pre;
  }
  __syncthreads();
  {
    uint32_t c[NW], sum = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      c[w] = dt < D ? wc[w][dt] : 0u;
      sum += c[w];
    }
    const uint32_t slot0 = (uint32_t)radix_block_scan<RADIX_NT, OffT>((OffT)sum, red);
    if (Src::FILTERED && dt == RADIX_NT - 1) kept = (int)(slot0 + sum);
    if (dt < D) {
      gb[dt] = dstart + dbefore - slot0;
      uint32_t run = slot0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        wc[w][dt] = (uint16_t)run;
        run += c[w];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r) {
    if (wbase + r * 64 + lane < total && radix_keeps(src, it[r])) {
      const uint32_t d = (uint32_t)(it[r].key() >> shift) & mask;
      const uint32_t slot = wc[wave][d] + rank[r];
      const uint32_t* w = reinterpret_cast<const uint32_t*>(&it[r]);
#pragma unroll
      for (int q = 0; q < W; ++q) stage[q][slot] = w[q];
    }
  }
  __syncthreads();
  const int64_t rest = total - base;
  const int tile_n = Src::FILTERED ? kept : rest < RADIX_TILE ? (int)rest : RADIX_TILE;
#pragma unroll
  for (int r = 0; r < RADIX_IPT; ++r) {
    const int j = r * RADIX_NT + (int)threadIdx.x;
    if (j < tile_n) {
      Item x;
      uint32_t* w = reinterpret_cast<uint32_t*>(&x);
#pragma unroll
      for (int q = 0; q < W; ++q) w[q] = stage[q][j];
      const uint32_t d = (uint32_t)(x.key() >> shift) & mask;
      dst.store((int64_t)(OffT)(gb[d] + (OffT)j), x);
    }
  }
}

template <int LOGD, int IPT, typename Src, typename Dst, typename OffT>
hipError_t radix_pass_t(const Src& src, const Dst& dst, int64_t total, int shift, int width, void* scratch, hipStream_t s) {
  const int64_t nt = radix_tiles<typename Src::Item>(total);
  OffT* cnt = static_cast<OffT*>(scratch);
  OffT* tot = cnt + nt * ((int64_t)1 << LOGD);
  const uint32_t mask = (1u << width) - 1u;
  hipLaunchKernelGGL((radix_hist_kernel<LOGD, IPT, Src, OffT>), dim3((unsigned)nt), dim3(RADIX_NT), 0, s, src, total,
                     shift, mask, cnt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((radix_scan_kernel<LOGD, OffT>), dim3((1 << LOGD) / 16), dim3(1024), 0, s, cnt, nt, tot);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((radix_scatter_kernel<LOGD, IPT, Src, Dst, OffT>), dim3((unsigned)nt), dim3(RADIX_NT), 0, s, src,
                     dst, total, shift, mask, cnt, tot);
  return hipGetLastError();
}

// One stable pass over digit (key >> shift) of `width` <= 9 bits of the `total` > 0
// items of src.
template <typename Src, typename Dst>
hipError_t radix_pass(const Src& src, const Dst& dst, int64_t total, int shift, int width, void* scratch, hipStream_t s) {
  if (radix_ipt<typename Src::Item>(total) == 8) {
    if (width <= 8) return radix_pass_t<8, 8, Src, Dst, uint32_t>(src, dst, total, shift, width, scratch, s);
    return radix_pass_t<9, 8, Src, Dst, uint32_t>(src, dst, total, shift, width, scratch, s);
  }
  if (total < ((int64_t)1 << 32)) {
    if (width <= 8) return radix_pass_t<8, 16, Src, Dst, uint32_t>(src, dst, total, shift, width, scratch, s);
    return radix_pass_t<9, 16, Src, Dst, uint32_t>(src, dst, total, shift, width, scratch, s);
  }
  if (width <= 8) return radix_pass_t<8, 16, Src, Dst, uint64_t>(src, dst, total, shift, width, scratch, s);
  return radix_pass_t<9, 16, Src, Dst, uint64_t>(src, dst, total, shift, width, scratch, s);
}

}  // namespace
}  // namespace gcn
