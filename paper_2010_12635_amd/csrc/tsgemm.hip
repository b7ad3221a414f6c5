// Tall-skinny products of the layer, C (n x N) = A (n x K) . B (K x N) with
// n large and K, N <= a few hundred:
//   S = H W                        (B(k, n) = W[k][n])
//   dZ_below = (G_S W^T) * mask    (B(k, n) = W[n][k])
// Both are bound by streaming A and C through HBM (arithmetic intensity
// <= 64 flop/byte in 16-bit storage), so the kernel is organised around the
// stream:
//  * a workgroup stages its block of B (up to 128 columns x K, k-contiguous,
//    zero-padded to the MFMA k chunk) in LDS once;
//  * each of its 4 waves owns TM x 16 consecutive rows of A and reads their
//    MFMA operand fragments straight from global memory (rows are adjacent,
//    so a wave's loads stay inside one compact region), with a 3-deep
//    register ring of chunks in flight; B fragments come from LDS;
//  * the output of each 16-row tile is staged, 128 bytes of a row at a time,
//    through a per-wave LDS buffer and written as 16-byte row-contiguous
//    vectors after the epilogue (plain store, or the ReLU/dropout derivative
//    read from H).  The buffer is kept that small, and the column blocks that
//    narrow, so that two workgroups (two waves per SIMD) share a compute unit.
#include "internal.h"
#include "xpose.h"

#include <algorithm>

namespace gcn {

namespace {

template <typename T> struct TsMfma;
template <> struct TsMfma<f16> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct TsMfma<bf16> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct TsMfma<float> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

constexpr int TS_LDS_B_BYTES = 80 * 1024;   // cap of the B block in LDS

struct TsParams {
  const void* A; int64_t lda;
  const void* B; int64_t ldb;
  int64_t M, N, K;
  int64_t kpad;            // K rounded up to the k chunk
  int nblk;                // columns per workgroup (multiple of 16)
  Epilogue epi;
  float* colsum;           // CS: [gridDim.x][N] column sums of the stored C, one row per workgroup
};

// Staging of a wave: 16 rows of VPC output vectors, in fp32 where the epilogue
// still has to scale the sums, else already rounded to T.
template <typename T, bool DM, int TNW>
struct TsStage {
  static constexpr int OV = Vec<T>::N;
  static constexpr int VPC = TNW * 16 / OV < 8 ? TNW * 16 / OV : 8;     // vectors per row and step (at most 128 bytes)
  static constexpr int NCH = (TNW * 16 / OV + VPC - 1) / VPC;            // steps per 16-row tile
  static constexpr int NT = VPC * OV / 16;                               // 16-column tiles per step
  static constexpr int IT = VPC < 4 ? 1 : VPC / 4;                       // vectors per lane and step
  static constexpr int ROW = DM ? (VPC * OV + 4) * 4 : (VPC * OV + 16 / (int)sizeof(T)) * (int)sizeof(T);   // bytes
  static constexpr int BYTES = 16 * ROW;
};

// Dynamic LDS: B block [nblk][kpad + VE] (T), then 4 per-wave staging buffers.
// DM: epilogue multiplies by the ReLU/dropout derivative read from H
// (EPI_DMASK with relu); otherwise a plain store.
// CS: the workgroup also sums the stored values (as stored, i.e. rounded to
// T) of each of its columns: a lane stores the same column vectors of every
// tile and sums them in registers (tiles in order); at the end the lanes of
// equal columns, then the four waves in wave order, are added into the
// workgroup's row of p.colsum (bias gradient of the layer below, without a
// pass of its own over C).
template <typename T, bool BKC, bool DM, bool CS, int TM, int TNW>
__global__ __launch_bounds__(256) void tsgemm_kernel(TsParams p) {
  using St = TsStage<T, DM, TNW>;
  constexpr int VE = Vec<T>::N;
  constexpr int KC = 4 * VE;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = p.nblk;
  const int64_t ldsb = p.kpad + VE;                 // LDS row stride of B (elements)
  T* sB = reinterpret_cast<T*>(smem);
  unsigned char* sC = smem + ((size_t)nblk * ldsb * sizeof(T) + 15) / 16 * 16;
  unsigned char* myC = sC + wave * St::BYTES;
  const int64_t n0 = (int64_t)blockIdx.y * nblk;
  const T* __restrict__ Bg = reinterpret_cast<const T*>(p.B);

  // ---- B block -> LDS, k-contiguous: sB[c][k] = B(k, n0 + c), zero outside.
  // Every load of a batch is issued (at an in-bounds address) before any is
  // used; out-of-range elements are zeroed afterwards with dword masks.
  if (BKC) {   // B(k, n) = Bg[n * ldb + k]: copy 16-byte vectors
    constexpr int TS_STAGE = 8;
    const int vpr = (int)(p.kpad / VE);
    const int total = nblk * vpr;
    for (int base = 0; base < total; base += 256 * TS_STAGE) {
      uint4 x[TS_STAGE];
#pragma unroll
      for (int u = 0; u < TS_STAGE; ++u) {
        const int v = base + u * 256 + (int)threadIdx.x;
        const int64_t n = n0 + v / vpr, k = (int64_t)(v % vpr) * VE;
        const bool ok = v < total && n < p.N && k < p.K;
        x[u] = ldg16(Bg + (ok ? n * p.ldb + k : 0));
      }
#pragma unroll
      for (int u = 0; u < TS_STAGE; ++u) {
        const int v = base + u * 256 + (int)threadIdx.x;
        if (v >= total) break;
        const int c = v / vpr;
        const int64_t n = n0 + c, k = (int64_t)(v % vpr) * VE;
        const int64_t nk = p.K - k;
        const int vk = (n >= p.N || nk <= 0) ? 0 : nk >= VE ? VE : (int)nk;
        *reinterpret_cast<uint4*>(sB + c * ldsb + k) = keep_first<T>(x[u], vk);
      }
    }
  } else {     // B(k, n) = Bg[k * ldb + n]: VE x VE blocks (VE k rows x VE columns) turned around in registers
    const int cpb = nblk / VE;                        // column blocks
    const int kpb = (int)(p.kpad / VE);               // k blocks
    const int total = cpb * kpb;
    for (int blk = threadIdx.x; blk < total; blk += 256) {
      const int kb = blk % kpb, cb = blk / kpb;       // consecutive threads: consecutive k blocks (LDS banks)
      const int64_t k0 = (int64_t)kb * VE, n = n0 + (int64_t)cb * VE;
      const int64_t nn = p.N - n;
      const int vc = nn <= 0 ? 0 : nn >= VE ? VE : (int)nn;
      const T* colp = Bg + (vc > 0 ? n : 0);         // n + VE <= round_up(N, 8) <= ldb
      uint4 in[VE], out[VE];
#pragma unroll
      for (int i = 0; i < VE; ++i) in[i] = ldg16(colp + (k0 + i < p.K ? k0 + i : 0) * p.ldb);
#pragma unroll
      for (int i = 0; i < VE; ++i) in[i] = keep_first<T>(in[i], k0 + i < p.K ? vc : 0);
      transpose_block(in, out, T());
#pragma unroll
      for (int j = 0; j < VE; ++j) *reinterpret_cast<uint4*>(sB + (cb * VE + j) * ldsb + k0) = out[j];
    }
  }
  __syncthreads();

  // ---- stream row tiles of A (4 waves x TM x 16 rows per tile), B stays in LDS
  const int64_t tile_rows = 4 * TM * 16;
  const int64_t ntiles = (p.M + tile_rows - 1) / tile_rows;
  const T* __restrict__ Ag = reinterpret_cast<const T*>(p.A);
  const T* bfrag = sB + (lane & 15) * ldsb + (lane >> 4) * VE;
  const int64_t nch = p.kpad / KC;
  const int64_t full = p.K / KC;                    // chunks with no k >= K
  const int tnw = min(TNW, nblk / 16);              // live column tiles of this block
  constexpr int OV = Vec<T>::N;
  const int sr = lane / St::VPC, sv = lane % St::VPC;   // this lane's row and vector of a staging step
  float creg[St::NCH][OV];                              // CS: sums of its column vectors
#pragma unroll
  for (int c = 0; c < St::NCH; ++c)
#pragma unroll
    for (int j = 0; j < OV; ++j) creg[c][j] = 0.f;

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = tile * tile_rows + (int64_t)wave * (TM * 16);
    const T* arow[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      int64_t r = r0 + tm * 16 + (lane & 15);
      if (r >= p.M) r = p.M - 1;                     // clamped rows are never stored
      arow[tm] = Ag + r * p.lda + (lane >> 4) * VE;
    }
    f32x4 acc[TM][TNW];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TNW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto loadA = [&](uint4* a, int64_t c) {
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) a[tm] = ldg16(arow[tm] + c * KC);
    };
    auto compute = [&](const uint4* a, int64_t c) {
#pragma unroll
      for (int tn = 0; tn < TNW; ++tn) {
        if (tn < tnw) {
          const uint4 b = *reinterpret_cast<const uint4*>(bfrag + tn * 16 * ldsb + c * KC);
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) acc[tm][tn] = TsMfma<T>::run(a[tm], b, acc[tm][tn]);
        }
      }
    };
    // The ReLU/dropout derivative of the epilogue reads H: for 16-bit types
    // the wave's H vectors are requested together with its A fragments, so
    // the tile costs one memory latency.
    constexpr bool dmask = DM;
    constexpr bool HPRE = DM && sizeof(T) == 2;          // H prefetched into registers
    constexpr int EIT = HPRE ? St::NCH * St::IT : 1;     // vectors per lane per 16 rows
    uint4 hv[TM][EIT];
    auto prefetch_h = [&]() {
      if constexpr (HPRE) {
        const T* hm = reinterpret_cast<const T*>(p.epi.hmask);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int it = 0; it < EIT; ++it) {
            const int rr = sr + (64 / St::VPC) * (it % St::IT), cv = sv + St::VPC * (it / St::IT);
            const int64_t row = r0 + tm * 16 + rr, col = n0 + cv * OV;
            const bool ok = rr < 16 && cv * OV < nblk && row < p.M && col < p.N;
            hv[tm][it] = ldg16(hm + (ok ? row * p.epi.ldh + col : 0));
          }
      }
    };
#define TS_FENCE() __builtin_amdgcn_sched_barrier(0)
    uint4 a0[TM], a1[TM], a2[TM], a3[TM];
    if (nch <= 4) {
      // The whole K range fits the four fragment sets: every load of the
      // tile is issued before the first is used (one memory latency per
      // tile).  Vectors at or past K read the row start and are zeroed.
      const int64_t kl0 = (lane >> 4) * VE;
      auto loadw = [&](uint4* a, int64_t c) {
        const int64_t off = c * KC + kl0 < p.K ? c * KC : -kl0;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) a[tm] = ldg16(arow[tm] + off);
      };
      auto maskw = [&](uint4* a, int64_t c) {
        const int64_t nk = p.K - (c * KC + kl0);
        const int vk = nk <= 0 ? 0 : nk >= VE ? VE : (int)nk;
        if (vk < VE) {
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) a[tm] = keep_first<T>(a[tm], vk);
        }
      };
      loadw(a0, 0);
      if (nch > 1) loadw(a1, 1);
      if (nch > 2) loadw(a2, 2);
      if (nch > 3) loadw(a3, 3);
      prefetch_h();   // after the A loads: waiting for A does not wait for H
      TS_FENCE();
      maskw(a0, 0); compute(a0, 0);
      if (nch > 1) { maskw(a1, 1); compute(a1, 1); }
      if (nch > 2) { maskw(a2, 2); compute(a2, 2); }
      if (nch > 3) { maskw(a3, 3); compute(a3, 3); }
    } else {
      prefetch_h();
      int64_t c = 0;
      if (full >= 3) {
        loadA(a0, 0); loadA(a1, 1); loadA(a2, 2);
        TS_FENCE();
        for (; c + 7 <= full; c += 4) {
          loadA(a3, c + 3); TS_FENCE(); compute(a0, c); TS_FENCE();
          loadA(a0, c + 4); TS_FENCE(); compute(a1, c + 1); TS_FENCE();
          loadA(a1, c + 5); TS_FENCE(); compute(a2, c + 2); TS_FENCE();
          loadA(a2, c + 6); TS_FENCE(); compute(a3, c + 3); TS_FENCE();
        }
        compute(a0, c); compute(a1, c + 1); compute(a2, c + 2);
        c += 3;
      }
      for (; c < full; ++c) { loadA(a0, c); compute(a0, c); }
      if (c < nch) {   // the chunk that straddles K: mask k >= K (B rows there are zero too)
        const int64_t kl = c * KC + (lane >> 4) * VE;
        // a vector starting below K ends inside the row (lda >= K rounded up to 8)
        const int64_t nk = p.K - kl;
        const int vk = nk <= 0 ? 0 : nk >= VE ? VE : (int)nk;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) a0[tm] = ldg16(arow[tm] + (vk > 0 ? c * KC : -(lane >> 4) * VE));
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) a0[tm] = keep_first<T>(a0[tm], vk);
        compute(a0, c);
      }
    }
#undef TS_FENCE

    // ---- epilogue: per 16-row tile and step, MFMA layout -> LDS -> row vectors
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
      for (int c = 0; c < St::NCH; ++c) {
#pragma unroll
        for (int q = 0; q < St::NT; ++q) {
          const int tn = c * St::NT + q;
          if (tn < TNW && tn < tnw) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              unsigned char* at = myC + ((lane >> 4) * 4 + v) * St::ROW;
              const int cc = q * 16 + (lane & 15);
              const float x = acc[tm][tn < TNW ? tn : 0][v];
              if constexpr (dmask) reinterpret_cast<float*>(at)[cc] = x;
              else reinterpret_cast<T*>(at)[cc] = from_f32<T>(x);
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int it = 0; it < St::IT; ++it) {
          const int rr = sr + (64 / St::VPC) * it, cv = sv + St::VPC * c;
          const int64_t row = r0 + tm * 16 + rr, col = n0 + cv * OV;
          if (rr >= 16 || cv * OV >= nblk || row >= p.M || col >= p.N) continue;
          const unsigned char* at = myC + rr * St::ROW;
          const int64_t nl = p.N - col;
          const int live = nl >= OV ? OV : (int)nl;        // columns >= N are stored as 0
          uint4 o;
          if constexpr (dmask) {
            float v[OV], h[OV];
#pragma unroll
            for (int j = 0; j < OV; ++j) v[j] = reinterpret_cast<const float*>(at)[sv * OV + j];
            if constexpr (HPRE) unpack<T>(hv[tm][c * St::IT + it], h);
            else unpack<T>(ldg16(reinterpret_cast<const T*>(p.epi.hmask) + row * p.epi.ldh + col), h);
#pragma unroll
            for (int j = 0; j < OV; ++j) v[j] = h[j] > 0.f ? v[j] * p.epi.keep_scale : 0.f;
            o = pack<T>(v);
          } else {
            o = *reinterpret_cast<const uint4*>(at + sv * 16);
          }
          o = keep_first<T>(o, live);
          stg16(reinterpret_cast<T*>(p.epi.out) + row * p.epi.ldo + col, o);
          float st[OV];
          unpack<T>(o, st);
          bool bad = false;
#pragma unroll
          for (int j = 0; j < OV; ++j) bad |= !finite_f32(st[j]);
          if (bad) raise_flag(p.epi.flag);
          if constexpr (CS) {
#pragma unroll
            for (int j = 0; j < OV; ++j) creg[c][j] += st[j];
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  }
  if constexpr (CS) {
    // lanes sv, sv + VPC, sv + 2 VPC, ... hold the same columns: butterfly
#pragma unroll
    for (int off = 32; off >= St::VPC; off >>= 1)
#pragma unroll
      for (int c = 0; c < St::NCH; ++c)
#pragma unroll
        for (int j = 0; j < OV; ++j) creg[c][j] += __shfl_xor(creg[c][j], off);
    __syncthreads();
    float* sum = reinterpret_cast<float*>(sC);              // [4][nblk]
    if (lane < St::VPC) {
#pragma unroll
      for (int c = 0; c < St::NCH; ++c)
        if ((sv + St::VPC * c) * OV < nblk)
#pragma unroll
          for (int j = 0; j < OV; ++j) sum[wave * nblk + (sv + St::VPC * c) * OV + j] = creg[c][j];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < nblk; c += 256) {
      if (n0 + c < p.N) {
        float a = sum[c];
        a += sum[nblk + c];
        a += sum[2 * nblk + c];
        a += sum[3 * nblk + c];
        p.colsum[(int64_t)blockIdx.x * p.N + n0 + c] = a;
      }
    }
  }
}

// Dynamic LDS of one workgroup: the B block, then the four staging buffers
// (at most 128 bytes of output, or 256 of fp32 sums, and 16 more per row).
template <typename T>
size_t ts_lds_bytes(int64_t nblk, int64_t kpad, bool dm) {
  const int64_t w = std::min<int64_t>(8, (nblk <= 16 ? 16 : nblk <= 32 ? 32 : 64) / Vec<T>::N) * Vec<T>::N;
  const size_t row = dm ? (w + 4) * 4 : w * sizeof(T) + 16;
  return ((size_t)nblk * (kpad + Vec<T>::N) * sizeof(T) + 15) / 16 * 16 + 4 * 16 * row;
}

// Half of a gfx950 compute unit's 160 KB of LDS.
constexpr size_t TS_LDS_TWO_WG = 80 * 1024;

// Workgroups per column block: enough to fill every CU twice, and a multiple of
// the dies, so that the column blocks of a row tile run on the same die and
// share A's lines in its L2.
int64_t ts_wgs_per_col(int64_t nb) { return std::max<int64_t>(XCDS, 512 / nb / XCDS * XCDS); }

// Columns of a block: equal blocks (every block gets as many workgroups), and
// narrow enough (us, with one workgroup per compute unit -> now: fp16 n =
// 131072, 256 -> 256 72.8 -> 40.0, 500 -> 64 43.6 -> 33.1; n = 1 M, 256 -> 256
// 481 -> 262, 128 -> 128 118 -> 99; n = 2048, 400 -> 150 11.2 -> 7.6; fp32 n = 1
// M, 256 -> 256 1379 -> 1149)
//  * for the B block's cap and for two workgroups per compute unit: with one
//    wave per SIMD the matrix instructions wait on each B read from LDS, and
//    the loads of A on the epilogue, with no other wave to issue;
//  * where the rows are few, for a workgroup per compute unit (not below 32
//    columns: each block reads all of A).
template <typename T>
int ts_nblk(int64_t M, int64_t N, int64_t kpad, bool dm) {
  auto block = [&](int64_t parts) { return ((N + parts - 1) / parts + 15) / 16 * 16; };
  const int64_t cap = std::max<int64_t>(TS_LDS_B_BYTES / ((kpad + Vec<T>::N) * (int64_t)sizeof(T)) / 16 * 16, 16);
  int64_t parts = (N + 127) / 128;
  while (block(parts) > 16 && (block(parts) > cap || ts_lds_bytes<T>(block(parts), kpad, dm) > TS_LDS_TWO_WG)) ++parts;
  while (block(parts + 1) >= 32 && (M + 63) / 64 * parts < 256) ++parts;
  return (int)block(parts);
}

template <typename T, bool BKC, bool DM, bool CS, int TM>
hipError_t launch_tm(const TsParams& p, int* grid_rows, hipStream_t s) {
  const int tnw = p.nblk / 16;
  const size_t lds = ts_lds_bytes<T>(p.nblk, p.kpad, DM);
  // persistent workgroups: enough to fill every CU twice, each looping over row tiles
  const int64_t nb = (p.N + p.nblk - 1) / p.nblk;
  const int64_t ntiles = (p.M + 64 * TM - 1) / (64 * TM);
  const int64_t per_col = ts_wgs_per_col(nb);
  dim3 grid((unsigned)std::min<int64_t>(ntiles, per_col), (unsigned)nb);
  if (grid_rows) *grid_rows = (int)grid.x;
#define TS_L(TNW_)                                                                                          \
  do {                                                                                                      \
    if (lds > 65536) {                                                                                      \
      hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&tsgemm_kernel<T, BKC, DM, CS, TM, TNW_>),\
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);           \
      if (ea != hipSuccess) return ea;                                                                      \
    }                                                                                                       \
    hipLaunchKernelGGL((tsgemm_kernel<T, BKC, DM, CS, TM, TNW_>), grid, dim3(256), lds, s, p);                \
  } while (0)
  if (tnw <= 1) TS_L(1);
  else if (tnw <= 2) TS_L(2);
  else if (tnw <= 4) TS_L(4);
  else TS_L(8);
#undef TS_L
  return hipGetLastError();
}

template <typename T, bool BKC, bool DM, bool CS>
hipError_t launch_b(TsParams p, int* grid_rows, hipStream_t s) {
  constexpr int KC = 4 * Vec<T>::N;
  p.kpad = (p.K + KC - 1) / KC * KC;
  p.nblk = ts_nblk<T>(p.M, p.N, p.kpad, DM);
  // rows per wave: 32 (each B fragment read from LDS then serves two MFMAs)
  // unless 16 leave the fullest workgroup less to do, as where the rows are
  // few or the last round of tiles is nearly empty
  // (TM = 4 would need more than 256 registers per lane with the whole-K
  // fragment sets, i.e. one wave per SIMD; TM = 2 keeps two)
  // (the H-mask epilogue with 128-column blocks holds another 32 registers:
  // one row tile per wave keeps two waves per SIMD there)
  const int64_t wgs = ts_wgs_per_col((p.N + p.nblk - 1) / p.nblk);
  auto most = [&](int64_t tm) { return ((p.M + 64 * tm - 1) / (64 * tm) + wgs - 1) / wgs * tm; };
  const bool two = 10 * most(2) <= 12 * most(1) && !(DM && p.nblk > 64);
  return two ? launch_tm<T, BKC, DM, CS, 2>(p, grid_rows, s) : launch_tm<T, BKC, DM, CS, 1>(p, grid_rows, s);
}

// Column sums (CS) are only asked of dZ_below = (G_S W^T) * mask, whose B
// is k-contiguous.
template <typename T>
hipError_t launch_t(const TsParams& p, bool bkc, int* grid_rows, hipStream_t s) {
  const bool dm = p.epi.mode == EPI_DMASK && p.epi.relu;
  if (p.colsum) {
    if (!bkc) return hipErrorInvalidValue;
    return dm ? launch_b<T, true, true, true>(p, grid_rows, s) : launch_b<T, true, false, true>(p, grid_rows, s);
  }
  if (!bkc && !dm) return launch_b<T, false, false, false>(p, grid_rows, s);
  if (!dm) return launch_b<T, true, false, false>(p, grid_rows, s);
  return bkc ? launch_b<T, true, true, false>(p, grid_rows, s) : launch_b<T, false, true, false>(p, grid_rows, s);
}

}  // namespace

bool tsgemm_supported(int prec, int64_t K) {
  const int64_t kc = prec == 0 ? 16 : 32;
  const int64_t kpad = (K + kc - 1) / kc * kc;
  const int64_t s = prec == 0 ? 4 : 2;
  return (kpad + 16 / s) * s * 16 <= TS_LDS_B_BYTES;   // at least one 16-column block fits
}

int tsgemm_colsum_rows_max() { return 512; }

hipError_t tsgemm_launch(int prec, const void* A, int64_t lda, const void* B, int64_t ldb, bool b_kc, int64_t M,
                         int64_t N, int64_t K, const Epilogue& epi, hipStream_t s, float* colsum, int* colsum_rows) {
  TsParams p;
  p.A = A; p.lda = lda; p.B = B; p.ldb = ldb; p.M = M; p.N = N; p.K = K; p.kpad = 0; p.nblk = 0; p.epi = epi;
  p.colsum = colsum;
  switch (prec) {
    case 0: return launch_t<float>(p, b_kc, colsum_rows, s);
    case 1: return launch_t<f16>(p, b_kc, colsum_rows, s);
    case 2: return launch_t<bf16>(p, b_kc, colsum_rows, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gcn
