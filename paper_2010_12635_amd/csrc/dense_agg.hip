// Dense-A_hat aggregation Y = epilogue(A_hat X) for A_hat stored as a dense
// n x n matrix (the paper's own storage: every tensor cast to dense,
// Section "Reduced Precision Changes").  With the feature width F <= 64 the
// product is bound by streaming A_hat from HBM (s * n^2 bytes against
// 2 * n^2 * F flops), so the kernel is built around that stream:
//
//  * Operand order.  MFMA 16x16 operands take, in lane l, 16 bytes of row
//    l % 16 at k-group l / 16.  In the tiled layout every 16-row x KC-column
//    piece (KC = 4 x 16 bytes of k) is one contiguous 1 KiB block in exactly
//    that lane order, and the four 16-row pieces of a 64-row block follow
//    each other, so each operand load is one contiguous 1 KiB and a wave's
//    k range is one contiguous stream (row-major rows give 16 short runs per
//    load, which measured far below the stream rate on MI355X).  Tiled
//    A_hat is read once per call, with non-temporal loads (measured 7-13 %
//    faster at n = 16384, F = 64 and 32; Xt, which every workgroup re-reads,
//    keeps ordinary loads).  Row-major A_hat does not: each of its 128-byte
//    lines serves two consecutive chunks, and with non-temporal loads the
//    line is gone before the second (O1 training 23 % slower).
//    X is transposed into the same tiled layout (Xt) before the product.
//  * A workgroup owns 64 rows and a 64-column block; its 8 waves split the
//    k range in 8 contiguous parts, each keeping its partial 64 x 64 tile in
//    MFMA accumulators, with a 3-deep register ring of loads in flight.
//  * The 8 partial tiles are summed through LDS in a fixed order (wave w
//    adds wave w + 4, then the four sums are added in wave order), then the
//    fused epilogue (bias, ReLU, dropout, cast, overflow flag) stores
//    16-byte vectors row by row.  No global partial sums, one launch.
#include "internal.h"
#include "xpose.h"

#include <algorithm>

namespace gcn {

namespace {

constexpr int DA_BM = 64;     // rows per workgroup
constexpr int DA_BN = 64;     // columns per workgroup (column block of Xt)
constexpr int DA_WAVES = 8;   // waves per workgroup, one k range each

// Tiled offset (elements) of entry (i, j) of an R x K matrix in operand
// order: 64-row blocks, KC-column chunks, 16-row pieces of 1 KiB.
template <typename T>
__host__ __device__ __forceinline__ int64_t tiled_off(int64_t i, int64_t j, int64_t nc) {
  constexpr int VE = Vec<T>::N, KC = 4 * VE;
  return (((i / 64) * nc + j / KC) * 4 + (i % 64) / 16) * (16 * KC) + ((j % KC) / VE * 16 + i % 16) * VE + j % VE;
}
template <typename T> constexpr int tile_kc() { return 4 * Vec<T>::N; }

// Xt = tiled(X^T): X is n x F (ldx); Xt has Fp = ceil(F / 64) * 64 rows
// and kpad = nc * KC columns; entries outside F x n are zero.  Each thread
// turns one VE x VE block (VE vertices x VE features) around in registers:
// VE 16-byte row loads, a register transpose, VE 16-byte stores, each of
// VE consecutive vertices of one feature, i.e. one contiguous piece of the
// tiled layout.  A wave covers 64 features x XB_K vertices, a workgroup four
// waves along the vertices.  With colsum != NULL the kernel also sums each
// feature over the workgroup's vertices (fixed order: block rows, a xor
// butterfly over the wave's vertex blocks, then the four waves in order)
// and writes row blockIdx.x of colsum ([gridDim.x][F] floats).
template <typename T>
struct XpGeom {
  static constexpr int VE = Vec<T>::N;
  static constexpr int FB = 64 / VE;          // feature blocks per wave
  static constexpr int KB = 64 / FB;          // vertex blocks per wave
  static constexpr int WAVE_K = KB * VE;      // vertices per wave
  static constexpr int WG_K = 4 * WAVE_K;     // vertices per workgroup
};

template <typename T>
__global__ __launch_bounds__(256) void transpose_tiled_kernel(const T* __restrict__ X, int64_t ldx, int64_t n, int64_t F,
                                                              T* __restrict__ Xt, int64_t nc, float* __restrict__ colsum) {
  using G = XpGeom<T>;
  constexpr int VE = G::VE, KC = 4 * VE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fb = lane % G::FB, kb = lane / G::FB;
  const int64_t f0 = (int64_t)blockIdx.y * 64 + fb * VE;
  const int64_t k0 = (int64_t)blockIdx.x * G::WG_K + wave * G::WAVE_K + kb * VE;
  const int64_t kpad = nc * KC;
  // all VE loads go out before any is used: rows >= n and feature blocks
  // >= F read row 0 / column 0 (in bounds) and are zeroed afterwards
  const int64_t nf = F - f0;
  const int vc = nf <= 0 ? 0 : nf >= VE ? VE : (int)nf;
  const T* colp = X + (vc > 0 ? f0 : 0);         // f0 + VE <= round_up(F, 8) <= ldx
  uint4 in[VE];
#pragma unroll
  for (int i = 0; i < VE; ++i) in[i] = ldg16(colp + (k0 + i < n ? k0 + i : 0) * ldx);
#pragma unroll
  for (int i = 0; i < VE; ++i) in[i] = keep_first<T>(in[i], k0 + i < n ? vc : 0);
  uint4 out[VE];
  transpose_block(in, out, T());
  if (k0 < kpad) {
#pragma unroll
    for (int j = 0; j < VE; ++j) stg16(Xt + tiled_off<T>(f0 + j, k0, nc), out[j]);
  }
  if (!colsum) return;
  __shared__ float red[4][64];
  float cs[VE];
#pragma unroll
  for (int j = 0; j < VE; ++j) {
    float v[VE];
    unpack<T>(out[j], v);
    float a = v[0];
#pragma unroll
    for (int i = 1; i < VE; ++i) a += v[i];
    cs[j] = a;
  }
#pragma unroll
  for (int off = G::FB; off < 64; off <<= 1)
#pragma unroll
    for (int j = 0; j < VE; ++j) cs[j] += __shfl_xor(cs[j], off);
  if (kb == 0) {
#pragma unroll
    for (int j = 0; j < VE; ++j) red[wave][fb * VE + j] = cs[j];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int64_t f = (int64_t)blockIdx.y * 64 + threadIdx.x;
    float a = red[0][threadIdx.x] + red[1][threadIdx.x];
    a += red[2][threadIdx.x];
    a += red[3][threadIdx.x];
    if (f < F) colsum[(int64_t)blockIdx.x * F + f] = a;
  }
}

template <typename T> struct DaMfma;
template <> struct DaMfma<f16> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct DaMfma<bf16> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct DaMfma<float> {
  static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

struct DaParams {
  const void* A; int64_t lda;     // dense A_hat, n x lda
  const void* Xt; int64_t ldt;    // Fp x ldt
  int64_t n;
  int64_t F;                      // logical output width
  Epilogue epi;
};

// One k chunk (4 lane groups x VE) of operand fragments.
template <int TN>
struct Frag {
  uint4 a[4];
  uint4 b[TN];
};

// In chunk c lane group g (= lane / 16) holds k = c * KC + g * VE + [0, VE)
// of A_hat and of Xt alike, so the MFMA sums over exactly the same k.
template <typename T, int TN, bool TILED>
__global__ __launch_bounds__(64 * DA_WAVES) void dense_agg_kernel(DaParams p) {
  constexpr int VE = Vec<T>::N;
  constexpr int KC = 4 * VE;                 // k per chunk: 32 (16-bit) / 16 (fp32)
  constexpr int PIECE = 16 * KC;             // elements of one 16-row piece (1 KiB)
  constexpr int LDR = DA_BN + 4;             // LDS row stride (floats)
  __shared__ float red[4][DA_BM * LDR];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * DA_BM;
  const int64_t c0 = (int64_t)blockIdx.y * DA_BN;
  const int64_t nc = (p.n + KC - 1) / KC;
  const T* __restrict__ A = reinterpret_cast<const T*>(p.A);
  const T* __restrict__ Xt = reinterpret_cast<const T*>(p.Xt);

  // Operand base pointers; fragment (chunk c, tile t) is at base + c * step + t * tstep.
  const T* abase[4];
  int64_t astep;
  if (TILED) {
    const T* blk = A + (int64_t)blockIdx.x * nc * 4 * PIECE + lane * VE;
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) abase[tm] = blk + tm * PIECE;
    astep = 4 * PIECE;
  } else {
    // rows beyond n read row n-1 (their results are never stored)
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
      int64_t r = m0 + tm * 16 + (lane & 15);
      if (r >= p.n) r = p.n - 1;
      abase[tm] = A + r * p.lda + (lane >> 4) * VE;
    }
    astep = KC;
  }
  const T* bbase = Xt + (int64_t)blockIdx.y * nc * 4 * PIECE + lane * VE;

  const int64_t cb = nc * wave / DA_WAVES, ce = nc * (wave + 1) / DA_WAVES;
  const int64_t full_end = TILED ? ce : min(ce, p.n / KC);   // chunks needing no mask

  f32x4 acc[4][TN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto load = [&](Frag<TN>& f, int64_t c) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
      f.a[tm] = TILED ? ldg16_nt(abase[tm] + c * astep) : ldg16(abase[tm] + c * astep);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) f.b[tn] = ldg16(bbase + c * 4 * PIECE + tn * PIECE);
  };
  auto compute = [&](const Frag<TN>& f) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = DaMfma<T>::run(f.a[tm], f.b[tn], acc[tm][tn]);
  };
  // keep the scheduler from moving MFMAs ahead of the loads issued before them
#define DA_FENCE() __builtin_amdgcn_sched_barrier(0)

  // full chunks: 4-deep ring of fragments (3 chunks in flight while computing)
  Frag<TN> f0, f1, f2, f3;
  int64_t c = cb;
  if (c + 3 <= full_end) {
    load(f0, c);
    load(f1, c + 1);
    load(f2, c + 2);
    DA_FENCE();
    // A step issues the 4 + TN loads of one chunk spread among the MFMAs of
    // another, one load before every NM / NL MFMAs, so that the matrix pipe
    // and the loads overlap (fp32, where the MFMAs dominate: 375 -> 274 us at
    // n = 16384, F = 64, 201 -> 170 us at F = 32; 16-bit unchanged, bound by
    // the stream).  With fewer MFMAs than loads the loads go first.
    constexpr int NL = 4 + TN, NM = 4 * TN * (sizeof(T) == 4 ? 4 : 1), PER = NM / NL;
#define DA_STEP(FL, CL, FC)                                                            \
    if (PER >= 1) {                                                                    \
      load(FL, CL); compute(FC);                                                       \
      _Pragma("unroll") for (int q_ = 0; q_ < NL; ++q_) {                              \
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   /* vector-memory read */  \
        __builtin_amdgcn_sched_group_barrier(0x008, PER >= 1 ? PER : 1, 0); /* MFMA */ \
      }                                                                                \
    } else {                                                                           \
      load(FL, CL); DA_FENCE(); compute(FC);                                           \
    }                                                                                  \
    DA_FENCE();
    for (; c + 7 <= full_end; c += 4) {
      DA_STEP(f3, c + 3, f0)
      DA_STEP(f0, c + 4, f1)
      DA_STEP(f1, c + 5, f2)
      DA_STEP(f2, c + 6, f3)
    }
#undef DA_STEP
    // drain: f0, f1, f2 hold chunks c, c+1, c+2
    compute(f0);
    compute(f1);
    compute(f2);
    c += 3;
  }
  for (; c < full_end; ++c) {
    load(f0, c);
    compute(f0);
  }
#undef DA_FENCE
  // row-major A_hat only: the chunk that straddles n (last wave): mask k >= n
  if (!TILED && c < ce) {
    const int64_t kl = c * KC + (lane >> 4) * VE;   // first k of this lane's vector
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) f0.b[tn] = ldg16(bbase + c * 4 * PIECE + tn * PIECE);   // Xt is zero-padded
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
      // a vector starting below n ends inside the row (lda >= n rounded up
      // to 8); one starting at or beyond n is not loaded at all
      f0.a[tm] = kl < p.n ? ldg16(abase[tm] + c * astep) : make_uint4(0, 0, 0, 0);
      T* e = reinterpret_cast<T*>(&f0.a[tm]);
#pragma unroll
      for (int j = 0; j < VE; ++j)
        if (kl + j >= p.n) e[j] = T(0);
    }
    compute(f0);
  }

  // partial tiles -> LDS (MFMA layout: lane holds rows 4*(lane/16)+v of
  // column lane%16).  Stage 1: waves 4..7 park their tiles, waves 0..3 add
  // them; stage 2: waves 0..3 park the sums.
  auto lds_at = [&](int w, int tm, int tn, int v) -> float& {
    return red[w][(tm * 16 + (lane >> 4) * 4 + v) * LDR + tn * 16 + (lane & 15)];
  };
  if (wave >= 4) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 4; ++v) lds_at(wave - 4, tm, tn, v) = acc[tm][tn][v];
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[tm][tn][v] += lds_at(wave, tm, tn, v);
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 4; ++v) lds_at(wave, tm, tn, v) = acc[tm][tn][v];
  }
  __syncthreads();

  // fixed-order sum of the 4 partials, fused epilogue, 16-byte stores
  constexpr int OV = Vec<T>::N;              // output elements per vector
  constexpr int VPR = DA_BN / OV;            // vectors per row of the block
  for (int idx = threadIdx.x; idx < DA_BM * VPR; idx += 64 * DA_WAVES) {
    const int r = idx / VPR, cv = idx % VPR;
    const int64_t row = m0 + r, col = c0 + cv * OV;
    if (row >= p.n || col >= p.F || cv * OV >= TN * 16) continue;
    float v[OV];
#pragma unroll
    for (int j = 0; j < OV; ++j) {
      const int cc = cv * OV + j;
      v[j] = red[0][r * LDR + cc] + red[1][r * LDR + cc];
      v[j] += red[2][r * LDR + cc];
      v[j] += red[3][r * LDR + cc];
    }
    epi_store_vec<T>(p.epi, row, col, v);
  }
}

// ---------------------------------------------------------------------------
// Tiled A_hat, F <= 64.  What bounds the product is, in
// 16-bit storage, the stream of A_hat from HBM and, beside it, the X^T
// fragments that every workgroup re-reads from L2 (F / rows of its bytes); in
// fp32 the matrix units.  So:
//  * a workgroup owns 128 rows and all columns (16 TN <= 64);
//    its 4 waves (one per SIMD, up to 512 registers) split the k range, each
//    with the whole 128 x 16 TN accumulator tile, ST_DEPTH - 1 chunks of
//    loads in flight, the loads spread among the MFMAs;
//  * where the row blocks alone would leave compute units idle, or a last
//    round of workgroups nearly empty, the k range is also cut over `ksplit`
//    workgroups per row block (rule at dense_plan), whose fp32 partial tiles
//    mm_reduce_kernel adds in order;
//  * the four waves' tiles are added through LDS in a fixed order.
// ---------------------------------------------------------------------------
struct StreamParams {
  const void* A;      // tiled A_hat
  const void* Xt;     // tiled X^T
  int64_t n, F, nc;   // vertices, features, k chunks
  int64_t rblocks;    // 64-row blocks of A_hat
  int64_t rb0, rowb;  // 128-row blocks of this launch: the first, how many
  int64_t ksplit;
  float* part;        // ksplit > 1: fp32 partial products [ksplit][prows][ldp] of the launch's rows
  int64_t prows, ldp;
  Epilogue epi;
};

template <typename T, int TN, int DEPTH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void dense_stream_kernel(StreamParams p) {
  constexpr int VE = Vec<T>::N, KC = 4 * VE, PIECE = 16 * KC;
  constexpr int TM = 8;                            // 16-row tiles per wave
  constexpr int NC = 16 * TN;                      // columns
  constexpr int LDR = NC + 4;                      // LDS row stride (floats)
  __shared__ float red[2][16 * TM * LDR];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t rbk = p.rb0 + blockIdx.x % p.rowb, split = blockIdx.x / p.rowb;   // k ranges outermost
  const int64_t blk = p.nc * 4 * PIECE;            // elements of one 64-row block
  const T* __restrict__ A = reinterpret_cast<const T*>(p.A);
  const T* __restrict__ Xt = reinterpret_cast<const T*>(p.Xt);
  // blocks past the padded extent read the last one (never stored)
  const T* abase[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) abase[i] = A + min(rbk * 2 + i, p.rblocks - 1) * blk + lane * VE;
  const T* bbase = Xt + lane * VE;
  const int64_t s0 = p.nc * split / p.ksplit, s1 = p.nc * (split + 1) / p.ksplit;
  const int64_t cb = s0 + (s1 - s0) * wave / 4, ce = s0 + (s1 - s0) * (wave + 1) / 4;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct Fr { uint4 a[TM]; uint4 b[TN]; };
  const int64_t clast = ce > cb ? ce - 1 : (cb < p.nc ? cb : p.nc - 1);
  auto load = [&](Fr& f, int64_t c) {
    const int64_t off = (c < clast ? c : clast) * (4 * PIECE);   // past the end: in bounds, unused
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = ldg16_nt(abase[i / 4] + off + (i % 4) * PIECE);
#pragma unroll
    for (int t = 0; t < TN; ++t) f.b[t] = ldg16(bbase + off + t * PIECE);
  };
  auto compute = [&](const Fr& f) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = DaMfma<T>::run(f.a[i], f.b[j], acc[i][j]);
  };
  // a step's loads are spread among its MFMAs
  constexpr int NL = TM + TN, NM = TM * TN * (sizeof(T) == 4 ? 4 : 1), PER = NM / NL;
#define ST_STEP(FL, CL, FC)                                                          \
  load(FL, CL); compute(FC);                                                         \
  _Pragma("unroll") for (int q_ = 0; q_ < NL; ++q_) {                                \
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   /* vector-memory read */    \
    __builtin_amdgcn_sched_group_barrier(0x008, PER > 0 ? PER : 1, 0);   /* MFMA */  \
  }                                                                                  \
  __builtin_amdgcn_sched_barrier(0);
  Fr f[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) load(f[d], cb + d);
  __builtin_amdgcn_sched_barrier(0);
  int64_t c = cb;
  for (; c + DEPTH <= ce; c += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) { ST_STEP(f[(d + DEPTH - 1) % DEPTH], c + d + DEPTH - 1, f[d]) }
  }
#undef ST_STEP
  // the last chunks (fewer than DEPTH) are in flight already
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d)
    if (c + d < ce) compute(f[d]);

  auto lds_at = [&](int w, int i, int j, int v) -> float& {
    return red[w][(i * 16 + (lane >> 4) * 4 + v) * LDR + j * 16 + (lane & 15)];
  };
  if (wave >= 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) lds_at(wave - 2, i, j, v) = acc[i][j][v];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float& r = lds_at(wave, i, j, v);        // this lane's own slot of the other wave's tile
          r = acc[i][j][v] + r;
        }
  }
  __syncthreads();

  constexpr int OV = Vec<T>::N, VPR = NC / OV;     // output vectors per row of the block
  float bv[OV];
  const int64_t m0 = rbk * 128;
  for (int idx = threadIdx.x; idx < 128 * VPR; idx += 256) {
    const int r = idx / VPR, cv = idx % VPR;
    const int64_t row = m0 + r, col = cv * OV;
    if (row >= p.n || col >= p.F) continue;
    float v[OV];
#pragma unroll
    for (int e = 0; e < OV; ++e) v[e] = red[0][r * LDR + cv * OV + e] + red[1][r * LDR + cv * OV + e];
    if (p.ksplit > 1) {
      float4* o = reinterpret_cast<float4*>(p.part + (split * p.prows + row - p.rb0 * 128) * p.ldp + col);
#pragma unroll
      for (int e = 0; e < OV / 4; ++e) o[e] = make_float4(v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]);
    } else {
      epi_load_bias<T>(p.epi, col, bv);
      epi_store_vec_b<T>(p.epi, row, col, v, bv);
    }
  }
}

// ---------------------------------------------------------------------------
// Wide features (the large model sizes of the paper's Table 1): 2 n^2 F flops
// against s n^2 bytes of A_hat put the product above the ridge point from
// F of about 300 on, so this kernel is built around the matrix cores.
//  * A workgroup of 4 waves (2 x 2, one per SIMD) owns up to a 256 x 256
//    output tile, each wave a quarter of it (at most 8 x 8 MFMA 16x16 tiles,
//    256 fp32 accumulators per lane).
//  * Both operands are in MFMA operand order (tiled A_hat, tiled X^T), every
//    fragment one contiguous 1 KiB.  Read straight into registers, each went
//    through the vector cache twice per workgroup (two waves share it), and
//    that path, 64 KB per chunk at 80-100 GB/s per compute unit, bound the
//    kernel; so a chunk is now copied once, by global-to-LDS loads (up to 120
//    GB/s per compute unit from L2, no registers held), into a ring of up to
//    eight chunks in LDS, from which a wave reads its fragments one chunk
//    ahead of the MFMAs (lane order: no bank conflicts).  One barrier per
//    chunk.  n = 32768, F = 2048 fp16: 3.06 -> 2.49 ms (1.44 -> 1.77 PFLOP/s),
//    same bits.  What bounds it now: LDS (96 KB per chunk read and written,
//    0.31 us) beside 0.43 us of matrix instructions, issued by one wave.
//  * Tiles are dealt out XCD by XCD: workgroup b runs on XCD b % 8, and each
//    XCD takes a contiguous range of tiles in row-major order, so the column
//    tiles of a row block run together and share A_hat in that XCD's L2
//    (measured at n = 32768: 1-2 % over plain order, 4 % over column-major).
//  * The epilogue stages each 16-row strip of the wave's quarter through
//    LDS and stores rows as 16-byte vectors through the fused epilogue
//    (with the bias of a lane's columns loaded once per tile).
// ---------------------------------------------------------------------------
constexpr int MM_LDR = 128 + 4;   // LDS stride (floats) of a staged strip
// Each wave stages through its own LDS area, so a strip needs no workgroup
// barrier: the wave's own LDS operations complete in order, and waiting for
// them (with a compiler memory fence) orders the writes of one lane before
// the reads of another (measured 2-5 % faster at F = 512 and 1024).
#define MM_SYNC() asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory")

// Up to 256 bytes, four lines of the scalar cache: with a fifth, which the
// epilogue alone reads, n = 8192, F = 512 in bf16 took 92.0 us instead of 90.6.
struct MmParams {
  const void* A;      // tiled A_hat
  const void* Xt;     // tiled X^T
  int64_t n, F, nc;   // vertices, features, k chunks
  int rblocks;        // 64-row blocks of A_hat
  int fblocks;        // 64-row blocks of X^T
  int tr0;            // first row of tiles of this launch
  int tiles, cb, per_xcd;
  int ksplit, kc;     // k ranges of kc chunks (the last one shorter), one per workgroup of a tile
  int chain;          // CHAINS: chunks (even) added to an accumulator before it is added to the sums
  float* part;        // ksplit > 1: fp32 partial products [ksplit][prows][ldp] of the launch's rows
  int64_t row0, prows;
  int64_t ldp;        // F rounded up to a whole output vector
  Epilogue epi;
};
static_assert(sizeof(MmParams) <= 256, "kernel arguments");

// Rows row0 .. row0 + 15, columns col0 .. col0 + W - 1 of the output from a
// staged strip (16 x W fp32, stride MM_LDR), through the fused epilogue.
// Where 64 is a multiple of W / Vec<T>::N a lane stores the same vector of
// columns in every row it takes, whose bias bv the caller loads once per tile.
template <typename T, int W>
__device__ __forceinline__ void mm_store_strip(const MmParams& p, const float* st, int lane, int64_t row0, int64_t col0,
                                               const float (&bv)[Vec<T>::N]) {
  constexpr int OV = Vec<T>::N;
  constexpr int VPR = W / OV;                      // vectors per strip row
#pragma unroll 1
  for (int k = 0; k < 16 * VPR / 64; ++k) {
    const int idx = k * 64 + lane;
    const int r = idx / VPR, cv = idx % VPR;
    const int64_t row = row0 + r, col = col0 + cv * OV;
    if (row >= p.n || col >= p.F) continue;
    float v[OV];
#pragma unroll
    for (int e = 0; e < OV; ++e) v[e] = st[r * MM_LDR + cv * OV + e];
    // (three quarters of a power of two: the vector differs from row to row)
    if constexpr (64 % VPR == 0) epi_store_vec_b<T>(p.epi, row, col, v, bv);
    else epi_store_vec<T>(p.epi, row, col, v);
  }
}

// The same strip as fp32 partial products of k range `split`, for the
// fixed-order reduction that applies the epilogue.
template <int W, int OV>
__device__ __forceinline__ void mm_store_strip_part(const MmParams& p, const float* st, int lane, int64_t row0,
                                                    int64_t col0, int64_t split) {
  constexpr int VPR = W / OV;
  float* part = p.part + (split * p.prows - p.row0) * p.ldp;
#pragma unroll 1
  for (int k = 0; k < 16 * VPR / 64; ++k) {
    const int idx = k * 64 + lane;
    const int r = idx / VPR, cv = idx % VPR;
    const int64_t row = row0 + r, col = col0 + cv * OV;
    if (row >= p.n || col >= p.F) continue;
    float4* o = reinterpret_cast<float4*>(part + row * p.ldp + col);
#pragma unroll
    for (int e = 0; e < OV / 4; ++e)
      o[e] = make_float4(st[r * MM_LDR + cv * OV + 4 * e], st[r * MM_LDR + cv * OV + 4 * e + 1],
                         st[r * MM_LDR + cv * OV + 4 * e + 2], st[r * MM_LDR + cv * OV + 4 * e + 3]);
  }
}

// Sum of the k ranges' partials in range order, one output vector per
// thread, through the vector epilogue (one Philox block per 8 outputs); the
// partials are those of rows row0 .. row0 + n - 1.
template <typename T>
__global__ __launch_bounds__(256) void mm_reduce_kernel(const float* __restrict__ part, int64_t ksplit, int64_t row0,
                                                        int64_t n, int64_t ldp, Epilogue epi) {
  constexpr int VE = Vec<T>::N;
  const int64_t vpr = ldp / VE;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n * vpr) return;
  const int64_t row = idx / vpr, col0 = (idx - row * vpr) * VE;
  float acc[VE];
#pragma unroll
  for (int i = 0; i < VE; ++i) acc[i] = 0.f;
  for (int64_t k = 0; k < ksplit; ++k) {
    const float4* q = reinterpret_cast<const float4*>(part + (k * n + row) * ldp + col0);
#pragma unroll
    for (int e = 0; e < VE / 4; ++e) {
      const float4 v = q[e];
      acc[4 * e] += v.x; acc[4 * e + 1] += v.y; acc[4 * e + 2] += v.z; acc[4 * e + 3] += v.w;
    }
  }
  epi_store_vec<T>(epi, row0 + row, col0, acc);
}

// 1 KiB from global memory straight into LDS (64 lanes x 16 bytes, lane order
// kept): lane l's 16 bytes at base + voff go to lds + 16 l.  Counted by vmcnt;
// written as asm because the compiler otherwise waits for every such load
// before any LDS read.  No register is written.
__device__ __forceinline__ void dma_1k(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}

// A wave owns TM x TN 16 x 16 tiles, the workgroup's 2 x 2 waves (32 TM) x
// (32 TN) of the output; S stages of one k chunk each in the LDS ring.  CHAINS:
// after every p.chain chunks the accumulators are added to a second set of sums,
// so that no addition meets more roundings than that (rule at dense_plan; at
// most 128 accumulators per lane leave registers for it).
template <typename T, int TM, int TN, int S, bool CHAINS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void dense_mm_kernel(MmParams p) {
  constexpr int VE = Vec<T>::N, KC = 4 * VE, PIECE = 16 * KC;
  constexpr int RB = TM / 2, CB = TN / 2;          // 64-row blocks of A_hat and of X^T per workgroup
  constexpr int NP = 4 * (RB + CB);                // 1 KiB pieces of a chunk
  constexpr int LPW = NP / 4;                      // and per wave
  static_assert(TM % 2 == 0 && TN % 2 == 0 && LPW <= TM && TN <= TM, "pieces and fragments spread over the TM tile rows");
  constexpr int RING = S * NP * 1024, EPI = 4 * 16 * MM_LDR * 4;
  __shared__ __align__(1024) unsigned char ring[RING > EPI ? RING : EPI];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = blockIdx.x;
  // units are (k range, tile), k range outermost, so that the workgroups of
  // one die (consecutive units) share rows of A_hat as before
  const int64_t tiles = p.tiles, cb = p.cb, rblocks = p.rblocks, fblocks = p.fblocks;
  const int64_t u = (b & 7) * p.per_xcd + (b >> 3);
  if (u >= tiles * p.ksplit) return;
  const int64_t split = u / tiles;
  const int64_t t = u - split * tiles;
  const int64_t tr = p.tr0 + t / cb, tc = t - (t / cb) * cb;
  const int64_t c_lo = split * p.kc;                  // this workgroup's k chunks: [c_lo, c_lo + nc)
  const int nc = (int)(min(p.nc, c_lo + p.kc) - c_lo);
  const int64_t blk = p.nc * 4 * PIECE;               // elements of one 64-row block
  const T* __restrict__ A = reinterpret_cast<const T*>(p.A);
  const T* __restrict__ Xt = reinterpret_cast<const T*>(p.Xt);
  // this wave's pieces of a chunk; blocks past the padded extent read the
  // last one (never stored)
  const T* src[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int pc = wave * LPW + j;
    const bool isa = pc < 4 * RB;
    const int q = isa ? pc : pc - 4 * RB;
    const int64_t bi = isa ? min(tr * RB + q / 4, rblocks - 1) : min(tc * CB + q / 4, fblocks - 1);
    src[j] = (isa ? A : Xt) + bi * blk + c_lo * 4 * PIECE + (q % 4) * PIECE;
  }
  const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  struct Fr { uint4 a[TM]; uint4 b[TN]; };
  // fragments of this wave in a stage: its TM pieces of A_hat, its TN of X^T
  const unsigned char* afrag = ring + (wave >> 1) * TM * 1024 + lane * 16;
  const unsigned char* bfrag = ring + (4 * RB + (wave & 1) * TN) * 1024 + lane * 16;
  auto issue = [&](int j, int c, int stage) {      // piece j of chunk c (past the end: in bounds, unused)
    const int cc = c < nc ? c : nc - 1;
    dma_1k(src[j], (uint32_t)cc * (4 * PIECE * sizeof(T)) + lane * 16, ring0 + stage * (NP * 1024) + (wave * LPW + j) * 1024);
  };
  auto read_a = [&](Fr& f, int i, int stage) {
    f.a[i] = *reinterpret_cast<const uint4*>(afrag + stage * (NP * 1024) + i * 1024);
  };
  auto read_b = [&](Fr& f, int i, int stage) {
    f.b[i] = *reinterpret_cast<const uint4*>(bfrag + stage * (NP * 1024) + i * 1024);
  };
#define MM_FENCE() __builtin_amdgcn_sched_barrier(0)
  // every wave's loads but those of the newest `chunks` chunks have landed,
  // and every wave holds what it read from LDS so far in registers
#define MM_LANDED(chunks)                                                                    \
  do {                                                                                       \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((chunks) * LPW) : "memory");         \
    __builtin_amdgcn_s_barrier();                                                            \
    MM_FENCE();                                                                              \
  } while (0)
  // chunk c is in F; chunk c + 1 (stage s1) goes to G, chunk c + S into the
  // stage s0 that chunk c was read from
  auto step = [&](const Fr& F, Fr& G, int c, int s0, int s1) {
    MM_LANDED(S - 2);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i < LPW) issue(i, c + S, s0);
      read_a(G, i, s1);
      if (i < TN) read_b(G, i, s1);
      MM_FENCE();
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = DaMfma<T>::run(F.a[i], F.b[j], acc[i][j]);
      MM_FENCE();
    }
  };
  auto next = [&](int s) { return s + 1 < S ? s + 1 : 0; };
  f32x4 sum[CHAINS ? TM : 1][CHAINS ? TN : 1];
  int left = p.chain;
  if constexpr (CHAINS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int d = 0; d < S; ++d)
#pragma unroll
    for (int j = 0; j < LPW; ++j) issue(j, d, d);
  MM_LANDED(S - 1);
  Fr f0, f1;
  // An odd chunk is done first, so that nothing follows the loop: with a
  // compute after it the register allocator rotates the accumulators on
  // every trip.  The launch guarantees nc >= 8, so the loop runs at least
  // once (a path around it made the allocator spill accumulators).
  int c = 0, s0 = 0;
  if (nc & 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(f1, i, 0);
#pragma unroll
    for (int i = 0; i < TN; ++i) read_b(f1, i, 0);
    step(f1, f0, 0, 0, 1);
    c = 1;
    s0 = 1;
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(f0, i, 0);
#pragma unroll
    for (int i = 0; i < TN; ++i) read_b(f0, i, 0);
  }
  do {
    const int s1 = next(s0), s2 = next(s1);
    step(f0, f1, c, s0, s1);
    step(f1, f0, c + 1, s1, s2);
    s0 = s2;
    c += 2;
    if constexpr (CHAINS) {
      left -= 2;
      if (left <= 0) {
        left = p.chain;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            sum[i][j] += acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  } while (c < nc);
  if constexpr (CHAINS) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += sum[i][j];
  }
  MM_LANDED(0);                                    // the ring becomes the epilogue's staging area
#undef MM_FENCE
#undef MM_LANDED

  // epilogue: one 16-row strip of the wave's block at a time (the strip
  // index is spelled out so that every accumulator index is static); with
  // k ranges the strips go out as fp32 partials instead
  float* st = reinterpret_cast<float*>(ring) + wave * (16 * MM_LDR);
  const int64_t row0 = (tr * 2 + (wave >> 1)) * (16 * TM), col0 = (tc * 2 + (wave & 1)) * (16 * TN);
  float bv[VE];
  epi_load_bias<T>(p.epi, col0 + (lane % (16 * TN / VE)) * VE, bv);
  const bool partial = p.ksplit > 1;
#define MM_STRIP(R)                                                                             \
  if ((R) < TM) {                                                                               \
    MM_SYNC();                                                                                  \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                              \
      _Pragma("unroll") for (int v = 0; v < 4; ++v)                                             \
        st[((lane >> 4) * 4 + v) * MM_LDR + j * 16 + (lane & 15)] = acc[(R) < TM ? (R) : 0][j][v]; \
    MM_SYNC();                                                                                  \
    if (partial) mm_store_strip_part<16 * TN, VE>(p, st, lane, row0 + (R) * 16, col0, split);   \
    else mm_store_strip<T, 16 * TN>(p, st, lane, row0 + (R) * 16, col0, bv);                    \
  }
  MM_STRIP(0) MM_STRIP(1) MM_STRIP(2) MM_STRIP(3) MM_STRIP(4) MM_STRIP(5) MM_STRIP(6) MM_STRIP(7)
#undef MM_STRIP
}

int64_t xt_elems(int prec, int64_t n, int64_t F) {
  const int64_t kc = prec == 0 ? 16 : 32;
  const int64_t nc = (n + kc - 1) / kc;
  return ((F + 63) / 64) * 64 * nc * kc;
}

// Bytes of the transposed X, rounded up to 256 (the partials follow it).
size_t xt_bytes(int prec, int64_t n, int64_t F) {
  return ((size_t)xt_elems(prec, n, F) * (prec == 0 ? 4 : 2) + 255) / 256 * 256;
}

// How one product is cut: which kernel, its tile, its k ranges.  Every
// candidate is priced in microseconds and the cheapest taken (one of the other
// two kernels only where it is 7 % below the 64-row blocks).  What the prices
// rest on, measured on MI355X:
//  * a round of workgroups (one per compute unit) costs as much as its longest;
//  * dense_agg_kernel and dense_stream_kernel, whose waves read fragments
//    straight into registers: a compute unit brings in at most about 48 GB/s
//    through its vector cache, A_hat and X^T together (46-50 GB/s for 47 to 256
//    workgroups, F = 16 and 64 alike), or works at the matrix rate; the chip is
//    held to the stream rate of A_hat, once per column block of 64;
//  * dense_mm_kernel, 16-bit: a k chunk takes `near` us while A_hat fits the 256
//    MB cache behind the L2s (up to NEAR_BYTES) and is there from the call
//    before, as from layer to layer of an epoch (a matrix just written, or called
//    for the first time, comes from HBM and takes longer), else `far` + `s` / (column
//    tiles), column tiles sharing a chunk of A_hat in L2, and at least `h` /
//    (column tiles), the rate at which the bytes that the LDS ring keeps in
//    flight come from HBM; fp32: `w32`, the matrix instructions;
//  * a round costs its start and end (`fixed`; 4 to 7 us for 64-row blocks of several column blocks),
//    k ranges the reduction launch and the partials' traffic; they are bounded
//    by DP_MAX_SPLIT, eight chunks each and the bytes of the partials;
//  * fp32 results show the rounding of the additions, and the more chains an
//    output is summed in the smaller it is (16-bit results do not show it:
//    2.078e-4 with one chain or eight).  The prices know nothing of it, so fp32
//    keeps to eight chains below F = 192, as the eight waves of the 64-row
//    blocks sum them, and above to as many, up to eight, as tiles of 128 x 128
//    need to fill the compute units; the streaming kernel's four waves take two
//    ranges at least.
//    They are ranges, or, up to 256 x 128, chains within a range, which cost
//    2 % of the time; a wider tile takes the ranges whatever their bytes.
//    Relative error on a full A_hat, one chain per range -> now: n = 8192 F =
//    128 8.1e-7 -> 5.8e-7 in 0.16 ms, n = 24000 F = 160 1.24e-6 -> 9.8e-7, 1.66
//    -> 1.58 ms, n = 12000 F = 190 8.8e-7 -> 6.2e-7, 0.44 -> 0.46 ms.
// One call with the transposition (us, before -> with the LDS ring of
// dense_mm_kernel, dense_stream_kernel and this rule), 16-bit: n = 16384 F =
// 128 191 -> 124, F = 384 357 -> 190; n = 8192 F = 512 90 -> 64; n = 24000 F =
// 256 539 -> 298; n = 32768 F = 160 1106 -> 406, F = 2048 3040 -> 2550; n =
// 20000 F = 64 202 -> 157; fp32: n = 2048 F = 64 40 -> 23, n = 6001 99 -> 56, n
// = 9000 F = 192 545 -> 245, n = 24000 F = 384 5598 -> 3261.
constexpr int64_t DP_MAX_SPLIT = 16;
constexpr int64_t DP_PART_BYTES = (int64_t)96 << 20;
constexpr int64_t ST_PART_BYTES = (int64_t)24 << 20;
enum DenseKind { DK_ROWS64, DK_STREAM, DK_MM };
struct DensePlan {
  DenseKind kind;
  int tile;             // DK_MM: index of MM_TILES
  int64_t ksplit, kc;   // k ranges, chunks per range
  int chain;            // DK_MM: chunks of a chain (0: one chain per range)
};
constexpr int MM_CHAIN_TILE = 2;   // the first of MM_TILES whose waves have registers for chains
struct MmTile { int rows, cols; double near, far, s, h, w32, fixed; };
constexpr MmTile MM_TILES[] = {
    {256, 256, 0.56, 0.55, 0.12, 0.80, 3.55, 9.0},
    {256, 192, 0.41, 0.45, 0.20, 0.72, 2.66, 8.5},
    {256, 128, 0.30, 0.38, 0.30, 0.74, 1.78, 7.0},
    {128, 128, 0.19, 0.24, 0.10, 0.39, 0.90, 5.5},
};
constexpr double NEAR_BYTES = 2e8;

double price_rounds(int64_t units) { return (double)((units + 255) / 256); }

// `rows` rows of the product through tile t, S ranges of kc chunks (us).
double mm_price(int prec, int64_t n, int64_t rows, int64_t F, const MmTile& t, int64_t S, int64_t kc) {
  const int64_t ct = (F + t.cols - 1) / t.cols, tiles = (rows + t.rows - 1) / t.rows * ct;
  const bool near = (double)n * (double)n * (prec == 0 ? 4 : 2) <= NEAR_BYTES;
  const double chunk = prec == 0 ? std::max(t.w32, t.h / ct) : near ? t.near : std::max(t.far + t.s / ct, t.h / ct);
  return price_rounds(tiles * S) * (kc * chunk + t.fixed) + (S > 1 ? 6.0 + 8.0 * S * (double)rows * F / 9e6 : 0.0);
}

DensePlan dense_plan(int prec, int64_t n, int64_t F, bool tiled, bool split) {
  const int64_t nc = (n + (prec == 0 ? 15 : 31)) / (prec == 0 ? 16 : 32);
  DensePlan pl{DK_ROWS64, 0, 1, nc, 0};
  if (!tiled) return pl;
  const double es = prec == 0 ? 4 : 2, dn = (double)n;
  const double cu_bytes = 4.8e4, chip = dn * dn * es / 6.8e6;                      // per us
  auto unit = [&](double rows, double cols, double cu_flops) {
    return std::max((rows + cols) * dn * es / cu_bytes, 2 * rows * dn * cols / cu_flops);
  };
  const int64_t cb64 = (F + 63) / 64, ldp = (F + 7) / 8 * 8;
  const double cols = F > 64 ? 64.0 : 16.0 * ((F + 15) / 16);
  const double ends = F <= 64 ? 0.0 : prec == 0 ? 7.0 : 4.0;
  double best = 0.93 * std::max(price_rounds((n + 63) / 64 * cb64) * (unit(64, cols, prec == 0 ? 4.8e5 : 4.8e6) + ends), chip * cb64);
  if (best < 8.0) return pl;                            // less than any other candidate's start and end
  auto offer = [&](double t, DenseKind kind, int tile, int64_t S, int64_t kc, int chain) {
    if (t < best) { best = t; pl = DensePlan{kind, tile, S, kc, chain}; }
  };
  if (F <= 64) {
    const int64_t blocks = (n + 127) / 128, least = prec == 0 ? 2 : 1;   // 4 waves: 8 chains
    for (int64_t S = 1; S <= DP_MAX_SPLIT; ++S) {
      if (S > 1 && (!split || nc < 8 * S || (S > least && S * n * ldp * 4 > ST_PART_BYTES))) break;
      if (S < least) continue;
      offer(std::max(price_rounds(blocks * S) * (unit(128, cols, prec == 0 ? 5.1e5 : 5.1e6) / S + 4.0), chip) +
                (S > 1 ? 7.0 + 8.0 * S * dn * F / 3e6 : 0.0),
            DK_STREAM, 0, S, 0, 0);
    }
    return pl;
  }
  int64_t need = 1;                                    // fp32: chains of additions per output
  if (prec == 0) {
    const int64_t few = (n + 127) / 128 * ((F + 127) / 128);
    while (need < 8 && (F < 192 || few * need < 256) && nc >= 12 * need) need *= 2;
  }
  for (int i = 0; nc >= 8 && i < 4; ++i) {
    const bool chains = i >= MM_CHAIN_TILE;
    for (int64_t S = 1; S <= DP_MAX_SPLIT; ++S) {
      const int64_t kc = (nc + S - 1) / S;
      if (S > 1 && (!split || kc < 8 || (S > (chains ? 1 : need) && S * n * ldp * 4 > DP_PART_BYTES))) break;
      if ((S < need && !chains) || nc - (S - 1) * kc < 8) continue;
      const double t = mm_price(prec, n, n, F, MM_TILES[i], S, kc);
      offer(S < need ? 1.02 * t : t, DK_MM, i, S, kc, S < need ? (int)(nc / need / 2 * 2) : 0);
    }
  }
  return pl;
}

// With less scratch than the partials of all rows need, the product takes its
// rows in several launches, each followed by its reduction.  The k ranges stay
// and with them every bit: the order in which an output is summed depends on the
// ranges and chains, not on the tile that holds it, so each launch takes the tile that is
// cheapest for its rows.  (All rows with one tile left compute units idle: n =
// 16384, F = 512, 16-bit, two ranges through the 64 MiB of
// gcn_layer_bwd_noalloc 400 us, 313 with the rows and tiles priced.)
size_t dense_part_bytes(const DensePlan& pl, int64_t rows, int64_t F) {
  return pl.ksplit > 1 ? (size_t)pl.ksplit * (size_t)rows * (size_t)((F + 7) / 8 * 8) * sizeof(float) : 0;
}
int64_t dense_row_step(const DensePlan& pl) { return pl.kind == DK_MM ? 256 : 128; }   // whole tiles, whichever

int cheapest_tile(int prec, const DensePlan& pl, int64_t n, int64_t rows, int64_t F, double* price) {
  int best = pl.tile;
  *price = mm_price(prec, n, rows, F, MM_TILES[best], pl.ksplit, pl.kc);
  for (int i = pl.chain ? MM_CHAIN_TILE : 0; i < 4; ++i) {
    const double t = mm_price(prec, n, rows, F, MM_TILES[i], pl.ksplit, pl.kc);
    if (t < *price) { *price = t; best = i; }
  }
  return best;
}

// Rows of a launch (the last one takes the rest): all where their partials fit.
int64_t dense_rows_per_launch(int prec, const DensePlan& pl, int64_t n, int64_t F, size_t part_bytes) {
  if (part_bytes >= dense_part_bytes(pl, n, F)) return n;
  const int64_t step = dense_row_step(pl), most = (int64_t)(part_bytes / dense_part_bytes(pl, 1, F)) / step * step;
  if (pl.kind != DK_MM) return most;
  int64_t best = most;
  double best_t = 0.0;
  for (int64_t per = most; per > most / 2; per -= step) {
    double whole, last = 0.0;
    cheapest_tile(prec, pl, n, per, F, &whole);
    if (n % per) cheapest_tile(prec, pl, n, n % per, F, &last);
    const double t = (double)(n / per) * whole + last;
    if (per == most || t < best_t) { best_t = t; best = per; }
  }
  return best;
}

template <typename T, int TN, int DEPTH>
void stream_launch(const StreamParams& q, hipStream_t s) {
  hipLaunchKernelGGL((dense_stream_kernel<T, TN, DEPTH>), dim3((unsigned)(q.rowb * q.ksplit)), dim3(256), 0, s, q);
}

// Rows row0 .. row0 + rows - 1: row0 a multiple of dense_row_step, rows too
// except for the last ones of the product.
template <typename T>
hipError_t launch_rows(const DensePlan& pl, const void* A, int64_t n, const T* Xt, int64_t F, int64_t nc, int64_t row0,
                       int64_t rows, const Epilogue& epi, float* part, hipStream_t s) {
  const int64_t ldp = (F + Vec<T>::N - 1) / Vec<T>::N * Vec<T>::N;
  const int64_t step = pl.kind == DK_MM ? MM_TILES[pl.tile].rows : 128, steps = (rows + step - 1) / step;
  if (pl.kind == DK_MM) {
    const int64_t cb = (F + MM_TILES[pl.tile].cols - 1) / MM_TILES[pl.tile].cols;
    const int64_t units = steps * cb * pl.ksplit;
    if (units > INT32_MAX / 2) return hipErrorInvalidValue;      // more than 8 TB of A_hat or X
    MmParams q;
    q.A = A; q.Xt = Xt; q.n = n; q.F = F; q.nc = nc;
    q.rblocks = (int)((n + 63) / 64);
    q.fblocks = (int)((F + 63) / 64);
    q.tr0 = (int)(row0 / step);
    q.cb = (int)cb;
    q.tiles = (int)(steps * cb);
    q.ksplit = (int)pl.ksplit;
    q.kc = (int)pl.kc;
    q.chain = pl.chain;
    q.part = part;
    q.row0 = row0;
    q.prows = rows;
    q.ldp = ldp;
    q.per_xcd = (int)((units + 7) / 8);
    q.epi = epi;
    const dim3 g((unsigned)(8 * q.per_xcd));
#define MM_LAUNCH(TM_, TN_, S_, C_) \
  hipLaunchKernelGGL((dense_mm_kernel<T, TM_, TN_, S_, C_>), g, dim3(256), 0, s, q)
    if constexpr (sizeof(T) == 4) {
      if (pl.chain && pl.tile == MM_CHAIN_TILE) MM_LAUNCH(8, 4, 6, true);
      else if (pl.chain) MM_LAUNCH(4, 4, 8, true);
    }
    if (!pl.chain) {
      switch (pl.tile) {
        case 0: MM_LAUNCH(8, 8, 4, false); break;
        case 1: MM_LAUNCH(8, 6, 5, false); break;
        case 2: MM_LAUNCH(8, 4, 6, false); break;
        default: MM_LAUNCH(4, 4, 8, false); break;
      }
    }
#undef MM_LAUNCH
  } else {
    StreamParams q;
    q.A = A; q.Xt = Xt; q.n = n; q.F = F; q.nc = nc;
    q.rblocks = (n + 63) / 64;
    q.rb0 = row0 / step;
    q.rowb = steps;
    q.ksplit = pl.ksplit;
    q.part = part;
    q.prows = rows;
    q.ldp = ldp;
    q.epi = epi;
    switch ((F + 15) / 16) {
      case 1: stream_launch<T, 1, 8>(q, s); break;
      case 2: stream_launch<T, 2, 8>(q, s); break;
      case 3: stream_launch<T, 3, 6>(q, s); break;
      default: stream_launch<T, 4, 6>(q, s); break;
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || pl.ksplit == 1) return e;
  // the k ranges' partials, added in range order, through the epilogue
  const int64_t vecs = rows * (ldp / Vec<T>::N);
  hipLaunchKernelGGL(mm_reduce_kernel<T>, dim3((unsigned)((vecs + 255) / 256)), dim3(256), 0, s, part, pl.ksplit, row0,
                     rows, ldp, epi);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const void* A, int64_t lda, bool tiled, int64_t n, const void* X, int64_t ldx, int64_t F,
                    const Epilogue& epi, void* ws, size_t ws_bytes, float* colsum, bool split, hipStream_t s) {
  constexpr int KC = tile_kc<T>();
  constexpr int PREC = sizeof(T) == 4 ? 0 : 1;
  const int64_t nc = (n + KC - 1) / KC;
  const int64_t fblocks = (F + 63) / 64;
  DensePlan pl = dense_plan(PREC, n, F, tiled, split);
  const size_t xb = xt_bytes(PREC, n, F);
  const int64_t per = ws_bytes < xb ? 0 : dense_rows_per_launch(PREC, pl, n, F, ws_bytes - xb);
  if (per <= 0) return hipErrorInvalidValue;
  T* Xt = reinterpret_cast<T*>(ws);
  dim3 tg((unsigned)((nc * KC + XpGeom<T>::WG_K - 1) / XpGeom<T>::WG_K), (unsigned)fblocks);
  hipLaunchKernelGGL(transpose_tiled_kernel<T>, tg, dim3(256), 0, s, reinterpret_cast<const T*>(X), ldx, n, F, Xt, nc,
                     colsum);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (pl.kind != DK_ROWS64) {
    float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + xb);
    for (int64_t r = 0; r < n; r += per) {
      const int64_t rows = std::min(per, n - r);
      double price;
      if (per < n && pl.kind == DK_MM) pl.tile = cheapest_tile(PREC, pl, n, rows, F, &price);
      e = launch_rows<T>(pl, A, n, Xt, F, nc, r, rows, epi, part, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  DaParams p;
  p.A = A; p.lda = lda; p.Xt = Xt; p.ldt = 0; p.n = n; p.F = F; p.epi = epi;
  dim3 grid((unsigned)((n + DA_BM - 1) / DA_BM), (unsigned)fblocks);
  const int tn = F > 48 ? 4 : (int)((F + 15) / 16);
  const dim3 blk(64 * DA_WAVES);
#define DA_LAUNCH(TN_)                                                                          \
  if (tiled) hipLaunchKernelGGL((dense_agg_kernel<T, TN_, true>), grid, blk, 0, s, p);          \
  else hipLaunchKernelGGL((dense_agg_kernel<T, TN_, false>), grid, blk, 0, s, p);
  switch (tn) {
    case 1: DA_LAUNCH(1) break;
    case 2: DA_LAUNCH(2) break;
    case 3: DA_LAUNCH(3) break;
    default: DA_LAUNCH(4) break;
  }
#undef DA_LAUNCH
  return hipGetLastError();
}

// Dense form of a CSR A_hat: one wave per row scatters its entries.
template <typename T, typename IdxT, bool TILED>
__global__ __launch_bounds__(256) void densify_kernel(int64_t n, const IdxT* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colidx, const T* __restrict__ values,
                                                      const float* __restrict__ dinv, T* __restrict__ dense,
                                                      int64_t ld, int64_t nc) {
  const int lane = threadIdx.x & 63;
  for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
    const float dr = values ? 0.f : dinv[r];
    for (int64_t k = (int64_t)rowptr[r] + lane; k < (int64_t)rowptr[r + 1]; k += 64) {
      const int32_t c = colidx[k];
      const T v = values ? values[k] : from_f32<T>(dr * dinv[c]);
      dense[TILED ? tiled_off<T>(r, c, nc) : r * ld + c] = v;
    }
  }
}

template <typename T>
hipError_t densify_t(const CsrView& A, bool tiled, void* dense, int64_t ld, hipStream_t s) {
  constexpr int KC = tile_kc<T>();
  const int64_t nc = (A.n + KC - 1) / KC;
  const size_t bytes = tiled ? (size_t)((A.n + 63) / 64) * 64 * nc * KC * sizeof(T) : (size_t)A.n * ld * sizeof(T);
  hipError_t e = fill_zero(dense, bytes, s);
  if (e != hipSuccess) return e;
  const dim3 g((unsigned)std::min<int64_t>((A.n + 3) / 4, 1 << 20));   // the kernel loops over rows
  const T* vals = reinterpret_cast<const T*>(A.values);
  T* d = reinterpret_cast<T*>(dense);
  if (A.idx64) {
    const int64_t* rp = reinterpret_cast<const int64_t*>(A.rowptr);
    if (tiled) hipLaunchKernelGGL((densify_kernel<T, int64_t, true>), g, dim3(256), 0, s, A.n, rp, A.colidx, vals, A.dinv, d, ld, nc);
    else hipLaunchKernelGGL((densify_kernel<T, int64_t, false>), g, dim3(256), 0, s, A.n, rp, A.colidx, vals, A.dinv, d, ld, nc);
  } else {
    const int32_t* rp = reinterpret_cast<const int32_t*>(A.rowptr);
    if (tiled) hipLaunchKernelGGL((densify_kernel<T, int32_t, true>), g, dim3(256), 0, s, A.n, rp, A.colidx, vals, A.dinv, d, ld, nc);
    else hipLaunchKernelGGL((densify_kernel<T, int32_t, false>), g, dim3(256), 0, s, A.n, rp, A.colidx, vals, A.dinv, d, ld, nc);
  }
  return hipGetLastError();
}

}  // namespace

size_t dense_agg_workspace_bytes(int prec, int64_t n, int64_t F, bool tiled, bool split) {
  return xt_bytes(prec, n, F) + dense_part_bytes(dense_plan(prec, n, F, tiled, split), n, F);
}

size_t dense_agg_min_bytes(int prec, int64_t n, int64_t F, bool tiled) {
  const DensePlan pl = dense_plan(prec, n, F, tiled, true);
  return xt_bytes(prec, n, F) + dense_part_bytes(pl, std::min(n, dense_row_step(pl)), F);
}

void dense_plan_query(int prec, int64_t n, int64_t F, int64_t out[6]) {
  const DensePlan pl = dense_plan(prec, n, F, true, true);
  const bool mm = pl.kind == DK_MM;
  out[0] = pl.kind;
  out[1] = mm ? MM_TILES[pl.tile].rows : pl.kind == DK_STREAM ? 128 : 64;
  out[2] = mm ? MM_TILES[pl.tile].cols : 64;
  out[3] = pl.ksplit;
  out[4] = mm ? pl.kc : (n + (prec == 0 ? 15 : 31)) / (prec == 0 ? 16 : 32);
  out[5] = pl.chain;
}

int64_t dense_tiled_elems(int prec, int64_t n) {
  const int64_t kc = prec == 0 ? 16 : 32;
  return ((n + 63) / 64) * 64 * ((n + kc - 1) / kc) * kc;
}

hipError_t dense_agg_launch(int prec, const void* A, int64_t lda, bool tiled, int64_t n, const void* X, int64_t ldx,
                            int64_t F, const Epilogue& epi, void* ws, size_t ws_bytes, float* colsum, hipStream_t s,
                            bool split) {
  switch (prec) {
    case 0: return launch_t<float>(A, lda, tiled, n, X, ldx, F, epi, ws, ws_bytes, colsum, split, s);
    case 1: return launch_t<f16>(A, lda, tiled, n, X, ldx, F, epi, ws, ws_bytes, colsum, split, s);
    case 2: return launch_t<bf16>(A, lda, tiled, n, X, ldx, F, epi, ws, ws_bytes, colsum, split, s);
  }
  return hipErrorInvalidValue;
}

int64_t dense_agg_colsum_rows(int prec, int64_t n) {
  const int64_t kc = prec == 0 ? 16 : 32;
  const int64_t wg_k = prec == 0 ? XpGeom<float>::WG_K : XpGeom<f16>::WG_K;
  return ((n + kc - 1) / kc * kc + wg_k - 1) / wg_k;
}

hipError_t densify_launch(const CsrView& A, int prec, bool tiled, void* dense, int64_t ld, hipStream_t s) {
  switch (prec) {
    case 0: return densify_t<float>(A, tiled, dense, ld, s);
    case 1: return densify_t<f16>(A, tiled, dense, ld, s);
    case 2: return densify_t<bf16>(A, tiled, dense, ld, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gcn
