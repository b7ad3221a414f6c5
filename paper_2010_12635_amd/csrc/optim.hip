// Optimiser step with fp32 master weights and dynamic loss scaling, the O2
// scheme of the paper's Section "Background and Motivation": gradients of
// the scaled loss are checked for overflow, unscaled, and applied by Adam
// (Kingma & Ba) to fp32 masters, whose 16-bit copies feed the next forward
// pass.  All state stays on the device: three launches, no host sync.
#include "internal.h"

namespace gcn {

namespace {

// Both kernels stream: E = 4 consecutive elements per thread and round, one
// 16-byte load per fp32 array (8 bytes of 16-bit working copies), or E = 1
// for arrays off those boundaries and for short ones (ADAM_WIDE).  The
// elements past the last whole four go to the first threads one by one.
// 8.4 M parameters with 16-bit copies, 252 MB: 60.7 -> 56.4 us a step (4.5
// TB/s; the three launches alone are 13 us up to a million parameters).
template <int E>
__global__ __launch_bounds__(256) void grad_check_kernel(int64_t count, const float* __restrict__ g, int32_t* flag) {
  bool bad = false;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t whole = count / E;
  for (int64_t i = first; i < whole; i += stride) {
    if constexpr (E == 4) {
      float x[4];
      unpack<float>(ldg16(g + 4 * i), x);
#pragma unroll
      for (int k = 0; k < 4; ++k) bad |= !finite_f32(x[k]);
    } else {
      bad |= !finite_f32(g[i]);
    }
  }
  if (first < count - whole * E) bad |= !finite_f32(g[whole * E + first]);
  if (bad) raise_flag(flag);
}

struct AdamStep {
  AdamHyper hp;
  float inv_scale, bc1, bc2;
};

// One element: its moments and master in place.
__device__ __forceinline__ void adam_element(const AdamStep& a, float g, float& w, float& m, float& v) {
  const float gi = g * a.inv_scale;
  m = a.hp.beta1 * m + (1.f - a.hp.beta1) * gi;
  v = a.hp.beta2 * v + (1.f - a.hp.beta2) * gi * gi;
  w = w - a.hp.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.hp.eps);
}

template <typename T>
__device__ __forceinline__ void adam_one(const AdamStep& a, int64_t i, float* w, const float* g, float* m, float* v,
                                         T* working) {
  float wi = w[i], mi = m[i], vi = v[i];
  adam_element(a, g[i], wi, mi, vi);
  m[i] = mi;
  v[i] = vi;
  w[i] = wi;
  if (working) working[i] = from_f32<T>(wi);
}

template <typename T, int E>
__global__ __launch_bounds__(256) void adam_kernel(int64_t count, float* __restrict__ w, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, T* __restrict__ working,
                                                   AdamHyper hp, const ScalerState* __restrict__ st,
                                                   const int32_t* __restrict__ flag) {
  if (*flag) return;
  const float t = (float)(st->step + 1);
  const AdamStep a{hp, 1.f / st->scale, 1.f - powf(hp.beta1, t), 1.f - powf(hp.beta2, t)};
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t whole = count / E;
  for (int64_t i = first; i < whole; i += stride) {
    if constexpr (E == 4) {
      const uint4 rg = ldg16(g + 4 * i), rw = ldg16(w + 4 * i), rm = ldg16(m + 4 * i), rv = ldg16(v + 4 * i);
      float gx[4], wx[4], mx[4], vx[4];
      unpack<float>(rg, gx);
      unpack<float>(rw, wx);
      unpack<float>(rm, mx);
      unpack<float>(rv, vx);
#pragma unroll
      for (int k = 0; k < 4; ++k) adam_element(a, gx[k], wx[k], mx[k], vx[k]);
      stg16(m + 4 * i, pack<float>(mx));
      stg16(v + 4 * i, pack<float>(vx));
      stg16(w + 4 * i, pack<float>(wx));
      if (working) {
        typedef T t4 __attribute__((ext_vector_type(4)));
        t4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = from_f32<T>(wx[k]);
        *reinterpret_cast<t4*>(working + 4 * i) = o;
      }
    } else {
      adam_one<T>(a, i, w, g, m, v, working);
    }
  }
  if (first < count - whole * E) adam_one<T>(a, whole * E + first, w, g, m, v, working);
}

__global__ void scaler_kernel(AdamHyper hp, ScalerState* st, int32_t* flag) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  ScalerState s = *st;
  if (*flag) {
    s.scale = fmaxf(s.scale * hp.backoff, hp.min_scale);
    s.good_steps = 0;
    s.skipped += 1;
  } else {
    s.step += 1;
    s.good_steps += 1;
    if (s.good_steps >= hp.interval) {
      s.scale = fminf(s.scale * hp.growth, hp.max_scale);
      s.good_steps = 0;
    }
  }
  *st = s;
  *flag = 0;
}

}  // namespace

namespace {

// Elements from which the 4-wide kernels are taken: below, one element per
// thread spreads the work over more compute units.  The launches hide the
// difference up to 2^20 (13.4 us either way from 2^18 to 2^20); 2^22 takes
// 27.6 us one by one, 24.5 four at a time.
constexpr int64_t ADAM_WIDE = 1 << 18;

bool on_boundary(const void* p, size_t bytes) { return reinterpret_cast<uintptr_t>(p) % bytes == 0; }

template <typename T, int E>
hipError_t launch_step(int64_t count, float* master, const float* grad, float* m, float* v, T* working,
                       const AdamHyper& hp, ScalerState* state, int32_t* flag, hipStream_t s) {
  int64_t blocks = (count + 256 * E - 1) / (256 * E);
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL((grad_check_kernel<E>), dim3((unsigned)blocks), dim3(256), 0, s, count, grad, flag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((adam_kernel<T, E>), dim3((unsigned)blocks), dim3(256), 0, s, count, master, grad, m, v, working,
                     hp, state, flag);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(scaler_kernel, dim3(1), dim3(64), 0, s, hp, state, flag);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_prec(int64_t count, float* master, const float* grad, float* m, float* v, void* working,
                       const AdamHyper& hp, ScalerState* state, int32_t* flag, hipStream_t s) {
  T* wk = static_cast<T*>(working);
  const bool wide = count >= ADAM_WIDE && on_boundary(master, 16) && on_boundary(grad, 16) && on_boundary(m, 16) &&
                    on_boundary(v, 16) && on_boundary(working, 4 * sizeof(T));
  return wide ? launch_step<T, 4>(count, master, grad, m, v, wk, hp, state, flag, s)
              : launch_step<T, 1>(count, master, grad, m, v, wk, hp, state, flag, s);
}

}  // namespace

hipError_t optimizer_launch(int64_t count, float* master, const float* grad, float* m, float* v, void* working,
                            int prec, const AdamHyper& hp, ScalerState* state, int32_t* flag, hipStream_t s) {
  switch (prec) {
    case 0: return launch_prec<float>(count, master, grad, m, v, working, hp, state, flag, s);
    case 1: return launch_prec<f16>(count, master, grad, m, v, working, hp, state, flag, s);
    case 2: return launch_prec<bf16>(count, master, grad, m, v, working, hp, state, flag, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gcn
