// Rader passes (rader.h states the identity) of compiled primes N <= 1009
// with both FFTs of length L = N - 1 = A B in two register steps.
//
// The tile's inputs go to LDS with lanes along each pencil.  Step 1:
// butterfly t (t < B) of a pencil gathers a[t + r B] = x[g^(t + r B)] (r <
// A) from there, transforms with DFT_A and leaves output r at row r, column
// t of the pencil's table, over the inputs (a barrier lies between).  Step
// 2: butterfly tm takes row tm through the twiddles and DFT_B to the
// frequencies tm + A k, keeps frequency 0 for y[0], multiplies by FFT_L(b) /
// L and goes straight on through DFT_B of the second transform and the
// twiddles back to its own row.  Step 3: butterfly t takes column t through
// DFT_A and stores x[0] + output t + B j at row g^(t + B j): the rotated
// store writes a row segment of consecutive pencils whatever the row, so
// the output permutation costs nothing.
//
// Against the staged pass (an LDS round trip and two barriers a radix, and a
// scatter through LDS), MI355X: see kernels_rader_two_step.hip.
//
// PassArgs fields used: pencil fields and element strides as for every
// pass, res_mask = N, res_shift = A, twp_mask = the radix code of L.
// Tables: tw[tm B + j] = w_L^{tm j}; twp = FFT_L(b) / L as filt[tm B + k] =
// (FFT_L(b) / L)[tm + A k] (L entries), then g^j mod N (j < L) as 32-bit
// integers.
#pragma once

#include "rader.h"
#include "two_step_kernel.h"

namespace dft3d {

template <int N, int A, int T> constexpr int rader_two_step_stride() {
  constexpr int table = two_step_stride(A, (N - 1) / A), row = N | 1;
  return table > row ? table : row;
}

template <int N, int A, int T>
__device__ __forceinline__ void rader_two_step_kernel_run(
    const float2* src, float2* dst, const float2* __restrict__ tw,
    const float2* __restrict__ twp, const PassArgs& a) {
  constexpr int L = N - 1, B = L / A, TH = two_step_threads(A > B ? A : B, T);
  constexpr int pitch = two_step_pitch(B), sq = rader_two_step_stride<N, A, T>();
  static_assert(A * B == L, "split of N - 1");
  __shared__ float2 lds[T * sq];
  __shared__ float2 x0s[T], dcs[T];
  const float2* __restrict__ filt = twp;
  const int* __restrict__ perm = reinterpret_cast<const int*>(twp + L);
  const int tid = threadIdx.x;
  const int64_t tile = tile_index(blockIdx.x, gridDim.x, a.xcd_remap);
  {  // inputs, lanes along the pencils; those past the end of a ragged last
     // tile read the last pencil
    constexpr int I = (T * N + TH - 1) / TH;
    float2 x[I];
#pragma unroll
    for (int i = 0; i < I; ++i) {
      const int e = tid + TH * i < T * N ? tid + TH * i : T * N - 1;
      int64_t b = tile * T + e / N;
      b = b < a.B ? b : a.B - 1;
      x[i] = src[pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.is0, a.is1, a.is2) +
                 e % N * a.ijs];
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
      const int e = tid + TH * i;
      if (e < T * N) {
        if (a.conj_in) x[i].y = -x[i].y;
        lds[e / N * sq + e % N] = x[i];
        if (e % N == 0) x0s[e / N] = x[i];
      }
    }
  }
  __syncthreads();  // inputs in LDS
  {
    const int q = tid / B, t = tid % B;
    float2 v[A];
    if (tid < T * B) {
#pragma unroll
      for (int r = 0; r < A; ++r) v[r] = lds[q * sq + perm[t + r * B]];
      dft_mixed<A>(v);
    }
    __syncthreads();  // every input is read
    if (tid < T * B) {
#pragma unroll
      for (int r = 0; r < A; ++r) lds[q * sq + r * pitch + t] = v[r];
    }
  }
  __syncthreads();  // step 1 is in LDS
  if (tid < T * A) {
    const int q = tid % T, tm = tid / T;
    float2* row = lds + q * sq + tm * pitch;
    int at = tm * B;
    float2 v[B];
    v[0] = row[0];
#pragma unroll
    for (int j = 1; j < B; ++j) v[j] = cmul(row[j], tw[at + j]);
    dft_mixed<B>(v);
    if (tm == 0) dcs[q] = v[0];
    // read where used, not held over a DFT (as in bluestein_two_step.h)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int j = 0; j < B; ++j) v[j] = cmul(v[j], filt[at + j]);
    dft_mixed<B>(v);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : "+v"(at));
    row[0] = v[0];  // its own row: no other thread reads it in this step
#pragma unroll
    for (int j = 1; j < B; ++j) row[j] = cmul(v[j], tw[at + j]);
  }
  __syncthreads();  // every row is transformed
  if (tid < T * B) {
    const int q = tid % T, t = tid / T;
    float2 v[A];
#pragma unroll
    for (int r = 0; r < A; ++r) v[r] = lds[q * sq + r * pitch + t];
    dft_mixed<A>(v);
    const int64_t b = tile * T + q;
    if (b < a.B) {
      float2* d = dst + pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.os0, a.os1, a.os2);
      const float2 x0 = x0s[q];
#pragma unroll
      for (int j = 0; j < A; ++j) {
        float2 y = cadd(x0, v[j]);
        if (a.conj_out) y.y = -y.y;
        d[perm[t + B * j] * a.oks] = y;
      }
      if (t == 0) {
        float2 y = cadd(x0, dcs[q]);
        if (a.conj_out) y.y = -y.y;
        d[0] = y;
      }
    }
  }
}

template <int N, int A, int T>
__global__ void __launch_bounds__((two_step_threads(A > (N - 1) / A ? A : (N - 1) / A, T)))
rader_two_step_kernel(const PassLaunch la) {
  rader_two_step_kernel_run<N, A, T>(la.src, la.dst, la.tw, la.twp, la.a);
}

template <int N, int A, int T>
hipError_t launch_rader_two_step(const PassArgs& a, const float2* src, float2* dst,
                                 const float2* tw, const float2* twp, hipStream_t stream) {
  constexpr int B = (N - 1) / A;
  const int64_t blocks = (a.B + T - 1) / T;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  if (a.res_mask != N || a.res_shift != A) return hipErrorInvalidValue;
  hipLaunchKernelGGL((rader_two_step_kernel<N, A, T>), dim3((unsigned)blocks),
                     dim3(two_step_threads(A > B ? A : B, T)), 0, stream,
                     PassLaunch{src, dst, tw, twp, a});
  return hipGetLastError();
}

template <int N, int A, int T>
KernelInfo kernel_info_rader_two_step() {
  constexpr int B = (N - 1) / A, TH = two_step_threads(A > B ? A : B, T);
  constexpr int LDS = (T * rader_two_step_stride<N, A, T>() + 2 * T) * 8;
  static_assert(LDS <= 160 * 1024 && TH <= 1024, "tile fits");
  KernelInfo k{N + 1, T, MODE_ROW, MODE_COL, 0, TH, LDS, &launch_rader_two_step<N, A, T>, 0, 0};
  k.rader = 1;
  k.two_step = A;
  k.fixed_n = N;
  k.fixed_code = mixed_radix_code(N - 1);
  return k;
}

}  // namespace dft3d
