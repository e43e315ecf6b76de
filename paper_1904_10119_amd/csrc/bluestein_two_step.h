// Bluestein axes of length n <= 1024 with a convolution length m = A B that
// is not a power of two but the next of a ladder of products at least 2 n
// (bluestein.h states the identity and the power-of-two form, which runs the
// longer lengths): both FFTs of length m in two register steps, two
// exchanges through LDS in all.
//
// Step 1: butterfly t (t < B) of a pencil loads its points t + r B times the
// chirp.  A is even and n <= m / 2, so only r < A / 2 are loaded and DFT_A
// runs as two DFT_{A/2} (its radix-2 step has one zero operand).  Step 2:
// butterfly tm (tm < A) takes row tm of the A x B table, times w_m^{tm t},
// through DFT_B to the frequencies tm + A k, times H / m, and straight on
// through DFT_B of the inverse transform (real and imaginary parts swapped:
// IDFT(x) = swap(DFT(swap(x)))), times w_m^{tm r}, back to its own row.
// Step 3: butterfly t takes column t through DFT_A, of whose outputs t + B j
// only the lower half (j < A / 2) can lie below n, times the chirp, to
// memory.
//
// What bounds it: instruction issue.  At n = 251, m = 504 = 24 x 21 the vector
// units issued in 80 % of the cycles, 96 instructions a point of m; twiddle-
// free index maps in the register DFTs, m = 512 = 16 x 32 and pointer steps
// instead of products brought 99 to 85 us a pass.  Tiles of 16 pencils up to
// m = 256 and of 8 above, where 16 leave two workgroups a CU (163^3 81 / 68
// us, 211^3 217 / 160, 263^3 385 / 316; 83^3 19.8 / 20.1, 101^3 30.4 / 31.1),
// and of 4 above m = 1024, where the registers (118 to 150) leave three
// wavefronts a SIMD and 4 pencils three workgroups a CU (8 / 4 pencils: 613 x
// 613 x 64 514 / 404 us, 699 x 699 x 64 637 / 518, 557 x 557 x 64 333 / 338;
// 6: 418 and 618; below m = 1024 8 pencils are 5 to 10 % ahead of 4).
// Against the power-of-two form (MI355X, three passes): 61^3 24.5 -> 14.9 us,
// 131^3 97.6 -> 48.7, 199^3 253 -> 131, 251^3 460 -> 254, 263^3 840 -> 316,
// 379^3 2.07 -> 0.96 ms, 509^3 4.35 -> 2.46 ms, 557 x 557 x 64 714 -> 338
// us, 699 x 699 x 64 990 -> 518, 839 x 839 x 64 1324 -> 829, 1021 x 1021 x 64
// 1785 -> 1196.
//
// PassArgs fields used: pencil fields and element strides as for every
// pass, res_mask = n, res_shift = A.  Tables: tw[tm B + j] = w_m^{tm j};
// twp = the chirp (n entries), then the filter as filt[tm B + k] = H[tm + A
// k] / m; all from FP64.
#pragma once

#include "two_step_kernel.h"

namespace dft3d {

// DFT of length A of x[0..A/2) followed by zeros.
template <int A>
__device__ __forceinline__ void dft_half_in(const float2 (&x)[A / 2], float2 (&y)[A]) {
  constexpr int H = A / 2;
  float2 e[H], o[H];
  static_for<H>([&](auto ri) {
    constexpr int r = decltype(ri)::value;
    e[r] = x[r];
    o[r] = mul_root<r, A>(x[r]);
  });
  dft_mixed<H>(e);
  dft_mixed<H>(o);
#pragma unroll
  for (int i = 0; i < H; ++i) {
    y[2 * i] = e[i];
    y[2 * i + 1] = o[i];
  }
}

// Outputs 0..A/2-1 of the DFT of length A of x.
template <int A>
__device__ __forceinline__ void dft_half_out(const float2 (&x)[A], float2 (&y)[A / 2]) {
  constexpr int H = A / 2;
  float2 e[H], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    e[i] = x[2 * i];
    o[i] = x[2 * i + 1];
  }
  dft_mixed<H>(e);
  dft_mixed<H>(o);
  static_for<H>([&](auto ki) {
    constexpr int k = decltype(ki)::value;
    y[k] = cadd(e[k], mul_root<k, A>(o[k]));
  });
}

constexpr int bluestein_two_step_threads(int a, int b, int t) {
  return two_step_threads(a > b ? a : b, t);
}

template <int A, int B, int NMIN, int T, int LM>
__device__ __forceinline__ void bluestein_two_step_kernel_run(
    const float2* src, float2* dst, const float2* __restrict__ tw,
    const float2* __restrict__ twp, const PassArgs& a) {
  constexpr int H = A / 2;
  constexpr int pitch = two_step_pitch(B), sq = two_step_stride(A, B);
  __shared__ float2 lds[T * sq];
  const int n = (int)a.res_mask;
  const float2* __restrict__ chirp = twp;
  const float2* __restrict__ filt = twp + n;
  const int tid = threadIdx.x;
  const int64_t tile = tile_index(blockIdx.x, gridDim.x, a.xcd_remap);

  if (tid < T * B) {
    const int q = LM == MODE_ROW ? tid / B : tid % T;
    const int t = LM == MODE_ROW ? tid % B : tid / T;
    // pencils past the end of a ragged last tile read the last pencil
    int64_t b = tile * T + q;
    b = b < a.B ? b : a.B - 1;
    const float2* s =
        src + pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.is0, a.is1, a.is2);
    // points below NMIN exist at every length of this kernel; those above
    // read the pencil's last point and are set to zero
    float2 x[H], c[H];
    const float2* u = s + t * a.ijs;
    const int64_t step = B * a.ijs;
#pragma unroll
    for (int r = 0; r < H; ++r) {
      if ((r + 1) * B <= NMIN) {
        x[r] = u[r * step];
        c[r] = chirp[t + r * B];
      } else {
        const int j = t + r * B < n ? t + r * B : n - 1;
        x[r] = s[j * a.ijs];
        c[r] = chirp[j];
      }
    }
#pragma unroll
    for (int r = 0; r < H; ++r) {
      if (a.conj_in) x[r].y = -x[r].y;
      x[r] = cmul(x[r], c[r]);
      if ((r + 1) * B > NMIN && t + r * B >= n) x[r] = make_float2(0.f, 0.f);
    }
    float2 y[A];
    dft_half_in<A>(x, y);
    float2* w = lds + q * sq + t;
#pragma unroll
    for (int r = 0; r < A; ++r) w[r * pitch] = y[r];
  }
  __syncthreads();  // the table of every pencil is in LDS
  if (tid < T * A) {
    const int q = tid % T, tm = tid / T;
    float2* row = lds + q * sq + tm * pitch;
    int at = tm * B;
    float2 v[B];
    v[0] = row[0];
#pragma unroll
    for (int j = 1; j < B; ++j) v[j] = cmul(row[j], tw[at + j]);
    dft_mixed<B>(v);
    // the filter and the second twiddles are read where they are used (the
    // table offset made opaque): held over a DFT they cost 2 B registers
    // and the CU its second workgroup
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const float2 g = cmul(v[j], filt[at + j]);
      v[j] = make_float2(g.y, g.x);
    }
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
    const float2* w = lds + q * sq + t;
    float2 v[A], y[H];
#pragma unroll
    for (int r = 0; r < A; ++r) v[r] = w[r * pitch];
    dft_half_out<A>(v, y);
    const int64_t b = tile * T + q;
    if (b < a.B) {
      float2* d = dst + pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.os0, a.os1, a.os2);
      d += t * a.oks;
      const int64_t step = B * a.oks;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const int k = t + B * j;
        if ((j + 1) * B <= NMIN || k < n) {
          float2 o = cmul(make_float2(y[j].y, y[j].x), chirp[k]);
          if (a.conj_out) o.y = -o.y;
          d[j * step] = o;
        }
      }
    }
  }
}

template <int A, int B, int NMIN, int T, int LM>
__global__ void __launch_bounds__(bluestein_two_step_threads(A, B, T))
bluestein_two_step_kernel(const PassLaunch la) {
  bluestein_two_step_kernel_run<A, B, NMIN, T, LM>(la.src, la.dst, la.tw, la.twp, la.a);
}

template <int A, int B, int NMIN, int T, int LM>
hipError_t launch_bluestein_two_step(const PassArgs& a, const float2* src, float2* dst,
                                     const float2* tw, const float2* twp, hipStream_t stream) {
  const int64_t blocks = (a.B + T - 1) / T;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  if (a.res_mask < NMIN || 2 * a.res_mask > A * B || a.res_shift != A) return hipErrorInvalidValue;
  hipLaunchKernelGGL((bluestein_two_step_kernel<A, B, NMIN, T, LM>), dim3((unsigned)blocks),
                     dim3(bluestein_two_step_threads(A, B, T)), 0, stream, PassLaunch{src, dst, tw, twp, a});
  return hipGetLastError();
}

template <int A, int B, int NMIN, int T, int LM>
KernelInfo kernel_info_bluestein_two_step(int smode) {
  constexpr int LDS = T * two_step_stride(A, B) * 8;
  constexpr int TH = bluestein_two_step_threads(A, B, T);
  static_assert(A % 2 == 0 && LDS <= 160 * 1024 && TH <= 1024, "tile fits");
  KernelInfo k{A * B, T, LM, smode, 0, TH, LDS, &launch_bluestein_two_step<A, B, NMIN, T, LM>, 0, 0};
  k.bluestein = 1;
  k.two_step = A;
  return k;
}

// The convolution lengths A B: up to 1024 those products (A even, both at
// most 32) whose operations a pencil no longer one undercuts, above it eleven
// whose factors the registers take (A up to 64, of which half is zero or not
// wanted; B, whose DFT runs whole and twice, up to 32).
constexpr int kBluesteinLadder[][2] = {
    {8, 8}, {6, 12}, {8, 10}, {8, 12}, {10, 10}, {12, 9}, {14, 8},
    {12, 10}, {16, 8}, {12, 12}, {16, 10}, {12, 14}, {16, 12}, {10, 20},
    {12, 18}, {16, 14}, {12, 20}, {16, 16}, {24, 12}, {16, 20}, {24, 14},
    {24, 15}, {16, 24}, {20, 20}, {24, 18}, {24, 20}, {16, 32}, {24, 24},
    {24, 25}, {32, 20}, {24, 28}, {24, 30}, {24, 32}, {28, 28}, {28, 30},
    {32, 28}, {32, 30}, {32, 32}, {36, 30}, {48, 24}, {40, 30}, {40, 32},
    {48, 28}, {48, 30}, {48, 32}, {56, 30}, {56, 32}, {60, 32}, {64, 32}};
constexpr int kBluesteinLadderSize = sizeof(kBluesteinLadder) / sizeof(kBluesteinLadder[0]);

// The kernels of ladder entries LO <= i < HI, for every order: lanes along
// the pencil on load (rotating and row passes) or across the pencils (column
// passes), across the pencils on store.
template <int LO, int HI>
void add_bluestein_two_step(std::vector<KernelInfo>& v) {
  if constexpr (HI - LO > 1) {
    add_bluestein_two_step<LO, (LO + HI) / 2>(v);
    add_bluestein_two_step<(LO + HI) / 2, HI>(v);
  } else {
    constexpr int A = kBluesteinLadder[LO][0], B = kBluesteinLadder[LO][1];
    // shorter lengths take the entry before
    constexpr int NMIN =
        LO == 0 ? 1 : kBluesteinLadder[LO ? LO - 1 : 0][0] * kBluesteinLadder[LO ? LO - 1 : 0][1] / 2 + 1;
    constexpr int T = A * B <= 256 ? 16 : A * B <= 1024 ? 8 : 4;
    v.push_back(kernel_info_bluestein_two_step<A, B, NMIN, T, MODE_ROW>(MODE_COL));
    v.push_back(kernel_info_bluestein_two_step<A, B, NMIN, T, MODE_ROW>(MODE_ROW));
    v.push_back(kernel_info_bluestein_two_step<A, B, NMIN, T, MODE_COL>(MODE_COL));
  }
}

}  // namespace dft3d
