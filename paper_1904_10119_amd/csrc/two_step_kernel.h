// Mixed-radix passes in two register steps: a length n = A B with A <= B,
// both free of prime factors above 13, is transformed with one exchange
// through LDS (the four-step identity of eq. (3) with the whole inner DFTs
// in registers).
//
// Step 1: butterfly t (t < B) of a pencil reads its points t + r B (r < A)
// straight from global memory, transforms them with DFT_A and leaves output
// r at row r, column t of the pencil's A x B table in LDS.  Step 2:
// butterfly tm (tm < A) reads row tm, multiplies entry j by w_n^{tm j},
// transforms with DFT_B and stores output j as point k = tm + A j straight
// to global memory.  Against the staged pass (mixed_kernel.h: an LDS round
// trip and two barriers a radix) every point crosses LDS once and each
// thread has its A loads in flight together.
//
// The butterflies of a tile of T pencils are numbered through, one of step 1
// and at most one of step 2 a thread.  ROW orders run lanes along the pencil (t, tm
// fastest), COL orders across the pencils.  LDS rows have an odd pitch and
// pencils an odd stride in 8-byte units, so neither order has bank
// conflicts beyond the 2-way split of a 64-lane 8-byte access.
//
// What bounds it: memory from about 10^7 points up (57 VALU instructions a
// point at n = 375, half of what the card issues at the copy rate), launch and
// load latency below.  The tile is 16 pencils so that a COL row segment is
// one 128-byte line: 400^3 takes 603 us so, 762 us in tiles of 8 pencils
// (64-byte segments) and 629 us in tiles of 32 (fewer workgroups a CU);
// two_step_tile says where 8 are taken, two_step_wide_tile and
// two_step_misaligned_tile where more than 16.
// Against the staged pass (same orders, MI355X): 96^3 25.0 -> 17.9 us, 90^3
// 30.4 -> 18.7, 150^3 62.9 -> 32.6, 252^3 209 -> 141 (5.4 TB/s a pass),
// 324^3 462 -> 326, 540^3 2370 -> 1481, 900^3 10.3 -> 8.6 ms, 640^3 2.95 ->
// 2.75 ms, 1050 x 1050 x 64 847 -> 710 us, 1078 x 1078 x 64 1088 -> 777, 1536 x
// 1536 x 64 2501 -> 1697; no faster at 1000^3 in the rotation's order (11.4 / 11.5 ms; 10.1
// in the cycle, against 10.3).  A kernel for any length with a radix switch
// took 177 us at 250^3 where the compiled lengths take 142: it holds the
// registers of the largest radix (120 against 93).
//
// PassArgs fields used: pencil fields and element strides as for every
// pass, res_mask = n, twp_mask = the length's radix code (as the staged
// pass), res_shift = A.  Table: tw[tm B + j] = w_n^{tm j}, from FP64.
#pragma once

#include "mixed_kernel.h"

namespace dft3d {

__host__ __device__ constexpr int two_step_pitch(int b) { return b | 1; }
__host__ __device__ constexpr int two_step_stride(int a, int b) {
  return (a * two_step_pitch(b)) | 1;
}

// FORM bits of a two-step kernel: kRoots reads w_n^{tm j} from a table of the
// roots of length n at tm j (the power-of-two passes, whose tables the other
// power-of-two kernels share); kMove leaves the DFTs and twiddles out (the
// move-only option).
constexpr int kRoots = 1, kMove = 2;

// Step 1 of radix R over the tile: B butterflies a pencil, one a thread.
template <int R, int B, int T, int LM, int FORM>
__device__ __forceinline__ void two_step_first(const float2* src, const PassArgs& a,
                                               int64_t tile, float2* lds, int tid) {
  constexpr int pitch = two_step_pitch(B), sq = two_step_stride(R, B);
  if (tid >= T * B) return;
  const int q = LM == MODE_ROW ? tid / B : tid % T;
  const int t = LM == MODE_ROW ? tid % B : tid / T;
  // pencils past the end of a ragged last tile read the last pencil
  int64_t b = tile * T + q;
  b = b < a.B ? b : a.B - 1;
  const float2* s = src + pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.is0, a.is1, a.is2);
  float2 v[R];
  if constexpr (LM == MODE_ROW) {
    s += t;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[r * B];
  } else {
    s += t * a.ijs;
    const int64_t step = B * a.ijs;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[r * step];
  }
  if (a.conj_in) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r].y = -v[r].y;
  }
  if constexpr (!(FORM & kMove)) dft_mixed<R>(v);
  float2* w = lds + q * sq + t;
#pragma unroll
  for (int r = 0; r < R; ++r) w[r * pitch] = v[r];
}

// Step 2 of radix R over the tile (A butterflies a pencil, one a thread) and
// the store.  The twiddles are read before the barrier that ends step 1
// where they fit in registers beside the data.
template <int A, int R, int T, int SM, int FORM>
__device__ __forceinline__ void two_step_second(float2* dst, const float2* __restrict__ tw,
                                                const PassArgs& a, int64_t tile,
                                                const float2* lds, int tid) {
  constexpr bool MV = (FORM & kMove) != 0, EARLY = R <= 16 && !MV;
  constexpr int pitch = two_step_pitch(R), sq = two_step_stride(A, R);
  const int q = SM == MODE_ROW ? tid / A : tid % T;
  const int tm = SM == MODE_ROW ? tid % A : tid / T;
  float2 w[R];
  auto twiddles = [&] {
#pragma unroll
    for (int j = 1; j < R; ++j) w[j] = tw[(FORM & kRoots) ? tm * j : tm * R + j];
  };
  if constexpr (EARLY) {
    if (tid < T * A) twiddles();
  }
  __syncthreads();  // every output of step 1 is in LDS
  if (tid >= T * A) return;
  if constexpr (!EARLY && !MV) twiddles();
  const float2* row = lds + q * sq + tm * pitch;
  float2 v[R];
  v[0] = row[0];
#pragma unroll
  for (int j = 1; j < R; ++j) v[j] = MV ? row[j] : cmul(row[j], w[j]);
  if constexpr (!MV) dft_mixed<R>(v);
  if (a.conj_out) {
#pragma unroll
    for (int j = 0; j < R; ++j) v[j].y = -v[j].y;
  }
  const int64_t b = tile * T + q;
  if (b < a.B) {
    float2* d = dst + pencil_offset_any(b, a.m0, a.m1, a.s0, a.s1, a.os0, a.os1, a.os2);
    if constexpr (SM == MODE_ROW) {
      d += tm;
#pragma unroll
      for (int j = 0; j < R; ++j) d[j * A] = v[j];
    } else {
      d += tm * a.oks;
      const int64_t step = A * a.oks;
#pragma unroll
      for (int j = 0; j < R; ++j) d[j * step] = v[j];
    }
  }
}

// One workgroup per tile of T pencils; the length A * B, the tile and the
// orders are compile-time constants (sizes and LDS offsets fold, no radix
// switch, and each length has its own register count).
template <int A, int B, int T, int TH, int LM, int SM, int FORM>
__device__ __forceinline__ void fft_two_step_kernel_run(
    const float2* src, float2* dst, const float2* __restrict__ tw,
    const float2* __restrict__ twp, const PassArgs& a) {
  __shared__ float2 lds[T * two_step_stride(A, B)];
  const int tid = threadIdx.x;
  const int64_t tile = tile_index(blockIdx.x, gridDim.x, a.xcd_remap);
  two_step_first<A, B, T, LM, FORM>(src, a, tile, lds, tid);
  two_step_second<A, B, T, SM, FORM>(dst, tw, a, tile, lds, tid);
}

template <int A, int B, int T, int TH, int LM, int SM, int FORM>
__global__ void __launch_bounds__(TH)
fft_two_step_kernel(const PassLaunch la) {
  fft_two_step_kernel_run<A, B, T, TH, LM, SM, FORM>(la.src, la.dst, la.tw, la.twp, la.a);
}

// Threads of a two-step workgroup: a butterfly of step 1 for each (at most
// 16 x 64 = 1024).
constexpr int two_step_threads(int b, int t) { return (t * b + 63) / 64 * 64; }

template <int A, int B, int T, int LM, int SM, int FORM>
hipError_t launch_two_step(const PassArgs& a, const float2* src, float2* dst, const float2* tw,
                           const float2* twp, hipStream_t stream) {
  const int64_t blocks = (a.B + T - 1) / T;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  if (FORM == 0 && (a.res_shift != A || a.res_mask != A * B)) return hipErrorInvalidValue;
  constexpr int TH = two_step_threads(B, T);
  hipLaunchKernelGGL((fft_two_step_kernel<A, B, T, TH, LM, SM, FORM>), dim3((unsigned)blocks),
                     dim3(TH), 0, stream, PassLaunch{src, dst, tw, twp, a});
  return hipGetLastError();
}

template <int A, int B, int T, int LM, int SM>
KernelInfo kernel_info_two_step() {
  constexpr int LDS = T * two_step_stride(A, B) * 8, TH = two_step_threads(B, T);
  static_assert(LDS <= 160 * 1024 && TH <= 1024, "tile fits");
  // n: a length bound above the kernel's length, as for the staged kernels
  KernelInfo k{A * B + 1, T, LM, SM, 0, TH, LDS, &launch_two_step<A, B, T, LM, SM, 0>, 0, 0};
  k.mixed = mixed_variant(mixed_radix_code(A * B));
  k.two_step = A;
  k.fixed_n = A * B;
  return k;
}

// The same kernel as an FP32 pass of a power of two (roots table), with its
// move-only form; registry.cpp says where it is taken and what it measured.
template <int N, int T, int LM, int SM>
void add_two_step_power(std::vector<KernelInfo>& v) {
  constexpr int A = two_step_split(N), B = N / A;
  KernelInfo k{N, T, LM, SM, 0, two_step_threads(B, T), T * two_step_stride(A, B) * 8,
               &launch_two_step<A, B, T, LM, SM, kRoots>, 0, 0};
  k.two_step = A;
  k.r0 = A;
  k.r1 = B;
  k.r2 = 1;
  v.push_back(k);
  k.launch = &launch_two_step<A, B, T, LM, SM, kRoots | kMove>;
  k.move_only = 1;
  v.push_back(k);
}
template <int N, int T>
void add_two_step_powers(std::vector<KernelInfo>& v) {
  add_two_step_power<N, T, MODE_ROW, MODE_COL>(v);
  add_two_step_power<N, T, MODE_ROW, MODE_ROW>(v);
  add_two_step_power<N, T, MODE_COL, MODE_COL>(v);
}

template <int A, int B, int T>
void add_two_step_modes(std::vector<KernelInfo>& v) {
  v.push_back(kernel_info_two_step<A, B, T, MODE_ROW, MODE_COL>());
  v.push_back(kernel_info_two_step<A, B, T, MODE_ROW, MODE_ROW>());
  v.push_back(kernel_info_two_step<A, B, T, MODE_COL, MODE_COL>());
}

// The kernels of the lengths LO <= n < HI that split, for every order, in the
// tiles find_two_step_kernel picks from.
template <int LO, int HI>
void add_two_step_kernels(std::vector<KernelInfo>& v) {
  if constexpr (HI - LO > 1) {
    add_two_step_kernels<LO, (LO + HI) / 2>(v);
    add_two_step_kernels<(LO + HI) / 2, HI>(v);
  } else if constexpr (two_step_split(LO) > 0) {
    constexpr int A = two_step_split(LO), B = LO / A, T = two_step_tile(LO);
    add_two_step_modes<A, B, T>(v);
    if constexpr (T == 16 && two_step_idle_tiles(LO) > 0) add_two_step_modes<A, B, 8>(v);
    // the wide tiles of the smallest and of the largest grids that have one
    constexpr int W0 = two_step_wide_tile(LO, kTwoStepWidePencils);
    constexpr int W1 = two_step_wide_tile(LO, int64_t(1) << 40);
    if constexpr (W0 > 0) add_two_step_modes<A, B, W0>(v);
    if constexpr (W1 != W0) add_two_step_modes<A, B, W1>(v);
    constexpr int M0 = two_step_misaligned_tile(LO, kTwoStepMisalignedPencils);
    constexpr int M1 = two_step_misaligned_tile(LO, int64_t(1) << 40);
    if constexpr (M0 > 0) v.push_back(kernel_info_two_step<A, B, M0, MODE_ROW, MODE_COL>());
    if constexpr (M1 != M0) v.push_back(kernel_info_two_step<A, B, M1, MODE_ROW, MODE_COL>());
  }
}

}  // namespace dft3d
