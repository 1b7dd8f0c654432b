// Device helpers shared by the kernel files (kernels_bf16.hip, kernels_xcache.hip, kernels_xfused.hip, kernels_f32.hip,
// kernels_generic.hip): vector types, the clamped sequence length, a barrier for LDS exchanges, the in-register 8 x 8 transposition that turns a lane's block of a
// row-major tile into MFMA operands, and loop helpers whose register buffers are picked at compile time.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

namespace slim {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr float NEG_INF = -INFINITY;

__device__ __forceinline__ int seq_len_of(const int32_t* lens, int b, int T) {
  if (!lens) return T;
  const int n = lens[b];
  return n < 0 ? 0 : (n > T ? T : n);
}

// Partials that a later launch reads, stored through the L2s to the memory side: what is left dirty there is written back between the
// launches, and the next one starts that much later (4 us after 9 MB).  For instructions that store runs of 256 bytes and more (they need not
// begin or end with a line: fp32 rows of 40 columns, units of heads of 80): pieces of 16 bytes took 12 % longer, and the partials of the
// by-sequence stream and of the wide path's weighted sum, which leave while others still stream or in such pieces, 1-3 %.  (The s_nops: a store of more than 64 bits still reads its data registers in the wait states after it issues, and the compiler,
// which pads its own stores, is free to overwrite the inputs of an asm statement with the very next vector instruction.)
__device__ __forceinline__ void store_through(float* p, f32x4 v) {
  asm volatile("s_nop 1\n\tglobal_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

// Workgroup barrier for data exchanged through LDS only: waits for this wave's LDS operations, not for its
// global loads (__syncthreads() would also drain the tiles that are being prefetched from HBM).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// v + (v of the lane selected by a DPP control inside the 16-lane row); one v_add_f32_dpp
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// max over the 32 lanes that share lane / 32: four DPP steps inside the 16-lane row (lane ^ 1, lane ^ 2,
// the other quad of the 8-lane half, the other half of the row), then the row 16 lanes away by a register swap
template <int CTRL>
__device__ __forceinline__ float dpp_max(float v) {
  return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ float max_over_32(float v) {
  v = dpp_max<0xB1>(v);
  v = dpp_max<0x4E>(v);
  v = dpp_max<0x141>(v);
  v = dpp_max<0x140>(v);
  const unsigned u = __float_as_uint(v);
  const auto sw = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// sum over the 32 lanes that share lane / 32, the same bits as a __shfl_xor butterfly from 1 to 16
__device__ __forceinline__ float sum_over_32(float v) {
  v = dpp_add<0xB1>(v);
  v = dpp_add<0x4E>(v);
  v = dpp_add<0x141>(v);
  v = dpp_add<0x140>(v);
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// max / sum over the whole wave, the same in every lane: DPP inside the 16-lane rows, register swaps across them (a
// __shfl_xor butterfly goes through LDS six times, a tenth of a microsecond each)
__device__ __forceinline__ float max_over_wave(float v) {
  v = max_over_32(v);
  const unsigned u = __float_as_uint(v);
  const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}
__device__ __forceinline__ float sum_over_wave(float v) {
  v = dpp_add<0xB1>(v);
  v = dpp_add<0x4E>(v);
  v = dpp_add<0x141>(v);
  v = dpp_add<0x140>(v);
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned w = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// v of the lanes up to and including this one added up: inside the 16-lane rows, then row by row.  By shuffles through LDS it took 0.2 to
// 0.4 us of a launch, all six steps (1 x 200 rows x 32 heads x 128 19.9 us, now 19.6) or as a loop over the steps that there are sequences for
// (165 x 92 x 4 x 64 16.0 us and six steps 15.65, now 15.3; 64 x 448 x 6 x 64 22.2 and 21.95, now 21.5).
__device__ __forceinline__ int prefix_over_wave(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);     // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);     // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);     // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15: rows 0 and 2 into 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31: rows 0 and 1 into 2 and 3
  return v;
}

// The lane, made where it is asked for: the compiler cannot keep it, or what follows from it, through the stream.
__device__ __forceinline__ int fresh_lane() {
  int ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  return ln;
}

// v of the lanes l, l^16, l^32, l^48 added up, the same in all four and the same bits as a __shfl_xor butterfly over 16 and 32: each
// sum has the same two terms
__device__ __forceinline__ float sum_over_row_groups(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned w = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// 8 rows x 8 bf16 columns per lane  ->  8 operands (one per column), each 8 rows of that column.
__device__ __forceinline__ void transpose8x8(const u32x4 (&kt)[8], u32x4 (&a)[8]) {
#pragma unroll
  for (int jp = 0; jp < 4; ++jp) {
    const u32x4 lo = kt[2 * jp], hi = kt[2 * jp + 1];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      a[2 * c][jp] = __builtin_amdgcn_perm(hi[c], lo[c], 0x05040100u);      // even column: low halves
      a[2 * c + 1][jp] = __builtin_amdgcn_perm(hi[c], lo[c], 0x07060302u);  // odd column: high halves
    }
  }
}

// Workgroup i of a one-dimensional launch -> (unit, inner): a unit is a set of `ninner` workgroups that read
// the same data (a sequence's q~ or scores, the same rows of X).  Workgroups are dealt to the 8 XCDs round
// robin, each with an L2 of its own, so with `colocate` a unit's workgroups are the ones with the same
// i % 8 and consecutive i / 8: what they share is fetched into one L2 instead of up to eight.  (Where the
// dealing differs the mapping is still a bijection: only the sharing is lost.)  False: no such unit.
__device__ __forceinline__ bool unit_of_workgroup(int i, int ninner, int nunits, bool colocate, int& unit, int& inner) {
  if (colocate) {
    const int slot = i >> 3;
    unit = (slot / ninner) * 8 + (i & 7);
    inner = slot % ninner;
  } else {
    unit = i / ninner;
    inner = i % ninner;
  }
  return unit < nunits;
}

// f(k + I, integral_constant<I>) for I = 0 .. N-1 while k + I < end: loop bodies whose register
// buffers are chosen by a compile-time index.
template <int I, int N, class F>
__device__ __forceinline__ void unrolled_steps(int k, int end, F& f) {
  if constexpr (I < N) {
    if (k + I < end) f(k + I, std::integral_constant<int, I>{});
    unrolled_steps<I + 1, N>(k, end, f);
  }
}

// The same without the bound checks, for whole groups of N steps (straight-line code: the compiler can
// then count the loads in flight across steps).
template <int I, int N, class F>
__device__ __forceinline__ void full_steps(int k, F& f) {
  if constexpr (I < N) {
    f(k + I, std::integral_constant<int, I>{});
    full_steps<I + 1, N>(k, f);
  }
}

}  // namespace slim
