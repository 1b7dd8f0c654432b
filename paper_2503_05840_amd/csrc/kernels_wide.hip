// Scores of a bf16 K-cache whose layer the stream kernel of kernels_bf16.hip does not take (more than 32 heads, more
// than 1024 sequences, heads of 8 columns): s[b][h][t] = q_h . K[t, head h] in the log2 domain, fp32 arithmetic.  The
// weighted sum that follows reads K a second time (kernels_xcache.hip, weights in full fp32 precision).
#include "slim_kernels.h"
#include "device_common.h"

namespace slim {
namespace {

// A wave takes 16 rows of 64 / LPHP neighbouring heads (LPHP lanes per head, 8 columns each: up to 1 KB of
// consecutive bytes per row), all 16 loads in flight at once, sums each row over the head's lanes with DPP adds and
// leaves with consecutive rows of a head on the head's lanes.  Bound by HBM: one load, 16 multiply-adds and the
// reduction per 16 bytes and lane are a fifth of what the vector ALU does in the time the bytes take.  (One wave per
// row with per-head sums through LDS, as the plain kernel does it: 67 us for 6503 rows of 5120 columns, 67 MB; this one
// 15.4 us, 4.3 TB/s with the launch.)
constexpr int KS_ROWS = 16, KS_WAVES = 4;

template <int LPHP, bool ROPE>
__global__ __launch_bounds__(KS_WAVES * 64) void kscores_kernel(const float* __restrict__ q, const uint16_t* __restrict__ K,
                                                                long k_bstride, const int32_t* __restrict__ seq_lens, int T,
                                                                int H, int d, int d_k, float scale_log2,
                                                                const float* __restrict__ rope, float* __restrict__ S,
                                                                int* counters, int ncounters) {
  constexpr int HPP = 64 / LPHP;                        // heads per wave
  const int npiece = (H + HPP - 1) / HPP;
  const int rb = blockIdx.x / npiece, piece = blockIdx.x - rb * npiece, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // (the arrival counters of the projection that ends this call start at 0)
  if (blockIdx.x == 0 && b == 0)
    for (int i = tid; i < ncounters; i += KS_WAVES * 64) counters[i] = 0;
  const int len = seq_len_of(seq_lens, b, T);
  const int r0 = (rb * KS_WAVES + w) * KS_ROWS;
  if (r0 >= len) return;
  const int hl = lane / LPHP, li = lane % LPHP;
  const int h = piece * HPP + hl;
  const bool live = h < H, act = live && li * 8 < d_k;
  const int col = act ? h * d_k + li * 8 : 0;           // (idle lanes read the row's first columns against a zero query)
  const char* Kb = reinterpret_cast<const char*>(K + (size_t)b * k_bstride + col);
  u32x4 kr[KS_ROWS];
#pragma unroll
  for (int j = 0; j < KS_ROWS; ++j)
    kr[j] = *reinterpret_cast<const u32x4*>(Kb + (size_t)min(r0 + j, len - 1) * ((size_t)d * 2));
  float qv[8];
  {
    const f32x4* src = reinterpret_cast<const f32x4*>(q + (size_t)b * d + col);
    const f32x4 x0 = src[0], x1 = src[1];
#pragma unroll
    for (int c = 0; c < 8; ++c) qv[c] = act ? (c < 4 ? x0[c] : x1[c - 4]) * scale_log2 : 0.f;
  }
  float s[KS_ROWS];
#pragma unroll
  for (int j = 0; j < KS_ROWS; ++j) {
    float cs[8];
    if constexpr (ROPE) {
      const f32x4* rp = reinterpret_cast<const f32x4*>(rope + (size_t)min(r0 + j, len - 1) * d_k + (act ? li * 8 : 0));
      const f32x4 y0 = rp[0], y1 = rp[1];
#pragma unroll
      for (int c = 0; c < 8; ++c) cs[c] = c < 4 ? y0[c] : y1[c - 4];
    }
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const unsigned kw = kr[j][c];
      const float x1 = __uint_as_float(kw << 16), x2 = __uint_as_float(kw & 0xffff0000u);
      if constexpr (ROPE) {
        // with (y1, y2) = (x1 c + x2 s, -x1 s + x2 c):  q1 y1 + q2 y2 = c (q1 x1 + q2 x2) + s (q1 x2 - q2 x1)
        v = fmaf(cs[2 * c], fmaf(qv[2 * c], x1, qv[2 * c + 1] * x2), v);
        v = fmaf(cs[2 * c + 1], fmaf(qv[2 * c], x2, -qv[2 * c + 1] * x1), v);
      } else {
        v = fmaf(qv[2 * c], x1, v);
        v = fmaf(qv[2 * c + 1], x2, v);
      }
    }
    if constexpr (LPHP > 1) v = dpp_add<0xB1>(v);       // lane ^ 1
    if constexpr (LPHP > 2) v = dpp_add<0x4E>(v);       // lane ^ 2
    if constexpr (LPHP > 4) v = dpp_add<0x141>(v);      // other quad of the 8-lane half
    if constexpr (LPHP > 8) v = dpp_add<0x140>(v);      // other half of the 16-lane row
    s[j] = v;
  }
  const int Tp = (T + 31) / 32 * 32;
  float* dst = S + ((size_t)b * H + (live ? h : 0)) * Tp + r0 + li;
#pragma unroll
  for (int g = 0; g < KS_ROWS; g += LPHP) {             // lane li of a head stores row g + li
    float v = s[g];
#pragma unroll
    for (int j = 1; j < LPHP; ++j) v = li == j ? s[g + j] : v;
    if (live && r0 + g + li < len) dst[g] = v;
  }
}

}  // namespace

// Whole 128-column blocks for the weighted sum, heads of whole 16-byte pieces up to 128 columns, and a sequence's
// rows within 32-bit byte offsets.  (Rows that end inside a block take the plain kernels, at three times the time:
// 1 x 2000 rows x 36 heads x 80 = 2880 columns 108 us.  The weighted sum has no masked column block.)
bool wide_ok(int dtype, int T, int d, int d_k) {
  return dtype == DT_BF16 && d % 128 == 0 && d < (1 << 22) && d_k % 8 == 0 && d_k <= 128 && T < (1 << 24) &&
         (size_t)T * d * 2 < ((size_t)1 << 32);
}

void launch_kscores(const float* q, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int d_k,
                    float scale_log2, const float* rope, float* S, int* counters, int ncounters, int B, hipStream_t st) {
  int lphp = 1;
  while (lphp < d_k / 8) lphp <<= 1;
  const int npiece = (H + 64 / lphp - 1) / (64 / lphp), nrb = (T + KS_WAVES * KS_ROWS - 1) / (KS_WAVES * KS_ROWS);
  dim3 grid((unsigned)npiece * nrb, B);
  auto go = [&](auto lp, auto rp) {
    hipLaunchKernelGGL((kscores_kernel<decltype(lp)::value, decltype(rp)::value>), grid, dim3(KS_WAVES * 64), 0, st, q,
                       (const uint16_t*)K, k_bstride, seq_lens, T, H, d, d_k, scale_log2, rope, S, counters, ncounters);
  };
  auto with_rope = [&](auto lp) {
    if (rope) go(lp, std::true_type{});
    else go(lp, std::false_type{});
  };
  switch (lphp) {
    case 1: with_rope(std::integral_constant<int, 1>{}); break;
    case 2: with_rope(std::integral_constant<int, 2>{}); break;
    case 4: with_rope(std::integral_constant<int, 4>{}); break;
    case 8: with_rope(std::integral_constant<int, 8>{}); break;
    default: with_rope(std::integral_constant<int, 16>{}); break;
  }
}

}  // namespace slim
