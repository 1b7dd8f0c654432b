// fp32 K-cache, rows of up to 1024 columns and up to 32 heads (gfx950): scores, softmax numerators and
// the full-width weighted sum of one (sequence, context split) in one kernel, K read from memory once;
// everything in fp32, the contraction P^T K on v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// What bounds it: latency.  The caches of this range are a few MB, so what counts is how few dependent
// round trips lie between the launch and the partial's stores, and that every compute unit takes part.
// A workgroup therefore keeps its H x d accumulators in registers for its whole row range (64 KB at 16 x
// 1024), takes 32 rows per step, and the context is cut into as many splits as there are tiles or compute
// units.  Before (scores written out by one kernel, a vector-ALU weighted sum of 2 columns per thread that
// filled 2 to 24 workgroups): 49.8 us at 1 x 256 rows x 512 columns and 80.6 us at 4 ragged sequences of
// 300..1500 rows x 1024 columns; this kernel takes 6.0 and 13.8 us there.
#include "slim_kernels.h"
#include "device_common.h"

namespace slim {
namespace {

constexpr int FS_ROWS = 32;              // rows per step
constexpr int FS_PP = 17;                // floats per row of the numerators (16 heads + 1: no bank conflicts)

__host__ __device__ inline int fs_pitch(int d) { return (d + 63) / 64 * 64 + 4; }     // floats per parked row
__host__ __device__ inline int fs_part_pitch(int d) { return d / 16 + 1; }            // floats per row of partial dots

// CI: 256-column pieces of a row (a wave loads a row in CI instructions of 16 bytes per lane); a wave owns
// (CI + 1) / 2 blocks of 64 columns in the weighted sum.  NT: head tiles of 16.
//   1. wave w holds rows 4 w .. 4 w + 3 of the tile in registers: dot products with the query (in registers as
//      well) per lane, summed over four lanes = 16 columns, to LDS; the rows to LDS; the next tile requested
//   2. lane (row, half) of wave w adds up the pieces of head 2 w + half (+ 16), numerators against the head's
//      running maximum, rescale factors
//   3. MFMA: M = columns (lane idx holds columns 4 idx .. +3 of a 64-column block, one MFMA per column of the
//      four), N = heads, K = 4 rows per instruction
// (CI = 4 with two head tiles and rotary keys does not fit 256 registers: 52 bytes of scratch per lane.)
template <int CI, int NT, bool ROPE>
__global__ __launch_bounds__(512) void f32_stream_kernel(const float* __restrict__ q, const float* __restrict__ K, long k_bstride,
                                                         const int32_t* __restrict__ seq_lens, int T, int H, int d, int d_k,
                                                         int nsplit, float scale, const float* __restrict__ rope,
                                                         float* __restrict__ Cpart, float* __restrict__ mpart,
                                                         float* __restrict__ lpart, int* counters, int ncounters) {
  constexpr int CB = (CI + 1) / 2;
  extern __shared__ __align__(16) float smem[];
  __shared__ float P_s[NT][FS_ROWS][FS_PP];
  __shared__ float alpha_s[NT * 16];
  const int s = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int idx = lane & 15, kg = lane >> 4;
  // (the arrival counters of the projection that follows start at 0)
  if (s == 0 && b == 0)
    for (int i = tid; i < ncounters; i += 512) counters[i] = 0;
  const int pitch = fs_pitch(d), pp = fs_part_pitch(d);
  float* const tile = smem;                            // [FS_ROWS][pitch]
  float* const part = smem + FS_ROWS * pitch;          // [FS_ROWS][pp]
  const int len = seq_len_of(seq_lens, b, T);
  const int per = f32_rows_per_split(len, nsplit);
  const int r_lo = s * per, r_hi = min(len, r_lo + per);
  if (r_lo >= r_hi) return;                            // (the merge knows which splits of a sequence exist)
  const int ntile = (r_hi - r_lo + FS_ROWS - 1) / FS_ROWS;

  const float* Kb = K + (size_t)b * k_bstride;
  f32x4 kr[4][CI], rr[ROPE ? 4 : 1][ROPE ? CI : 1], qv[CI];
  bool act[CI];
  int ropecol[CI];
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    const int c = (i * 64 + lane) * 4;
    act[i] = c < d;
    ropecol[i] = act[i] ? c % d_k : 0;                 // (cos, sin pairs: two floats per two columns)
  }
  // (rows past the end re-read the last row and get no weight; lanes past the row re-read its first columns)
  auto load = [&](int k) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = min(r_lo + k * FS_ROWS + w * 4 + j, r_hi - 1);
      const float* src = Kb + (size_t)row * d;
#pragma unroll
      for (int i = 0; i < CI; ++i) {
        kr[j][i] = *reinterpret_cast<const f32x4*>(src + (act[i] ? (i * 64 + lane) * 4 : 0));
        if constexpr (ROPE) rr[j][i] = *reinterpret_cast<const f32x4*>(rope + (size_t)row * d_k + ropecol[i]);
      }
    }
  };
  load(0);
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    qv[i] = *reinterpret_cast<const f32x4*>(q + (size_t)b * d + (act[i] ? (i * 64 + lane) * 4 : 0));
    qv[i] *= scale;
  }

  f32x4 acc[CB][NT][4];
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[i][t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int row = lane & 31, half = lane >> 5;         // step 2: this lane's row and head of the pair
  const int npk = d_k / 16;                            // pieces of 16 columns per head
  float m[NT], l[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) { m[t] = NEG_INF; l[t] = 0.f; }

  for (int k = 0; k < ntile; ++k) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < CI; ++i) {
        const f32x4 kv = kr[j][i];
        float p;
        if constexpr (ROPE) {
          // with (y1, y2) = (x1 c + x2 s, -x1 s + x2 c):  q1 y1 + q2 y2 = c (q1 x1 + q2 x2) + s (q1 x2 - q2 x1)
          const f32x4 cs = rr[j][i], qq = qv[i];
          p = cs[0] * fmaf(qq[0], kv[0], qq[1] * kv[1]);
          p = fmaf(cs[1], fmaf(qq[0], kv[1], -qq[1] * kv[0]), p);
          p = fmaf(cs[2], fmaf(qq[2], kv[2], qq[3] * kv[3]), p);
          p = fmaf(cs[3], fmaf(qq[2], kv[3], -qq[3] * kv[2]), p);
        } else {
          p = fmaf(kv[3], qv[i][3], fmaf(kv[2], qv[i][2], fmaf(kv[1], qv[i][1], kv[0] * qv[i][0])));
        }
        p = dpp_add<0xB1>(p);                          // lane ^ 1
        p = dpp_add<0x4E>(p);                          // lane ^ 2
        if (act[i]) {
          if ((lane & 3) == 0) part[(w * 4 + j) * pp + i * 16 + (lane >> 2)] = p;
          *reinterpret_cast<f32x4*>(tile + (size_t)(w * 4 + j) * pitch + (i * 64 + lane) * 4) =
              r_lo + k * FS_ROWS + w * 4 + j < r_hi ? kv : f32x4{0.f, 0.f, 0.f, 0.f};     // (0 x what a repeated row holds may be no 0)
        }
      }
    if (k + 1 < ntile) load(k + 1);
    lds_barrier();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int h = t * 16 + 2 * w + half;
      float sc = NEG_INF;
      if (h < H && r_lo + k * FS_ROWS + row < r_hi) {
        sc = 0.f;
#pragma unroll 4
        for (int j = 0; j < npk; ++j) sc += part[row * pp + h * npk + j];
      }
      const float mn = fmaxf(m[t], max_over_32(sc));
      const float ref = (mn == NEG_INF) ? 0.f : mn;
      const float alpha = __expf(m[t] - ref);          // 0 the first time
      const float pw = __expf(sc - ref);
      l[t] = fmaf(l[t], alpha, pw);
      m[t] = mn;
      P_s[t][row][2 * w + half] = pw;
      if (row == 0) alpha_s[t * 16 + 2 * w + half] = alpha;
    }
    lds_barrier();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float al = alpha_s[t * 16 + idx];
      if (k > 0 && __any(al != 1.f)) {
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[i][t][c] *= al;
      }
    }
#pragma unroll
    for (int ks = 0; ks < FS_ROWS / 4; ++ks) {
      float pv[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) pv[t] = P_s[t][ks * 4 + kg][idx];
#pragma unroll
      for (int i = 0; i < CB; ++i) {
        const int c0 = (w + 8 * i) * 64;
        if (c0 < d) {                                  // (wave-uniform; columns past d inside the block: never stored)
          const f32x4 kv = *reinterpret_cast<const f32x4*>(tile + (size_t)(ks * 4 + kg) * pitch + c0 + idx * 4);
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[i][t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[c], pv[t], acc[i][t][c], 0, 0, 0);
        }
      }
    }
    if (k + 1 < ntile) lds_barrier();                  // the tile and the numerators are overwritten next
  }

  // The partial leaves by way of the idle tile, a wave's 16 heads x 64 columns at a time, so that a head's 256 bytes lie on sixteen
  // neighbouring lanes, and through the L2s (store_through).  Straight from the accumulators an instruction stored 64 pieces of 16 bytes,
  // and what the L2s held was written back before the merge could start: 4 x 300..1500 rows x 1024 columns 23.2 -> 20.6 us, 8 x 100..1000
  // 26.4 -> 22.0, 32 x 500 36.8 -> 31.2; by way of the tile alone 20.9, 22.5 and 31.9.
  constexpr int OP = 64 + 4;                           // floats per head (padding: no bank conflicts)
  float* const ob = smem + w * (16 * OP);              // (a wave with columns has 64 floats of 32 rows there)
  lds_barrier();                                       // (the other waves have read the tile)
  const size_t pid = (size_t)b * nsplit + s;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int c0 = (w + 8 * i) * 64;
      if (c0 >= d) continue;                           // (wave-uniform)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(ob + idx * OP + (kg * 4 + r) * 4) = f32x4{acc[i][t][0][r], acc[i][t][1][r], acc[i][t][2][r], acc[i][t][3][r]};
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (LDS operations of one wave complete in order)
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) {
        const int hl = 4 * k2 + kg, h = t * 16 + hl, c = c0 + idx * 4;
        const f32x4 v = *reinterpret_cast<const f32x4*>(ob + hl * OP + idx * 4);
        if (h < H && c < d) store_through(Cpart + (pid * H + h) * d + c, v);
      }
    }
    const float lt = sum_over_32(l[t]);
    const int h2 = t * 16 + 2 * w + half;
    if (row == 0 && h2 < H) {
      mpart[pid * H + h2] = m[t];
      lpart[pid * H + h2] = lt;
    }
  }
}

}  // namespace

// Rows of up to 1024 columns (the tile and its partial dots fill 148 of the 160 KB of LDS there), whole pieces
// of 16 columns per head, at most two head tiles (32 heads: 128 accumulator registers).
bool f32_stream_ok(int dtype, int H, int d, int d_k) { return dtype == DT_F32 && d <= 1024 && d_k % 16 == 0 && H <= 32; }

// One split per 32 rows until every compute unit has one, at most what one wave of the merge looks after: a split
// costs a partial of H x d floats, but a compute unit without rows costs more (141 of 188 workgroups with rows at 4
// ragged sequences: 13.8 us, the whole step 26.5 us against 128.7 with at most 12 splits and the separate kernels).
int f32_stream_splits(int B, int T) {
  int s = (T + FS_ROWS - 1) / FS_ROWS;
  const int fill = (256 + B - 1) / B;
  if (s > fill) s = fill;
  if (s > MERGE_MAX_SPLITS) s = MERGE_MAX_SPLITS;
  return s < 1 ? 1 : s;
}

void launch_f32_stream(const float* q, const float* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int d_k,
                       int nsplit, float scale, const float* rope, float* Cpart, float* mpart, float* lpart, int* counters,
                       int ncounters, int B, hipStream_t st) {
  const size_t smem = sizeof(float) * FS_ROWS * (size_t)(fs_pitch(d) + fs_part_pitch(d));
  auto go = [&](auto ci, auto nt, auto rp) {
    auto* kern = f32_stream_kernel<decltype(ci)::value, decltype(nt)::value, decltype(rp)::value>;
    if (smem > 65536) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    hipLaunchKernelGGL(kern, dim3(nsplit, B), dim3(512), smem, st, q, K, k_bstride, seq_lens, T, H, d, d_k, nsplit, scale, rope,
                       Cpart, mpart, lpart, counters, ncounters);
  };
  auto with_nt = [&](auto ci) {
    auto with_rope = [&](auto nt) {
      if (rope) go(ci, nt, std::true_type{});
      else go(ci, nt, std::false_type{});
    };
    if (H <= 16) with_rope(std::integral_constant<int, 1>{});
    else with_rope(std::integral_constant<int, 2>{});
  };
  if (d <= 256) with_nt(std::integral_constant<int, 1>{});
  else if (d <= 512) with_nt(std::integral_constant<int, 2>{});
  else if (d <= 768) with_nt(std::integral_constant<int, 3>{});
  else with_nt(std::integral_constant<int, 4>{});
}

}  // namespace slim
