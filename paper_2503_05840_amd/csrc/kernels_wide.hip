// bf16 K-caches whose layer the stream kernel of kernels_bf16.hip does not take (more than 32 heads, more than 1024
// sequences, heads of 8 columns), in two passes over K:
//   kscores_kernel   : scores q_h . K[t, head h] in the log2 domain, fp32 arithmetic, and from them the softmax numerators
//                      against the maximum of each 64-row block, with the maxima and the sums of every block
//   kweighted_kernel : per context split the weighted sum of the rows, weights in full fp32 precision
#include "slim_kernels.h"
#include "device_common.h"

namespace slim {
namespace {

// A wave takes 16 rows of 64 / LPHP neighbouring heads (LPHP lanes per head, 8 columns each: up to 1 KB of
// consecutive bytes per row), all 16 loads in flight at once, sums each row over the head's lanes with DPP adds and
// leaves with consecutive rows of a head on the head's lanes.  Bound by HBM: one load, 16 multiply-adds and the
// reduction per 16 bytes and lane are a fifth of what the vector ALU does in the time the bytes take.  (One wave per
// row with per-head sums through LDS, as the plain kernel does it: 67 us for 6503 rows of 5120 columns, 67 MB; this one
// 16.3 us, numerators included: 4.1 TB/s with the launch.)
// With rotary keys the table's entries of four rows travel beside the 16 rows, and where numerators follow four waves per SIMD are
// asked for (three with heads of 8 columns, 133 registers): left to itself the compiler takes 62 to 67 registers for eight, the rows
// alone being 64, and loads a few rows at a time (the step with 2 x 3000 rows x 40 heads x 64: 37.3 us, with these registers
// 34.9; 1 x 700 x 40 x 128 33.8 and 31.1; before there were numerators 35.4 and 31.4).
constexpr int KS_ROWS = 16, KS_WAVES = 4, KS_BLOCK = KS_ROWS * KS_WAVES;
constexpr int ks_waves(int lphp, bool fixed, int otherwise) { return fixed ? (lphp == 1 ? 3 : 4) : otherwise; }

// NUM: leaves with numerators p = 2^(s - ref) of its 64 rows, ref = the block's largest score of the head rounded up to a
// whole number, and with ref and the sum of p per (block, head): the weighted sum's workgroups, one per 128 columns of K,
// would each take every exponential again (40 times at 5120 columns).  A whole ref makes the weighted sum's change to a
// common one a change of exponent.  Rows past the end up to the next multiple of 32 get weight 0.  Without NUM: the scores.
template <int LPHP, bool ROPE, bool NUM>
__global__ __launch_bounds__(KS_WAVES * 64) __attribute__((amdgpu_waves_per_eu(ks_waves(LPHP, ROPE && NUM, 1), ks_waves(LPHP, ROPE && NUM, 8)))) void kscores_kernel(const float* __restrict__ q, const uint16_t* __restrict__ K,
                                                                long k_bstride, const int32_t* __restrict__ seq_lens, int T,
                                                                int H, int d, int d_k, float scale_log2,
                                                                const float* __restrict__ rope, float* __restrict__ S,
                                                                float* __restrict__ blocks, int* counters, int ncounters) {
  constexpr int HPP = 64 / LPHP;                        // heads per wave
  const int npiece = (H + HPP - 1) / HPP;
  const int rb = blockIdx.x / npiece, piece = blockIdx.x - rb * npiece, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // (the arrival counters of the projection that ends this call start at 0)
  if (blockIdx.x == 0 && b == 0)
    for (int i = tid; i < ncounters; i += KS_WAVES * 64) counters[i] = 0;
  const int len = seq_len_of(seq_lens, b, T);
  const int r0 = (rb * KS_WAVES + w) * KS_ROWS;
  if (NUM ? rb * KS_BLOCK >= len : r0 >= len) return;    // (NUM: the workgroup's waves meet)
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
  float mx = NEG_INF, ref = 0.f, sum = 0.f;
  __shared__ float m_s[NUM ? KS_WAVES : 1][64], l_s[NUM ? KS_WAVES : 1][64];
  if constexpr (NUM) {
#pragma unroll
    for (int j = 0; j < KS_ROWS; ++j) {
      if (r0 + j >= len) s[j] = NEG_INF;
      mx = fmaxf(mx, s[j]);
    }
    if (li == 0) m_s[w][hl] = mx;
    lds_barrier();
#pragma unroll
    for (int ww = 0; ww < KS_WAVES; ++ww) mx = fmaxf(mx, m_s[ww][hl]);
    mx = ceilf(mx);
    ref = mx == NEG_INF ? 0.f : mx;
  }
  const int end = NUM ? (len + 31) / 32 * 32 : len;
#pragma unroll
  for (int g = 0; g < KS_ROWS; g += LPHP) {             // lane li of a head stores row g + li
    float v = s[g];
#pragma unroll
    for (int j = 1; j < LPHP; ++j) v = li == j ? s[g + j] : v;
    if constexpr (NUM) {
      v = __builtin_amdgcn_exp2f(v - ref);
      sum += v;
    }
    if (live && r0 + g + li < end) dst[g] = v;
  }
  if constexpr (NUM) {
    if constexpr (LPHP > 1) sum = dpp_add<0xB1>(sum);
    if constexpr (LPHP > 2) sum = dpp_add<0x4E>(sum);
    if constexpr (LPHP > 4) sum = dpp_add<0x141>(sum);
    if constexpr (LPHP > 8) sum = dpp_add<0x140>(sum);
    if (li == 0) l_s[w][hl] = sum;
    lds_barrier();
    if (w == 0 && li == 0 && live) {
      float l = 0.f;
#pragma unroll
      for (int ww = 0; ww < KS_WAVES; ++ww) l += l_s[ww][hl];
      const int nblk = (T + KS_BLOCK - 1) / KS_BLOCK;
      float* at = blocks + ((size_t)b * nblk + rb) * H + h;
      at[0] = mx;                                       // (-inf: no row counts)
      at[(size_t)gridDim.y * nblk * H] = l;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Weighted sum of the rows of K for one (sequence, context split, group of 16 NT heads, block of 128 columns) from the
// numerators of kscores_kernel.  The 8 waves split the rows (wave w takes 32-row tiles w, w + 8, ...) and are summed
// through LDS at the end.  Register tile and MFMA layout as in the stream kernel: lane (idx = l % 16, rg = l / 16) holds
// 16 bytes of rows rg*8 .. rg*8+7 and transposes its 8 x 8 block into 8 A operands; B = the weights, lane (head, rg), as
// three bf16 terms (8 + 8 + 8 bits: exactly the fp32 value, three MFMAs where one would do: the matrix cores are idle most
// of the time).  All waves weigh against one reference, the largest of the split's blocks, so nothing is rescaled on the
// way: a tile's numerators are multiplied by 2^(its block's reference - that one).
// What bounds it: the trip of a tile of K, which comes from the memory-side cache, one tile ahead at three head tiles (two do
// not fit the registers): 24.6 us at 40 heads x 5120 columns, 6503 rows (67 MB), where taking the numerators in every
// workgroup, 130 vector operations and 8 exponentials per tile and head tile, took 27.8.  The whole step 60.6 -> 57.7 us
// there, 140.6 -> 128.1 at 12 ragged sequences of 300..3000 rows, 163.3 -> 156.0 at 4 x 6000 rows x 48 heads x 128; with
// contexts of a few hundred rows it is the same (27.7 and 27.6 us at 2 x 250..500 x 40 x 96).
// ------------------------------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(512) void kweighted_kernel(const float* __restrict__ P, const float* __restrict__ blocks,
                                                        const uint16_t* __restrict__ K, long k_bstride,
                                                        const int32_t* __restrict__ seq_lens, int T, int B, int H, int d, int nsplit,
                                                        float* __restrict__ Cpart, float* __restrict__ mpart,
                                                        float* __restrict__ lpart, int colocate) {
  constexpr int NW = 8, HG = NT * 16, PARTS = 512 / HG;
  __shared__ float red[NW][4][8][64];                  // one head tile at a time: [wave][r][i][lane]
  __shared__ float bsh[PARTS][HG];
  const int ncb = d / 128;
  // unit = (sequence, context split): its workgroups read the same rows of K and the same numerators
  int unit, inner;
  if (!unit_of_workgroup(blockIdx.x, ((H + HG - 1) / HG) * ncb, B * nsplit, colocate != 0, unit, inner)) return;
  const int b = unit / nsplit, s = unit - b * nsplit;
  const int cbk = inner % ncb, hg = inner / ncb;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = lane & 15, rg = lane >> 4;
  const int col0 = cbk * 128;
  const int len = seq_len_of(seq_lens, b, T);
  const int rows_per = ((len + nsplit - 1) / nsplit + KS_BLOCK - 1) / KS_BLOCK * KS_BLOCK;   // (whole blocks)
  const int r_lo = s * rows_per, r_hi = min(len, r_lo + rows_per);
  const int ntile_all = r_lo < r_hi ? (r_hi - r_lo + 31) / 32 : 0;
  const int ntile = ntile_all > w ? (ntile_all - w + NW - 1) / NW : 0;   // this wave's tiles: w, w + 8, ...
  auto row_of = [&](int k) { return r_lo + 32 * (w + NW * k); };
  const int nblk = (T + KS_BLOCK - 1) / KS_BLOCK, Tp = (T + 31) / 32 * 32;
  const float* refs = blocks + (size_t)b * nblk * H;
  const float* sums = refs + (size_t)B * nblk * H;

  // Rows by 32-bit byte offsets from the sequence's base (wide_ok); rows past the end re-read the last row, weight 0.
  const char* Kb = reinterpret_cast<const char*>(K + (size_t)b * k_bstride + col0 + n * 8);
  const unsigned pitchB = (unsigned)d * 2u;
  auto load_tile = [&](u32x4 (&t)[8], int r0) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      t[j] = *reinterpret_cast<const u32x4*>(Kb + __umul24((unsigned)min(r0 + rg * 8 + j, len - 1), pitchB));
  };
  int hl[NT];                                          // this lane's heads (a padded one: the last, its results are not stored)
#pragma unroll
  for (int t = 0; t < NT; ++t) hl[t] = min(hg * HG + t * 16 + n, H - 1);
  struct Num { f32x4 p[NT][2]; float ref[NT]; };
  auto load_num = [&](Num& x, int r0) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float* src = P + ((size_t)b * H + hl[t]) * Tp + r0 + rg * 8;
      x.p[t][0] = *reinterpret_cast<const f32x4*>(src);
      x.p[t][1] = *reinterpret_cast<const f32x4*>(src + 4);
      x.ref[t] = refs[(size_t)(r0 / KS_BLOCK) * H + hl[t]];
    }
  };
  // K tiles and numerators travel D steps ahead; past the end the last tile again (unused), so that every step issues the
  // same loads and the compiler waits for exactly the ones it needs.
  constexpr int D = NT <= 2 ? 2 : 1, UN = 2;
  u32x4 kt[D][8];
  Num nm[D];
  if (ntile > 0) {
#pragma unroll
    for (int j = 0; j < D; ++j) load_tile(kt[j], row_of(min(j, ntile - 1)));
#pragma unroll
    for (int j = 0; j < D; ++j) load_num(nm[j], row_of(min(j, ntile - 1)));
  }
  // the split's reference per head: the largest of its blocks'
  const int b_lo = r_lo / KS_BLOCK, b_hi = r_lo < r_hi ? (r_hi + KS_BLOCK - 1) / KS_BLOCK : b_lo;
  const int hs = tid % HG, part = tid / HG, hsc = min(hg * HG + hs, H - 1);
  float mx = NEG_INF;
  if (part < PARTS) {
    for (int k = b_lo + part; k < b_hi; k += PARTS) mx = fmaxf(mx, refs[(size_t)k * H + hsc]);
    bsh[part][hs] = mx;
  }
  lds_barrier();
  auto reference = [&](int h) {
    float m = NEG_INF;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) m = fmaxf(m, bsh[q][h]);
    return m;
  };
  float mref[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    mref[t] = reference(t * 16 + n);
    if (mref[t] == NEG_INF) mref[t] = 0.f;
  }
  if (cbk == 0) {                                      // one workgroup per head group also leaves with reference and sum
    const float m = reference(hs), ref = m == NEG_INF ? 0.f : m;
    lds_barrier();
    float l = 0.f;
    if (part < PARTS) {
      for (int k = b_lo + part; k < b_hi; k += PARTS)
        l = fmaf(sums[(size_t)k * H + hsc], __builtin_amdgcn_exp2f(refs[(size_t)k * H + hsc] - ref), l);
      bsh[part][hs] = l;
    }
    lds_barrier();
    if (tid < HG && hg * HG + tid < H) {
      float all = 0.f;
#pragma unroll
      for (int q = 0; q < PARTS; ++q) all += bsh[q][tid];
      const size_t at = (size_t)(b * nsplit + s) * H + hg * HG + tid;
      mpart[at] = m;
      lpart[at] = all;
    }
  }

  f32x4 acc[8][NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int k, auto SI) {
    constexpr int si = decltype(SI)::value % D;
    u32x4 am[8];
    transpose8x8(kt[si], am);
    load_tile(kt[si], row_of(min(k + D, ntile - 1)));
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float f = __builtin_amdgcn_exp2f(nm[si].ref[t] - mref[t]);
      u32x4 pb[3];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float p0 = nm[si].p[t][j >> 2][j & 3] * f, p1 = nm[si].p[t][j >> 2][(j & 3) + 1] * f;
        unsigned u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
        pb[0][j / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);          // the upper halves: the value truncated to 8 bits
        const float q0 = p0 - __uint_as_float(u0 & 0xffff0000u), q1 = p1 - __uint_as_float(u1 & 0xffff0000u);
        u0 = __float_as_uint(q0); u1 = __float_as_uint(q1);
        pb[1][j / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        const float o0 = q0 - __uint_as_float(u0 & 0xffff0000u), o1 = q1 - __uint_as_float(u1 & 0xffff0000u);
        pb[2][j / 2] = __builtin_amdgcn_perm(__float_as_uint(o1), __float_as_uint(o0), 0x07060302u);   // (8 bits are left)
      }
#pragma unroll
      for (int o = 2; o >= 0; --o)                        // (the smallest terms first)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, am[i]), __builtin_bit_cast(bf16x8, pb[o]),
                                                              acc[i][t], 0, 0, 0);
    }
    load_num(nm[si], row_of(min(k + D, ntile - 1)));
  };
  int k = 0;
  for (; k + UN <= ntile; k += UN) full_steps<0, UN>(k, step);
  unrolled_steps<0, UN>(k, ntile, step);

  // ---- sum the 8 waves, a head tile at a time: thread (w, lane) takes four of the eight columns of group rg*4 + w%4 ---
  // (The lane made here again: two addresses that waited in scratch through the steps, 8 bytes a lane, cost 2 x 4001 rows x 40 heads x 128
  // 57.5 us instead of 56.2 and 4 x 6000 121.1 instead of 119.2.)
  const int ln = fresh_lane(), wv = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t > 0) lds_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wv][r][i][ln] = acc[i][t][r];
    lds_barrier();
    const int i0 = (wv >> 2) * 4, r = wv & 3, h = hg * HG + t * 16 + (ln & 15);
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) o[i] += red[ww][r][i0 + i][ln];
    if (h < H) *reinterpret_cast<f32x4*>(Cpart + ((size_t)(b * nsplit + s) * H + h) * d + col0 + ((ln >> 4) * 4 + r) * 8 + i0) = o;
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

// Head tiles per workgroup.  Three where that saves a pass over K (33..48, 65..96 heads, ...), else two, which leaves
// registers for a second tile in flight.
int kweighted_tiles(int H) {
  const int tiles = (H + 15) / 16;
  return (tiles + 2) / 3 < (tiles + 1) / 2 ? 3 : 2;
}

// One round of workgroups (one per compute unit: 8 waves of 256 registers), eight tiles of rows each at least.
int kweighted_splits(int B, int H, int T, int d) {
  const int nt = kweighted_tiles(H);
  const long per = (long)B * ((H + nt * 16 - 1) / (nt * 16)) * (d / 128 > 0 ? d / 128 : 1);
  int s = (int)(256 / per);
  const int cap = (T + 255) / 256;
  if (s > cap) s = cap;
  if (s > PROJ_MAX_PARTS) s = PROJ_MAX_PARTS;
  return s < 1 ? 1 : s;
}

size_t kscores_block_floats(int B, int H, int T) { return 2 * (size_t)B * H * ((T + KS_BLOCK - 1) / KS_BLOCK); }

void launch_kscores(const float* q, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int d_k,
                    float scale_log2, const float* rope, float* S, float* blocks, int* counters, int ncounters, int B, hipStream_t st) {
  int lphp = 1;
  while (lphp < d_k / 8) lphp <<= 1;
  const int npiece = (H + 64 / lphp - 1) / (64 / lphp), nrb = (T + KS_BLOCK - 1) / KS_BLOCK;
  dim3 grid((unsigned)npiece * nrb, B);
  auto go = [&](auto lp, auto rp, auto num) {
    hipLaunchKernelGGL((kscores_kernel<decltype(lp)::value, decltype(rp)::value, decltype(num)::value>), grid, dim3(KS_WAVES * 64), 0, st, q,
                       (const uint16_t*)K, k_bstride, seq_lens, T, H, d, d_k, scale_log2, rope, S, blocks, counters, ncounters);
  };
  auto with_num = [&](auto lp, auto rp) {
    if (blocks) go(lp, rp, std::true_type{});
    else go(lp, rp, std::false_type{});
  };
  auto with_rope = [&](auto lp) {
    if (rope) with_num(lp, std::true_type{});
    else with_num(lp, std::false_type{});
  };
  switch (lphp) {
    case 1: with_rope(std::integral_constant<int, 1>{}); break;
    case 2: with_rope(std::integral_constant<int, 2>{}); break;
    case 4: with_rope(std::integral_constant<int, 4>{}); break;
    case 8: with_rope(std::integral_constant<int, 8>{}); break;
    default: with_rope(std::integral_constant<int, 16>{}); break;
  }
}

void launch_kweighted(const float* P, const float* blocks, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d,
                      int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st) {
  const int nt = kweighted_tiles(H);
  const int ninner = ((H + nt * 16 - 1) / (nt * 16)) * (d / 128), colocate = colocate_units(B * nsplit);
  dim3 grid(unit_grid(B * nsplit, ninner, colocate));
  auto go = [&](auto tiles) {
    hipLaunchKernelGGL((kweighted_kernel<decltype(tiles)::value>), grid, dim3(512), 0, st, P, blocks, (const uint16_t*)K, k_bstride,
                       seq_lens, T, B, H, d, nsplit, Cpart, mpart, lpart, colocate);
  };
  if (nt == 3) go(std::integral_constant<int, 3>{});
  else go(std::integral_constant<int, 2>{});
}

}  // namespace slim
