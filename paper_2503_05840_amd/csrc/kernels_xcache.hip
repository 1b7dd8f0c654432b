// bf16 fast path of the X-cache scheme (non-square section, Fig. 4; also the encoder-cache option of
// the encoder-decoder section): the cache holds the layer input X [T][d_model]; K and V are never formed.
//
//   xq_tilde_kernel   : q~_h = q_h W_K,h^T, scaled, as bf16 hi + lo in MFMA operand order (W_K read once)
//   xscores_kernel    : s[h][t] = q~_h . X[t]        [B][H][T padded to 32], log2 domain, on MFMA
//   xweighted_kernel  : per context split, m = reference, l = sum 2^(s-m), C_h = sum_t 2^(s-m) X[t]
//                       on MFMA, one contraction for 32 heads at a time
// followed by the merge + projection of the K-cache path with W_V in place of W_KV.
//
// All heads use the full row of X here (no per-head column slice), so the scores are a plain
// dense product over d_model; they are written out (H x T x 4 bytes per sequence, small next to the
// 2 x e-wide caches the scheme avoids) and the weighted sum is a second pass over X.
#include "slim_kernels.h"

#include "device_common.h"

#include <algorithm>

namespace slim {
namespace {

// 8 fp32 values -> bf16 hi and bf16 lo (x = hi + lo up to 2^-17 relative)
__device__ __forceinline__ void split_hi_lo(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const __bf16 h = (__bf16)x[j];
    hi[j] = h;
    lo[j] = (__bf16)(x[j] - (float)h);
  }
}

// ------------------------------------------------------------------------------------------------
// q~[b][h][c] = scale * sum_j q[b][h d_k + j] W_K[c][h d_k + j]   (scale = log2(e) / sqrt(d_k)), written
// as two bf16 arrays, hi = bf16(q~) and lo = bf16(q~ - hi), in the order the scores kernel's MFMA B operands
// take them: [b][tile of 16 heads][k-step of 32 columns][lane = (column / 8 % 4) * 16 + head % 16][8 columns],
// so that a wave reads one operand as 1 KB of consecutive bytes.
// grid (H / XQ_HEADS, d_model / 128, batch chunks of 16); a wave owns 16 rows c of W_K for XQ_HEADS heads.
// MFMA: A = W_K block (M = 16 rows c, K = the head's columns j), B = q^T (N = sequences) as hi + lo.
// The 8 waves share their B operands: the workgroup fetches its slice of q once (consecutive threads on
// consecutive floats), splits it and lays the operands out in LDS.  (Fetched per wave in operand order --
// a lane per sequence, rows of q 4 e bytes apart -- q cost more time than W_K: 16 lines per instruction that
// fall on few L2 channels, and every workgroup of a head asks for the same ones.)
// ------------------------------------------------------------------------------------------------
constexpr int XQ_HEADS = 4;
constexpr int XQ_QROW = 16 * 16 + 16;    // bytes per (head, k-step, k-group) of B operands in LDS: 16 sequences x 16 bytes + padding

template <bool ONCE>
__global__ __launch_bounds__(512) void xq_tilde_kernel(const float* q, const uint16_t* Wk, uint16_t* qt, int B,
                                                       int H, int d_k, int dm, int e, float scale, int* counters,
                                                       int ncounters) {
  __shared__ __align__(16) unsigned char qs[2][XQ_HEADS * 4 * 4 * XQ_QROW];   // hi, lo
  // (the arrival counters of the projection that ends this call start at 0)
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
    for (int i = threadIdx.x; i < ncounters; i += 512) counters[i] = 0;
  const int bbase = blockIdx.z * 16;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int c0 = (blockIdx.y * 8 + w) * 16;            // (d_model is a multiple of 128: every wave has rows)
  const int h0 = blockIdx.x * XQ_HEADS;
  const int b = bbase + n;
  const int nks = d_k / 32;                            // 1..4 k-steps per head
  // all loads of W_K are issued before anything else: they come from HBM
  u32x4 av[XQ_HEADS][4];
#pragma unroll
  for (int hh = 0; hh < XQ_HEADS; ++hh) {
    const int h = min(h0 + hh, H - 1);
    const uint16_t* wrow = Wk + (size_t)(c0 + n) * e + (size_t)h * d_k + kq * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const u32x4* const src = reinterpret_cast<const u32x4*>(wrow + min(ks, nks - 1) * 32);
      if constexpr (ONCE) av[hh][ks] = __builtin_nontemporal_load(src);
      else av[hh][ks] = *src;
    }
  }
  // q of the workgroup's heads and sequences: 16 x XQ_HEADS d_k floats = nks pieces of 4 floats per thread
  {
    const int upq = d_k / 4;                           // pieces per head
    f32x4 qraw[4];
    int off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      qraw[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      off[i] = 0;
      if (i < nks) {
        const int g = i * 512 + tid, bl = g / d_k, rem = g - bl * d_k, hh = rem / upq, j0 = (rem - hh * upq) * 4;
        // (heads past H and sequences past B: zeros)
        if (bbase + bl < B && h0 + hh < H)
          qraw[i] = *reinterpret_cast<const f32x4*>(q + (size_t)(bbase + bl) * e + (size_t)(h0 + hh) * d_k + j0);
        off[i] = ((hh * 4 + (j0 >> 5)) * 4 + ((j0 & 31) >> 3)) * XQ_QROW + bl * 16 + (j0 & 7) * 2;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < nks) {
        unsigned hw[2], lw[2];
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const float x0 = qraw[i][r], x1 = qraw[i][r + 1];
          const __bf16 hb0 = (__bf16)x0, hb1 = (__bf16)x1;
          const __bf16 l0 = (__bf16)(x0 - (float)hb0), l1 = (__bf16)(x1 - (float)hb1);
          hw[r / 2] = (unsigned)__builtin_bit_cast(uint16_t, hb0) | ((unsigned)__builtin_bit_cast(uint16_t, hb1) << 16);
          lw[r / 2] = (unsigned)__builtin_bit_cast(uint16_t, l0) | ((unsigned)__builtin_bit_cast(uint16_t, l1) << 16);
        }
        *reinterpret_cast<uint2*>(&qs[0][off[i]]) = make_uint2(hw[0], hw[1]);
        *reinterpret_cast<uint2*>(&qs[1][off[i]]) = make_uint2(lw[0], lw[1]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int hh = 0; hh < XQ_HEADS; ++hh) {
    const int h = h0 + hh;
    if (h >= H) break;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks < nks) {
        const int qo = ((hh * 4 + ks) * 4 + kq) * XQ_QROW + n * 16;
        const bf16x8 hi = *reinterpret_cast<const bf16x8*>(&qs[0][qo]);
        const bf16x8 lo = *reinterpret_cast<const bf16x8*>(&qs[1][qo]);
        const bf16x8 a8 = __builtin_bit_cast(bf16x8, av[hh][ks]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, hi, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, lo, acc, 0, 0, 0);
      }
    }
    // D: column n = sequence, rows kq*4 + r = c0 + ...; stored scaled, as bf16 hi and lo halves
    if (b < B) {
      unsigned hw[2], lw[2];
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const float x0 = acc[r] * scale, x1 = acc[r + 1] * scale;
        const __bf16 hb0 = (__bf16)x0, hb1 = (__bf16)x1;
        const __bf16 l0 = (__bf16)(x0 - (float)hb0), l1 = (__bf16)(x1 - (float)hb1);
        hw[r / 2] = (unsigned)__builtin_bit_cast(uint16_t, hb0) | ((unsigned)__builtin_bit_cast(uint16_t, hb1) << 16);
        lw[r / 2] = (unsigned)__builtin_bit_cast(uint16_t, l0) | ((unsigned)__builtin_bit_cast(uint16_t, l1) << 16);
      }
      // B-operand order of the scores kernel: [b][head tile][k-step of 32 columns][lane (kq, n)][8]
      const int c = c0 + kq * 4, nht = (H + 15) / 16;
      const size_t at = ((((size_t)b * nht + h / 16) * (dm / 32) + c / 32) * 64 + ((c % 32) / 8) * 16 + h % 16) * 8 + c % 8;
      *reinterpret_cast<uint2*>(qt + at) = make_uint2(hw[0], hw[1]);
      *reinterpret_cast<uint2*>(qt + (size_t)B * nht * 16 * dm + at) = make_uint2(lw[0], lw[1]);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Both passes over X share one layout: a workgroup stages tiles of X in LDS with coalesced loads
// (every element of X leaves HBM once per pass) and its 8 waves split the HEADS: wave w owns head
// tile (16 heads) w % P of the P tiles in flight, P = 1, 2, 4 or 8, and shares the rest of the work
// with the 8 / P waves of the same head tile.  More than 16 P heads: several passes.
//
// xscores: s[b][h][t] = sum_c X[b][t][c] q~[b][h][c]   (log2 domain; q~ arrives scaled)
// grid (blocks of 128 rows, B).  X is staged in chunks of 256 columns (double-buffered: the next chunk
// travels HBM -> registers while this one is used, then registers -> LDS).  Per chunk a wave holds the
// B operands of its head tile (hi + lo, 8 k-steps) in registers and runs over its M tiles of 16 rows:
// A operands come from LDS (16 bytes per lane: row m, columns ks*32 + kq*8).
// ------------------------------------------------------------------------------------------------
constexpr int XL_RB = 128;               // rows per workgroup
constexpr int XL_KC = 128;               // columns per chunk
constexpr int XL_KS = XL_KC / 32;        // k-steps per chunk
constexpr int XL_PITCH = XL_KC + 8;      // bf16 elements per staged row (16 bytes of padding)
constexpr int XL_AHEAD = 4;              // chunks of X in flight from HBM (register sets)

template <int P>
__global__ __launch_bounds__(512) void xscores_kernel(const uint16_t* qt, const uint16_t* X, long x_bstride,
                                                      const int32_t* seq_lens, int T, int B, int H, int dm, float* S,
                                                      int colocate) {
  __shared__ __align__(16) uint16_t xs[2][XL_RB * XL_PITCH];
  constexpr int RS = 8 / P;                            // waves per head tile = row subsets
  constexpr int D = XL_AHEAD;
  // unit = sequence (its row blocks read the same q~), inner = block of XL_RB rows
  int b, rbk;
  if (!unit_of_workgroup(blockIdx.x, (T + XL_RB - 1) / XL_RB, B, colocate != 0, b, rbk)) return;
  const int row_base = rbk * XL_RB;
  const int len = seq_len_of(seq_lens, b, T);
  if (row_base >= len) return;                         // (workgroup-uniform)
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int htl = w % P, rs = w / P;
  const int NHT = (H + 15) / 16;
  const int nkc = dm / XL_KC, npass = (NHT + P - 1) / P;   // (dm is a multiple of 128)
  const int total = npass * nkc;
  const uint16_t* Xb = X + (size_t)b * x_bstride;
  const size_t lo_off = (size_t)B * NHT * 16 * dm;     // the lo halves follow the hi halves
  const int Tp = (T + 31) / 32 * 32;                   // rows of S are padded to whole tiles

  // staging: thread t moves 16-byte column chunk t % 16 of rows t / 16 + 32 i
  const int srow = tid >> 4, scol = (tid & 15) * 8;
  u32x4 stg[D][4];
  auto issue_x = [&](u32x4 (&g)[4], int it) {
    const int col = (it % nkc) * XL_KC + scol;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = min(row_base + srow + 32 * i, len - 1);   // rows past the end: any finite values, never stored
      g[i] = *reinterpret_cast<const u32x4*>(Xb + (size_t)r * dm + col);
    }
  };
  auto commit_x = [&](const u32x4 (&g)[4], int it) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<u32x4*>(&xs[it & 1][(srow + 32 * i) * XL_PITCH + scol]) = g[i];
  };
  // B operands of iteration it (head tile and chunk): 1 KB of consecutive bytes per operand
  auto load_b = [&](u32x4 (&bh)[XL_KS], u32x4 (&bl)[XL_KS], int it) {
    const int ht = min((it / nkc) * P + htl, NHT - 1), kc = it % nkc;
    const uint16_t* src = qt + ((((size_t)b * NHT + ht) * (dm / 32) + (size_t)kc * XL_KS) * 64 + lane) * 8;
#pragma unroll
    for (int ks = 0; ks < XL_KS; ++ks) {
      bh[ks] = *reinterpret_cast<const u32x4*>(src + ks * 512);
      bl[ks] = *reinterpret_cast<const u32x4*>(src + lo_off + ks * 512);
    }
  };

  f32x4 acc[P];
  u32x4 bh[XL_KS], bl[XL_KS], nh[XL_KS], nl[XL_KS];
#pragma unroll
  for (int j = 0; j < D; ++j) issue_x(stg[j], min(j, total - 1));
  load_b(bh, bl, 0);
  commit_x(stg[0], 0);
  lds_barrier();
  // One chunk; SI is it % D as a type: the register set whose chunk (it) has already gone to LDS.
  auto step = [&](int it, auto SI) {
    constexpr int si = decltype(SI)::value;
    const int hp = it / nkc, kc = it % nkc;
    const bool more = it + 1 < total;
    // (a wave's loads complete in issue order: what the next chunk needs goes first, so that waiting for it
    //  does not wait for the X chunk that is D chunks away)
    // Issued unconditionally (past the end: the last chunk again, unused) so that the compiler can count
    // the loads in flight and wait for exactly the ones a step needs.
    load_b(nh, nl, min(it + 1, total - 1));
    issue_x(stg[si], min(it + D, total - 1));
    const int ht = hp * P + htl;
    if (kc == 0) {
#pragma unroll
      for (int mi = 0; mi < P; ++mi) acc[mi] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (ht < NHT) {
      const uint16_t* xa = &xs[it & 1][n * XL_PITCH + kq * 8];
#pragma unroll
      for (int mi = 0; mi < P; ++mi) {
        const int mt = rs + mi * RS;                   // this wave's M tiles: rs, rs + RS, ...
#pragma unroll
        for (int ks = 0; ks < XL_KS; ++ks) {
          const bf16x8 a8 = *reinterpret_cast<const bf16x8*>(xa + mt * 16 * XL_PITCH + ks * 32);
          acc[mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, __builtin_bit_cast(bf16x8, bh[ks]), acc[mi], 0, 0, 0);
          acc[mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, __builtin_bit_cast(bf16x8, bl[ks]), acc[mi], 0, 0, 0);
        }
      }
      if (kc == nkc - 1) {                             // D: column n = head, rows kq*4 + r
        const int h = ht * 16 + n;
        if (h < H) {
#pragma unroll
          for (int mi = 0; mi < P; ++mi) {
            const int t0 = row_base + (rs + mi * RS) * 16 + kq * 4;
            float* dst = S + ((size_t)b * H + h) * Tp + t0;
            if (t0 + 3 < len) {                         // (rows of S are padded to 32: 16-byte aligned)
              *reinterpret_cast<f32x4*>(dst) = acc[mi];
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (t0 + r < len) dst[r] = acc[mi][r];
            }
          }
        }
      }
    }
    if (more) {
      commit_x(stg[(si + 1) % D], it + 1);
#pragma unroll
      for (int ks = 0; ks < XL_KS; ++ks) { bh[ks] = nh[ks]; bl[ks] = nl[ks]; }
    }
    lds_barrier();
  };
  int it = 0;
  for (; it + D <= total; it += D) full_steps<0, D>(it, step);
  unrolled_steps<0, D>(it, total, step);
}

// ------------------------------------------------------------------------------------------------
// Weighted sum of the rows of X for one (sequence, context split, group of 32 heads, block of 128
// columns).  The 8 waves of the workgroup split the ROWS of the split (wave w takes 32-row tiles w,
// w + 8, ...) and merge their (m, l, C) through LDS at the end, so one partial leaves per workgroup:
// splitting the context across workgroups instead costs H x d_model x 4 bytes of partial per split and
// sequence, which at 8 splits was four times the bytes of X itself.
// Register tile and MFMA layout as in the K-cache stream kernel: lane (idx = l % 16, rg = l / 16)
// loads 16 bytes of rows rg*8 .. rg*8+7, transposes its 8x8 block into 8 A operands; B = weights
// P^T (lane (n = head, kg = row group) reads 8 consecutive scores of head n).
// Writes Cpart[(b nsplit + s)][h][c] (unnormalised), mpart (log2 domain) and lpart.
// ------------------------------------------------------------------------------------------------
constexpr float XW_SLACK = 6.0f;

// NT: head tiles of 16 per workgroup.  FULL: the weights enter the matrix product as three bf16 terms (8 + 8 + 8
// bits: exactly the fp32 value) and their sum is taken in fp32 on the vector ALU -- K-caches whose weights are fp32, where
// the scratch has no room for what kweighted_kernel (kernels_wide.hip) needs (heads of 8 columns with 321 to 511 rows, say, or
// 1100 sequences of 4300 rows and more x 8 heads of 64 columns); otherwise rounded to bf16 once.  (FULL is 3 MFMAs where there was one; the
// matrix cores are idle most of the time here.)  At 8 sequences of 500 rows, 48 heads x 8 columns: 10.9 us, where the vector-ALU
// kernel takes 58.4.
template <int NT, bool FULL>
__global__ __launch_bounds__(512) void xweighted_kernel(const float* S, const uint16_t* X, long x_bstride,
                                                        const int32_t* seq_lens, int T, int B, int H, int dm, int nsplit,
                                                        float* Cpart, float* mpart, float* lpart, int colocate) {
  constexpr int NW = 8;
  constexpr int TP = NT <= 2 ? NT : 1;                 // head tiles merged at once: 64 KB of LDS each
  static_assert(NT <= 3, "registers");
  __shared__ float red[NW][TP][4][8][64];              // [wave][head tile][r][i][lane]
  __shared__ float msh[NW][NT * 16], lsh[NW][NT * 16];
  // unit = (sequence, context split): its workgroups read the same rows of X (one column block each, for
  // every head group) and the same scores (one head group each, for every column block)
  const int ncb = dm / 128;
  int unit, inner;
  if (!unit_of_workgroup(blockIdx.x, ((H + NT * 16 - 1) / (NT * 16)) * ncb, B * nsplit, colocate != 0, unit, inner)) return;
  const int b = unit / nsplit, s = unit - b * nsplit;
  const int cbk = inner % ncb, hg = inner / ncb;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int idx = lane & 15, rg = lane >> 4;
  const int n = idx, kg = rg;
  const int col0 = cbk * 128;
  const int len = seq_len_of(seq_lens, b, T);
  const int rows_per = ((len + nsplit - 1) / nsplit + 31) / 32 * 32;
  const int r_lo = s * rows_per, r_hi = min(len, r_lo + rows_per);
  const int pid = b * nsplit + s;
  const int ntile_all = r_lo < r_hi ? (r_hi - r_lo + 31) / 32 : 0;
  const int ntile = ntile_all > w ? (ntile_all - w + NW - 1) / NW : 0;   // this wave's tiles: w, w + 8, ...
  auto row_of = [&](int k) { return r_lo + 32 * (w + NW * k); };

  float m[NT];
  f32x4 acc[8][NT], accl[NT];                          // (FULL: accl[t][0] is this lane's share of the sum)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    m[t] = NEG_INF;
    accl[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Rows are addressed by 32-bit byte offsets from the sequence's base (a sequence of X is below 4 GB:
  // checked on the host); rows past the end re-read the last row and weigh nothing (their scores are masked).
  const char* Xb = reinterpret_cast<const char*>(X + (size_t)b * x_bstride + col0 + idx * 8);
  const unsigned pitchB = (unsigned)dm * 2u;
  auto load_tile = [&](u32x4 (&t)[8], int r0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned off = __umul24((unsigned)min(r0 + rg * 8 + j, len - 1), pitchB);
      t[j] = *reinterpret_cast<const u32x4*>(Xb + off);
    }
  };
  // scores of a tile: lane (n, kg) takes rows r0 + kg*8 .. +7 of heads hg*32 + t*16 + n.  The rows of S
  // are padded to a multiple of 32 floats, so the 32 bytes are always there; what lies past the end of
  // the split (or belongs to a padded head) is replaced, not computed with.
  const int Tp = (T + 31) / 32 * 32;
  auto load_scores = [&](f32x4 (&x)[NT][2], int r0) {    // (raw: masked when used, so that nothing waits here)
    const int row = r0 + kg * 8;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int h = min(hg * (NT * 16) + t * 16 + n, H - 1);
      const float* src = S + ((size_t)b * H + h) * Tp + row;
      x[t][0] = *reinterpret_cast<const f32x4*>(src);
      x[t][1] = *reinterpret_cast<const f32x4*>(src + 4);
    }
  };
  // X tiles travel HBM/L2 -> registers D tiles ahead, scores DS tiles ahead (register sets chosen by a
  // compile-time index).  A step's work is short next to the latency of a load, so what it needs must
  // have been requested several steps earlier.  Loads past the end re-read the last tile (unused) so that
  // every step issues the same loads and the compiler can wait for exactly the ones a step needs.
  // Three head tiles leave registers for one set of each; a step is long enough there (2000 cycles a wave).  With three
  // terms per weight both tile counts are past the 256 registers by ten (44 bytes of scratch per lane).
  constexpr int D = NT <= 2 ? 2 : 1, DS = D, UN = 2;   // X sets, score sets, steps per unrolled group (a common multiple)
  u32x4 xt[D][8];
  f32x4 sc[DS][NT][2];
  if (ntile > 0) {
#pragma unroll
    for (int j = 0; j < DS; ++j) load_scores(sc[j], row_of(min(j, ntile - 1)));
#pragma unroll
    for (int j = 0; j < D; ++j) load_tile(xt[j], row_of(min(j, ntile - 1)));
  }
  // weights of head tile t from its scores (first row of the lane: row), the state of its softmax moved on
  auto weights = [&](int t, const f32x4 (&sx)[2], int row, u32x4 (&pb)[FULL ? 3 : 1]) {
    const int live = (hg * (NT * 16) + t * 16 + n < H) ? r_hi - row : 0;   // rows of this lane that count
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = j < live ? sx[j >> 2][j & 3] : NEG_INF;
    float tmax = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    // The reference the weights are taken against moves only when the maximum has grown by more than
    // XW_SLACK (log2 domain): weights stay below 2^XW_SLACK, which costs bf16 and the fp32 sums nothing,
    // and the accumulators are rescaled rarely instead of at nearly every tile.
    const float mn = (tmax > m[t] + XW_SLACK) ? tmax : m[t];
    const float ref = (mn == NEG_INF) ? 0.f : mn;
    const float alpha = __builtin_amdgcn_exp2f(m[t] - ref);
    float psum = 0.f;
    if constexpr (FULL) {
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const float p0 = __builtin_amdgcn_exp2f(x[j] - ref), p1 = __builtin_amdgcn_exp2f(x[j + 1] - ref);
        psum += p0 + p1;
        unsigned u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
        pb[0][j / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);          // the upper halves: the value truncated to 8 bits
        const float q0 = p0 - __uint_as_float(u0 & 0xffff0000u), q1 = p1 - __uint_as_float(u1 & 0xffff0000u);
        u0 = __float_as_uint(q0); u1 = __float_as_uint(q1);
        pb[1][j / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        const float o0 = q0 - __uint_as_float(u0 & 0xffff0000u), o1 = q1 - __uint_as_float(u1 & 0xffff0000u);
        pb[2][j / 2] = __builtin_amdgcn_perm(__float_as_uint(o1), __float_as_uint(o0), 0x07060302u);   // (8 bits are left)
      }
    } else {
      bf16x8 pv;
#pragma unroll
      for (int j = 0; j < 8; ++j) pv[j] = (__bf16)__builtin_amdgcn_exp2f(x[j] - ref);
      pb[0] = __builtin_bit_cast(u32x4, pv);
    }
    m[t] = mn;
    if (__any(alpha != 1.f)) {
      accl[t] *= alpha;
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i][t] *= alpha;
    }
    if constexpr (FULL) accl[t][0] += psum;
  };
  auto step = [&](int k, auto SI) {
    constexpr int si = decltype(SI)::value;
    u32x4 (&cur)[8] = xt[si % D];
    f32x4 (&sx)[NT][2] = sc[si % DS];
    const int row = row_of(k) + kg * 8;
    u32x4 am[8];
    if constexpr (FULL) {
      // one head tile after the other: only its own terms of the weights are live
      transpose8x8(cur, am);
      load_tile(cur, row_of(min(k + D, ntile - 1)));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        u32x4 pb[3];
        weights(t, sx[t], row, pb);
#pragma unroll
        for (int o = 2; o >= 0; --o)                      // (the smallest terms first)
#pragma unroll
          for (int i = 0; i < 8; ++i)
            acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, am[i]), __builtin_bit_cast(bf16x8, pb[o]),
                                                                acc[i][t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      load_scores(sx, row_of(min(k + DS, ntile - 1)));
    } else {
      u32x4 pb[NT][1];
#pragma unroll
      for (int t = 0; t < NT; ++t) weights(t, sx[t], row, pb[t]);
      transpose8x8(cur, am);
      // both sets are free again: the scores of the wave's tile k + DS first, then X of its tile k + D
      load_scores(sx, row_of(min(k + DS, ntile - 1)));
      load_tile(cur, row_of(min(k + D, ntile - 1)));
      const u32x4 ones_bits = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
      const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        accl[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pb[t][0]), accl[t], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, am[i]), __builtin_bit_cast(bf16x8, pb[t][0]),
                                                              acc[i][t], 0, 0, 0);
    }
  };
  int k = 0;
  for (; k + UN <= ntile; k += UN) full_steps<0, UN>(k, step);
  unrolled_steps<0, UN>(k, ntile, step);

  // ---- merge the 8 waves: common maximum per head, rescale, sum through LDS ---------------------
  // (a lane's accumulators of head tile t all belong to head t*16 + n: the D operand's column)
  if (kg == 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t) msh[w][t * 16 + n] = m[t];
  }
  __syncthreads();
  float mall[NT], wsc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float mm = NEG_INF;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) mm = fmaxf(mm, msh[ww][t * 16 + n]);
    mall[t] = mm;
    wsc[t] = (m[t] == NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(m[t] - mm);
    float lw = accl[t][0] * wsc[t];
    if constexpr (FULL) {                               // the four row groups' shares
      lw += __shfl_xor(lw, 16);
      lw += __shfl_xor(lw, 32);
    }
    if (kg == 0) lsh[w][t * 16 + n] = lw;
  }
#pragma unroll
  for (int t0 = 0; t0 < NT; t0 += TP) {
    if (t0 > 0) __syncthreads();                        // (the tiles before have been read)
#pragma unroll
    for (int tt = 0; tt < TP; ++tt)
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[w][tt][r][i][lane] = acc[i][t0 + tt][r] * wsc[t0 + tt];
    __syncthreads();
    // thread (tt, r, lane): columns col0 + (rg*4 + r)*8 .. +7 of head tile t0 + tt, head n; with one tile at a time the
    // two halves of the waves take four of the eight columns each
    constexpr int IC = TP == 2 ? 8 : 4;
    const int tt = TP == 2 ? w >> 2 : 0, i0 = TP == 2 ? 0 : (w >> 2) * 4, r = w & 3;
    const int h = hg * (NT * 16) + (t0 + tt) * 16 + n;
    float o[IC];
#pragma unroll
    for (int i = 0; i < IC; ++i) {
      float sum = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) sum += red[ww][tt][r][i0 + i][lane];
      o[i] = sum;
    }
    if (h < H) {
      float* dst = Cpart + ((size_t)pid * H + h) * dm + col0 + (rg * 4 + r) * 8 + i0;
      *reinterpret_cast<f32x4*>(dst) = f32x4{o[0], o[1], o[2], o[3]};
      if constexpr (IC == 8) *reinterpret_cast<f32x4*>(dst + 4) = f32x4{o[4], o[5], o[6], o[7]};
      if (cbk == 0 && r == 0 && kg == 0 && i0 == 0) {
        float l = 0.f, mh = NEG_INF;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) l += lsh[ww][(t0 + tt) * 16 + n];
#pragma unroll
        for (int t = 0; t < NT; ++t) mh = t == t0 + tt ? mall[t] : mh;
        mpart[(size_t)pid * H + h] = mh;
        lpart[(size_t)pid * H + h] = l;
      }
    }
  }
}


}  // namespace

// Head tiles in flight for H heads: 1, 2, 4 or 8.
static int head_tiles_in_flight(int H) {
  const int nht = (H + 15) / 16;
  int p = 1;
  while (p < nht && p < 8) p *= 2;
  return p;
}
// (heads of at most 128 columns: q~ holds four k-steps of a head's columns, the projection a head's output block in one
// tile of 128)
bool xcache_fast_ok(int dtype, int H, int d_model, int d_k) {
  return dtype == DT_BF16 && d_model % 128 == 0 && d_k % 32 == 0 && d_k >= 32 && d_k <= 128 && H >= 1 && d_model < (1 << 22);
}

int xcache_splits(int B, int H, int T, int d_model) {
  // The weighted sum runs one workgroup per (split, 32 heads, 128 columns, sequence): split the context
  // across workgroups only as far as it takes to fill the chip (every split costs a partial).
  const int per = B * ((H + 31) / 32) * (d_model >= 128 ? d_model / 128 : 1);
  int s = (256 + per - 1) / per;
  const int cap = (T + 255) / 256;
  if (s > cap) s = cap;
  if (s > PROJ_MAX_PARTS) s = PROJ_MAX_PARTS;
  return s < 1 ? 1 : s;
}

// Two passes over X: the second finds X in the memory-side cache, and nontemporal weights gain nothing beside it (64 heads x 8 x
// 8192 rows x 2048 columns 178.4 -> 179.0 us).
bool xcache_read_once(int B, int T, int d_model, int e, bool ragged, bool one_pass) {
  return one_pass && read_once(4 * (size_t)e * d_model, ragged ? 0 : 2 * (size_t)B * T * d_model);
}

void launch_xq_tilde(const float* q, const void* Wk, float* qt, int B, int H, int d_k, int d_model, int e,
                     float scale, bool once, int* counters, int ncounters, hipStream_t st) {
  dim3 grid((H + XQ_HEADS - 1) / XQ_HEADS, (d_model + 127) / 128, (B + 15) / 16);
  auto go = [&](auto nt) {
    hipLaunchKernelGGL(xq_tilde_kernel<decltype(nt)::value>, grid, dim3(512), 0, st, q, (const uint16_t*)Wk, (uint16_t*)qt, B, H, d_k,
                       d_model, e, scale, counters, ncounters);
  };
  if (once && grid.z == 1) go(std::true_type{});
  else go(std::false_type{});
}

void launch_xscores(const float* qt, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H,
                    int d_model, float* S, int B, hipStream_t st) {
  const int ninner = (T + XL_RB - 1) / XL_RB, colocate = colocate_units(B);
  dim3 grid(unit_grid(B, ninner, colocate));
  const uint16_t* q16 = (const uint16_t*)qt;
  const uint16_t* X16 = (const uint16_t*)X;
  switch (head_tiles_in_flight(H)) {
    case 1: hipLaunchKernelGGL(xscores_kernel<1>, grid, dim3(512), 0, st, q16, X16, x_bstride, seq_lens, T, B, H, d_model, S, colocate); break;
    case 2: hipLaunchKernelGGL(xscores_kernel<2>, grid, dim3(512), 0, st, q16, X16, x_bstride, seq_lens, T, B, H, d_model, S, colocate); break;
    case 4: hipLaunchKernelGGL(xscores_kernel<4>, grid, dim3(512), 0, st, q16, X16, x_bstride, seq_lens, T, B, H, d_model, S, colocate); break;
    default: hipLaunchKernelGGL(xscores_kernel<8>, grid, dim3(512), 0, st, q16, X16, x_bstride, seq_lens, T, B, H, d_model, S, colocate); break;
  }
}

void launch_xweighted(const float* S, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H,
                      int d_model, int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st) {
  const int ninner = ((H + 31) / 32) * (d_model / 128), colocate = colocate_units(B * nsplit);
  dim3 grid(unit_grid(B * nsplit, ninner, colocate));
  hipLaunchKernelGGL((xweighted_kernel<2, false>), grid, dim3(512), 0, st, S, (const uint16_t*)X, x_bstride, seq_lens, T, B, H,
                     d_model, nsplit, Cpart, mpart, lpart, colocate);
}

void launch_xweighted_full(const float* S, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int nsplit,
                           float* Cpart, float* mpart, float* lpart, int B, hipStream_t st) {
  const int nt = kweighted_tiles(H);
  const int ninner = ((H + nt * 16 - 1) / (nt * 16)) * (d / 128), colocate = colocate_units(B * nsplit);
  dim3 grid(unit_grid(B * nsplit, ninner, colocate));
  if (nt == 3)
    hipLaunchKernelGGL((xweighted_kernel<3, true>), grid, dim3(512), 0, st, S, (const uint16_t*)K, k_bstride, seq_lens, T, B, H, d,
                       nsplit, Cpart, mpart, lpart, colocate);
  else
    hipLaunchKernelGGL((xweighted_kernel<2, true>), grid, dim3(512), 0, st, S, (const uint16_t*)K, k_bstride, seq_lens, T, B, H, d,
                       nsplit, Cpart, mpart, lpart, colocate);
}

}  // namespace slim
