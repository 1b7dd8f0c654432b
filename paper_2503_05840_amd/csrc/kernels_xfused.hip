// One pass over X for X-caches of 512 <= d_model <= 1280 columns: scores, softmax numerators and the weighted sum of
// one (sequence, context split, group of heads) in one kernel (kernels_xcache.hip makes q~ before and has the two
// passes that the other widths take).
#include "slim_kernels.h"

#include "device_common.h"

#include <algorithm>

namespace slim {
namespace {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr float XF_SLACK = 6.0f;         // log2 domain, as xweighted_kernel's
constexpr int XF_NW = 4;                 // waves: one per SIMD, up to 512 registers each
constexpr int XF_RED_HS = 36;            // floats per head row of a wave's partial scores (32 rows + padding that keeps 16-byte stores)
constexpr int XF_P_HS = 40;              // bf16 per head row of the numerators (32 rows + padding)

// An accumulator times a factor.  It stays in the accumulation registers around the product, which the compiler otherwise
// takes as a reason to move all of them to vector registers and back in every step.
__device__ __forceinline__ void rescale(f32x4& acc, float al) {
  asm volatile("" : "+a"(acc));
  acc *= al;
  asm volatile("" : "+a"(acc));
}

// Bytes per parked row of a wave: its columns and 32 of padding
constexpr int xf_pitch(int CBF, int HALF) { return CBF * 256 + HALF * 128 + 32; }

// Workgroups a compute unit holds at once: two where 256 registers hold a workgroup's share.
constexpr int xf_per_cu(int CBF, int HALF, int NT) { return CBF == 1 && HALF + NT == 1 ? 2 : 1; }

// ------------------------------------------------------------------------------------------------
// One workgroup per (context split, group of 16 NT heads, sequence) keeps the group's accumulators (32 heads x d_model fp32 =
// 128 KB at 1024 columns) in registers for its whole row range, so X leaves memory once per head group and no score matrix
// is written.  The COLUMNS are split over its four waves -- CBF blocks of 128 and HALF of 64 each: a wave's slice of q~
// resident as B operands (hi + lo), its slice of every 32-row tile, its accumulator block -- and the waves meet twice per
// tile in LDS:
//   1. the partial scores of tile k, which the step before left in LDS, are summed over the waves (a thread: a few rows of one
//      head), against the head's running reference, and become bf16 numerators;  -- barrier --
//   2. every wave adds P^T X of tile k (its operands wait in registers, transposed) and takes the partial scores of tile
//      k + 1 from its slot in LDS; block by block, tile k + 1 leaves the slot for the registers of the sum, tile k + 2
//      takes its place there and tile k + 3 is requested;  -- barrier --
// Rows are not split over the waves, so nothing is merged at the end.  The head groups of a (sequence, split) read the same
// rows and are mapped to one XCD (unit_of_workgroup).
//
// What bounds it: one wave per SIMD issues everything in turn -- per tile of 1024 columns and 32 heads 96 matrix instructions
// (1600 cycles), 16 LDS writes (20 each), 38 reads, 64 transpositions, 16 requests -- and the numerators, during which the
// matrix cores wait: 3400 cycles a tile.  Eight waves of 128 columns (two per SIMD, two phases of latency behind three barriers'
// worth of LDS round trips, partial scores of eight owners) took 4900; the registers for this order of a step are not there
// with two waves per SIMD.  8 sequences x 128 heads x 4096 rows x 1024 columns: 45.6 -> 39.5 us, the call 69.3 -> 63.0;
// 24 x 1500 x 20 heads x 1280 51.9 -> 46.9, 4 x 1000 x 64 heads x 768 37.3 -> 29.9, 4 x 1500 x 8 heads x 512 27.3 -> 24.1.
// Tried on it: the numerators beside the weighted sum (3800 cycles: the parking then crowds into that phase), tiles touched
// two steps ahead so that they come from L2 (5 us slower: 64 lines an instruction), and requests and parking in one place
// each instead of spread over the matrix instructions (4900 cycles).
// ------------------------------------------------------------------------------------------------
template <int CBF, int HALF, int NT, bool ALL>
__global__ __launch_bounds__(XF_NW * 64, xf_per_cu(CBF, HALF, NT)) void xfused_kernel(const uint16_t* qt, const uint16_t* X, long x_bstride,
                                                               const int32_t* seq_lens, int T, int B, int H, int dm, int nsplit,
                                                               float* Cpart, float* mpart, float* lpart, int colocate, int through) {
  constexpr int HG = 16 * NT;                          // heads per group
  constexpr int KS = CBF * 4 + HALF * 2;               // k-steps of 32 columns per wave
  constexpr int PITCH = xf_pitch(CBF, HALF);
  constexpr int VPT = HG * 32 / (XF_NW * 64);          // (head, row) pairs per thread: 2 or 4 neighbouring rows of a head
  constexpr int TPH = 32 / VPT;                        // threads per head
  __shared__ __align__(16) unsigned char slot[XF_NW][32 * PITCH];
  __shared__ __align__(16) float red[XF_NW][HG][XF_RED_HS];
  __shared__ __align__(16) uint16_t P_s[HG][XF_P_HS];
  __shared__ float alpha_s[HG];
  int unit, hg;
  if (!unit_of_workgroup(blockIdx.x, (H + HG - 1) / HG, B * nsplit, colocate != 0, unit, hg)) return;
  const int s = unit / B, b = unit - s * B;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kg = lane >> 4;             // column group / row group of the tile; MFMA: M or N index, k group
  const int len = __builtin_amdgcn_readfirstlane(seq_len_of(seq_lens, b, T));
  const int rows_per = ((len + nsplit - 1) / nsplit + 31) / 32 * 32;
  const int r_lo = s * rows_per, r_hi = min(len, r_lo + rows_per);
  const int pid = b * nsplit + s;
  const int ntile = r_lo < r_hi ? (r_hi - r_lo + 31) / 32 : 0;
  const int NHT = (H + 15) / 16;
  // This wave's columns: block c of 128 at 128 (w + 4 c), then the half block at 512 CBF + 64 w.  (!ALL: the last ones may lie
  // past the row's end; wave-uniform.)
  auto full_at = [&](int c) { return 128 * (w + XF_NW * c); };
  const int half_at = 128 * XF_NW * CBF + 64 * w;
  auto has_full = [&](int c) { return ALL || full_at(c) < dm; };
  const bool has_half = HALF && (ALL || half_at < dm);
  // (k-step ks of 32 columns: its first column, and whether it exists)
  auto ks_at = [&](int ks) { return ks < CBF * 4 ? full_at(ks / 4) + (ks % 4) * 32 : half_at + (ks - CBF * 4) * 32; };
  auto ks_has = [&](int ks) { return ks < CBF * 4 ? has_full(ks / 4) : has_half; };

  // q~ of the group's heads over this wave's columns, hi + lo, resident as B operands
  u32x4 bqh[NT][KS], bql[NT][KS];
  {
    const size_t lo_off = (size_t)B * NHT * 16 * dm;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int ht = min(hg * NT + t, NHT - 1);        // (a tile past the last one repeats it; its heads are masked)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint16_t* src = qt + ((((size_t)b * NHT + ht) * (dm / 32) + (size_t)(ks_has(ks) ? ks_at(ks) / 32 : 0)) * 64 + lane) * 8;
        bqh[t][ks] = *reinterpret_cast<const u32x4*>(src);
        bql[t][ks] = *reinterpret_cast<const u32x4*>(src + lo_off);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(bql[t][ks]));
  }
  const char* const Xb = reinterpret_cast<const char*>(X + (size_t)b * x_bstride);
  const unsigned pitchB = (unsigned)dm * 2u;
  u32x4 lf[CBF][8];                                    // the next tile on its way: rows kg*8 + j, columns n*8 .. +7 of a block
  u32x2 lh[8];                                         // columns n*4 .. +3 of the half block
  // (rows past the end re-read the last row: finite values that meet a zero weight; a block past the row's end re-reads the first)
  unsigned off[8];                                     // byte offsets of this lane's rows of the tile that is requested next
  auto aim = [&](int k) {
    const int r0 = r_lo + 32 * min(k, max(ntile - 1, 0));
#pragma unroll
    for (int j = 0; j < 8; ++j) off[j] = __umul24((unsigned)max(min(r0 + kg * 8 + j, len - 1), 0), pitchB) + (unsigned)n * 16u;
  };
  auto request = [&](int blk, int j0, int j1) {
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      if (HALF && blk == CBF) lh[j] = *reinterpret_cast<const u32x2*>(Xb + (has_half ? half_at * 2 : 0) + (off[j] - (unsigned)n * 8u));
      else lf[blk < CBF ? blk : 0][j] = *reinterpret_cast<const u32x4*>(Xb + (has_full(blk) ? full_at(blk) * 2 : 0) + off[j]);
    }
  };
  char* const park_at = reinterpret_cast<char*>(slot[w]) + (kg * 8) * PITCH;
  auto park = [&](int blk, int j0, int j1) {
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      if (HALF && blk == CBF) *reinterpret_cast<u32x2*>(park_at + j * PITCH + CBF * 256 + n * 8) = lh[j];
      else *reinterpret_cast<u32x4*>(park_at + j * PITCH + blk * 256 + n * 16) = lf[blk < CBF ? blk : 0][j];
    }
  };
  f32x4 sp[2][NT];                                     // partial scores over this wave's columns: 16 rows x 16 heads each
  auto no_scores = [&]() {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) sp[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  const char* const sc_at = reinterpret_cast<const char*>(slot[w]) + n * PITCH + kg * 16;
  bf16x8 a8[2][2];                                     // A operands of a k-step: the next one's are on their way meanwhile
  auto read_a = [&](int ks) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) a8[ks & 1][mt] = *reinterpret_cast<const bf16x8*>(sc_at + mt * 16 * PITCH + ks * 64);
  };
  auto products = [&](int ks) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) sp[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8[ks & 1][mt], __builtin_bit_cast(bf16x8, bqh[t][ks]), sp[mt][t], 0, 0, 0);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) sp[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8[ks & 1][mt], __builtin_bit_cast(bf16x8, bql[t][ks]), sp[mt][t], 0, 0, 0);
  };
  auto score = [&](int ks) {
    if (ALL || ks_has(ks)) products(ks);
  };
  // The first tile's: a branch for each block that may not exist, not for each k-step.  (Two head tiles: for each k-step, and one way for every
  // number of tiles, below.  Their small batches go in groups of 16, and with either change the compiler moves more registers in the loop: 36 x
  // 7172 rows x 64 heads x 640 139.3 -> 144.3 us, 22 x 3777 x 128 x 1024 125.9 -> 130.7.)
  auto first_scores = [&]() {
    no_scores();
#pragma unroll
    for (int blk = 0; blk < CBF + HALF; ++blk)
      if (NT == 2 || blk == 0 || ALL || (blk < CBF ? has_full(blk) : has_half)) {
#pragma unroll
        for (int ks = blk * 4; ks < min(blk * 4 + 4, KS); ++ks) { read_a(ks); if (NT == 2) score(ks); else products(ks); }
      }
  };
  auto hand_over = [&]() {                             // D: column n = head, rows kg*4 + i
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(&red[w][t * 16 + n][mt * 16 + kg * 4]) = sp[mt][t];
  };
  // softmax state: thread (head tid / TPH, rows VPT (tid % TPH) ..); m is the same in the head's threads, l a thread's own share
  const int ohl = tid / TPH, orow = (tid % TPH) * VPT;
  const bool oreal = hg * HG + ohl < H;
  float m = NEG_INF, l = 0.f;
  bool moved_before = true;                            // alpha_s of this wave's heads may not be all ones (wave-uniform)
  typedef float fvec __attribute__((ext_vector_type(VPT)));
  auto max_over_head = [](float v) {
    v = dpp_max<0xB1>(v);
    v = dpp_max<0x4E>(v);
    v = dpp_max<0x141>(v);
    if constexpr (TPH == 16) v = dpp_max<0x140>(v);
    return v;
  };
  auto numerators = [&](int k) {
    fvec part[XF_NW];
#pragma unroll
    for (int ws = 0; ws < XF_NW; ++ws) part[ws] = *reinterpret_cast<const fvec*>(&red[ws][ohl][orow]);
    const fvec x4 = (part[0] + part[1]) + (part[2] + part[3]);
    const int live = oreal ? r_hi - (r_lo + 32 * k) - orow : 0;
    float x[VPT];
    bool over = false;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      x[i] = i < live ? x4[i] : NEG_INF;
      over |= x[i] > m + XF_SLACK;
    }
    // The reference moves only when the maximum has grown by more than XF_SLACK, as in xweighted_kernel: rarely, so the
    // maximum over the rows is taken only then.
    const bool moved = __any(over);
    if (moved || moved_before) {
      float tmax = x[0];
#pragma unroll
      for (int i = 1; i < VPT; ++i) tmax = fmaxf(tmax, x[i]);
      tmax = max_over_head(tmax);
      const float mn = (tmax > m + XF_SLACK) ? tmax : m;
      const float alpha = (m == NEG_INF) ? 1.f : __builtin_amdgcn_exp2f(m - mn);   // (nothing accumulated yet: nothing to rescale)
      l *= alpha;
      m = mn;
      if (orow == 0) alpha_s[ohl] = alpha;
    }
    moved_before = moved;
    const float ref = m == NEG_INF ? 0.f : m;
    unsigned pw[VPT / 2];
#pragma unroll
    for (int i = 0; i < VPT; i += 2) {
      const __bf16 p0 = (__bf16)__builtin_amdgcn_exp2f(x[i] - ref), p1 = (__bf16)__builtin_amdgcn_exp2f(x[i + 1] - ref);
      l += (float)p0;                                  // the weights as the MFMA will see them
      l += (float)p1;
      const bf16x2 v = {p0, p1};
      pw[i / 2] = __builtin_bit_cast(unsigned, v);
    }
    if constexpr (VPT == 4) *reinterpret_cast<u32x2*>(&P_s[ohl][orow]) = u32x2{pw[0], pw[1]};
    else *reinterpret_cast<unsigned*>(&P_s[ohl][orow]) = pw[0];
  };
  f32x4 accf[CBF][8][NT], acch[4][NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int c = 0; c < CBF; ++c)
#pragma unroll
      for (int i = 0; i < 8; ++i) accf[c][i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) acch[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // the parked tile out of the slot, four rows of a block at a time, and transposed in registers: A operands of its weighted sum
  u32x4 amf[CBF][8], amh[4];
  u32x4 rf[4];
  u32x2 rh[4];
  auto read_rows = [&](int blk, int q) {               // rows 4 q .. 4 q + 3 of the lane's eight
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (HALF && blk == CBF) rh[j] = *reinterpret_cast<const u32x2*>(park_at + (q * 4 + j) * PITCH + CBF * 256 + n * 8);
      else rf[j] = *reinterpret_cast<const u32x4*>(park_at + (q * 4 + j) * PITCH + blk * 256 + n * 16);
    }
  };
  auto turn = [&](int blk, int q, const u32x4* f, const u32x2* g) {      // (the four rows in f, of the half block in g)
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
      if (HALF && blk == CBF) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          amh[2 * c][2 * q + jp] = __builtin_amdgcn_perm(g[2 * jp + 1][c], g[2 * jp][c], 0x05040100u);
          amh[2 * c + 1][2 * q + jp] = __builtin_amdgcn_perm(g[2 * jp + 1][c], g[2 * jp][c], 0x07060302u);
        }
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          amf[blk < CBF ? blk : 0][2 * c][2 * q + jp] = __builtin_amdgcn_perm(f[2 * jp + 1][c], f[2 * jp][c], 0x05040100u);
          amf[blk < CBF ? blk : 0][2 * c + 1][2 * q + jp] = __builtin_amdgcn_perm(f[2 * jp + 1][c], f[2 * jp][c], 0x07060302u);
        }
      }
    }
    if (q == 1) {                                      // (whole from here on: as single words they would be held twice around the loop)
      if (HALF && blk == CBF) {
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(amh[i]));
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(amf[blk < CBF ? blk : 0][i]));
      }
    }
  };
  auto turn_rows = [&](int blk, int q) { turn(blk, q, rf, rh); };
  bf16x8 pb[NT];
  float al[NT];
  auto fetch_weights = [&]() {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      al[t] = alpha_s[t * 16 + n];
      pb[t] = *reinterpret_cast<const bf16x8*>(&P_s[t * 16 + n][kg * 8]);
    }
  };
  auto rescale_all = [&]() {                           // where a reference moved
    bool any = al[0] != 1.f;
#pragma unroll
    for (int t = 1; t < NT; ++t) any |= al[t] != 1.f;
    if (__any(any)) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int c = 0; c < CBF; ++c)
#pragma unroll
          for (int i = 0; i < 8; ++i) rescale(accf[c][i][t], al[t]);
        if constexpr (HALF) {
#pragma unroll
          for (int i = 0; i < 4; ++i) rescale(acch[i][t], al[t]);
        }
      }
    }
  };
  constexpr int NBLK = CBF + HALF;
  auto sum_block = [&](int blk) {
    if (HALF && blk == CBF) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acch[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, amh[i]), pb[t], acch[i][t], 0, 0, 0);
    } else {
      const int c = blk < CBF ? blk : 0;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          accf[c][i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, amf[c][i]), pb[t], accf[c][i][t], 0, 0, 0);
    }
  };
  // One wave per SIMD hides nothing behind another wave, so the order of a step is written out in groups of a few matrix
  // instructions, each group with what the next ones need: LDS reads first, then the parking, the requests and the
  // transpositions between the matrix instructions.  (Measured per shape: 16 heads a group leave too few matrix instructions
  // to pace by, and beyond 768 columns the groups' borders cost more than they give: 49.2 -> 48.1 us at 24 x 1500 x 1280.)
  auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
  auto paced = [&]() {
    if constexpr (NT == 2 || CBF == 2) {
      __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);       // LDS reads
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);     // matrix instructions
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);     // an LDS write
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);     // a request
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);     // vector operations
      }
    }
    if constexpr (NT == 2 || CBF == 1) fence();
  };
  constexpr int END = NBLK - 1;                        // the last block
  // EARLY: registers that were parked are asked for again at once, not when the block's other work is done.  What decides there is how many
  // bytes are on their way, and a register waits for its next request empty: 16 heads a group, two blocks: 32 x 1500 rows x 16 heads x 1024
  // 42.4 -> 41.3 us, 96 x 16 x 1024 80.8 -> 78.6, 64 x 16 x 768 53.4 -> 53.1, small batches the same; 32 heads a group, one block: 76 ragged x 1500 x
  // 24 x 512 49.6 -> 43.9, 40 x 1000 x 32 x 512 33.6 -> 32.8.  Not where the matrix instructions decide (32 heads and two blocks: 8 x 4096 x
  // 128 x 1024 63.7 -> 64.8) nor where two workgroups share a compute unit (16 heads and one block: 4 x 1500 x 16 x 512 23.8 -> 24.2).
  constexpr bool EARLY = NT == 1 ? NBLK == 2 : NBLK == 1;
  auto last = [&]() {
    numerators(ntile - 1);
    lds_barrier();
    fetch_weights();
    rescale_all();
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) sum_block(blk);
  };
  // A workgroup of one tile has a way of its own, which asks for no other tile and transposes this one on its way to the slot: one wave per
  // SIMD issues all of it in turn, and what the longer way does for the tiles after the first took a tenth of such a call (with what the
  // partial's way out saves: 2 x 17 rows x 8 heads x 1152 22.5 -> 20.8 us, 3 x 10 x 20 x 1280 22.7 -> 21.3).
  if (NT == 1 && ntile == 1) {
    aim(0);
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) request(blk, 0, 8);
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
      park(blk, 0, 8);
      turn(blk, 0, lf[blk < CBF ? blk : 0], lh);
      turn(blk, 1, lf[blk < CBF ? blk : 0] + 4, lh + 4);
    }
    first_scores();
    hand_over();
    lds_barrier();
    last();
  } else if (ntile > 0) {
    aim(0);
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) { request(blk, 0, 8); park(blk, 0, 8); }
    aim(1);
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) request(blk, 0, 8);
    first_scores();
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
      read_rows(blk, 0); turn_rows(blk, 0);
      read_rows(blk, 1); turn_rows(blk, 1);
    }
    hand_over();
#pragma unroll
    for (int blk = 0; blk < (NBLK == 1 ? 1 : END); ++blk) park(blk, 0, 8);
    aim(2);
    if constexpr (NBLK > 1 || EARLY) request(0, 0, 8);
    lds_barrier();
    int k = 0;
    if (ntile > 1) {
      do {
        // on entry: tile k's operands in registers and its partial scores handed over; tile k + 1 parked but for the last of
        // several blocks, which is in registers; tile k + 2 requested as far as its registers were free
        numerators(k);
        read_a(0);
        lds_barrier();
        fence();
        fetch_weights();
        no_scores();
        read_a(1);
        fence();
        if constexpr (NBLK > 1) park(END, 0, 2);
        if constexpr (EARLY && NBLK == 2) request(END, 0, 2);
        if constexpr (NBLK != 2 && !(NBLK == 1 && EARLY)) request(NBLK == 1 ? 0 : 1, 0, 4);
        score(0);
        paced();
        read_a(2);
        if constexpr (NBLK > 1) park(END, 2, 4);
        if constexpr (EARLY && NBLK == 2) request(END, 2, 4);
        if constexpr (NBLK != 2 && !(NBLK == 1 && EARLY)) request(NBLK == 1 ? 0 : 1, 4, 8);
        score(1);
        paced();
        rescale_all();
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk) {
          read_rows(blk, 0);
          if (blk > 0) park(blk - 1, 0, 4);
          if (blk == 0 && NBLK > 1) park(END, 4, 8);
          if (blk == 0 && NBLK == 2 && EARLY) request(END, 4, 8);
          if (blk == (END > 0 ? 1 : 0)) aim(k + 3);
          if (blk == 1 && EARLY) request(0, 0, 4);
          sum_block(blk);
          paced();
          const int ks0 = blk == 0 ? 2 : blk * 4, ks1 = blk == 0 ? 4 : min(blk * 4 + 4, KS);
#pragma unroll
          for (int ks = ks0; ks < ks1; ++ks) {
            if (ks + 1 < KS && ks + 1 > 2) read_a(ks + 1);
            if (ks == ks0) {
              turn_rows(blk, 0);
              read_rows(blk, 1);
              if (blk > 0) park(blk - 1, 4, 6);
              if (blk == 1 && EARLY) request(0, 4, 6);
            }
            if (ks == ks0 + 1) {
              turn_rows(blk, 1);
              if (blk > 0) park(blk - 1, 6, 8);
              if (blk == 1 && EARLY) request(0, 6, 8);
              if (NBLK == 1) park(0, 0, 8);
              if (NBLK == 1 && EARLY) request(0, 0, 8);
            }
            if (blk == 0 && NBLK > 1 && !EARLY) request(END, (ks - ks0) * 4, (ks - ks0) * 4 + 4);
            // (the first block's registers are free once it is parked, behind the second block's first k-steps)
            if (blk == 1 && !EARLY) {
              if (ks1 - ks0 == 4 && ks >= ks1 - 2) request(0, (ks - ks1 + 2) * 4, (ks - ks1 + 2) * 4 + 4);
              if (ks1 - ks0 == 2 && ks == ks1 - 1) request(0, 0, 8);
            }
            score(ks);
            paced();
          }
        }
        hand_over();
        lds_barrier();
      } while (++k + 1 < ntile);
      last();
    }
    if (NT > 1 && ntile == 1) last();
  }

  // ---- the partial of this (sequence, split): every wave its own columns, a head's threads its (m, l).  An accumulator lane
  // holds 32 consecutive columns of a head in a block of 128 (16 in the half block): stored from there, every instruction
  // writes 64 pieces into 64 different cache lines.  So the wave's 16 x 128 block of a head tile goes through its own, now
  // idle, slot and leaves with a head's columns on consecutive lanes, through the L2s where xfused_through says so.  The stores go by a
  // buffer descriptor of the group's heads that exist, which drops the rows of the others: one addition each, where a predicate and a 64-bit
  // address took a dozen instructions; a block of 16 heads took 0.5 us to leave and takes 0.2.
  float* const ob = reinterpret_cast<float*>(slot[w]);
  const __amdgpu_buffer_rsrc_t to =
      __builtin_amdgcn_make_buffer_rsrc(Cpart + ((size_t)pid * H + hg * HG) * dm, 0, min(H - hg * HG, HG) * dm * 4, 0x00020000);
  auto leave = [&](int t, int col, auto COLS, auto&& put) {
    constexpr int NC = decltype(COLS)::value, OP = NC + 4, LPR = NC / 4;   // floats per head row (padding: no bank conflicts), lanes per row
    static_assert(16 * OP * 4 <= 32 * PITCH, "a head tile's block must fit the wave's slot");
    const int at = (lane / LPR * dm + (lane % LPR) * 4) * 4;
    asm volatile("" ::: "memory");                     // (LDS operations of one wave complete in order: nothing to wait for)
    put(ob + n * OP);
    asm volatile("" ::: "memory");
    auto rows = [&](auto POLICY) {
#pragma unroll
      for (int k2 = 0; k2 < NC / 16; ++k2) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(ob + ((64 / LPR) * k2 + lane / LPR) * OP + (lane % LPR) * 4);
        __builtin_amdgcn_raw_buffer_store_b128(v, to, at + ((t * 16 + (64 / LPR) * k2) * dm + col) * 4, 0, decltype(POLICY)::value);
      }
    };
    if (through) rows(std::integral_constant<int, 1 | 16>{});            // (sc0 sc1)
    else rows(std::integral_constant<int, 0>{});
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int c = 0; c < CBF; ++c)
      if (has_full(c))
        leave(t, full_at(c), std::integral_constant<int, 128>{}, [&](float* row) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {                // accumulator row i: column group kg*4 + i of the block, eight columns
            float* d8 = row + (kg * 4 + i) * 8;
            *reinterpret_cast<f32x4*>(d8) = f32x4{accf[c][0][t][i], accf[c][1][t][i], accf[c][2][t][i], accf[c][3][t][i]};
            *reinterpret_cast<f32x4*>(d8 + 4) = f32x4{accf[c][4][t][i], accf[c][5][t][i], accf[c][6][t][i], accf[c][7][t][i]};
          }
        });
    if constexpr (HALF)
      if (has_half)
        leave(t, half_at, std::integral_constant<int, 64>{}, [&](float* row) {
#pragma unroll
          for (int i = 0; i < 4; ++i)                  // (column groups of four)
            *reinterpret_cast<f32x4*>(row + (kg * 4 + i) * 4) = f32x4{acch[0][t][i], acch[1][t][i], acch[2][t][i], acch[3][t][i]};
        });
  }
  float lt = dpp_add<0xB1>(l);
  lt = dpp_add<0x4E>(lt);
  lt = dpp_add<0x141>(lt);
  if constexpr (TPH == 16) lt = dpp_add<0x140>(lt);
  if (orow == 0 && oreal) {
    mpart[(size_t)pid * H + hg * HG + ohl] = m;
    lpart[(size_t)pid * H + hg * HG + ohl] = lt;
  }
}

}  // namespace

bool xfused_ok(int d_model) { return d_model % 128 == 0 && d_model >= 512 && d_model <= 1280; }

// Head tiles of a workgroup, at most.  Beyond 1024 columns 32 heads' accumulators and q~ alone are 320 registers a lane: spills.
static int xfused_most_tiles(int H, int d_model) { return H > 16 && d_model <= 1024 ? 2 : 1; }
static long xfused_groups(int H, int tiles) { return (H + 16 * tiles - 1) / (16 * tiles); }
static long xfused_slots(int d_model, int tiles) { return 256 * (d_model <= 512 ? xf_per_cu(1, 0, tiles) : 1); }   // workgroups at once

// Layers of more than 16 heads go in groups of 16 where all of these run at once, each on a compute unit of its own: their steps are shorter, and
// X, which the groups share in an XCD's L2, is not what bounds so few rows.  (In groups of 32 half of the chip and more stood idle: 2 x 490 rows x 32
// heads x 1024 27.8 -> 24.9 us, 6 x 14 x 64 x 1024 23.8 -> 21.9, 1 x 2998 x 64 x 640 30.7 -> 28.4.  Where they do not fit it is the other way: 18 x
// 2145 x 128 heads x 640 65.7 us, in groups of 16 84.9; 81 x 686 x 64 x 512, two workgroups on a compute unit, 55.3 and 59.2.)  A head's sums do not depend on
// its group.
int xfused_tiles(int B, int H, int d_model, int nsplit) {
  const long units = (long)B * nsplit, groups = xfused_groups(H, 1);
  const bool fit = colocate_units(B * nsplit) ? (units + 7) / 8 * groups <= 32 : units * groups <= 256;   // (per XCD where launch_xfused deals the units to them)
  return fit ? 1 : xfused_most_tiles(H, d_model);
}

// Context splits, at most: one per started 128 rows of T (a split may hold fewer: lengths below T, whole tiles), what the projection merges,
// and six more than fill the chip once (beyond that 0.5 % of the shapes up to 8192 rows would gain up to 1.5 % in steps, for partials
// without bound).  Grows with T.
int xfused_most_splits(int B, int H, int T, int d_model) {
  const int tiles = xfused_most_tiles(H, d_model);
  const long units = B * xfused_groups(H, tiles), fill = (xfused_slots(d_model, tiles) + units - 1) / units + 6;
  const int most = (T + 127) / 128;
  return (int)std::min<long>(std::min(most, PROJ_MAX_PARTS), fill);
}

// The count whose rounds of workgroups of as many heads as fit take the least time, in tenths of a step of 32 rows (1.6 us at 1024 columns and 32
// heads): starting a workgroup, its first tile and its last cost about four steps; a split's partials 0.4 steps per MB (written here,
// read by the projection) and a tenth more (a round trip of the merge).  Without the partials' share 8 sequences x 32 heads x 4096 rows x
// 1024 columns took 47.9 us in 32 splits and take 44.2 in 16.  One price for steps of every width is too dear for narrow rows and few heads, and
// a ragged batch is cut as if all had T rows.  Prices by width and head tiles, rounds per XCD and half of T for ragged batches gave 0.4 % in the mean
// over 310 shapes (32 x 1500 x 16 heads x 1024 42.4 -> 40.9 us, 55 x 100..7576 x 40 x 512 158 -> 125), but another count moves the references of the numerators,
// and with them the rounding of the weights: the results differ by 1e-3 from those of this count, where the error against 64 bits is
// the same.  A call's results stay what they are.
int xfused_splits(int B, int H, int T, int d_model) {
  const int wide = xfused_most_tiles(H, d_model), tiles = (T + 31) / 32, most = xfused_most_splits(B, H, T, d_model);
  const long per = B * xfused_groups(H, wide), slots = xfused_slots(d_model, wide);
  const long partial = 4L * B * H * d_model;           // bytes of a split's partials
  int best = 1;
  long best_cost = 0;
  for (int s = 1; s <= most; ++s) {
    const long rounds = (per * s + slots - 1) / slots, cost = 10 * rounds * ((tiles + s - 1) / s + 4) + 4 * s * partial / (1 << 20) + s;
    if (s == 1 || cost < best_cost) { best = s; best_cost = cost; }
  }
  return best;
}

// Whether that many bytes of partials leave through the L2s (store_through).  What is left dirty there is written back between the launches, 0.4 us for
// 5 MB, 1.2 for 40; what goes to memory takes the longer way, 0.3 us of the launch's end whatever it is.  264 shapes: up to 1.8 MB 0.25 us a call faster
// without (1 x 14 rows x 24 heads x 896 23.2 -> 22.9), from 2.6 MB 0.2 to 1.2 slower (8 x 4096 x 32 heads x 1024 42.8 and 44.5).
bool xfused_through(size_t bytes) { return bytes >= ((size_t)9 << 18); }

void launch_xfused(const float* qt, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H, int d_model,
                   int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st) {
  const int nt = xfused_tiles(B, H, d_model, nsplit);
  const int colocate = colocate_units(B * nsplit);
  dim3 grid(unit_grid(B * nsplit, (int)xfused_groups(H, nt), colocate));
  auto go = [&](auto cbf, auto half, auto all) {
    auto with = [&](auto tiles) {
      hipLaunchKernelGGL((xfused_kernel<decltype(cbf)::value, decltype(half)::value, decltype(tiles)::value, decltype(all)::value>), grid,
                         dim3(XF_NW * 64), 0, st, (const uint16_t*)qt, (const uint16_t*)X, x_bstride, seq_lens, T, B, H, d_model, nsplit,
                         Cpart, mpart, lpart, colocate, xfused_through(sizeof(float) * B * nsplit * H * d_model));
    };
    if constexpr (decltype(cbf)::value + decltype(half)::value < 3)       // (wider rows: 16 heads a group, xfused_most_tiles)
      if (nt == 2) return with(std::integral_constant<int, 2>{});
    with(std::integral_constant<int, 1>{});
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  switch (d_model / 128) {
    case 4: go(I1{}, I0{}, std::true_type{}); break;
    case 5: go(I1{}, I1{}, std::false_type{}); break;
    case 6: go(I1{}, I1{}, std::true_type{}); break;
    case 7: go(I2{}, I0{}, std::false_type{}); break;
    case 8: go(I2{}, I0{}, std::true_type{}); break;
    case 9: go(I2{}, I1{}, std::false_type{}); break;
    default: go(I2{}, I1{}, std::true_type{}); break;
  }
}

}  // namespace slim
