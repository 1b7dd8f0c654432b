// bf16 fast path of the slim-attention decode step for gfx950 (MI355X).
//
//   fused_stream_kernel : one pass over the K-cache.  Softmax arguments (eq. 2), online softmax
//                         and the full-width weighted sum [softmax(.) K] of eq. 7 option 2, the
//                         latter as one MFMA contraction for all heads at once (the text under
//                         eq. 7 points out that the heads need not be handled one by one).  K is
//                         read from HBM once.
//   project_mfma_kernel : log-sum-exp merge of the context splits and the per-head product with
//                         W_KV,i (eq. 7 option 2, second factor) on MFMA; W_KV is read once.
//
// Why workgroups exchange scores.  The weighted sum keeps H x d fp32 accumulators per sequence
// (512 KB for H=32, d=4096: a whole CU's register file), so the row width has to be split over
// workgroups; but head h's weights need columns [h d_k, (h+1) d_k) only, which one column owner
// holds, while every column owner needs every head's weights.  A "group" of G workgroups (one per
// column unit of <=128 columns) therefore walks the same rows together; wave w of every workgroup of
// the group takes the same 32-row tiles: it computes the scores of the heads inside its unit, turns them
// into softmax numerators against the head's running reference, parks the tile in LDS and publishes
// 16-byte words {tag, reference, 4 bf16 numerators} to a small ring in global memory; one step later it
// gathers all heads' words of that tile, takes the tile out of LDS and feeds it to the MFMA.  No fences
// are needed: every 16-byte word (written by one store) carries the tile's tag, so a reader either
// sees the values of this tile or gathers again.  Every wait is bounded in real time; a time-out raises
// an error word instead of hanging.
//
// Register tile.  A wave owns 32 rows x 128 columns: lane l loads 16 bytes (8 columns) of 8 rows,
// column group l%16; the rows are 4 j + l/16 (one load instruction = four consecutive rows) or, with
// rotary keys, 8 (l/16) + j.  Both MFMA contractions take their operands from the tile's LDS
// copy.  Scores (v_mfma_f32_16x16x32_bf16, contraction over columns): A = 16 rows x 32 columns read
// straight in operand layout, B = the unit's queries.  Weighted sum (contraction over rows): a lane reads
// its 8 x 8 block back and transposes it in registers (v_perm_b32) into 8 A-operands, one per column:
// A_i[m = l%16][k = 8 rows of lane group l/16] = K[row][col (l%16)*8 + i]; the B-operand is P^T: lane
// (n = l%16, l/16) holds the weights of head n for the same 8 rows.
#include "slim_kernels.h"
#include "device_common.h"

#include <math.h>
#include <type_traits>

namespace slim {
namespace {

constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float bf16_lo(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(unsigned x) { return __uint_as_float(x & 0xffff0000u); }

// max over the four lanes l, l^16, l^32, l^48 (the same column group in the four row groups).
// Register swaps (v_permlane32_swap / v_permlane16_swap), no LDS traffic.
__device__ __forceinline__ float max_over_row_groups(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float h = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const unsigned w = __float_as_uint(h);
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Score exchange accesses.  Readers load at agent scope (never served by the CU's own vector L1).
// Writers have two flavours, chosen per launch:
//  * XCD-local (the normal case): all workgroups of a group run on one XCD (workgroup i is
//    dispatched to XCD i % 8, which the host verifies once per device), so that XCD's L2 is their
//    meeting point: a plain store (the vector L1 is write-through) is enough and the words never
//    leave the L2.
//  * system scope (fallback): write-through stores that also reach the memory side, for groups
//    whose workgroups may sit on different XCDs.
// 16-byte accesses: a wave's gather of one tile is a handful of fully coalesced 1 KB loads.
__device__ __forceinline__ u32x4 ld_exch(const u32x4* p) {
  u32x4 v;
  asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ void st_exch(u32x4* p, u32x4 v, bool xcd_local) {
  // The s_nops matter: a store of more than 64 bits still reads its data registers in the wait
  // states after it issues, and the compiler (which pads its own stores) is free to overwrite
  // the inputs of an asm statement with the very next VALU instruction.
  if (xcd_local) asm volatile("s_nop 1\n\tglobal_store_dwordx4 %0, %1, off\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  else asm volatile("s_nop 1\n\tglobal_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
// Results other workgroups of the same launch will read (write_through): stored at system scope.
__device__ __forceinline__ void st_result(float* p, float v, bool write_through) {
  if (write_through) asm volatile("global_store_dword %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
  else *p = v;
}
__device__ __forceinline__ void st_result(int* p, int v, bool write_through) {
  if (write_through) asm volatile("global_store_dword %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
  else *p = v;
}

__device__ __forceinline__ void st_result4(float* p, f32x4 v, bool write_through) {
  if (write_through) store_through(p, v);
  else *reinterpret_cast<f32x4*>(p) = v;
}

__device__ __forceinline__ unsigned my_xcc() { return __builtin_amdgcn_s_getreg((31 << 11) | 20) & 7; }   // HW_REG_XCC_ID

// Tiles of 32 rows: prefix[b] = number of tiles of sequences 0..b-1; lens_s[b] (if given) = rows of
// sequence b.  The first wave takes 64 sequences at a time, one per lane (one memory round trip per 64
// sequences instead of one per sequence), and adds them up with a scan over the lanes (prefix_over_wave).
__device__ void build_tile_prefix(int* prefix, int* lens_s, const int32_t* lens, int B, int T) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int carry = 0;
    for (int b0 = 0; b0 < B; b0 += 64) {
      const int b = b0 + lane;
      const int len = b < B ? seq_len_of(lens, b, T) : 0;
      const int v = prefix_over_wave((len + TILE_ROWS - 1) / TILE_ROWS);
      if (b < B) {
        prefix[b + 1] = carry + v;
        if (lens_s) lens_s[b] = len;
      }
      carry += __builtin_amdgcn_readlane(v, 63);
    }
    if (lane == 0) prefix[0] = 0;
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// merge + projection:  out[b][h d_k + j] = sum_c Cn[b][h][c] W[c][h d_k + j]
// One workgroup (8 waves) per (head h, row split cs of W, batch chunk bz of 16*NBT sequences).  The
// wave tile is the same 32 x 128 register tile as above (rows = c, columns = the head's output
// columns), A = W tile transposed, B = merged, normalised C^T split in bf16 hi + lo.
// What bounds it is the chain of dependent round trips around its bytes, so everything that can be asked for at once
// is: two tiles of W per wave, then the maxima and sums of all partials.
// COH: the partials come from other workgroups of the same launch (loads at agent scope, each a trip to the memory
// side): they are asked for together with their maxima and sums, a lane four consecutive rows c of one sequence and
// eight loads in flight, and the merged C goes to LDS in B-operand order (up to PROJ_STAGED_ROWS rows, in the place
// of the cross-wave sum).  Merged per tile in operand layout instead, as a launch of its own does it, that is a trip per
// tile more: 13 us instead of 10 from the last arrival to the end at 16 sequences x 4096 columns.  (As a launch of its own
// the staged form takes longer, 13.6 against 12.3 us at 64 sequences x 1280 columns with 3 partials each.)
// ------------------------------------------------------------------------------------------------
template <int NBT>
struct ProjShared {
  int pid0s[16 * NBT], nps[16 * NBT];
  float wpid[16 * NBT][PROJ_MAX_PARTS];
  float obuf[16 * NBT][128];
  int is_last;
};

template <bool COH>
__device__ __forceinline__ float ld_part(const float* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
template <bool COH>
__device__ __forceinline__ int ld_err(const int* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
// a pointer the compiler can keep in scalar registers (it is the same in every lane, which it cannot always see)
__device__ __forceinline__ const float* uniform_ptr(const float* p) {
  const unsigned long long u = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u), hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
  return (const float*)(((unsigned long long)hi << 32) | lo);
}
// eight 16-byte loads in flight together, p[q] wave-uniform, byte offsets o0 for the first four and o1 for the others, at
// agent scope: loads and their wait in one asm block
__device__ __forceinline__ void ld_part8(const float* const (&p)[8], unsigned o0, unsigned o1, f32x4 (&x)[8]) {
  asm volatile("global_load_dwordx4 %0, %8, %10 sc1\n\tglobal_load_dwordx4 %1, %8, %11 sc1\n\t"
                 "global_load_dwordx4 %2, %8, %12 sc1\n\tglobal_load_dwordx4 %3, %8, %13 sc1\n\t"
                 "global_load_dwordx4 %4, %9, %14 sc1\n\tglobal_load_dwordx4 %5, %9, %15 sc1\n\t"
                 "global_load_dwordx4 %6, %9, %16 sc1\n\tglobal_load_dwordx4 %7, %9, %17 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                 : "v"(o0), "v"(o1), "s"(p[0]), "s"(p[1]), "s"(p[2]), "s"(p[3]), "s"(p[4]), "s"(p[5]), "s"(p[6]), "s"(p[7])
                 : "memory");
}

// `red`: 64 KB of LDS: the merged C, later the cross-wave sum.
// `after_w_issue` runs (all threads) once the first tile of W is in flight and before any partial
// is read: the place to build the tile prefix, or to wait for the other workgroups' partials (false: this one has no part
// in a result, which is NaN).
// DENSE: plain products out_m = x W_m for up to three matrices that share x (ProjArgs::Wm); hx counts
// (matrix, head) column blocks.  The result leaves as fp32, or -- the new token's rows -- rotated to
// the append position and/or stored into the caches (ProjArgs::role).
// ONCE: W is read once per launch and is large: its loads ask to be let go of first (nontemporal).
// FEW: up to four sequences in a launch of its own.
template <int NBT, bool COH, bool DENSE, bool ONCE, bool FEW, class Hook>
__device__ __forceinline__ void project_work(const ProjArgs& a, int hx, int cs, int bz, const int* prefix,
                                             ProjShared<NBT>& sm, float* red, Hook&& after_w_issue) {
  const int mtx = DENSE ? hx / a.H : 0;
  const int h = DENSE ? hx - mtx * a.H : hx;
  const uint16_t* const Wmat = DENSE ? a.Wm[mtx] : a.W;
  float* const outp = DENSE ? a.outm[mtx] : a.out;
  // a head's partial sums: eight elements i of its column groups, padded to whole fours (proj_part_row)
  const int lph = a.d_k / 8, lph4 = (lph + 3) & ~3, part_row = a.H * lph4 * 8;
  float* const outpart = DENSE ? a.outpart + (size_t)mtx * a.csw * a.B * part_row : a.outpart;
  const int bbase = bz * 16 * NBT;
  const int nb = min(16 * NBT, a.B - bbase);
  constexpr int NW = 8, NTHR = 512;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int idx = lane & 15, rg = lane >> 4;
  const int n = idx, kg = rg;

  const int nhx = DENSE ? a.H * a.nmat : a.H;          // units per batch chunk
  const bool col_active = idx < lph;
  const uint16_t* Wh = Wmat + (size_t)h * a.d_k + idx * 8;
  const int c_lo = cs * a.crows, c_hi = min(a.rows, c_lo + a.crows);
  const int ntile = (c_hi - c_lo + TILE_ROWS - 1) / TILE_ROWS;
  auto load_w = [&](u32x4 (&wt)[8], int ct) {
    const int c0 = c_lo + ct * TILE_ROWS;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = min(c0 + rg * 8 + j, a.rows - 1);
      const u32x4* const src = reinterpret_cast<const u32x4*>(Wh + (size_t)r * a.e);
      if constexpr (ONCE) wt[j] = col_active ? __builtin_nontemporal_load(src) : u32x4{0u, 0u, 0u, 0u};
      else wt[j] = col_active ? *src : u32x4{0u, 0u, 0u, 0u};
    }
  };
  // DENSE: the B operand is a slice of x, known from the start: requested first, one tile ahead.
  f32x4 xc[NBT][2], xn[NBT][2];
  auto load_x = [&](f32x4 (&x)[NBT][2], int ct) {
    const int c = min(c_lo + ct * TILE_ROWS + kg * 8, a.rows - 8);
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
      const float* src = a.Cpart + (size_t)min(bbase + t * 16 + n, a.B - 1) * a.rows + c;
      x[t][0] = *reinterpret_cast<const f32x4*>(src);
      x[t][1] = *reinterpret_cast<const f32x4*>(src + 4);
    }
  };
  // DENSE, a new token's rows: where a thread's elements go (and the rotation they get) depends on their sequences' lengths.
  // Asked for behind the first tiles of W, and the rotations behind the products, so that the workgroup that finishes a unit
  // does not go to memory for one and then for the other once per element: block of 16 ragged sequences x 4096 columns with
  // rotary positions 108.9 -> 107.4 us, of 12 x 1280 columns 46.0 -> 45.6; a few sequences or no rotation: the same.
  constexpr int NE = DENSE && NBT == 1 ? 4 : 1;       // elements tid + 512 u of 16 sequences x 128 columns
  constexpr bool AHEAD = DENSE && NBT == 1;
  const int role = DENSE ? a.role[mtx] : 0;
  const bool turned = DENSE && a.rope && (role == 1 || (role == 2 && a.rotate_k));
  int el_bl[NE] = {}, el_j[NE] = {}, el_len[NE] = {};
  float el_c[NE] = {}, el_s[NE] = {};
  auto rotation = [&](int pos, int j, float& c, float& s) {
    const float* cs = a.rope + ((size_t)max(pos, 0) * (a.d_k / 2) + j / 2) * 2;
    c = cs[0]; s = cs[1];
  };
  auto row_of_len = [&](int n) { return min(max(n, 0), a.T) - 1; };     // (as seq_len_of)
  // (raised by an earlier launch; the single launch reads the word when its own waits are over)
  const int err_early = !COH && a.err_before ? ld_err<true>(a.err) : 0;
  if constexpr (DENSE) load_x(xc, min(w, max(ntile - 1, 0)));
  u32x4 wt[8], wn[8];
  if (w < ntile) load_w(wt, w);                      // in flight while the merge weights are built
  if (w + NW < ntile) load_w(wn, w + NW);
  if constexpr (AHEAD) {
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      if (u * NTHR >= nb * a.d_k) break;               // (few sequences: one element a thread, or two)
      const int v = min(tid + u * NTHR, nb * a.d_k - 1);
      el_bl[u] = v / a.d_k;
      el_j[u] = v - el_bl[u] * a.d_k;
      el_len[u] = a.T;
      if (role != 0 && a.seq_lens) el_len[u] = a.seq_lens[bbase + el_bl[u]];
    }
  }

  // Which partials belong to which sequence: in mode 1 nsplit each; in mode 0 from the tile prefix, looked up once and
  // kept in LDS (single-launch mode: before the wait for the other workgroups, whose barrier it shares).
  auto look_up = [&]() {
    if (w == 0) {                                     // (16 NBT <= 64 sequences: one wave)
      const int b = bbase + min(lane, nb - 1);
      const int VT = prefix[a.B];
      const int Qt = (VT + a.NG - 1) / a.NG;
      const int gf = prefix[b] / Qt, gl = (prefix[b + 1] - 1) / Qt;
      const int np = min(gl - gf + 1, PROJ_MAX_PARTS);
      if (lane < nb) {
        sm.pid0s[lane] = min(b + gf, a.B + a.NG - 2);  // (a sequence without rows has no partial)
        sm.nps[lane] = np;
      }
    }
  };
  if constexpr (COH && !DENSE) look_up();
  const bool all_well = after_w_issue();

  // One finished output element (sequence bbase + bl, column j of the head); `other` is column j ^ 1.  u: which of the
  // thread's elements it is, where their lengths and rotations are at hand (AHEAD).
  auto emit = [&](int bl, int j, float val, float other, bool bad, int u) {
    const size_t b = (size_t)(bbase + bl);
    const int col = h * a.d_k + j;
    if (bad) val = other = NAN;
    if constexpr (!DENSE) {
      outp[b * a.e + col] = val;
    } else {
      if (role == 0) { outp[b * a.e + col] = val; return; }
      // the new token of sequence b sits at row / position len_b - 1
      const int pos = AHEAD && u >= 0 ? row_of_len(el_len[AHEAD ? u : 0]) : seq_len_of(a.seq_lens, (int)b, a.T) - 1;
      if (pos < 0) return;
      float r = val;
      if (turned) {
        float c, s;
        if constexpr (AHEAD) {
          if (u >= 0) { c = el_c[u]; s = el_s[u]; }
          else rotation(pos, j, c, s);
        } else {
          rotation(pos, j, c, s);
        }
        r = (j & 1) ? fmaf(val, c, -other * s) : fmaf(val, c, other * s);
      }
      if (role == 1) { outp[b * a.e + col] = r; return; }
      // (banded K-cache: bands of 32 rows, a head's 32 x d_k block contiguous inside its band)
      const size_t at = (role == 2 && a.k_banded)
                            ? ((size_t)(pos >> 5) * a.H + h) * (32 * (size_t)a.d_k) + (size_t)(pos & 31) * a.d_k + j
                            : (size_t)pos * a.e + col;
      uint16_t* dst = (role == 2 ? a.Kc : a.Vc) + b * a.c_bstride + at;
      *dst = __builtin_bit_cast(uint16_t, (__bf16)r);
    }
  };
  // all elements of a unit, from sm.obuf
  auto emit_all = [&](bool bad) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int u = 0; u < NE; ++u)
        if (tid + u * NTHR < nb * a.d_k) emit(el_bl[u], el_j[u], sm.obuf[el_bl[u]][el_j[u]], sm.obuf[el_bl[u]][el_j[u] ^ 1], bad, u);
    } else {
      for (int v = tid; v < nb * a.d_k; v += NTHR) {
        const int bl = v / a.d_k, j = v % a.d_k;
        emit(bl, j, sm.obuf[bl][j], sm.obuf[bl][j ^ 1], bad, -1);
      }
    }
  };
  auto no_result = [&]() {
    for (int v = tid; v < nb * a.d_k; v += NTHR) emit(v / a.d_k, v % a.d_k, NAN, NAN, true, -1);
  };
  if (COH && !all_well) {                              // (the unit's workgroups are apart: all of them know)
    if (tid == 0) st_result(a.err, (int)a.launch_id, true);
    no_result();
    return;
  }
  // In a launch of its own: who takes part in this unit, and where (see the hand-over); on its way to the memory side and
  // back while W and the partials travel.
  const bool xl = a.xcd_local != 0;
  const unsigned long long my_place = COH ? 0 : 1ull << (8 * (my_xcc() ^ (a.apart ? cs & 1 : 0)));
  unsigned long long places = 0;
  // With a.flags (an attention block's first launch: nothing has cleared any words for it) as a flag instead.
  const bool by_flags = DENSE && a.flags != nullptr;
  const int unit_at = (bz * nhx + hx) * a.csw, flag_id = (int)(a.launch_id << 3);
  const int place_flag = DENSE ? flag_id | (int)((my_xcc() ^ (a.apart ? cs & 1 : 0))) : 0;
  if (by_flags && xl && a.csw > 1 && tid == 0) st_result(a.flags + PROJ_MAX_FLAGS + unit_at + cs, place_flag, true);
  else if (!COH && xl && a.csw > 1 && tid == 0)
    places = __hip_atomic_fetch_add(a.places + (bz * nhx + hx), my_place, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + my_place;

  const bool even = a.mode == 1;
  if constexpr (!COH && !DENSE) {
    if (!even) {
      look_up();
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
  }
  // (bl: wave-uniform)
  auto first_part = [&](int bl) { return even ? (bbase + bl) * a.nsplit : __builtin_amdgcn_readfirstlane(sm.pid0s[bl]); };
  auto num_parts = [&](int bl) { return even ? min(a.nsplit, PROJ_MAX_PARTS) : __builtin_amdgcn_readfirstlane(sm.nps[bl]); };

  // The merged C in LDS: 8 rows of 16 sequences after the other, a sequence's 8 values as 16 bytes; hi halves, then lo
  static_assert(!COH || NBT == 1, "the single launch has at most 16 sequences");
  uint16_t* const cs_hi = reinterpret_cast<uint16_t*>(red);
  uint16_t* const cs_lo = cs_hi + PROJ_STAGED_ROWS * 16;
  const int rows4 = ntile * TILE_ROWS / 4;            // (crows <= PROJ_STAGED_ROWS: checked on the host)
  // A wave merges whole sequences, a lane four consecutive rows c: 8 / wps sequences at a time, each by wps waves (all in
  // shifts and wave-uniform addresses: this code is a good part of what stands between the partials and the product).
  // One round trip takes RI x 256 rows of a wave and 8 / RI of a sequence's partials.
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int lg = nb >= 5 ? 0 : nb >= 3 ? 1 : nb == 2 ? 2 : 3;     // log2(wps)
  const int seq0 = wu >> lg, lane0 = (wu & ((1 << lg) - 1)) * 64;
  f32x4 px[8];
  auto fetch = [&](auto RI_, int bl, int v, int pb) {
    constexpr int RI = decltype(RI_)::value, Q = 8 / RI;
    const int p0 = first_part(bl), np = num_parts(bl);
    const float* p[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      p[q] = uniform_ptr(a.Cpart + ((size_t)(p0 + min(pb + q % Q, max(np - 1, 0))) * a.H + h) * a.rows + c_lo);
    const int top = a.rows - 4 - c_lo;
    ld_part8(p, (unsigned)min((v + lane) * 4, top) * 4u, (unsigned)min((v + lane + (RI == 2 ? 64 << lg : 0)) * 4, top) * 4u, px);
  };
  auto merge = [&](auto RI_, bool fetched) {
    constexpr int RI = decltype(RI_)::value, Q = 8 / RI;
    for (int bl = seq0; bl < nb; bl += 8 >> lg) {
      const int np = num_parts(bl);
      for (int v = lane0; v < rows4; v += (64 << lg) * RI) {
        f32x4 cn[RI];
#pragma unroll
        for (int i = 0; i < RI; ++i) cn[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int pb = 0; pb < np; pb += Q) {
          if (!(fetched && bl == seq0 && v == lane0 && pb == 0)) fetch(RI_, bl, v, pb);
#pragma unroll
          for (int pq = 0; pq < Q; ++pq)
            if (pb + pq < np) {
              const float wgt = sm.wpid[bl][pb + pq];
#pragma unroll
              for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) cn[i][j] = fmaf(wgt, px[i * Q + pq][j], cn[i][j]);
            }
        }
#pragma unroll
        for (int i = 0; i < RI; ++i) {
          const int ve = v + lane + i * (64 << lg), r = ve * 4;
          if (ve < rows4) {
            if (c_lo + r >= c_hi) cn[i] = f32x4{0.f, 0.f, 0.f, 0.f};  // (rows of the last tile past the end of W)
            unsigned hw[2], lw[2];
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
              const __bf16 h0 = (__bf16)cn[i][j], h1 = (__bf16)cn[i][j + 1];
              const bf16x2 hv = {h0, h1}, lv = {(__bf16)(cn[i][j] - (float)h0), (__bf16)(cn[i][j + 1] - (float)h1)};
              hw[j / 2] = __builtin_bit_cast(unsigned, hv);
              lw[j / 2] = __builtin_bit_cast(unsigned, lv);
            }
            const int at = ((r >> 3) * 16 + bl) * 8 + (r & 7);
            *reinterpret_cast<uint2*>(cs_hi + at) = make_uint2(hw[0], hw[1]);
            *reinterpret_cast<uint2*>(cs_lo + at) = make_uint2(lw[0], lw[1]);
          }
        }
      }
    }
  };
  // (few sequences: their rows are spread over several waves and one round trip takes eight partials)
  auto with_rows = [&](auto&& f) {
    if (lg > 0) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 2>{});
  };
  // A launch of its own makes the merged C of a tile's rows in B-operand layout, a lane eight rows c of sequence n.  FEW: from
  // four partials per round trip, the first four of a tile asked for ahead -- behind the maxima and sums for the first tile, behind
  // the products of the one before for the others -- because a trip is what takes the time there (X-cache of 1 x 4096 rows x 32 heads x
  // 1024 columns 34.5 -> 32.6 us, 1 x 4096 x 128 heads 46.2 -> 44.3, wide K-cache of 2 x 4001 x 40 heads x 128 56.2 -> 55.5).  More
  // sequences: one or two at a time, since there the lines of the partials do, 16 for 16 sequences, and what is fetched beyond
  // the last partial costs (24 x 1500 x 20 heads x 1280 48.1 us, with four per trip 49.6; 8 x 4096 x 64 heads x 768 44.1 and 45.7).
  // In a kernel of its own, because the others paid for what they do not run: 64 x 448 rows x 6 heads x 64 22.4 -> 22.2 us.
  constexpr int QMOST = 4;
  f32x4 pt[FEW ? QMOST : 1][2];
  int pn0 = 0, pnn = 0, most = 0;                     // this lane's sequence: first partial, how many; the most of any lane
  auto ask_parts = [&](auto Q_, int ct, int p) {
    constexpr int Q = decltype(Q_)::value;
    const int c = min(c_lo + ct * TILE_ROWS + kg * 8, a.rows - 8);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float* src = a.Cpart + ((size_t)(pn0 + min(p + q, max(pnn - 1, 0))) * a.H + h) * a.rows + c;
      pt[q][0] = *reinterpret_cast<const f32x4*>(src);
      pt[q][1] = *reinterpret_cast<const f32x4*>(src + 4);
    }
  };
  // (a partial that does not exist is a repeated load of one that does: one, two or four per trip by how many there are)
  auto with_parts = [&](auto&& f) {
    if (most <= 1) f(std::integral_constant<int, 1>{});
    else if (most == 2) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, QMOST>{});
  };
  if constexpr (!DENSE) {
    // ---- merge weights for head h: one wave per sequence, one lane per partial; the first partials
    //      themselves are asked for behind the maxima and sums ----------------------------------------
    constexpr int SW = 2 * NBT;                       // sequences per wave
    float mp[SW], lp[SW];
#pragma unroll
    for (int i = 0; i < SW; ++i) {
      const int bl = wu + NW * i;
      mp[i] = NEG_INF; lp[i] = 0.f;
      if (bl < nb && lane < num_parts(bl)) {
        mp[i] = ld_part<COH>(a.mpart + (size_t)(first_part(bl) + lane) * a.H + h);
        lp[i] = ld_part<COH>(a.lpart + (size_t)(first_part(bl) + lane) * a.H + h);
      }
    }
    if constexpr (FEW) {
      const int bl = min(n, nb - 1);
      pn0 = even ? (bbase + bl) * a.nsplit : sm.pid0s[bl];
      pnn = even ? min(a.nsplit, PROJ_MAX_PARTS) : sm.nps[bl];
      most = even ? pnn : __builtin_amdgcn_readfirstlane((int)max_over_wave((float)pnn));
      if (w < ntile) with_parts([&](auto Q_) { ask_parts(Q_, w, 0); });
    }
    const bool fetched = COH && seq0 < nb && lane0 < rows4;
    if constexpr (COH)
      if (fetched) with_rows([&](auto RI_) { fetch(RI_, seq0, lane0, 0); });
#pragma unroll
    for (int i = 0; i < SW; ++i) {
      const int bl = wu + NW * i;
      if (bl >= nb) break;
      const float M = max_over_wave(mp[i]);
      const float wgt = (mp[i] == NEG_INF) ? 0.f : exp2f((mp[i] - M) * a.mscale);
      const float L = sum_over_wave(wgt * lp[i]);
      if (lane < num_parts(bl)) sm.wpid[bl][lane] = wgt / L;
    }
    // (barriers for LDS only: __syncthreads() would also wait for the tiles of W in flight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (COH) {
      with_rows([&](auto RI_) { merge(RI_, fetched); });
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
  }

  f32x4 acc[8][NBT];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int t = 0; t < NBT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int ct = w; ct < ntile; ct += NW) {
    const int c0 = c_lo + ct * TILE_ROWS;
    const bool more = ct + NW < ntile;
    // B operand: merged C for (b = bt*16 + n, rows c0 + kg*8 .. +8)
    bf16x8 bhi[NBT], blo[NBT];
    if constexpr (DENSE) {
      const int c = c0 + kg * 8;
      load_x(xn, min(ct + NW, ntile - 1));
#pragma unroll
      for (int t = 0; t < NBT; ++t) {
        const bool live = t * 16 + n < nb && c < c_hi;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float v = live ? xc[t][j >> 2][j & 3] : 0.f;
          const __bf16 hi = (__bf16)v;
          bhi[t][j] = hi;
          blo[t][j] = (__bf16)(v - (float)hi);
        }
      }
    } else if constexpr (COH) {
#pragma unroll
      for (int t = 0; t < NBT; ++t) {                // (columns of sequences past the last one: any values, never used)
        const int at = ((ct * 4 + kg) * 16 + n) * 8;
        bhi[t] = *reinterpret_cast<const bf16x8*>(cs_hi + at);
        blo[t] = *reinterpret_cast<const bf16x8*>(cs_lo + at);
      }
    } else if constexpr (FEW) {
      float cn[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) cn[j] = 0.f;
      with_parts([&](auto Q_) {
        constexpr int Q = decltype(Q_)::value;
        for (int p = 0; p < most; p += Q) {
          if (p > 0) ask_parts(Q_, ct, p);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const float wgt = p + q < pnn ? sm.wpid[min(n, nb - 1)][p + q] : 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) cn[j] = p + q < pnn ? fmaf(wgt, pt[q][j >> 2][j & 3], cn[j]) : cn[j];
          }
        }
        if (more) ask_parts(Q_, ct + NW, 0);
      });
      const bool live = n < nb && c0 + kg * 8 < c_hi;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = live ? cn[j] : 0.f;
        const __bf16 hi = (__bf16)v;
        bhi[0][j] = hi;
        blo[0][j] = (__bf16)(v - (float)hi);
      }
    } else {
      const int c = c0 + kg * 8;
#pragma unroll
      for (int t = 0; t < NBT; ++t) {
        float cn[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) cn[j] = 0.f;
        const int bl = t * 16 + n;
        if (bl < nb && c < c_hi) {
          const int p0 = even ? (bbase + bl) * a.nsplit : sm.pid0s[bl], np = even ? min(a.nsplit, PROJ_MAX_PARTS) : sm.nps[bl];
          for (int p = 0; p < np; ++p) {
            const float wgt = sm.wpid[bl][p];
            const float* src = a.Cpart + ((size_t)(p0 + p) * a.H + h) * a.rows + c;
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(src), x1 = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) { cn[j] = fmaf(wgt, x0[j], cn[j]); cn[4 + j] = fmaf(wgt, x1[j], cn[4 + j]); }
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const __bf16 hi = (__bf16)cn[j];
          bhi[t][j] = hi;
          blo[t][j] = (__bf16)(cn[j] - (float)hi);
        }
      }
    }
    u32x4 am[8];
    transpose8x8(wt, am);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bf16x8 av = __builtin_bit_cast(bf16x8, am[i]);
#pragma unroll
      for (int t = 0; t < NBT; ++t) {
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bhi[t], acc[i][t], 0, 0, 0);
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, blo[t], acc[i][t], 0, 0, 0);
      }
    }
    if (more) {
#pragma unroll
      for (int j = 0; j < 8; ++j) wt[j] = wn[j];
      if (ct + 2 * NW < ntile) load_w(wn, ct + 2 * NW);
    }
    if constexpr (DENSE) {
#pragma unroll
      for (int t = 0; t < NBT; ++t) { xc[t][0] = xn[t][0]; xc[t][1] = xn[t][1]; }
    }
  }
  if constexpr (COH) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (the merged C gives way to the sum)

  if constexpr (AHEAD) {
    if (turned) {
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        if (u * NTHR >= nb * a.d_k) break;
        rotation(row_of_len(el_len[u]), el_j[u], el_c[u], el_s[u]);
      }
    }
  }
  // Where the unit's workgroups run, all of whom have stored that by now if they started together (else asked again below);
  // this one's own flag is out.
  int place = place_flag;
  auto look_at_places = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane < a.csw) place = ld_err<true>(a.flags + PROJ_MAX_FLAGS + unit_at + lane);
  };
  if (by_flags && xl && a.csw > 1 && w == 0) look_at_places();

  // ---- sum the 8 waves, IPR of the 8 accumulator columns per pass through LDS: thread (ei, lane) ends up with
  //      accumulator element i0 + ei / NBT of batch tile ei % NBT as that lane of a wave held it ----------------
  constexpr int IPR = 8 / NBT;
  f32x4* const red4 = reinterpret_cast<f32x4*>(red);
  f32x4 osum[NBT];                                     // per pass: columns (kg*4 + r)*8 + i of sequence n of the batch tile
#pragma unroll
  for (int ps = 0; ps < NBT; ++ps) {
#pragma unroll
    for (int ii = 0; ii < IPR; ++ii)
#pragma unroll
      for (int t = 0; t < NBT; ++t) red4[(w * 8 + ii * NBT + t) * 64 + lane] = acc[ps * IPR + ii][t];
    __syncthreads();
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) sum += red4[(ww * 8 + w) * 64 + lane];
    osum[ps] = sum;
    if (ps + 1 < NBT) __syncthreads();
  }
  const int obl = (w % NBT) * 16 + n, omi = kg * 4;    // this thread's sequence and first column group
  auto oi = [&](int ps) { return ps * IPR + w / NBT; };
  const bool mine = obl < nb && omi < lph;
  auto to_obuf = [&]() {
    if (obl < nb) {
#pragma unroll
      for (int ps = 0; ps < NBT; ++ps)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (omi + r < lph) sm.obuf[obl][(omi + r) * 8 + oi(ps)] = osum[ps][r];
    }
    __syncthreads();
  };

  if (a.csw == 1) {
    const bool bad = a.err_before && (COH ? ld_err<true>(a.err) : err_early) == (int)a.launch_id;
    to_obuf();
    emit_all(bad);
    return;
  }
  // ---- several workgroups share the rows of W: last one to arrive adds the partial sums ---------
  // No cache-wide fences: the partial sums are stored and waited for before this workgroup's arrival is counted, and
  // the last workgroup reads them past its L1.  Where the workgroups of a head share an XCD (xcd_local: found by
  // the host at set-up) its L2 is their meeting point -- plain stores, an atomic that the L2 executes; otherwise the stores are
  // written through and the atomic has device scope: three round trips to the memory side instead of to the L2.
  // Whether they do share it they find out themselves on every launch.  In the single launch the arrival flags carry the XCD
  // of every workgroup.  In a launch of its own each adds its XCD to the unit's word, and the last one to do so sees them all:
  // if they are apart, none of the counts becomes complete, so that nobody else writes the result; it writes NaN and raises
  // the error word.  (The XCD that workgroup 0 runs on differs from queue to queue: the host has nothing to compare with.)
  // The partial sums of a head lie in accumulator order, [element i][column group], padded to whole fours of column groups,
  // so that they leave and come back 16 bytes at a time.  (Heads of 80 columns without the padding, one dword after the
  // other: 24.9 instead of 21.4 us at 1 x 300 rows x 32 heads.)
  // Dense products of up to 1024 elements (a few sequences) keep their columns in order instead, an element or two a thread:
  // they are finished from where they are read, without another pass through LDS (4 x 4096 x 4096: 12.0 against 12.8 us; two
  // elements: vanilla block of 12 x 300 rows x 20 heads x 64 43.5 against 44.6 us, of 8 x 500 x 32 x 128 74.1 against 74.8).
  if (!COH && a.err_before && err_early == (int)a.launch_id) {             // (then the control words may not be 0 either)
    no_result();
    return;
  }
  const int nel = nb * a.d_k;
  constexpr int IN_ORDER = NBT == 1 ? 2 : 1;            // elements per thread at most (more batch tiles: registers)
  const bool in_order = DENSE && nel <= IN_ORDER * NTHR;
  // (thread tid: elements tid and tid + NTHR, the second one in f<2> only)
  auto per_thread = [&](auto&& f) {
    if (IN_ORDER == 1 || nel <= NTHR) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, IN_ORDER>{});
  };
  auto part_at = [&](int sp, int ps) { return outpart + ((size_t)sp * a.B + bbase + obl) * part_row + (h * 8 + oi(ps)) * lph4 + omi; };
  if (in_order) {
    to_obuf();
    per_thread([&](auto NE) {
#pragma unroll
      for (int u = 0; u < decltype(NE)::value; ++u) {
        const int v = tid + u * NTHR, bl = v / a.d_k, j = v - bl * a.d_k;
        if (v < nel) st_result(outpart + ((size_t)cs * a.B + bbase + bl) * part_row + h * lph4 * 8 + j, sm.obuf[bl][j], !xl);
      }
    });
  } else if (mine) {
#pragma unroll
    for (int ps = 0; ps < NBT; ++ps) st_result4(part_at(cs, ps), osum[ps], !xl);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (by_flags) {
    // Arrival flags that carry the launch's id need no launch that clears them; this one takes longer by a round trip to L2 more
    // than counting costs, and the call gains 0.2 to 1.3 us.  A workgroup stores its flag, waits for that, and looks at all of the unit's: the last to store sees them
    // all.  Two that see them all both finish, with the same values.  The flags of where they run were stored before
    // anything else: seen by the last as well.
    if (w == 0) {
      if (lane == 0 && !(xl && a.apart && (cs & 1))) st_result(a.flags + unit_at + cs, flag_id, !xl);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      int arrived = flag_id;
      if (lane < a.csw) arrived = ld_err<true>(a.flags + unit_at + lane);
      if (!__all((unsigned)(place ^ flag_id) < 8u)) look_at_places();
      const bool all_here = __all(arrived == flag_id), all_placed = __all((unsigned)(place ^ flag_id) < 8u), together = __all(place == place_flag);
      if (lane == 0) sm.is_last = all_placed && !together ? 2 : (all_here && together);
    }
  } else if (tid == 0) {
    int* const counter = &a.counters[bz * nhx + hx];
    // (the sum of the bytes: how many had added themselves by then)
    const bool last_apart = !COH && (int)((places * 0x0101010101010101ull) >> 56) == a.csw && places != (unsigned long long)a.csw * my_place;
    int old = -1;
    if (!xl) old = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else if (COH || !(a.apart && (cs & 1))) old = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    sm.is_last = xl && last_apart ? 2 : (old == a.csw - 1);
  }
  __syncthreads();
  if (!sm.is_last) return;
  if (!COH && sm.is_last == 2) {                       // the last of a unit whose workgroups are apart
    if (tid == 0) st_result(a.err, (int)a.launch_id, true);
    no_result();
    return;
  }
  // (single launch: the error word travels with the partial sums, requested here, looked at behind their wait)
  const int errv = COH ? ld_err<true>(a.err) : err_early;
  if (in_order) {
    per_thread([&](auto NE) {
      constexpr int N = decltype(NE)::value;
      int bl[N], col[N];
      const float* src[N];
      float sum[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int v = min(tid + u * NTHR, nel - 1);
        bl[u] = v / a.d_k; col[u] = v - bl[u] * a.d_k; sum[u] = 0.f;
        src[u] = outpart + ((size_t)bbase + bl[u]) * part_row + h * lph4 * 8 + col[u];
      }
      for (int s0 = 0; s0 < a.csw; s0 += 8) {
        float part[N][8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int u = 0; u < N; ++u) part[u][q] = ld_part<true>(src[u] + (size_t)min(s0 + q, a.csw - 1) * a.B * part_row);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int u = 0; u < N; ++u) if (s0 + q < a.csw) sum[u] += part[u][q];
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const float other = __shfl_xor(sum[u], 1);       // (a pair's columns sit in neighbour lanes)
        if (tid + u * NTHR < nel) emit(bl[u], col[u], sum[u], other, false, AHEAD ? u : -1);
      }
    });
    if (tid == 0 && !by_flags) a.counters[bz * nhx + hx] = 0;
    return;
  }
  if (mine) {
#pragma unroll
    for (int ps = 0; ps < NBT; ++ps) {
      osum[ps] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int s0 = 0; s0 < a.csw; s0 += 8) {
        const float* src[8];
        f32x4 part[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) src[q] = uniform_ptr(outpart + (size_t)min(s0 + q, a.csw - 1) * a.B * part_row);
        const unsigned at = (unsigned)(part_at(0, ps) - outpart) * 4u;
        ld_part8(src, at, at, part);
#pragma unroll
        for (int q = 0; q < 8; ++q) if (s0 + q < a.csw) osum[ps] += part[q];
      }
    }
  }
  to_obuf();
  const bool bad = a.err_before && errv == (int)a.launch_id;              // NaN: the stream kernel gave up waiting
  emit_all(bad);
  if (tid == 0 && !by_flags) a.counters[bz * nhx + hx] = 0;
}

template <int NBT, bool DENSE, bool ONCE, bool FEW>
__global__ __launch_bounds__(512) void project_mfma_kernel(const ProjArgs a) {
  __shared__ int prefix[FUSED_MAX_B + 1];
  __shared__ ProjShared<NBT> sm;
  __shared__ __align__(16) float red[8 * 8 * 4 * 64];
  // unit = (head, batch chunk), for which csw workgroups share the rows of W: dealt to the XCDs so that they meet in one L2
  const int nhx = DENSE ? a.H * a.nmat : a.H;
  const int slot = blockIdx.x >> 3, unit = (slot / a.csw) * 8 + (blockIdx.x & 7);
  // (the launch the error word speaks of; an earlier launch of the call has written it already)
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.err && !a.err_before) st_result(a.err - 1, (int)a.launch_id, true);
  // (control words of the launches that follow: nothing of this launch uses them)
  if (DENSE && a.flags && blockIdx.x == 0)
    for (int i = threadIdx.x; i < PROJ_BLOCK_INTS; i += 512) a.counters[i] = 0;
  if (unit >= nhx * ((a.B + 16 * NBT - 1) / (16 * NBT))) return;
  project_work<NBT, false, DENSE, ONCE, FEW>(a, unit % nhx, slot % a.csw, unit / nhx, prefix, sm, red, [&]() {
    if (!DENSE && a.mode == 0) build_tile_prefix(prefix, nullptr, a.seq_lens, a.B, a.T);
    return true;
  });
}

// ------------------------------------------------------------------------------------------------
// fused stream kernel
//
// A workgroup is FUSED_WAVES waves that all do the same work on tiles of their own.  In step k a wave
//   1. parks tile k (in registers since two steps ago) in one of its two LDS slots and scores it from
//      there on MFMA (with rotary keys: on the vector ALU from the registers, before parking): scores of
//      its unit's heads, softmax numerators against the head's running maximum (bf16, the precision the
//      MFMA consumes anyway); publishes {tag, running max, 4 numerators} words,
//   2. requests all heads' words of its tile k-1 (published by the same wave of every workgroup of the
//      group one step earlier) and, behind them, tile k+2 into the registers that became free in 1,
//   3. takes tile k-1 out of its LDS slot while the words travel, waits for them (a wave's vector-memory
//      operations complete in issue order: the wait lets exactly the loads of tile k+2 stay in flight),
//      rescales its accumulators when a maximum moved and does the MFMA contraction.
// Every wave does both halves, so all eight waves of a compute unit share the scoring work and the
// loads.  A wave never waits for another wave of its workgroup.
// ------------------------------------------------------------------------------------------------
//
// ROPE (RoPE appendix, option 1): the cache holds raw keys and row t sits at position t.  The
// scoring rotates each key pair by its position for the score only; the tile that goes to the
// weighted sum stays raw.  With (y1, y2) = (x1 c + x2 s, -x1 s + x2 c) the pair's share of the
// score is c (q1 x1 + q2 x2) + s (q1 x2 - q2 x1): two dot products of the raw pair, with (q1, q2)
// and with (-q2, q1).  cos / sin of a lane's first row come from the table with the tile; the
// following seven rows advance by the one-position rotation (table row 1), kept in registers.
constexpr float SOFTMAX_SLACK = 6.0f;

// LPHP: lanes reserved per head: 16, 8, 4 or 2 (heads of up to 128, 64, 32 or 16 columns).  At compile time, because the
// divisions by it and what follows from them cost registers: with a run-time value for the two narrow classes, layers of 17
// to 32 such heads had 84 bytes of scratch per lane (108 with rotary keys) where the others had 56..60 (80..88; now none has any), and took
// 26.2 us at 1 x 4096 rows x 32 heads x 32 (now 25.8), 40.3 at 4 x 5000 with rotary keys (now 38.1).  BYSEQ: the by-sequence partition (a.by_sequence != 0), which has no merge of the
// waves and never runs the projection; an instantiation of its own keeps each partition's code out of the
// other's registers.
template <int NT, bool ROPE, int LPHP, bool BYSEQ>
__global__ __launch_bounds__(FUSED_WAVES * 64) void fused_stream_kernel(const FusedArgs a) {
  constexpr int NP = FUSED_WAVES, NS = FUSED_SLOTS, PD = FUSED_AHEAD;
  constexpr int NTHR = NP * 64;
  constexpr int HP = NT * 16;                       // heads padded to the MFMA N tile
  static_assert(NP == 8 && NS == 2 && PD == 2, "the step structure and the thread mappings below assume these");
  __shared__ int prefix[FUSED_MAX_B + 1];
  __shared__ int lens_s[FUSED_MAX_B];               // rows per sequence
  __shared__ __align__(16) float marr[NT][16][NP];  // (a head's eight waves side by side: two 16-byte reads)
  __shared__ __align__(16) float larr[NT][16][NP];
  // Per wave: NS landing slots of 8 KB for K tiles.  By-context partition: the end-of-share merge of
  // the waves goes through the (then idle) slots, which is why the array is a little larger than
  // the slots.  By-sequence partition: the other waves keep streaming; a wave writes its result
  // straight from its registers.  The projection of the single-launch mode runs after everything
  // else and reuses the slots and sbuf.
  constexpr int MERGE_PITCH = 132;                  // floats per head row of the merge buffer: 16-byte accesses without bank conflicts
  constexpr size_t SLOT_BYTES = (size_t)NP * NS * TILE_ROWS * 272, MERGE_BYTES = sizeof(float) * NP * HP * MERGE_PITCH;   // (272: a tile row and its padding)
  __shared__ __align__(16) unsigned char lds_main[SLOT_BYTES > MERGE_BYTES ? SLOT_BYTES : MERGE_BYTES];
  __shared__ __align__(16) float sbuf[sizeof(ProjShared<1>) / sizeof(float)];
  float* const mbuf = reinterpret_cast<float*>(lds_main);           // [NP][HP][MERGE_PITCH] floats
  float* const red = reinterpret_cast<float*>(lds_main);            // 64 KB for the projection's cross-wave sum
  static_assert(sizeof(float) * 8 * 8 * 4 * 64 <= sizeof(lds_main), "cross-wave sum must fit");

  // ---- which group / column unit is this workgroup -------------------------------------------
  int g = 0, u = 0;
  bool has_work = true;                             // (workgroup-uniform)
  {
    const int i = blockIdx.x;
    if (a.gpx > 0) {                                // groups packed inside one XCD (WG i -> XCD i % 8)
      const int x = i & 7, r = i >> 3;
      const int gx = r / a.G;
      if (gx >= a.gpx) has_work = false;
      g = x * a.gpx + gx;
      u = r % a.G;
    } else {
      g = i / a.G;
      u = i % a.G;
    }
    if (g >= a.NG) has_work = false;
  }
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int idx = lane & 15, rg = lane >> 4;        // column group / row group of the register tile
  const int n = idx, kg = rg;                       // head-in-tile / row group of the B operand
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int p = wu;                                 // this wave's team: wave p of every workgroup of the group

  const bool fuse = !BYSEQ && a.fuse != 0;
  // Single launch: this workgroup's (head, row split) of the projection, a head's workgroups on one XCD as in
  // project_mfma_kernel.  The arrival counters start at 0, a head's cleared by its first workgroup, in the L2 that counts.
  auto projection_share = [&](int& phead, int& psplit) {
    int i = blockIdx.x;
    asm volatile("" : "+s"(i));                       // (computed where it is used: not kept in registers through the stream)
    const int slot = i >> 3;
    psplit = slot % a.proj.csw;
    // Heads wider than a cache line whose rows of W are no whole lines share lines with their neighbours, so neighbours share
    // an XCD: dealt round robin, every XCD fetches those lines for itself (1 x 500..3000 rows x 32 heads x 96 columns: 23.7,
    // 25.4 and 26.1 us against 22.7, 24.3 and 24.9).  The others are dealt round robin, which is the faster one there
    // (128 columns: 25.5 against 25.9; 16..32 columns, a small W: up to 0.7 us).
    if (a.d_k > 64 && a.d_k % 64 != 0) {
      const int x = i & 7;
      phead = x * a.H / 8 + slot / a.proj.csw;
      if (phead >= (x + 1) * a.H / 8) phead = a.H;
    } else {
      phead = (slot / a.proj.csw) * 8 + (i & 7);
    }
  };
  if (fuse) {
    if (wu == NP - 1) {                               // (while the first wave builds the tile prefix)
      int phead, psplit;
      projection_share(phead, psplit);
      if (phead < a.proj.H && psplit == 0 && lane == 0) st_result(a.counters + phead, 0, a.proj.xcd_local == 0);
    }
  } else if (blockIdx.x == 0 && a.counters) {
    for (int i = tid; i < a.ncounters; i += NTHR) a.counters[i] = 0;
  }

  build_tile_prefix(prefix, lens_s, a.seq_lens, a.B, a.T);     // (ends with a workgroup barrier)
  const int VT = prefix[a.B];
  const int Qt = (VT + a.NG - 1) / a.NG;            // tiles per group
  const int v0 = g * Qt, v1 = min(VT, v0 + Qt);
  if (BYSEQ ? (g * NP >= a.B * a.by_sequence) : (v0 >= v1)) has_work = false;
  if (!has_work && !fuse) return;

  // ---- lane -> column mapping inside the unit --------------------------------------------------
  constexpr int lphp = LPHP;
  const int hh = idx / lphp, li = idx % lphp;
  const int myhead = u * a.hpu + hh;
  const bool col_active = (li < a.lph) && (hh < a.hpu) && (myhead < a.H);
  const int mycol = myhead * a.d_k + li * 8;        // first of this lane's 8 columns
  const bool pub_lane = col_active && (li == 0);    // one lane per head publishes its row group
  const int ucol0 = u * a.hpu * a.d_k;
  const int uwc = min(a.hpu * a.d_k, a.d - ucol0);  // columns of this unit
  // first unit-local column of column group mi (the A operand's M index), or -1
  auto col_of_group = [&](int mi) {
    const int h2 = mi / lphp, l2 = mi % lphp;
    return (l2 < a.lph && h2 < a.hpu && h2 * a.d_k + l2 * 8 < uwc) ? h2 * a.d_k + l2 * 8 : -1;
  };

  // A tile in its LDS slot: row r, 16-byte chunk c (8 columns) at byte r * ROW_PITCH + c * 16, with one
  // chunk of padding per row (17 chunks), so that all three access patterns are free of bank conflicts
  // and each is one per-lane base plus compile-time offsets: the store and the read for the weighted sum
  // (the 16 chunks of a row) and the A operands of the score MFMA (one chunk of 16 consecutive rows).
  //   store of register j (row j*RJ + rg*RR), chunk idx ....... wpos + j * RJ * ROW_PITCH
  //   score A operand, rows mt*16 + idx, chunk ks*4 + rg ...... spos + mt * 16 * ROW_PITCH + ks * 64
  //   sum, rows jh*16 + kg*4 + jl, chunk idx (no rotary keys) . ppos + (jh * 16 + jl) * ROW_PITCH
  constexpr unsigned ROW_PITCH = 272, SLOT_PITCH = TILE_ROWS * ROW_PITCH;
  // Which row of the tile a lane's register j holds: j * RJ + rg * RR.  With rotary keys the scores are taken
  // from the registers and a lane needs eight consecutive positions (rows rg*8 + j).  Otherwise the registers
  // only carry the tile to its slot, and row j*4 + rg makes one load instruction cover four consecutive rows:
  // in the banded cache 4 d_k x 2 contiguous bytes, whole cache lines that no other instruction touches
  // (with rows eight apart and d_k = 96, every second line is shared by two instructions).
  constexpr int RJ = ROPE ? 1 : 4, RR = ROPE ? 8 : 1;
  const unsigned wpos = (unsigned)(rg * RR) * ROW_PITCH + (unsigned)idx * 16u;
  const unsigned spos = (unsigned)idx * ROW_PITCH + (unsigned)rg * 16u;
  const unsigned ppos = (unsigned)(kg * 4) * ROW_PITCH + (unsigned)idx * 16u;
  // Scores on MFMA (no rotary keys): column n = 2 * (head in unit) + {0: query hi, 1: query lo}; the lane
  // with the even n publishes its head's words for its four-row groups.
  const int mhead = u * a.hpu + (idx >> 1);          // head of this lane's score column
  const bool mpub_lane = !(idx & 1) && (idx >> 1) < a.hpu && mhead < a.H;

  const bool xl = a.xcd_local != 0;
  const bool heads_full = (a.H == HP);               // no padded heads in the MFMA N tiles
  const unsigned pitchB = (unsigned)a.d * 2u;        // bytes per cache row
  u32x4* const team_ring = reinterpret_cast<u32x4*>(a.exch) + (size_t)(g * NP + p) * EXCH_SLOTS * (HP * 8);
  char* const myslots = reinterpret_cast<char*>(lds_main) + (size_t)p * NS * SLOT_PITCH;
  bool dead = false;                                // a wait timed out: stop waiting, just drain
  auto give_up = [&]() {
    if (!dead && lane == 0) atomicExch(a.err, (int)a.launch_id);
    dead = true;
  };
  // Every wait for another workgroup is bounded by the same budget of real time (the constant
  // 100 MHz counter), measured from the first failed check of that wait.
  auto out_of_time = [&](unsigned long long& since) {
    const unsigned long long now = __builtin_amdgcn_s_memrealtime();
    if (since == ~0ull) since = now;
    return now - since >= a.wait_ticks;
  };
  if (blockIdx.x == 0 && tid == 0) st_result(a.err - 1, (int)a.launch_id, true);   // the launch the error word speaks of

  // The work of this wave as a list of segments (a sequence or a share of one); tile k of a segment is
  // row tile t0 + k * stride (less `lead` from the second tile on) of sequence b.  Two partitions:
  //  * by context (default): the group's range of tiles [v0, v1) is cut at sequence boundaries and
  //    the waves take the tiles of a share round-robin, waves 0..3 with a tile's lead; the waves' results are merged at the
  //    end of each share and the groups' partials by the projection.  Balanced for any lengths.
  //  * by sequence: every sequence is cut into a.by_sequence equal shares and wave slot g * NP + p
  //    takes shares round-robin; no merge inside the workgroup, one partial per share.  For batches
  //    whose shares fill the slots evenly (many short sequences).
  struct Seg { int b, t0, stride, lead, ntl, len, pid; unsigned it0; const uint16_t* Kb; };   // it0: tiles of earlier segments
  constexpr bool by_seq = BYSEQ;
  int seg_b = by_seq ? g * NP + p : 0;
  unsigned seg_it = 0;                              // tiles this wave has been through so far
  if (has_work && !by_seq)
    while (prefix[seg_b + 1] <= v0) ++seg_b;
  auto next_segment = [&](Seg& sg) -> bool {
    if (by_seq) {
      const int shares = a.by_sequence;               // shares per sequence (equal runs of tiles)
      if (seg_b >= a.B * shares) return false;
      const int q = seg_b, b = q / shares, j = q - b * shares;
      seg_b += a.NG * NP;
      const int tiles_b = prefix[b + 1] - prefix[b], per = (tiles_b + shares - 1) / shares;
      sg.b = b; sg.t0 = j * per; sg.stride = 1; sg.lead = 0; sg.pid = q;
      sg.len = lens_s[b];
      sg.Kb = a.K + (size_t)b * a.k_bstride;
      sg.ntl = max(0, min(per, tiles_b - j * per));
      sg.it0 = seg_it;
      seg_it += (unsigned)sg.ntl;
      return true;
    }
    for (; seg_b < a.B && prefix[seg_b] < v1; ++seg_b) {
      const int b = seg_b;
      const int s0 = max(v0, prefix[b]) - prefix[b];
      const int s1 = min(v1, prefix[b + 1]) - prefix[b];
      if (s0 >= s1) continue;
      sg.b = b; sg.pid = b + g;
      // The first four tiles of a share go to waves 0..3, the rest to all eight in turn: every SIMD holds one of the first
      // four waves and one of the others, whose first tiles arrive about one and a half steps later (requested at 9 us
      // after the launch, not 4: the first burst is the memory's) and which so ended 5 us later with as many tiles.
      // 52.6 -> 52.0 us at 16384 rows x 4096 columns, 67.5 -> 66.8 on the ragged rotary batch.  (Shares of less than four
      // tiles per wave are over before that: there two tiles behind one another on half of the waves would be the longer.)
      const int ahead = s1 - s0 >= 4 * NP ? NP / 2 : 0;
      sg.stride = NP; sg.lead = p < ahead ? NP - ahead : 0;
      sg.t0 = s0 + p + (p < ahead ? 0 : ahead);        // (without the lead: s0 + p, s0 + p + NP, ...)
      sg.len = lens_s[b];
      sg.Kb = a.K + (size_t)b * a.k_bstride;
      sg.ntl = (p < ahead ? 1 : 0) + max(0, (s1 - s0 - ahead - p + NP - 1) / NP);
      sg.it0 = seg_it;                                // tile k carries tag tag_base + it0 + k + 1
      seg_it += (unsigned)sg.ntl;
      ++seg_b;
      return true;
    }
    return false;
  };
  // End of a share in the by-context partition, all threads: sum the waves' accumulators
  // out of mbuf[wave][head][col] (one thread per four columns of a head) and write the group's
  // partial for this sequence.
  // (ln: the lane, see fresh_lane)
  auto write_partial = [&](int pid, int ln) {
    if (u == 0 && wu == NP - 1 && ln < a.H) {         // (first: this workgroup is not to be later than the others for it)
      const f32x4* const mw = reinterpret_cast<const f32x4*>(marr[ln >> 4][ln & 15]);
      const f32x4* const lw = reinterpret_cast<const f32x4*>(larr[ln >> 4][ln & 15]);
      const f32x4 m0 = mw[0], m1 = mw[1], l0 = lw[0], l1 = lw[1];
      float mall = NEG_INF, l = 0.f;
#pragma unroll
      for (int ww = 0; ww < NP; ++ww) {
        mall = fmaxf(mall, ww < 4 ? m0[ww & 3] : m1[ww & 3]);
        l += ww < 4 ? l0[ww & 3] : l1[ww & 3];
      }
      st_result(a.mpart + (size_t)pid * a.H + ln, mall, fuse);
      st_result(a.lpart + (size_t)pid * a.H + ln, l, fuse);
    }
    const int oc4 = (ln & 31) * 4, oh0 = wu * 2 + (ln >> 5);         // four columns of heads oh0, oh0 + 16
    if (oc4 < uwc) {
      f32x4 part[HP / 16][NP];
#pragma unroll
      for (int jj = 0; jj < HP / 16; ++jj)
#pragma unroll
        for (int ww = 0; ww < NP; ++ww)
          part[jj][ww] = *reinterpret_cast<const f32x4*>(mbuf + ((size_t)ww * HP + oh0 + 16 * jj) * MERGE_PITCH + oc4);
#pragma unroll
      for (int jj = 0; jj < HP / 16; ++jj) {
        const int h = oh0 + 16 * jj;
        f32x4 osum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ww = 0; ww < NP; ++ww) osum += part[jj][ww];
        // (Through the L2s also where a launch of its own reads them, for two head tiles: 0.2 us of a call slower up to 7 MB of partials, the
        // same up to 12, 0.6 to 3 us faster from there (80 shapes; units that share lines, heads of 40 or 80 columns, no other than whole lines).
        // For one tile, up to 10 MB, the way to memory is the longer one: 0.3 to 1.8 us (129 shapes).  A choice by the bytes when the kernel runs
        // costs its calls 0.5 to 1 %, more than it gives.)
        if (h < a.H) st_result4(a.Cpart + ((size_t)pid * a.H + h) * a.d + ucol0 + oc4, osum, NT == 2 || fuse);
      }
    }
  };

  if (has_work) {
    Seg sg;
    // rotary table: this lane's 4 column pairs start at pair li * 4 of the head
    const float* rope_lane = nullptr;
    const unsigned rope_pitch = (unsigned)(a.d_k / 2) * 8u;   // bytes per table row
    float w1c[4], w1s[4];                           // rotation by one position
    if constexpr (ROPE) {
      rope_lane = a.rope + (size_t)(col_active ? li : 0) * 8;
      const f32x4* r1 = reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(rope_lane) + (size_t)min(1, a.T - 1) * rope_pitch);
      const f32x4 v0 = r1[0], v1 = r1[1];
      w1c[0] = v0[0]; w1s[0] = v0[1]; w1c[1] = v0[2]; w1s[1] = v0[3];
      w1c[2] = v1[0]; w1s[2] = v1[1]; w1c[3] = v1[2]; w1s[3] = v1[3];
    }
    while (next_segment(sg)) {
      const int ntl = sg.ntl, len = sg.len;
      const uint16_t* Kb = sg.Kb;
      // query for this lane's 8 columns: requested here, used only after the first tiles have been
      // requested (the wait for it then overlaps theirs)
      const u32x4* qsrc = reinterpret_cast<const u32x4*>(a.q + (size_t)sg.b * a.d + (col_active ? mycol : 0));
      const u32x4 qraw0 = qsrc[0], qraw1 = qsrc[1];
      unsigned qh[4], ql[4];
      // (lanes without live columns re-read the unit's first columns: finite values that meet a zero
      //  query in the scores and accumulator rows nobody reads in the weighted sum)
      // Byte offset of element (row r, this lane's first column) from the sequence's start:
      //   (r / 32) * bandB + (r % 32) * rowB + lane_col_off
      // row-major cache: rowB = the row pitch; banded cache (32-row bands, head-major inside a band: a
      // head's 32 x d_k block is contiguous): rowB = d_k * 2 and the head's block offset joins the lane's.
      const unsigned bandB = TILE_ROWS * pitchB;
      const unsigned rowB = a.k_banded ? (unsigned)a.d_k * 2u : pitchB;
      const int lane_head = col_active ? myhead : u * a.hpu, lane_li = col_active ? li : 0;
      const unsigned lane_col_off = a.k_banded ? (unsigned)lane_head * TILE_ROWS * (unsigned)a.d_k * 2u + (unsigned)lane_li * 16u
                                               : (unsigned)(col_active ? mycol : ucol0) * 2u;
      const unsigned lane_off = (unsigned)(rg * RR) * rowB + lane_col_off;
      float mrun = NEG_INF;                           // running maximum of this lane's head (log2 domain)
      bf16x8 bq[4];                                   // B operands of the score MFMA (filled below, behind the first tile requests)
      // softmax state of the weighted sum and its accumulators; accl: sum of the weights (an all-ones A operand)
      float m[NT];
      f32x4 acc[8][NT], accl[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        m[t] = NEG_INF;
        accl[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      // Tiles travel HBM -> registers (PD register sets: one tile being scored, the other in flight)
      // -> LDS slot, where the same wave picks them up one step later.
      u32x4 ts[PD][8];
      f32x4 tr[PD][2];                                // ROPE: {cos, sin} x 4 pairs at the lane's first row of the tile
      // Every call issues the same number of loads on every path (also for k past the end of the segment,
      // where all rows collapse onto the last one and nobody uses the result): the compiler's s_waitcnt
      // for the next tile's registers is then exact.
      auto load_tile = [&](u32x4 (&t)[8], f32x4 (&r)[2], int k) {
        const int st = __builtin_amdgcn_readfirstlane(sg.t0 + k * sg.stride - (k > 0 ? sg.lead : 0));
        if constexpr (ROPE) {
          const int row = min(st * TILE_ROWS + rg * 8, a.T - 1);
          const f32x4* rp = reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(rope_lane) + (size_t)row * rope_pitch);
          r[0] = rp[0];
          r[1] = rp[1];
        }
        if (k < ntl && (st + 1) * TILE_ROWS <= len) {
          // full tile: uniform row base + per-lane 32-bit offset
          const char* tb = reinterpret_cast<const char*>(Kb) + (size_t)st * bandB;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            t[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tb + (size_t)(j * RJ) * rowB + lane_off));
        } else {
          // last, partial tile (rows past the end re-read the last row; masked in the scores) or no tile
          const int r0 = st * TILE_ROWS + rg * RR;
          const char* cb = reinterpret_cast<const char*>(Kb) + lane_col_off;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int rr = max(min(r0 + j * RJ, len - 1), 0);
            t[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(cb + (size_t)(rr >> 5) * bandB + (size_t)(rr & 31) * rowB));
          }
        }
      };
      // ---- all heads' words of tile k: requested here, waited for in sum_step
      constexpr int GW = 2 * NT;                      // 16-byte words per lane and tile
      u32x4 gq[GW];
      auto gather = [&](int k) {
        const u32x4* base = team_ring + (size_t)((sg.it0 + (unsigned)k + 1u) & (EXCH_SLOTS - 1)) * (HP * 8) + (n * 4 + kg);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int t = 0; t < NT; ++t) gq[c * NT + t] = ld_exch(base + (c * HP + t * 16) * 4);
      };
      auto pin_gq = [&]() {                           // (the asm loads' results, as far as the compiler is concerned)
        if constexpr (NT == 1) asm volatile("" : "+v"(gq[0]), "+v"(gq[1]) : : "memory");
        else asm volatile("" : "+v"(gq[0]), "+v"(gq[1]), "+v"(gq[2]), "+v"(gq[3]) : : "memory");
      };
      // ---- tile k out of its registers into its LDS slot (the tile that was there has been summed in the
      //      step before); tile k+2 requested into the registers
      auto park = [&](int k, auto SI) {
        u32x4 (&cur)[8] = ts[decltype(SI)::value];
        char* sl = myslots + (k & (NS - 1)) * SLOT_PITCH + wpos;
#pragma unroll
        for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(sl + j * RJ * ROW_PITCH) = cur[j];
      };
      auto request = [&](int k, auto SI) { load_tile(ts[decltype(SI)::value], tr[decltype(SI)::value], k); };
      // ---- softmax numerators of the unit's heads from the 8 scores of a lane (row of score jj given by
      //      row_of), against the head's running maximum
      auto numerators = [&](int k, float (&sc)[8], unsigned (&pw)[4], auto&& row_of) {
        const int st = sg.t0 + k * sg.stride - (k > 0 ? sg.lead : 0);
        if ((st + 1) * TILE_ROWS > len) {             // last, partial tile: rows past the end weigh nothing
#pragma unroll
          for (int j = 0; j < 8; ++j) sc[j] = (st * TILE_ROWS + row_of(j) < len) ? sc[j] : NEG_INF;
        }
        float tmax = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
        tmax = max_over_row_groups(tmax);
        // The reference moves only when the maximum has grown by more than SOFTMAX_SLACK (log2 domain):
        // numerators stay below 2^SOFTMAX_SLACK, which costs bf16 and the fp32 sums nothing, and the
        // accumulators are rescaled rarely instead of at most early tiles.
        mrun = (tmax > mrun + SOFTMAX_SLACK) ? tmax : mrun;
        const float ref = (mrun == NEG_INF) ? 0.f : mrun;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bf16x2 v = {(__bf16)__builtin_amdgcn_exp2f(sc[2 * i] - ref), (__bf16)__builtin_amdgcn_exp2f(sc[2 * i + 1] - ref)};
          pw[i] = __builtin_bit_cast(unsigned, v);
        }
      };
      // ---- scores of tile k on MFMA, from its LDS slot: S[row][n] = sum_c K[row][c] q_n[c], two M tiles of
      //      16 rows, four k-steps of 32 columns.  A lane ends up with rows mt*16 + rg*4 + r of column idx.
      auto score_mfma = [&](int k, unsigned (&pw)[4]) {
        const char* sl = myslots + (k & (NS - 1)) * SLOT_PITCH + spos;
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(sl + ks * 64);
          const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(sl + ks * 64 + 16 * ROW_PITCH);
          s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bq[ks], s0, 0, 0, 0);
          s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bq[ks], s1, 0, 0, 0);
        }
        float sc[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {                 // query hi + lo: neighbour columns
          sc[r] = dpp_add<0xB1>(s0[r]);
          sc[4 + r] = dpp_add<0xB1>(s1[r]);
        }
        numerators(k, sc, pw, [&](int jj) { return (jj >> 2) * 16 + rg * 4 + (jj & 3); });
      };
      // ---- scores of tile k with rotary keys, on the vector ALU from the tile's registers; a lane ends up
      //      with rows rg*8 + j of its head
      auto score_rotary = [&](int k, auto SI, unsigned (&pw)[4]) {
        u32x4 (&cur)[8] = ts[decltype(SI)::value];
        f32x4 (&rot)[2] = tr[decltype(SI)::value];
        float sc[8];
        float cc[4] = {rot[0][0], rot[0][2], rot[1][0], rot[1][2]};
        float ss[4] = {rot[0][1], rot[0][3], rot[1][1], rot[1][3]};
        // (-q2, q1) of every pair, same hi + lo split: rebuilt for every tile (three operations per word) so
        // that the eight registers are free during the rest of the step; the empty asm keeps the compiler
        // from hoisting them out of the loop again
        unsigned ph[4], pl[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          unsigned h = qh[c], l = ql[c];
          asm volatile("" : "+v"(h), "+v"(l));
          ph[c] = ((h >> 16) ^ 0x8000u) | (h << 16);
          pl[c] = ((l >> 16) ^ 0x8000u) | (l << 16);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float sj = 0.f;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const unsigned kw = cur[j][c];             // (a scalar copy: bit_cast of a vector element picks lane 0)
            const bf16x2 kv = __builtin_bit_cast(bf16x2, kw);
            float da = __builtin_amdgcn_fdot2_f32_bf16(kv, __builtin_bit_cast(bf16x2, qh[c]), 0.f, false);
            da = __builtin_amdgcn_fdot2_f32_bf16(kv, __builtin_bit_cast(bf16x2, ql[c]), da, false);
            float db = __builtin_amdgcn_fdot2_f32_bf16(kv, __builtin_bit_cast(bf16x2, ph[c]), 0.f, false);
            db = __builtin_amdgcn_fdot2_f32_bf16(kv, __builtin_bit_cast(bf16x2, pl[c]), db, false);
            sj = fmaf(cc[c], da, sj);
            sj = fmaf(ss[c], db, sj);
            if (j < 7) {                              // on to the next row's position
              const float nc = fmaf(cc[c], w1c[c], -ss[c] * w1s[c]);
              ss[c] = fmaf(ss[c], w1c[c], cc[c] * w1s[c]);
              cc[c] = nc;
            }
          }
          sc[j] = sj;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {                 // sum over the head's lanes, all inside a 16-lane row
          if (lphp > 1) sc[j] = dpp_add<0xB1>(sc[j]);      // lane ^ 1   (a head spans lphp = 1, 2, 4, 8 or 16 lanes)
          if (lphp > 2) sc[j] = dpp_add<0x4E>(sc[j]);      // lane ^ 2
          if (lphp > 4) sc[j] = dpp_add<0x141>(sc[j]);     // other quad of the 8-lane half
          if (lphp > 8) sc[j] = dpp_add<0x140>(sc[j]);     // other half of the row
        }
        numerators(k, sc, pw, [&](int jj) { return rg * 8 + jj; });
      };
      // ---- publish tile k's words: {tag, running max, p0 p1, p2 p3} and {tag, 0, p4 p5, p6 p7} per row group
      auto publish = [&](int k, const unsigned (&pw)[4]) {
        const unsigned itk = sg.it0 + (unsigned)k + 1u;
        const unsigned tag = a.tag_base + itk;
        u32x4* ring = team_ring + (size_t)(itk & (EXCH_SLOTS - 1)) * (HP * 8);
        const int head = ROPE ? myhead : mhead;
        if (ROPE ? pub_lane : mpub_lane) {
          st_exch(ring + (head * 4 + rg), u32x4{tag, __float_as_uint(mrun), pw[0], pw[1]}, xl);
          st_exch(ring + ((HP + head) * 4 + rg), u32x4{tag, 0u, pw[2], pw[3]}, xl);
        }
      };
      // ---- the scoring half of a step: tile k parked, its numerators published
      auto score_tile = [&](int k, auto SI) {
        unsigned pw[4];
        if constexpr (ROPE) {
          score_rotary(k, SI, pw);
          park(k, SI);
        } else {
          park(k, SI);
          score_mfma(k, pw);
        }
        publish(k, pw);
      };
      // ---- weighted sum of tile k with the words gathered for it.  (k-slot jj of the operands is the row
      //      the numerators' jj stands for: rg*8 + jj with rotary keys, (jj / 4) * 16 + kg * 4 + jj % 4 otherwise.)
      //      HALF: the tile comes out of its slot in two halves of 64 columns (the first four and the last
      //      four columns of every lane), which keeps fewer registers live.
      auto tile_half = [&](int k, auto HALF, u32x4 (&am)[4]) {
        constexpr int hf = decltype(HALF)::value;
        const char* sl = myslots + (k & (NS - 1)) * SLOT_PITCH + (ROPE ? wpos : ppos) + hf * 8;
        unsigned lo[8], hi[8];                        // columns 4 hf + {0, 1} and 4 hf + {2, 3} of the lane's 8 rows
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
          const unsigned off = ROPE ? jj * ROW_PITCH : ((jj >> 2) * 16 + (jj & 3)) * ROW_PITCH;
          const auto v = *reinterpret_cast<const __attribute__((ext_vector_type(2))) unsigned*>(sl + off);
          lo[jj] = v[0];
          hi[jj] = v[1];
        }
#pragma unroll
        for (int jp = 0; jp < 4; ++jp) {                // (the 8 x 4 half of transpose8x8)
          am[0][jp] = __builtin_amdgcn_perm(lo[2 * jp + 1], lo[2 * jp], 0x05040100u);
          am[1][jp] = __builtin_amdgcn_perm(lo[2 * jp + 1], lo[2 * jp], 0x07060302u);
          am[2][jp] = __builtin_amdgcn_perm(hi[2 * jp + 1], hi[2 * jp], 0x05040100u);
          am[3][jp] = __builtin_amdgcn_perm(hi[2 * jp + 1], hi[2 * jp], 0x07060302u);
        }
      };
      // ---- every word of tile k must carry its tag; gather again while any is missing
      auto await_words = [&](int k) {
        const unsigned tag = a.tag_base + sg.it0 + (unsigned)k + 1u;
        pin_gq();
        unsigned long long since = ~0ull;
        for (;;) {
          unsigned bad = 0;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const unsigned bt = (gq[t][0] ^ tag) | (gq[NT + t][0] ^ tag);
            bad |= (heads_full || (t * 16 + n) < a.H) ? bt : 0u;
          }
          if (__all(bad == 0)) break;
          if (dead || out_of_time(since)) { give_up(); break; }
          __builtin_amdgcn_s_sleep(8);
          gather(k);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          pin_gq();
        }
      };
      auto sum_finish = [&](int k, u32x4 (&am)[4]) {    // am: the first half, already out of the slot
        bf16x8 pb[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const bool live = heads_full || (t * 16 + n) < a.H;      // padded head: no weights at all
          const float mn = live ? __uint_as_float(gq[t][1]) : NEG_INF;
          const float ref = (mn == NEG_INF) ? 0.f : mn;            // all -inf so far: exp2(-inf - 0) = 0
          const float alpha = __builtin_amdgcn_exp2f(m[t] - ref);
          m[t] = mn;
          const u32x4 pw = live ? u32x4{gq[t][2], gq[t][3], gq[NT + t][2], gq[NT + t][3]} : u32x4{0u, 0u, 0u, 0u};
          pb[t] = __builtin_bit_cast(bf16x8, pw);
          if (__any(alpha != 1.f)) {
            accl[t] *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i][t] *= alpha;
          }
        }
        const u32x4 ones_bits = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
        const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);
#pragma unroll
        for (int t = 0; t < NT; ++t) accl[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[t], accl[t], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bf16x8 av = __builtin_bit_cast(bf16x8, am[i]);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb[t], acc[i][t], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);            // (the second half's registers only after the first half's are dead)
        tile_half(k, std::integral_constant<int, 1>{}, am);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bf16x8 av = __builtin_bit_cast(bf16x8, am[i]);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[4 + i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb[t], acc[4 + i][t], 0, 0, 0);
        }
      };
      // One step (k >= 1).  Tile k is scored and published first; only then are the words of tile k-1
      // requested (every workgroup of the group published them a scoring time ago), and behind them
      // tile k+2 (LOADS_PER_TILE loads, the only vector-memory operations younger than the gather when it
      // is waited for).  The tile comes out of its slot while the words travel.  (Requesting the words
      // before the scoring instead, and tile k+2 only after they have been checked, was measured: no
      // faster at 8 tiles per wave, 4 % slower on long sequences.)
      constexpr int LOADS_PER_TILE = ROPE ? 10 : 8;
      auto step = [&](int k, auto SI) {
        u32x4 am[4];
        score_tile(k, SI);
        gather(k - 1);
        request(k + PD, SI);
        tile_half(k - 1, std::integral_constant<int, 0>{}, am);
        if constexpr (ROPE) asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        static_assert(LOADS_PER_TILE == (ROPE ? 10 : 8), "the wait above counts the loads of one tile");
        await_words(k - 1);
        sum_finish(k - 1, am);
      };

      f32x4 qx[4][2];                                 // the query columns behind bq, as loaded
      bool qlive[4];
      if constexpr (!ROPE) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const int C = ks * 4 + rg, hq = C / lphp, lq = C % lphp;
          qlive[ks] = lq < a.lph && hq < a.hpu && u * a.hpu + hq < a.H && (idx >> 1) == hq;
          const f32x4* src = reinterpret_cast<const f32x4*>(a.q + (size_t)sg.b * a.d + (qlive[ks] ? (u * a.hpu + hq) * a.d_k + lq * 8 : 0));
          qx[ks][0] = src[0];
          qx[ks][1] = src[1];
        }
      }
#pragma unroll
      for (int k = 0; k < PD; ++k) load_tile(ts[k], tr[k], k);
      // B operands of the score MFMA: k-step ks covers chunks ks*4 .. ks*4+3 of the unit; this lane holds
      // chunk ks*4 + rg of column n = idx: the head's query (pre-scaled, bf16 hi or lo) where the chunk
      // belongs to that head, zero elsewhere.  (Requested ahead of the first tiles, converted behind
      // their requests: the wait for it then overlaps theirs.)
      if constexpr (!ROPE) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const f32x4 x0 = qx[ks][0], x1 = qx[ks][1];
          const bool live = qlive[ks];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float f = live ? (i < 4 ? x0[i] : x1[i - 4]) * a.qscale : 0.f;
            const __bf16 h = (__bf16)f;
            bq[ks][i] = (idx & 1) ? (__bf16)(f - (float)h) : h;
          }
        }
      }
      // the query, pre-scaled (log2 domain), split into bf16 hi + lo pairs so that the dot products run
      // on v_dot2c_f32_bf16 without losing the fp32 query
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const unsigned r0 = c < 2 ? qraw0[2 * c] : qraw1[2 * c - 4], r1 = c < 2 ? qraw0[2 * c + 1] : qraw1[2 * c - 3];
        const float f0 = col_active ? __uint_as_float(r0) * a.qscale : 0.f;
        const float f1 = col_active ? __uint_as_float(r1) * a.qscale : 0.f;
        const __bf16 h0 = (__bf16)f0, h1 = (__bf16)f1;
        const bf16x2 hi = {h0, h1};
        const bf16x2 lo = {(__bf16)(f0 - (float)h0), (__bf16)(f1 - (float)h1)};
        qh[c] = __builtin_bit_cast(unsigned, hi);
        ql[c] = __builtin_bit_cast(unsigned, lo);
      }
      {
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        // (the request is unconditional: a path into the loop without it would make the compiler wait for
        //  every outstanding load at the top of each step)
        if (ntl > 0) score_tile(0, S0{});
        request(PD, S0{});
        // Whole rounds of PD steps without a condition between them (a step that may be skipped
        // inside the loop would make the compiler's waits for the tile registers conservative).
        int k = 1;
        for (; k + PD <= ntl; k += PD) {
          step(k, S1{});
          step(k + 1, S0{});
        }
        if (k < ntl) step(k, S1{});
        // the last tile: nothing left to score while its words travel
        if (ntl > 0) {
          u32x4 am[4];
          gather(ntl - 1);
          tile_half(ntl - 1, std::integral_constant<int, 0>{}, am);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          await_words(ntl - 1);
          sum_finish(ntl - 1, am);
        }
      }

      // ---- end of this sequence's share ---------------------------------------------------------------
      if (by_seq) {
        // the whole share was this wave's: its partial needs no merge.  A lane holds 8 consecutive columns
        // of a head per accumulator row; stored from there, an instruction writes 64 16-byte pieces into 64
        // different cache lines (7 of 71 us at 64 sequences of 1500 rows).  So head tile t goes through the
        // wave's (idle) slot t and leaves with a head's columns on consecutive lanes.
        constexpr int OP = 128 + 4;                     // floats per head row in the slot (padding: no bank conflicts)
        static_assert(16 * OP * 4 <= SLOT_PITCH && NT <= NS, "a head tile's block must fit one slot");
        // (Two head tiles: the lane made here, as below, because what waits for this in scratch delays the loads in flight.  One tile has
        // registers for it: 243 ragged x 165 rows x 16 heads x 72 57.0 us, with the lane made here 58.3.)
        const int ln = NT == 1 ? lane : fresh_lane(), nl = ln & 15, kl = ln >> 4;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float* const ob = reinterpret_cast<float*>(myslots + t * SLOT_PITCH) + nl * OP;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int oc = col_of_group(kl * 4 + r);
            if (oc < 0) continue;
            *reinterpret_cast<f32x4*>(ob + oc) = f32x4{acc[0][t][r], acc[1][t][r], acc[2][t][r], acc[3][t][r]};
            *reinterpret_cast<f32x4*>(ob + oc + 4) = f32x4{acc[4][t][r], acc[5][t][r], acc[6][t][r], acc[7][t][r]};
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (LDS operations of one wave complete in order)
        {
          // head hl of the block on lanes 32 (hl % 2) .. +31, four columns per lane; two heads per instruction
          const int c4 = (ln & 31) * 4;
          const float* src = reinterpret_cast<const float*>(myslots) + (ln >> 5) * OP + c4;
          float* dst = a.Cpart + ((size_t)sg.pid * a.H + (ln >> 5)) * a.d + ucol0 + c4;
          const int nh = min(a.H, HP);
#pragma unroll 1
          for (int hl = ln >> 5; hl < nh; hl += 2) {
            const int t = hl >> 4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(src + (t * (SLOT_PITCH / 4 - 16 * OP)));
            if (c4 < uwc) st_result4(dst, v, fuse);
            src += 2 * OP;
            dst += 2 * (size_t)a.d;
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the next share parks its tiles in these slots)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int h = t * 16 + nl;
          if (u == 0 && kl == 0 && h < a.H) {
            st_result(a.mpart + (size_t)sg.pid * a.H + h, m[t], fuse);
            st_result(a.lpart + (size_t)sg.pid * a.H + h, accl[t][0], fuse);
          }
        }
        continue;
      }
      // ---- by context: merge the waves and write one partial (every wave of the workgroup walks the
      //      same shares, so all of them meet at these barriers) -------------------------------------
      // What depends on the lane is made here, from a lane number made here, as in the by-sequence partial above: made before the
      // stream, it waited in scratch (60 bytes a lane, 88 with rotary keys), a round trip for each piece that is fetched
      // back.  Without any, and with what else is said here: 1 x 16384 rows x 32 heads x 128 51.8 -> 43.7 us, 1 x 200 22.9 -> 19.7,
      // 8 ragged x 5000 x 32 x 96 with rotary keys 66.6 -> 59.9, 16 ragged x 32768 (banded) 370 -> 351; 64 x 1500 x 20 x 64, 12
      // bytes before, 70.6 -> 69.1.  (Barriers for LDS only: __syncthreads() would also wait for the requests past the end and,
      // between shares, for the partial's write-through stores, whose arrival only the flag at the end of the launch depends on.)
      const int ln = fresh_lane(), nl = ln & 15, kl = ln >> 4;
      if (kl == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) marr[t][nl][p] = m[t];
      }
      lds_barrier();                                  // every slot is idle from here on
      {
        // accumulators -> mbuf[wave][head][col], in MFMA layout, scaled to the maximum over the waves
        f32x4 mw[NT][2];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i) mw[t][i] = *reinterpret_cast<const f32x4*>(&marr[t][nl][i * 4]);
        float wsc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float mall = NEG_INF;
#pragma unroll
          for (int ww = 0; ww < NP; ++ww) mall = fmaxf(mall, mw[t][ww >> 2][ww & 3]);
          wsc[t] = (m[t] == NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(m[t] - mall);
          if (kl == 0) larr[t][nl][p] = accl[t][0] * wsc[t];   // every accumulator row holds the same sum
        }
        float* mine = mbuf + (size_t)p * HP * MERGE_PITCH + nl * MERGE_PITCH;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int oc = col_of_group(kl * 4 + r);
          if (oc < 0) continue;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            f32x4* dst = reinterpret_cast<f32x4*>(mine + t * 16 * MERGE_PITCH + oc);
            dst[0] = f32x4{acc[0][t][r], acc[1][t][r], acc[2][t][r], acc[3][t][r]} * wsc[t];
            dst[1] = f32x4{acc[4][t][r], acc[5][t][r], acc[6][t][r], acc[7][t][r]} * wsc[t];
          }
        }
      }
      lds_barrier();
      write_partial(sg.pid, ln);
      lds_barrier();                                  // the slots are reused by the next share
    }
  }
  if (!fuse) return;

  // ========================= single-launch mode: merge + projection ===============================
  // This workgroup's partials are out (write-through stores, waited for) before its arrival flag: the launch's id, and in the
  // three lowest bits the XCD it runs on.
  int phead, psplit;
  projection_share(phead, psplit);
  const unsigned flag_id = a.launch_id << 3, xcc = my_xcc() ^ (a.proj.apart ? psplit & 1 : 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) st_result(reinterpret_cast<int*>(a.flags) + blockIdx.x, (int)(flag_id | xcc), true);
  if (phead >= a.proj.H) return;
  // (everything of the stream phase is over in this workgroup: its LDS is reused)
  ProjShared<1>& psm = *reinterpret_cast<ProjShared<1>*>(sbuf);
  project_work<1, true, false, false, false>(a.proj, phead, psplit, 0, prefix, psm, red, [&]() {
    // Every workgroup's partials must be out: all arrival flags carry this launch's id.  False: the workgroups of this head
    // are to meet in an XCD's L2, and do not run on one XCD.
    bool together = true;
    if (wu == 0) {
      unsigned long long since = ~0ull;
      for (;;) {
        // all flags of a poll in one round trip (a chain of "ok && load" would take one trip per 64 flags)
        unsigned seen[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          seen[j] = __hip_atomic_load(a.flags + min(lane + 64 * j, (int)gridDim.x - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned other = (seen[0] ^ flag_id) | (seen[1] ^ flag_id) | (seen[2] ^ flag_id) | (seen[3] ^ flag_id);
        static_assert(FUSED_MAX_GRID <= 256, "four flags per lane cover the grid");
        if (__all(other < 8)) {
          // (this head's workgroups: i % 8 as here, i / 8 in the csw slots of the head)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int i = lane + 64 * j, s0 = (int)(blockIdx.x >> 3) - psplit;
            if ((i & 7) == (int)(blockIdx.x & 7) && (unsigned)((i >> 3) - s0) < (unsigned)a.proj.csw) together &= (seen[j] & 7) == xcc;
          }
          together = __all(together) || a.proj.xcd_local == 0 || a.proj.csw == 1;
          break;
        }
        if (dead || out_of_time(since)) { give_up(); break; }
        __builtin_amdgcn_s_sleep(4);
      }
      if (lane == 0) psm.is_last = together;
    }
    __syncthreads();
    return psm.is_last != 0;
  });
}

// Records which XCD each workgroup of a 256-workgroup launch runs on.
__global__ __launch_bounds__(512) void xcc_probe_kernel(unsigned* out) {
  const unsigned xcc = my_xcc();
  if (threadIdx.x == 0) out[blockIdx.x] = xcc;
  for (int i = 0; i < 200; ++i) __builtin_amdgcn_s_sleep(10);        // stay resident while the rest start
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
bool fused_geometry(int B, int H, int T, int d, FusedGeom* g) {
  if (H < 1 || d % H != 0) return false;
  const int d_k = d / H;
  if (d_k % 8 != 0 || d_k < 16 || d_k > 128 || H > 32 || B > FUSED_MAX_B) return false;   // (16 score columns hold 8 heads of a unit, hi + lo)
  g->lph = d_k / 8;
  int lphp = 1;
  while (lphp < g->lph) lphp <<= 1;
  g->lphp = lphp;
  g->hpu = 16 / lphp;
  g->G = (H + g->hpu - 1) / g->hpu;
  g->NT = H <= 16 ? 1 : 2;
  g->NP = FUSED_WAVES;
  const int cus = FUSED_MAX_GRID;
  if (g->G > cus) return false;
  if (g->G <= 32) {
    g->gpx = 32 / g->G;
    if (g->gpx > 8) g->gpx = 8;                     // at most PROJ_MAX_PARTS groups
    g->NG = 8 * g->gpx;
    g->grid = cus;
  } else {
    g->gpx = 0;
    g->NG = cus / g->G;
    g->grid = g->NG * g->G;
  }
  g->nparts = B + g->NG - 1;
  return true;
}

// True when workgroups i and j of a 256-workgroup launch share an XCD exactly where i % 8 == j % 8: a probe
// launch on `st` that records each workgroup's XCD into `dev_buf` (device memory, 256 unsigned), read
// back with a blocking copy.  The caller caches the answer per device.
bool probe_xcd_round_robin(unsigned* dev_buf, hipStream_t st) {
  unsigned h[256];
  hipLaunchKernelGGL(xcc_probe_kernel, dim3(256), dim3(512), 0, st, dev_buf);
  bool ok = hipMemcpyAsync(h, dev_buf, sizeof(h), hipMemcpyDeviceToHost, st) == hipSuccess &&
            hipStreamSynchronize(st) == hipSuccess;
  if (ok)
    for (int i = 8; i < 256 && ok; ++i) ok = h[i] == h[i & 7];
  if (ok)
    for (int i = 1; i < 8 && ok; ++i)
      for (int j = 0; j < i; ++j) ok = ok && h[i] != h[j];
  (void)hipGetLastError();
  return ok;
}

// Workgroups of the stream kernel one compute unit can hold at once (0 on error): the launch is only
// safe when all of its workgroups are resident together.
int fused_blocks_per_cu(const FusedGeom& g, bool rope) {
  int n = 0;
  auto ask = [&](auto nt, auto rp, auto lp) {                 // (the smaller figure of the two partitions' instantiations)
    int n0 = 0, n1 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n0, fused_stream_kernel<decltype(nt)::value, decltype(rp)::value, decltype(lp)::value, false>,
                                                     g.NP * 64, 0) != hipSuccess) { n0 = 0; (void)hipGetLastError(); }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n1, fused_stream_kernel<decltype(nt)::value, decltype(rp)::value, decltype(lp)::value, true>,
                                                     g.NP * 64, 0) != hipSuccess) { n1 = 0; (void)hipGetLastError(); }
    n = n0 < n1 ? n0 : n1;
  };
  auto with_lphp = [&](auto nt, auto rp) {
    if (g.lphp == 16) ask(nt, rp, std::integral_constant<int, 16>{});
    else if (g.lphp == 8) ask(nt, rp, std::integral_constant<int, 8>{});
    else if (g.lphp == 4) ask(nt, rp, std::integral_constant<int, 4>{});
    else ask(nt, rp, std::integral_constant<int, 2>{});
  };
  auto with_rope = [&](auto nt) {
    if (rope) with_lphp(nt, std::true_type{});
    else with_lphp(nt, std::false_type{});
  };
  if (g.NT == 1) with_rope(std::integral_constant<int, 1>{});
  else with_rope(std::integral_constant<int, 2>{});
  return n;
}

// By-sequence partition: how many equal shares to cut every sequence into so that the shares fill
// the wave slots (groups x waves) evenly (1..4), or 0 to keep the balanced by-context partition.  Ragged
// batches qualify only with many shares per slot.
int fused_by_sequence(const FusedGeom& g, int B, bool ragged) {
  const long slots = (long)g.NG * FUSED_WAVES;
  int best = 0;
  double best_waste = 1.13;                           // at most 13 % idle slot-time
  for (int s = 1; s <= 4; ++s) {
    const long shares = (long)B * s, rounds = (shares + slots - 1) / slots;
    const double waste = (double)(rounds * slots) / (double)shares;
    if (ragged && shares < 4 * slots) continue;
    if (waste < best_waste - 0.04) { best = s; best_waste = waste; }
  }
  return best;
}

size_t fused_exch_bytes(const FusedGeom& g) {
  // per team and ring slot: two 16-byte words for each (padded head, row group of 8)
  return (size_t)g.NG * g.NP * EXCH_SLOTS * (g.NT * 16) * 8 * 16;
}

void launch_fused_stream(const FusedGeom& g, const FusedArgs& a, hipStream_t st) {
  dim3 grid(g.grid), block(g.NP * 64);
  auto go = [&](auto nt, auto rope, auto lphp) {
    if (a.by_sequence)
      hipLaunchKernelGGL((fused_stream_kernel<decltype(nt)::value, decltype(rope)::value, decltype(lphp)::value, true>), grid, block, 0, st, a);
    else
      hipLaunchKernelGGL((fused_stream_kernel<decltype(nt)::value, decltype(rope)::value, decltype(lphp)::value, false>), grid, block, 0, st, a);
  };
  auto with_lphp = [&](auto nt, auto rope) {
    if (g.lphp == 16) go(nt, rope, std::integral_constant<int, 16>{});
    else if (g.lphp == 8) go(nt, rope, std::integral_constant<int, 8>{});
    else if (g.lphp == 4) go(nt, rope, std::integral_constant<int, 4>{});
    else go(nt, rope, std::integral_constant<int, 2>{});
  };
  auto with_rope = [&](auto nt) {
    if (a.rope) with_lphp(nt, std::true_type{});
    else with_lphp(nt, std::false_type{});
  };
  if (g.NT == 1) with_rope(std::integral_constant<int, 1>{});
  else with_rope(std::integral_constant<int, 2>{});
}

// Sequences per workgroup of the projection, in MFMA N tiles of 16 (1, 2 or 4).  One tile keeps the
// kernel out of register spills and gives more workgroups; it costs one more pass over W_KV per 16
// sequences, which is only worth it while those passes stay small.
int proj_batch_tiles(int B, int rows, int e, int H) {
  if (B <= 16) return 1;
  const long w_bytes = (long)rows * e * 2;
  // One tile of 16 sequences per workgroup (no register spills, most workgroups) as long as one round of
  // workgroups, one per CU, covers every (head, batch chunk); W is read once per batch chunk (mostly from
  // L2), which bounds the number of chunks.  Measured at B = 64, H = 20: 14.8 us against 19.1 us with two tiles.
  for (int nbt = 1; nbt <= 2; nbt *= 2) {            // (four batch tiles per workgroup measured slower than two rounds)
    const long chunks = (B + 16 * nbt - 1) / (16 * nbt);
    if ((long)H * chunks <= 256 && w_bytes * chunks <= (64L << 20)) return nbt;
  }
  if (w_bytes * ((B + 15) / 16) <= (64L << 20)) return 1;
  return B <= 32 ? 2 : 4;
}

int proj_row_splits(int H, int rows, int e, int B) {
  // one 32-row tile of W per wave (8 waves = 256 rows per workgroup) unless that makes more
  // workgroups than CUs
  const int per = 16 * proj_batch_tiles(B, rows, e, H);
  const int zb = (B + per - 1) / per;
  const int csw = (rows + 8 * TILE_ROWS - 1) / (8 * TILE_ROWS), cap = proj_splits_per_unit(H * zb);
  return csw > cap ? cap : csw;
}

// Floats of a sequence's partial sums: every head's column groups of 8 in whole fours.
int proj_part_row(int H, int d_k) { return H * ((d_k + 31) / 32 * 32); }

int proj_rows_per_split(int rows, int csw) {
  return ((rows + csw - 1) / csw + TILE_ROWS - 1) / TILE_ROWS * TILE_ROWS;
}

// Whether a call's loads of its weight matrices are nontemporal (where one batch chunk reads a matrix): weights of at least 64 MB,
// in a call that is known to read 96 MB of what the memory-side cache (256 MB) would keep: its weights, and an X-cache that is
// read once.  Three such layers fill that cache, so a model's next token finds nothing of W there, and the loads are faster where
// they ask for no room in it.  us with temporal -> nontemporal loads, layers of together at least 0.9 GB in turn; three
// layers; one layer alone, whose weights the cache does keep and which is slower for it:
//   block, 16 sequences x 4096 columns, rotary  114.1 -> 111.3   113.6 -> 107.6   105.2 -> 106.5
//   block, 1 x 4096                              55.7 -> 52.7     55.0 -> 50.9     49.8 -> 51.9
//   block, 1 x 3584                              50.4 -> 47.8     49.4 -> 47.7     45.9 -> 46.9
//   vanilla block, 4 x 4096                      84.3 -> 80.5     89.0 -> 85.6     85.4 -> 86.7
//   64 heads x 8192 columns, 1 x 400 rows        45.7 -> 43.4     45.8 -> 43.5     38.5 -> 42.9   (2 x 4000: 98.9 -> 98.0)
//   X-cache, 128 heads, 8 x 4096 x 1024          71.4 -> 70.3     71.2 -> 69.4     66.0 -> 67.4   (16 x 4096: 103.1 -> 102.7)
// Below 96 MB three layers fit (block of 2 x 3072 columns, 75 MB of weights: 50.9 -> 49.6, but 47.9 -> 49.1 and 47.4 -> 48.8).
// Fewer weights gain nothing (X-cache, 80 heads, 8 x 4096 x 1280, 52 MB of weights: 81.9 -> 81.9, 81.6 -> 81.4, 71.5 -> 74.8), nor
// do several batch chunks, which share W in L2 (24 sequences x 4096: 72.5 -> 73.4).  Rows that a call may have but need not use do
// not count (X-cache, 64 heads, 400 of 4096 rows in use: 38.3 -> 39.1, 35.4 -> 36.2, 35.0 -> 39.9), nor do caches that are
// read twice, the second time from the memory-side cache (40 heads x 5120 columns, 4 ragged sequences of 3000..6000 rows: 121.3
// -> 129.2 with three layers or more; 2 ragged of 2500..4001 rows 58.2 -> 58.0).
bool read_once(size_t weight_bytes, size_t cache_bytes) {
  return weight_bytes >= ((size_t)64 << 20) && weight_bytes + cache_bytes >= ((size_t)96 << 20);
}

template <bool DENSE>
static void launch_product(const ProjArgs& a, int nbt, int units_per_chunk, hipStream_t st) {
  const int chunks = (a.B + 16 * nbt - 1) / (16 * nbt);
  dim3 grid(8u * a.csw * (((unsigned)units_per_chunk * chunks + 7) / 8)), block(512);
  auto launch = [&](auto nb, auto once) {
    if constexpr (!DENSE && decltype(nb)::value == 1)
      if (a.B <= 4) {                                  // (FEW: project_work)
        hipLaunchKernelGGL((project_mfma_kernel<1, false, decltype(once)::value, true>), grid, block, 0, st, a);
        return;
      }
    hipLaunchKernelGGL((project_mfma_kernel<decltype(nb)::value, DENSE, decltype(once)::value, false>), grid, block, 0, st, a);
  };
  auto go = [&](auto nb) {
    // (a block's matrices are at most 4096 columns wide: more than one batch tile always come in more than one chunk)
    if constexpr (!DENSE || decltype(nb)::value == 1)
      if (a.once && chunks == 1) return launch(nb, std::true_type{});
    launch(nb, std::false_type{});
  };
  if (nbt == 1) go(std::integral_constant<int, 1>{});
  else if (nbt == 2) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 4>{});
}

void launch_project_mfma(ProjArgs a, hipStream_t st) {
  const int nbt = proj_batch_tiles(a.B, a.rows, a.e, a.H);
  a.crows = proj_rows_per_split(a.rows, a.csw);
  launch_product<false>(a, nbt, a.H, st);
}

// out_m = x W_m for a.nmat matrices in one launch (a.Cpart = x, a.csw from dense_row_splits).
void launch_dense_mfma(ProjArgs a, hipStream_t st) {
  const int nbt = proj_batch_tiles(a.B, a.rows, a.e, a.H * a.nmat);
  a.crows = proj_rows_per_split(a.rows, a.csw);
  a.mode = 2;
  launch_product<true>(a, nbt, a.H * a.nmat, st);
}

int dense_row_splits(int H, int nmat, int rows, int e, int B) {
  return proj_row_splits(H * nmat, rows, e, B);
}

}  // namespace slim
