// Internal launch interface between the C-ABI layer (slim_api.hip) and the kernel files.
// Everything here is device-pointer based; shapes have been validated by the caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slim {

constexpr int DT_F32 = 0;
constexpr int DT_BF16 = 1;

inline int vec_elems(int dtype) { return dtype == DT_BF16 ? 8 : 4; }   // elements per 16-byte vector
inline int elem_bytes(int dtype) { return dtype == DT_BF16 ? 2 : 4; }

// ---- generic vector-ALU kernels (kernels_generic.hip) ------------------------------------------

// S[b][h][r] = scale * sum_j q[b][h*d_k + j] * M[b][r][h*d_k + j]   for r < rows_b
// (attention scores against a K-cache, eq. 2; also q_h W_K,h^T for the X-cache scheme with
//  M := W_K, rows := d_model, m_bstride := 0).  rope: nullable [rows][d_k/2] {cos, sin}; when set,
// row r is rotated by position r before the dot product (RoPE appendix, option 1).  Zeroes `ncounters` counters.
void launch_head_scores(int dtype, const float* q, long q_bstride, const void* M, long m_bstride,
                        long row_pitch, const int32_t* rows_per_b, int rows, int e, int H, int d_k,
                        float scale, float* S, long s_bstride, const float* rope, int* counters, int ncounters, int B,
                        hipStream_t st);

// S[b][h][t] = scale * sum_c qt[b][h][c] * X[b][t][c]   (X-cache scores, Fig. 4)
void launch_dense_scores(int dtype, const float* qt, const void* X, long x_bstride, int d_model,
                         const int32_t* seq_lens, int T, int H, float scale, float* S, int B,
                         hipStream_t st);

// Per (b, split): m = max_t S, l = sum_t exp(S - m), Cpart[h][c] = sum_t exp(S - m) M[t][c]
void launch_weighted_sum(int dtype, const float* S, const void* M, long m_bstride, int width,
                         const int32_t* seq_lens, int T, int H, int nsplit, float* Cpart,
                         float* mpart, float* lpart, int B, hipStream_t st);

// Splits of one sequence that one wave of the merge looks after (a lane per split).
constexpr int MERGE_MAX_SPLITS = 64;

// Merge + projection:  C[b][h] = sum_s e^{m_s - m} Cpart[b][s][h] / sum_s e^{m_s - m} l_s,
// out[b][n] = sum_c C[b][n / d_k][c] W[c][n],  W row-major [rows][e].  own_splits: sequence b has
// ceil(len_b / f32_rows_per_split(len_b)) splits (kernels_f32.hip), else nsplit.  The rows of W are shared by
// row_splits workgroups (merge_row_splits); with more than one, outpart [row_splits][B][e] and
// merge_counters(...) counters that are 0 on entry.
long merge_counters(int H, int d_k, int B);
int merge_row_splits(int H, int d_k, int rows, int B, int max_counters);
void launch_merge_project(int dtype, const float* Cpart, const float* mpart, const float* lpart, int nsplit, bool own_splits,
                          const int32_t* seq_lens, int T, const void* W, int rows, int e, int H, int d_k, float* out,
                          float* outpart, int row_splits, int* counters, int B, hipStream_t st);

// out[b][n] = sum_c x[b][c] W[c][n],  W row-major [rows][e]
void launch_project(int dtype, const float* x, const void* W, int rows, int e, float* out, int B, hipStream_t st);

// ---- fp32 caches of up to 1024 columns (kernels_f32.hip) ---------------------------------------
// Partials as launch_weighted_sum's (natural logarithms) from one kernel; zeroes `ncounters` counters.
bool f32_stream_ok(int dtype, int H, int d, int d_k);
int f32_stream_splits(int B, int T);
__host__ __device__ inline int f32_rows_per_split(int len, int nsplit) { return ((len + nsplit - 1) / nsplit + 31) / 32 * 32; }
void launch_f32_stream(const float* q, const float* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int d_k,
                       int nsplit, float scale, const float* rope, float* Cpart, float* mpart, float* lpart, int* counters,
                       int ncounters, int B, hipStream_t st);

// New token rows into the caches at row len_b - 1: K <- knew (rotated to that position when rope and
// rotate_k), V <- vnew (nullable: no V-cache); with rope, q [B][d] is rotated in place as well.
void launch_append(int dtype, const float* knew, const float* vnew, void* K, void* V, long bstride,
                   const int32_t* seq_lens, int T, int d, int d_k, const float* rope, float* q, int rotate_k,
                   int B, hipStream_t st);
void launch_zero_ints(int* p, int n, hipStream_t st);
// Plain streaming read of `bytes` (measurement only).
void launch_read_probe(const void* buf, size_t bytes, hipStream_t st);

// Vanilla K+V decode: partial (m, l, acc) per (b, split, head) then a merge.
int vanilla_heads_per_wave(int dtype, int d_k);   // heads a wave of the packed bf16 kernel covers (0: plain kernel)
void launch_vanilla(int dtype, const float* q, const void* K, const void* V, long bstride,
                    const int32_t* seq_lens, int T, int H, int d_k, int nsplit, float* acc,
                    float* mpart, float* lpart, float* out, int B, hipStream_t st);

// ---- bf16 fast path (kernels_bf16.hip) -----------------------------------------------------------
constexpr int TILE_ROWS = 32;        // cache rows per wave tile
constexpr int EXCH_SLOTS = 16;       // ring depth of the score exchange (a power of two >= 2 * FUSED_SLOTS)
constexpr int FUSED_MAX_B = 1024;    // sequences per call the fast path handles
constexpr int FUSED_MAX_GRID = 256;  // workgroups of a stream-kernel launch at most (one per compute unit)
constexpr int FUSED_WAVES = 8;       // waves per workgroup of the stream kernel, each with tiles of its own
constexpr int FUSED_SLOTS = 2;       // LDS landing slots (8 KB tiles) per wave
constexpr int FUSED_AHEAD = 2;       // register sets of a wave: one tile being scored, the other in flight
constexpr int PROJ_MAX_PARTS = 64;   // partials per sequence the projection merges
constexpr int PROJ_STAGED_ROWS = 1024;   // rows of W per workgroup of the single launch at most
// Control words of a projection whose rows of W are split, all 0 on entry: per (head, batch chunk) unit an arrival counter,
// which the last arriver leaves at 0, and in a launch of its own a 64-bit word of who takes part, a byte per XCD, which is
// used once (a block's second launch has a second set; leaving it at 0 as well, at the memory side, was 0.2 us of a launch).
// More units than this have no row splits (proj_splits_per_unit).
constexpr int PROJ_MAX_UNITS = 128;
constexpr int PROJ_CTRL_INTS = 3 * PROJ_MAX_UNITS;             // counters, words
constexpr int PROJ_SECOND_WORDS = PROJ_CTRL_INTS;              // (int offset of the second set, cleared by a block's first launch)
constexpr int PROJ_BLOCK_INTS = PROJ_SECOND_WORDS + 2 * PROJ_MAX_UNITS;
// A block's first launch finds nothing cleared: flags tagged with the launch's id, one per workgroup (row splits times units,
// a single round of workgroups at most), that it has arrived and, behind these, where it runs.
constexpr int PROJ_MAX_FLAGS = 256;
constexpr int PROJ_FLAGS_AT = 1024;                            // int offset in the control block
static_assert(PROJ_FLAGS_AT >= PROJ_BLOCK_INTS, "the flags are not among the words that are cleared");

// Row splits of `units` (head, batch chunk) pairs: a unit's workgroups share an XCD, which holds 32 of them at once
// (one per compute unit: a single round).
constexpr int proj_splits_per_unit(int units) {
  const int c = 32 / ((units + 7) / 8);
  return c < 1 ? 1 : c;
}
// Split units have a control word each, their workgroups a flag each, and a wave looks at a unit's flags a lane each.
constexpr bool proj_splits_fit() {
  for (int units = 1; units <= 16 * PROJ_MAX_UNITS; ++units) {
    const int c = proj_splits_per_unit(units);
    if (c > 1 && (units > PROJ_MAX_UNITS || units * c > PROJ_MAX_FLAGS || c > 64)) return false;
  }
  return true;
}
static_assert(proj_splits_fit(), "control words and flags of a projection whose rows of W are split");

struct FusedGeom {
  int lph, lphp, hpu;   // active lanes per head (d_k/8), lanes reserved per head, heads per unit
  int G, NG, gpx;       // column units per group, groups, groups per XCD (0 = not packed)
  int NT, NP, grid, nparts;   // MFMA head tiles, waves per workgroup
};

// The order of the fields decides which of them a kernel loads together, so has to hold together: with another eight bytes before
// csw the single launch of up to 16 heads kept ~390 scalars in lanes of vector registers and loaded arguments, which lie in
// host memory, once more on its way to the result; as it is, 86.  1 x 1500 rows x 8 heads x 64 22.4 -> 19.4 us, 1 x 1500 x 16 x 128 20.4 -> 18.1,
// 8 ragged x 2000 x 16 x 64 23.7 -> 22.6; 32 heads the same within 0.5 %, but for 17..32 heads of 64 columns: 21.9 -> 22.2 at 1 x 700.
struct ProjArgs {
  int* flags;                         // dense products, nullable: [2][PROJ_MAX_FLAGS], used instead of counters and places
  const float* Cpart; const float* mpart; const float* lpart;
  const uint16_t* W;                  // [rows][e] bf16
  float* out; float* outpart;         // [B][e], [csw][B][proj_part_row]
  int* counters; unsigned long long* places;       // [PROJ_MAX_UNITS] each
  int* err; unsigned launch_id;       // err: word raised (= launch_id) when the result cannot be had; err[-1]: launch it speaks of
  int err_before;                     // an earlier launch of this call may have raised err: then the result is NaN
  const int32_t* seq_lens;
  int B, T, H, d_k, rows, e;
  int NG, nsplit, mode;               // mode 0: partials laid out by the stream kernel; 1: [b][nsplit]
  float mscale;                       // 1 for log2-domain maxima, log2(e) for natural-log ones
  int csw, crows;                     // row splits of W across workgroups, rows per split
  // Workgroups i and j of a launch share an XCD where i % 8 == j % 8 (checked at set-up, and by the workgroups of a unit on
  // every launch): the row splits of a head meet in its L2.  0: not known, they meet at the memory side.
  int xcd_local;
  int apart;                          // (for tests: with xcd_local, every second row split behaves as if on another XCD)
  // Dense products (launch_dense_mfma): Cpart = x [B][rows], out_m = x W_m for nmat matrices.
  // role 0: fp32 result.  The new token's rows (it sits at row / position seq_lens[b] - 1):
  // role 1: query, fp32, rotated to that position when rope is set; role 2: key row into Kc (rotated
  // when rope and rotate_k); role 3: value row into Vc.
  int nmat;
  const uint16_t* Wm[3]; float* outm[3]; int role[3];
  uint16_t* Kc; uint16_t* Vc; long c_bstride;
  int k_banded;                       // Kc is a banded cache (see FusedArgs::k_banded)
  const float* rope; int rotate_k;
  bool once;                          // nontemporal loads of W where one batch chunk reads it (read_once)
};

struct FusedArgs {
  const float* q;
  const uint16_t* K;
  long k_bstride;
  int k_banded;                       // 0: [t][d] row-major per sequence; 1: [t / 32][H][32][d_k] (32-row bands, head-major)
  const int32_t* seq_lens;
  int T, B, H, d, d_k;
  int G, NG, gpx, lph, hpu;
  float qscale;                       // log2(e) / sqrt(d_k): scores live in the log2 domain
  unsigned long long* exch;           // [NG][NP][EXCH_SLOTS][2][16*NT][4] 16-byte words {tag, max, 4 bf16 weights}
  unsigned tag_base, launch_id;
  unsigned long long wait_ticks;      // budget of every wait for another workgroup, in ticks of the 100 MHz real-time counter
  float* Cpart;                       // [nparts][H][d]
  float* mpart;                       // [nparts][H]  running max, log2 domain
  float* lpart;                       // [nparts][H]
  int* err;                           // set to launch_id when a wait timed out; err[-1] receives launch_id at the start
  int* counters;                      // arrival counters of the projection, zeroed here
  int ncounters;
  int xcd_local;                      // 1: a group's workgroups share an XCD, the exchange stays in its L2
  // Single-launch mode: once all workgroups have written their partials (arrival flags, tagged
  // with launch_id), each takes a (head, row split) share of the merge + projection.
  const float* rope;                  // nullable [T][d_k/2] {cos, sin}: rotate key rows by position for the scores
  int by_sequence;                    // > 0: by-sequence partition with this many shares per sequence
  int fuse;
  unsigned* flags;                    // [grid]
  ProjArgs proj;                      // csw * H <= grid, B <= 16
};


bool fused_geometry(int B, int H, int T, int d, FusedGeom* g);
int fused_by_sequence(const FusedGeom& g, int B, bool ragged);
size_t fused_exch_bytes(const FusedGeom& g);
bool probe_xcd_round_robin(unsigned* dev_buf, hipStream_t st);
int fused_blocks_per_cu(const FusedGeom& g, bool rope);
void launch_fused_stream(const FusedGeom& g, const FusedArgs& a, hipStream_t st);
int proj_batch_tiles(int B, int rows, int e, int H);
int proj_row_splits(int H, int rows, int e, int B);
int proj_part_row(int H, int d_k);
bool read_once(size_t weight_bytes, size_t cache_bytes);
int proj_rows_per_split(int rows, int csw);
void launch_project_mfma(ProjArgs a, hipStream_t st);
int dense_row_splits(int H, int nmat, int rows, int e, int B);
void launch_dense_mfma(ProjArgs a, hipStream_t st);

// ---- bf16 fast path of the X-cache scheme (kernels_xcache.hip) -------------------------------------
bool xcache_fast_ok(int dtype, int H, int d_model, int d_k);
int xcache_splits(int B, int H, int T, int d_model);
void launch_xq_tilde(const float* q, const void* Wk, float* qt, int B, int H, int d_k, int d_model, int e,
                     float scale, bool once, int* counters, int ncounters, hipStream_t st);
void launch_xscores(const float* qt, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H,
                    int d_model, float* S, int B, hipStream_t st);
bool xfused_ok(int d_model);                 // (kernels_xfused.hip) one pass over X instead of xscores + xweighted
bool xcache_read_once(int B, int T, int d_model, int e, bool ragged, bool one_pass);   // (read_once)
int xfused_splits(int B, int H, int T, int d_model);
int xfused_most_splits(int B, int H, int T, int d_model);    // bound of the splits at T and every shorter context
int xfused_tiles(int B, int H, int d_model, int nsplit);     // head tiles of 16 in a workgroup
bool xfused_through(size_t bytes);           // whether that many bytes of partials leave through the L2s
void launch_xfused(const float* qt, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H, int d_model,
                   int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st);
void launch_xweighted(const float* S, const void* X, long x_bstride, const int32_t* seq_lens, int T, int H,
                      int d_model, int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st);

// ---- launches whose units of workgroups share what they read (unit_of_workgroup) -----------------------
// Units dealt to the 8 XCDs (unit_of_workgroup): only when they spread evenly, within a quarter
inline int colocate_units(int nunits) { return (nunits % 8 == 0 || nunits >= 32) ? 1 : 0; }
inline unsigned unit_grid(int nunits, int ninner, int colocate) {
  return colocate ? 8u * (unsigned)ninner * (unsigned)((nunits + 7) / 8) : (unsigned)nunits * (unsigned)ninner;
}

// ---- bf16 K-caches the stream kernel does not take (kernels_wide.hip; launch_xweighted_full in kernels_xcache.hip) ----
// [B][H][T padded to 32]: with `blocks` (kscores_block_floats) softmax numerators against a reference per head and 64
// rows, else scores in the log2 domain (scale_log2 = log2(e) / sqrt(d_k)); then per split the weighted sum with fp32
// weights, partials laid out [b][nsplit], maxima in the log2 domain.
bool wide_ok(int dtype, int T, int d, int d_k);
int kweighted_tiles(int H);
int kweighted_splits(int B, int H, int T, int d);
size_t kscores_block_floats(int B, int H, int T);
void launch_kscores(const float* q, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int d_k,
                    float scale_log2, const float* rope, float* S, float* blocks, int* counters, int ncounters, int B, hipStream_t st);
void launch_kweighted(const float* P, const float* blocks, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d,
                      int nsplit, float* Cpart, float* mpart, float* lpart, int B, hipStream_t st);
// the same from scores, the numerators taken by every workgroup for itself
void launch_xweighted_full(const float* S, const void* K, long k_bstride, const int32_t* seq_lens, int T, int H, int d, int nsplit,
                           float* Cpart, float* mpart, float* lpart, int B, hipStream_t st);

}  // namespace slim
