// Internal kernel argument blocks and launchers (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace trevs {

// ---------------------------------------------------------------- stage 1
struct PrepArgs {
  const void* cls;           // [B,H,N]
  int B, H, N, n_seg, seg_len;
  float2* row_stats;         // [B*H*n_seg]: (row max * log2 e, 1 / sum of exp)
  const void* text;          // [B,M_max,d]
  const int32_t* text_len;   // [B] or null
  int M_max, row_bytes;      // row_bytes = d * elem
  float* inv_tnorm;          // [B*M_max]: 1/max(||t_j||, 1e-12), 0 for j >= M_b
  int n_cls_blocks;          // blocks [0, n_cls_blocks) do [CLS] rows, the rest text rows
  int cls_vec16;             // every [CLS] segment row starts 16-byte aligned
};

struct RelArgs {
  const void* cls;
  const float2* row_stats;
  int H, n_seg, seg_len;
  const void* Z;             // [B,N,d]
  const void* T;             // [B,M_max,d]
  const int32_t* text_len;
  const float* inv_tnorm;
  int cls_vec16;             // every [CLS] segment row starts 16-byte aligned
  bool fused_stats;          // no prep: the launch forms row statistics and text norms itself
  int B, N, M_max, row_bytes, tiles_per_sample;
  float* sal;                // [B,N]
  float* rel;                // [B,N]
  // feature-dimension split (n_split > 1): workgroup (tile, split) covers
  // the 128-byte slabs [split*split_slabs, ...) and writes its partial dot
  // products t_j.z_i to part [B,n_split,M_max,N], its partial ||z_i||^2 to zpart
  // [B,n_split,N] and (first tile) ||t_j||^2 to tpart [B,n_split,M_max]; a merge
  // pass finishes Eq. (4)-(5)
  int n_split, split_slabs;
  float* part;
  float* zpart;
  float* tpart;
  float* inv_norm;           // [B,N] 1 / max(||z_i||, 1e-12), or null
};

// Launch shape of the relevance pass for one problem size.
struct RelPlan {
  bool tail;             // rows end inside a 128-byte slab
  int MT;                // text rows per tile (32, 64 or 128)
  int tile_tokens;       // visual tokens per workgroup
  int tiles_per_sample;
  int n_split, split_slabs;
  bool fused_stats;
  size_t part_floats() const;  // floats of part + zpart + tpart (0 without a split)
  int B, N, M_max;
};

struct NormArgs {
  const float* sal;
  const float* rel;
  int N;
  float* stats;              // [B,4]: Med(s^v), MAD(s^v), Med(s^t), MAD(s^t)
};

struct SelArgs {
  const float* sal;
  const float* rel;
  const float* stats;        // [B,4] from the robust-statistics kernel
  int N, K;
  int K_t;                   // budget-split mode: tokens taken by s^t first
  float wv, wt, tau_v, tau_t, lam, eps;
  float* score_out;          // [B,N] or null
  float* norm_stats;         // [B,4] or null
  int32_t* kept_idx;         // [B,K]
  // with a diversity set: the control words of its picks, zeroed here, and for
  // pool rounds the N - K other tokens, ascending (each null without)
  int32_t* pick_ctrl;
  int32_t* rest;
  uint32_t* rest_mx;         // [B,N - K], zeroed
};

// ---------------------------------------------------------------- stage 2
// The statistics and head passes of the two questions of the text sensitivity
// run in one launch (QuestionPair, the last grid dimension), and so does the
// profile pass.  Three launches less, and twice the workgroups of grids that
// fill the GPU once: 4 x 4096 visual tokens 147.4 -> 130.9 us a call (with the
// rank correlation), 12 x 72 57.2 -> 36.6.  Stage 2 has one question and takes
// its arguments as they are (with a choice between two: 4 x 4096 tokens 70.8 -> 71.1
// us a call).
struct StatsArgs {
  const void* q;             // [B,S,H_q,dh]
  const void* k;             // [B,S,H_kv,dh]
  int B, S, P, K_in, T_max, H_q, H_kv, G;
  float scale_log2e;         // scale * log2 e
  int n_split, split_len;    // visual columns per split (multiple of 32)
  int n_rgroups;             // workgroups along the (head-in-group, text row) axis
  float4* part;              // [B,H_q,T_max,n_split]: (max, sum e, sum e^2, -) in log2 units
  // Causal softmax domain: split s also reduces the non-visual causal keys
  // [s*rest_len, (s+1)*rest_len) of each text row (key j < P is prefix row j,
  // j >= P text row j - P, valid for text row q while j - P <= q).
  int rest_len;              // multiple of 32; 0 for the visual-only domain
  float4* part_rest;         // [B,H_q,T_max,n_split]: as part, over the non-visual keys
};

struct HeadArgs {
  const float4* part;
  int B, H_q, T_max, T_pad, K_in, n_split;
  const int32_t* text_len;
  const float* lse_rest;     // [B,H_q,T_max] natural log, or null
  const float4* part_rest;   // [B,H_q,T_max,n_split] non-visual causal statistics, or null
  float* lse2;               // [B,H_q,T_pad] row log-sum-exp in log2 units (T_pad = T_max rounded up to 32)
  float* head_var;           // [B,H_q] u_h
};

template <class A>
struct QuestionPair {
  A of[2];
};
template <class A>
__device__ __forceinline__ const A& question(const A& a, int) {
  return a;
}
template <class A>
__device__ __forceinline__ const A& question(const QuestionPair<A>& a, int c) {
  return a.of[c];
}

struct ScoreArgs {
  const void* q;
  const void* k;
  int B, S, P, K_in, T_max, T_pad, H_q, H_kv, G, n_keep;
  int n_vtiles;              // workgroups per sample (score_tile_tokens visual tokens each)
  float scale_log2e;
  const float* lse2;
  const float* head_var;     // [B,H_q] u_h
  int32_t* head_sel;         // [B,n_keep] H* ascending, or null
  const int32_t* text_len;
  float* p;                  // [B,K_in]
  // head split (n_hsplit > 1): workgroup (tile, split) sums the attention of
  // the selected heads [split*hps, (split+1)*hps) and writes it per (text
  // row, token) to hpart [B,n_hsplit,T_max,K_in]; a merge pass adds the
  // splits and takes the max over text rows
  int n_hsplit, hps;
  float* hpart;
};

// ---------------------------------------------------------------- diversity set
// Control words of one sample's picks, zeroed by the pivot selection.
// kCtrlPicks: tokens picked so far; kCtrlRound: picks before the last round;
// kCtrlBound: the largest distance (float bits) outside the round's pool, as
// the pool was selected (see norm_gap).
constexpr int kPickCtrl = 4;
enum { kCtrlPicks = 0, kCtrlRound = 1, kCtrlBound = 2 };

struct GramArgs {
  const void* Z;             // [B,N,d]
  int B, N, row_bytes;
  int n_tiles;               // tiles a side (set by the launchers, as n_rtiles and n_ctiles)
  float* G;                  // [B,n,ldg] fp32 dot products z_j . z_i of n tokens
  int ldg;                   // row stride of G, a multiple of 4
  // samples whose picks (ctrl, if not null) have reached K_d are skipped
  const int32_t* ctrl;
  int K_d;
  // products over lists of tokens
  const int32_t* rows;       // [B,n_rows]
  const int32_t* cols;       // [B,n_cols]
  int n_rows, n_cols;
  int n_rtiles, n_ctiles;
  bool natural;              // k order of the 256-row tiles (set by the launchers)
  float* inv_norm;           // [B,N] 1 / max(||z_i||, 1e-12); set from G by launch_gram_full
  const float* near_pick;    // [B,N] -inf: picked (launch_gram_next)
  uint32_t* mx;              // [B,n_cols] maxima, as keys (f2key), over 0 or what is there
  // pool: bit i of row j of mask [B,n_rows,mask_words] is set where token j may
  // bring token i nearer: its cosine to i is above that of the nearest selected
  // token, nearest [B,n_rows], less the share `margin` of it (see norm_gap)
  uint32_t* mask;
  int mask_words;
  const float* nearest;
  float margin;
};
// The first round knows most tokens' norms from the relevance pass only.  Such
// an inverse norm is within this share of
// the one from the Gram diagonal, which the picks use.  A sum of positive terms that pass n
// fp32 roundings each is within n 2^-24 of the exact one: at most d + 1 on the
// diagonal (a multiply of n products rounds at most n times, an fp32 product once
// more), d / 8 + 56 in the relevance pass (chunks of 16 bytes, one half-row a lane,
// 32 groups of splits).  The inverse norm has half of both, and four
// roundings of its own each; the rest is room for the few that cosines add.
// (Rows of equal magnitudes come to a tenth of this: their rounding errors
// have one sign.)
// Distances 1 - x, 1 - x' with x' within the share e of x: a token outside
// the pool, at most `bound` far by the relevance pass's norms, is at most
// bound + e |1 - bound| far by the Gram matrix's.  And pick j brings token i
// nearer only if their cosine c, off by 2 e |c|, is above i's, off by e |x|: if
// c > x - 3 e |x| / (1 - 2 e) by the relevance pass's norms.  Later rounds have
// every norm from the diagonal: only the order of a cosine's factors differs.
inline float norm_gap(int d) { return (0.6f * d + 64.f) * 5.9604645e-8f; }
constexpr int kNormGapMaxD = 1 << 18;  // a gap of 0.01
constexpr float kMaskMargin = 3.1f;    // 3 / (1 - 2 e)
constexpr float kCosRounding = 4 * 5.9604645e-8f;
bool gram256_ok(int dtype, int N, int row_bytes);  // 256-row tiles can be used
// G of all N tokens.
hipError_t launch_gram_full(const GramArgs& g, int dtype, hipStream_t s);
// G of the tokens that are no pivots (cols), and their inv_norm, in the samples
// that are not finished.
hipError_t launch_gram_rest(const GramArgs& g, int dtype, hipStream_t s);
// G of the listed tokens (rows).
hipError_t launch_gram_pool(const GramArgs& g, int dtype, hipStream_t s);
// Maxima, by tiles of 128 x 128, or, where gram256_ok, 256 x 256 or 256 x 192.
hipError_t launch_gram_max(const GramArgs& g, int rtile, int ctile, int dtype, hipStream_t s);
// Maxima over the last round's picks (of a.rows), as minus the least distance;
// inv_norm of the other columns, as launch_gram_full would set it.
hipError_t launch_gram_next(const GramArgs& g, int dtype, hipStream_t s);
// inv_norm of the listed bf16 tokens (rows), as launch_gram_full would set it.
hipError_t launch_gram_norms(const GramArgs& g, hipStream_t s);

// How the K_d picks are made (see pick_plan).
struct PickPlan {
  int rounds;                // pool rounds (0: none, and the Gram matrix of all tokens)
  int C, ldc;                // pool size, row stride of its Gram matrix
  int mask_words;            // 32-bit words of a row of its mask, a multiple of 4
  int row_tile, col_tile;    // tile of the first round's distances (later: 128 x 128)
  int n_gram, ldg;           // tokens of the Gram matrix without or after the rounds, its row stride
  int n_psplit;              // pivot splits of the initial distances over the full Gram matrix
  size_t gram_floats() const;  // floats of a sample's Gram matrix, of n_gram tokens or of the pool
};
constexpr int kRoundTile = 128;  // row tile of the products over pools and picks
PickPlan pick_plan(int B, int N, int K_r, int K_d, int dtype, int row_bytes);
struct PickArgs {
  PickPlan p;
  int B, N, K_r, K_d, R;     // R = N - K_r
  float gap;                 // norm_gap of the rows
  const int32_t* pivots;     // [B,K_r] ascending
  const int32_t* rest;       // [B,R] ascending, the other tokens (pool rounds)
  float* inv_norm;           // [B,N]
  float* G;                  // [B,n_gram,ldg], or [B,C,ldc]
  float* part;               // [n_psplit,B,N]: per split, max over its pivots j of G_ij / ||z_j||
  int32_t* ctrl;             // [B,kPickCtrl]
  // pool rounds
  uint32_t* mx;              // [B,R] keys, zeroed by the pivot selection
  float* near_piv;           // [B,N] max over the pivots j of G_ij / ||z_j||
  float* near_pick;          // [B,N] least distance to a pick of an earlier round, -inf once picked
  int32_t* cand;             // [B,C] pool tokens, ascending
  float* cand_piv;           // [B,C] their near_piv,
  float* cand_pick;          // [B,C] near_pick
  float* cand_cos;           // [B,C] and cosine to the nearest
  uint32_t* mask;            // [B,C,mask_words]
  int32_t* picks;            // [B,K_d]
  int32_t* kept_idx;         // [B,K_r+K_d] ascending
  int32_t* div_idx;          // [B,K_d] picks in pick order, or null
};
// The K_d picks and the kept list.
hipError_t launch_picks(const PickArgs& a, const void* Z, int row_bytes, int dtype, hipStream_t s);

// ---------------------------------------------------------------- analysis
struct ProfileArgs {
  const void* q[2];
  const void* k[2];
  int B, S, P, K_in, T_max, T_pad, H_q, H_kv, G;
  int n_split, split_len;    // visual columns per workgroup (multiple of 32, <= kProfileSplitMax)
  float scale_log2e;
  const float* lse2[2];         // [B,H_q,T_pad] row log-sum-exp in log2 units
  const int32_t* text_len[2];
  float* profile[2];            // [B,H_q,K_in] mean attention over the valid text rows
};
constexpr int kProfileSplitMax = 2048;
struct SensitivityArgs {
  const float* profile[2];   // [B,H_q,K_in] per question
  int H_q, K_in;
  float* ts;                 // [B,H_q]
};
struct SpearmanArgs {
  const float* sv;           // [B,N]
  const float* st;           // [B,N]
  const int32_t* idx;        // [B,K] the top-K saliency set
  int N, K, n_tiles;         // n_tiles = ceil(K / kRankTile)
  long long* part;           // [B,n_tiles,4] partial sums of the centred rank products
  double* rho;               // [B]
};
constexpr int kRankTile = 64;  // tokens ranked per workgroup (one per lane)
// Visual profiles of every head for one question, the sensitivity of each
// head between two questions, and the rank correlation within a top-K set.
hipError_t launch_profile(const ProfileArgs& a, int dtype, int dh, hipStream_t s);
hipError_t launch_sensitivity(const SensitivityArgs& a, int B, hipStream_t s);
// The top-K set (to idx, which a.idx also names) and its rank correlation.
hipError_t launch_topk_spearman(const SpearmanArgs& a, int B, int32_t* idx, hipStream_t s);

// ---------------------------------------------------------------- gather
constexpr int kGatherMaxTensors = 4;
struct GatherTensor {
  const uint8_t* src;
  uint8_t* dst;
  long long src_bstride, dst_bstride;  // bytes per sample
  int row_bytes;                       // multiple of 16
};
struct GatherArgs {
  GatherTensor t[kGatherMaxTensors];
  int n_tensors;
  const int32_t* idx;        // [B,n_kept] kept rows relative to the selected block
  int B, rows_out, P, K_in, n_kept;
  const int64_t* pos;        // [n_pos,B,S] or null
  int64_t* pos_out;          // [n_pos,B,rows_out]
  int n_pos, S;
};
constexpr int kGatherRowsPerBlock = 4;  // one row per wave
constexpr int kGatherThreads = 256;
constexpr int kGatherBatch = 8;  // 16-byte loads in flight per lane
constexpr int kGatherShortRows = 8;  // rows of at most 1 KB per wave

// Elements per thread of a 1024-thread selection workgroup over N values
// (a power of two, the template argument of the selection kernels).
inline int select_e(int N) {
  int e = 1;
  while (e * 1024 < N) e <<= 1;
  return e;
}

hipError_t launch_prep(const PrepArgs& a, int dtype, hipStream_t s);
RelPlan relevance_plan(int B, int N, int M_max, int row_bytes, int H, int n_seg);
hipError_t launch_relevance(const RelArgs& a, const RelPlan& p, int dtype, hipStream_t s);
hipError_t launch_norm_stats(const NormArgs& a, int B, hipStream_t s);
hipError_t launch_prellm_select(const SelArgs& a, int B, hipStream_t s);
// Budget-split selection: the K_t highest s^t, then the K - K_t highest s^v
// among the other tokens.
hipError_t launch_budget_select(const SelArgs& a, int B, hipStream_t s);
// Stable top-K per row; nonneg: every score is >= 0 (lets the selection skip
// its min/max reduction).
hipError_t launch_topk(const float* scores, int B, int N, int K, int32_t* out, hipStream_t s,
                       bool nonneg = false);
// (n questions of the same sizes, one or two)
hipError_t launch_stats(const StatsArgs* a, int n, int dtype, int dh, hipStream_t s);
hipError_t launch_heads(const HeadArgs* a, int n, hipStream_t s);
// u_h and the row log-sum-exps from the caller's per-row statistics
// [B,H_q,T_max,3] = (log-sum-exp, sum A, sum A^2) instead of the
// statistics pass.
hipError_t launch_heads_given(const float* row_stats, const HeadArgs& a, hipStream_t s);
hipError_t launch_score(const ScoreArgs& a, int dtype, int dh, hipStream_t s);
hipError_t launch_gather(const GatherArgs& a, hipStream_t s);

// Waves per workgroup of the statistics pass (column blocks of 32 rows).
int stats_waves(int G, int T_max);
// Visual tokens per workgroup of the token-score pass.
int score_tile_tokens(int dtype, int dh);
// Head splits of the token-score pass (1: none).
int score_head_splits(int B, int n_vtiles, int n_keep);

}  // namespace trevs
