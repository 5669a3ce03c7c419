// Scoring phases of the compression pass (Section 3.2: cross-modal attention entropy; Section 3.3:
// cumulative attention score).  The softmax normalisers of a window row are needed before any of its
// probabilities can be added to a column sum or to the head-averaged cross-modal matrix, so the keys
// are visited twice:
//   pass A  score_stats_kernel   row maxima and normalisers (all keys / vision keys / text keys),
//                                split over column chunks; also 1/|k| of every key (used by the merge)
//           score_stats_dma_kernel     the same for grouped heads and the row-block mode, fed by asynchronous copies
//           stats_combine_kernel merges the chunk partials of every row
//   pass B  score_accum_kernel   recomputes the logits, adds normalised probabilities into the column
//                                scores A_s and into the head-averaged cross-modal matrix, whose row
//                                entropies are reduced per tile
//           score_accum_dma_kernel     the same for grouped heads, fed by asynchronous copies
//           score_accum_blocks_kernel  the row-block mode (more than 128 scoring rows)
//   both    score_stats_direct_kernel, score_accum_direct_kernel  windows over few keys (score_direct.hip)
// Logits are kept in the base-2 domain: t = (q.k) * scale * log2(e), probabilities are exp2(t - max).
// This header holds what the passes share: the argument block and its filling from the plan.  Pass A and each form
// of pass B are translation units of their own (score_stats.hip, score_stats_dma.hip, score_accum.hip,
// score_accum_dma.hip, score_accum_blocks.hip, score_direct.hip): they sit at the edge of their register budgets and the compiler's allocation for one
// kernel shifted when another lived in the same module.
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "plan.hpp"

namespace meda {

// f(0), f(1), .. f(N-1) with the index as a compile-time constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

struct ScoreArgs {
  const char* q;
  const char* k;
  const uint8_t* mask;  // [N][Tk]: layer l belongs to sequence l / Lseq
  float4* stats_part;  // [L][Hq][stats_rows][NPART] (max, Z_vision, Z_text, -)
  float4* stats;       // [L][Hq][4][stats_rows] floats: planes of (max, 1/Z_all, coef for vision columns, coef for text
                       // columns), or of the form the row-block mode uses (stats_combine_kernel)
  float* inv_norm;     // [L][Hkv][T]
  float* col_scores;   // [L][Hkv][T]
  double* ent_part;    // [L][NT][2]
  int L, Hq, Hkv, G, T, W, RB, Wp;   // T keys and W query rows of this launch (the last W positions below T)
  int Lseq;        // layers per sequence
  int NCG, CS, CH, NPART, NT;
  int Tk;          // key rows per (layer, kv head) in memory (>= T)
  int q_rows;      // rows per (layer, head) in the query buffer
  int q_row0;      // first query row of this launch in the buffer
  int NTk;         // tiles per layer in ent_part
  int accumulate;  // add to col_scores / ent_part instead of storing
  // Row-block mode (blocks; q_rows scoring rows, the last positions of the sequence): the rows are cut
  // into blocks of row_block rows counted from the end; block bi holds the positions [Tb - Wb, Tb) with
  // Tb = Tk - bi * row_block, Wb = min(row_block, q_rows - bi * row_block), and sees only the keys below Tb, so it is
  // the window computation of the sequence cut at Tb.  The kernels derive T, W and q_row0 of their block themselves
  // (one launch covers all blocks).
  int blocks, row_block;
  int stats_rows;  // rows per (layer, head) in stats / stats_part (the padded window, or all q_rows rows)
  int stats_row0;  // first row of this launch's (or block's) rows in them
  float c;             // scale * log2(e)
};

// The arguments of row block bi (see ScoreArgs::blocks).
__device__ __forceinline__ void select_row_block(ScoreArgs& a, int bi) {
  a.T = a.Tk - bi * a.row_block;
  a.W = min(a.row_block, a.q_rows - bi * a.row_block);  // the first rows may leave the last block short
  a.q_row0 = a.q_rows - bi * a.row_block - a.W;
  a.stats_row0 = a.q_row0;
  a.accumulate = bi > 0;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// 1/|k| of the row whose fragment the two lane groups hold.
template <typename T, int D>
__device__ __forceinline__ float inverse_norm(const Frag<T, D>& f) {
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < Tile<T, D>::kFragChunks; ++i) ss += chunk_sumsq<T>(f.c[i]);
  ss += __shfl_xor(ss, 32, kWave);
  return 1.0f / fmaxf(sqrtf(ss), 1e-30f);
}

// Pass A with a lane per query row: adds the raw products of the row with 16 of a block's 32 keys (acc, register r is
// the key acc_row(r, kg)) to the row's running maximum m and normalisers zv (vision keys), zt (text keys).  mword: the
// modality bits of the block's keys.  Every key counts: the maximum is taken on the raw products (the scale is positive,
// so it commutes with the maximum) and the scale is folded into the exponent's multiply-add.
__device__ __forceinline__ void stats_add_plain(const f32x16_t& acc, float c, uint32_t mword, int kg, float& m, float& zv, float& zt) {
  float bm = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
#pragma unroll
  for (int r = 3; r < 15; r += 2) bm = fmaxf(fmaxf(bm, acc[r]), acc[r + 1]);
  bm = fmaxf(bm, acc[15]);
  const float mn = fmaxf(m, bm * c);
  const float sc = fast_exp2(m - mn);
  zv *= sc;
  zt *= sc;
  m = mn;
  float e[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) e[r] = fast_exp2(fmaf(acc[r], c, -mn));
  if (mword == 0u || mword == 0xffffffffu) {
    float t = e[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) t += e[r];
    zv += mword ? t : 0.f;
    zt += mword ? 0.f : t;
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool vis = (mword >> acc_row(r, kg)) & 1u;
      zv += vis ? e[r] : 0.f;
      zt += vis ? 0.f : e[r];
    }
  }
}

// The same where the row sees only the keys 0 .. last_seen of the block.
__device__ __forceinline__ void stats_add_masked(const f32x16_t& acc, float c, uint32_t mword, int kg, int last_seen, float& m,
                                                 float& zv, float& zt) {
  float t[16], bm = kNegBig;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    t[r] = acc_row(r, kg) <= last_seen ? acc[r] * c : kNegBig;
    bm = fmaxf(bm, t[r]);
  }
  const float mn = fmaxf(m, bm);
  const float sc = fast_exp2(m - mn);
  zv *= sc;
  zt *= sc;
  m = mn;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    // the exponent in the form pass B uses (one rounding, as in the plain path above): the probability of a row's largest
    // logit is then the same number in both passes, and a nearly one-hot row keeps its normaliser consistent with its
    // probabilities
    const float e = (t[r] > 0.5f * kNegBig) ? fast_exp2(fmaf(acc[r], c, -mn)) : 0.f;
    const bool vis = (mword >> acc_row(r, kg)) & 1u;
    zv += vis ? e : 0.f;
    zt += vis ? 0.f : e;
  }
}

// The two lane groups hold disjoint keys of the same row: its partial (max, Z_vision, Z_text, -) over both.
__device__ __forceinline__ float4 stats_merge_halves(float m, float zv, float zt) {
  const float mo = __shfl_xor(m, 32, kWave);
  const float zvo = __shfl_xor(zv, 32, kWave);
  const float zto = __shfl_xor(zt, 32, kWave);
  const float M = fmaxf(m, mo);
  const float f1 = fast_exp2(m - M), f2 = fast_exp2(mo - M);
  return make_float4(M, zv * f1 + zvo * f2, zt * f1 + zto * f2, 0.f);
}

inline ScoreArgs make_args(const Plan& p, const Buffers& b, bool pass_a = false) {
  ScoreArgs a;
  a.q = static_cast<const char*>(b.q);
  a.k = static_cast<const char*>(b.k);
  a.mask = b.mask;
  a.stats_part = reinterpret_cast<float4*>(b.ws + p.off_stats_part);
  a.stats = reinterpret_cast<float4*>(b.ws + p.off_stats);
  a.inv_norm = reinterpret_cast<float*>(b.ws + p.off_inv_norm);
  a.col_scores = reinterpret_cast<float*>(b.ws + p.off_col_scores);
  a.ent_part = reinterpret_cast<double*>(b.ws + p.off_ent_part);
  a.L = p.L; a.Hq = p.Hq; a.Hkv = p.Hkv; a.G = p.G; a.T = p.Tb; a.W = p.Wb; a.RB = p.RB; a.Wp = p.Wp;
  a.Lseq = p.Lseq; a.Tk = p.Tk; a.q_rows = p.R; a.q_row0 = p.q_row0; a.NTk = p.NTk; a.accumulate = p.accumulate;
  a.NCG = p.NCG; a.CS = p.CS; a.CH = p.CH; a.NPART = p.NPART; a.NT = p.NT;
  a.blocks = p.blocks; a.row_block = kScoreRowBlock;
  a.stats_rows = p.blocks ? p.R : p.Wp; a.stats_row0 = 0;
  if (pass_a) {  // pass A has its own row blocks when every prompt row scores
    a.RB = p.RBa;
    if (p.blocks) a.row_block = p.row_block_a;
  }
  a.c = p.scale_log2;
  return a;
}

// Both passes for windows over few keys (score_direct.hip); the statistics are merged by pass B itself.
hipError_t launch_score_stats_direct(const Plan& p, const Buffers& b, hipStream_t s);
hipError_t launch_score_accum_direct(const Plan& p, const Buffers& b, hipStream_t s);

// Pass A for grouped heads and the row-block mode, fed by asynchronous copies (score_stats_dma.hip).
bool score_stats_dma_supported(const Plan& p);
hipError_t launch_score_stats_dma(const Plan& p, const Buffers& b, hipStream_t s);

// Pass B when every prompt row scores, for shapes whose items fit a two-stage LDS ring (score_accum_blocks.hip);
// the other shapes take the row-block mode of score_accum_kernel.
bool score_accum_blocks_supported(const Plan& p);
hipError_t launch_score_accum_blocks(const Plan& p, const Buffers& b, hipStream_t s);

// Pass B of the window mode for grouped heads, fed by asynchronous copies (score_accum_dma.hip).
bool score_accum_dma_supported(const Plan& p);
hipError_t launch_score_accum_dma(const Plan& p, const Buffers& b, hipStream_t s);

}  // namespace meda
