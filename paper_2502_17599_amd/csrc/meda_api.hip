// C ABI of libmeda: parameter validation, workspace layout, the launch sequence of the compression
// pass, optional per-phase event timing.
#include <math.h>

#include <mutex>
#include <vector>

#include "plan.hpp"

namespace meda {

// Which windows go to the direct scoring kernels: those with few column tiles of 128 keys over all layers.  Both passes
// and the merge of the statistics, in us (kernels over LDS tiles / direct), 60 to 120 shapes at each number of tiles:
//   6 tiles   geometric mean of the ratio 1.87 (2 layers of 300, 8 heads per kv head, fp32: 139 / 45)
//   16        1.68 (2 layers of 1024 keys, 28 heads, bf16: 49 / 42), 32  1.67, 64  1.51 (0.95 at worst)
//   128       1.10: 0.73 to 1.04 for few heads and grouped bf16 rows of 256 bytes, 1.03 to 1.6 for the others
//   256       0.79 (a tile of 128 keys shares what a workgroup of 32 keys reads again), 512  0.69
// Up to four sequences, and no more than 128 tiles in all, go the way one of them would go alone, so that its sums are the
// same; 7 of 4 layers of 487 keys, 4 heads, 2 kv heads, 80 rows (112 tiles; whole pass) 77 / 91.
constexpr int64_t kDirectTiles = 64, kDirectTilesAll = 128;
constexpr int kDirectManyHeads = 28;

// (Head, 32-row block) pairs in all, every prompt row scoring, above which a pass-A workgroup takes more than four of them
// (bf16 rows of 256 bytes).  Pass A in us, workgroups of 4 / 8 / 12 / 16 pairs:
//   bf16, 256 bytes   1600 pairs (8 layers of 780, 8 heads)  28 / 34 / 43 / 59    9600 (24 of 1600, 8)   137 / 139 / 174 / 219
//                     16128 (8 of 2000, 32)  244 / 245 / 250 / 290                19200 (24 of 1600, 16 in 4) 225 / 205 / 211 / 215
//                     56000 (28 of 4000, 16 in 8) 1408 / 1347 / 1217 / 1366       131072 (32 of 4096, 32)  3370 / 3039 / 2858 / 2893
//                     110544 (28 of 4500, 28 in 4: 12 and 8 hold one row block)   2838 / 2814 / 2823 / 2632
//   bf16, 128 bytes   4800 (24 of 780, 8)  42 / 54 / 51 / 71    110544 (28 of 4500, 28 in 4)  1811 / 1824 / 1831 / 1996
//   fp32, 512 bytes   16128 (8 of 2000, 32)  1389 / 2385 / 2819 / 3021
// With a multiple of 8 kv heads 12 pairs are between 0.8 and 1.35 of the time of 16 (250 layers of 2000 and 1458, 8 heads: 1926 /
// 2545, 1435 / 1059), so those keep 16; the others, (layer, kv head) pairs dealt to the XCDs: 250 layers, 8 heads in 2, of 600,
// 1458, 2000, 3000: 12 pairs 214, 966, 1507, 3223, 16 pairs 216, 1000, 1674, 3243; in the order of the grid 12 pairs 213, 1428,
// 1477, 4076, 16 pairs 220, 1030, 2394, 3632.
constexpr int64_t kLargePairs = 12000;
// The same for observation windows of more than 128 rows, whose row blocks all walk nearly the whole prompt: up to which
// number of pairs a workgroup takes four, and eight, of them.  Pass A in us, workgroups of 4 / 8 / 16 pairs, 20000 keys:
//   bf16, 256 bytes   2048 pairs (64 pairs of kv heads, 1000 rows)   505 / 559 / 957    2240 (28 layers, 16 heads in 4, 129)  736 / 747 / 960
//                     3584 (28, 16 in 4, 256) 881 / 797 / 958         4096 (8, 32 in 8, 512)    907 / 833 / 953
//                     7168 (28, 16 in 4, 512) 1590 / 1485 / 1386      8192 (8, 32 in 8, 1000)   1684 / 1519 / 1449
//   bf16, 128 bytes   4096 659 / 645 / 783, 7168 1021 / 1097 / 1127, 8192 1132 / 1113 / 1136
constexpr int64_t kLongWindowPairs[2] = {2300, 6500};

// ---- similarity kernels

// bf16 problems for the direct kernel: short prompts whose tiled launch would leave most CUs empty: 16 pairs of 500
// positions 16 (packing 8) -> 6 us, of 1000 21 -> 13 us, of 2000 (128 workgroups) 27 -> 29 us; 2 pairs of 8000 53 -> 120 us
// (its key loads are not shared by the waves, so long sets stay with the tiled kernel).
constexpr int kSimDirectPositions = 2048;

// Where the resident-set kernel takes the layers that fit: a workgroup of it occupies a whole CU, so with one or two per CU
// its last round leaves most of the chip empty, and with long sets its few layers do not cover their own launch.  Tiled
// alone / both kernels, similarity in us, mean budget of a layer in brackets, prompts of 1000 to 3000:
//   256 bytes  256 pairs [375] 60 / 76, [750] 159 / 185, [1125] 297 / 334    384 [240] 148 / 139, [375] 91 / 101, [1125] 439 / 475
//              512 [240] 190 / 163, [675] 468 / 436, [1125] 576 / 622        1024 [240] 364 / 304, [750] 603 / 566, [1125] 1024 / 1025
//   128 bytes  256 [375] 37 / 44, [750] 93 / 125, 360 [701] 133 / 163        384 [240] 80 / 78, [750] 135 / 140, [1125] 241 / 270
//              512 [450] 146 / 142, [750] 180 / 174, [1125] 334 / 366        1024 [240] 209 / 198, [675] 481 / 475, [1125] 566 / 586
// Below 512 pairs it takes prompts long enough against the sets that its workgroups walk the rows for long:
//   256 bytes  448 of 3000 [120] 121 / 107, [330] 176 / 166, [600] 224 / 223, of 8000 [240] 356 / 303, [600] 585 / 567
//              384 of 3000 [120] 108 / 98, [240] 130 / 130, of 8000 [330] 359 / 333, [600] 505 / 521
//              256 of 3000 [60] 69 / 65, [120] 76 / 77, of 8000 [240] 219 / 211, [330] 243 / 250
//   128 bytes  448 of 3000 [330] 104 / 99, of 8000 [240] 206 / 199, [600] 342 / 347   384 of 8000 [120] 143 / 133, [330] 210 / 219
//              256 of 8000 [60] 89 / 85, [120] 100 / 104
constexpr long long kResidentKept = 900;
static bool resident_pays(const Plan& p, int64_t pairs) {
  if (pairs >= 512) return p.B <= kResidentKept * p.L;
  const int64_t times = pairs >= 448 ? 9 : p.d == 128 ? (pairs >= 384 ? 16 : 32) : (pairs >= 384 ? 32 : 100);
  return pairs >= kResidentPairs && p.B * times <= (int64_t)p.T * p.L;  // mean budget against positions
}

// fp32 problems for the split kernel, the others go to the direct one: from a number of positions over all (layer, head)
// pairs on that grows with the share kept, and where the direct kernel's waves, which share no loads, would walk too long
// a share of the set.  Below it the waves that take their blocks again, and the search for copies in the selection (2 to
// 8 us), cost more than the matrix instructions save.  Selection and similarity in us, direct kernel / split kernel, a
// tenth and three tenths kept:
//   rows of 256 bytes  32 pairs of 1200  31 / 34, 40 / 45   of 2000   46 / 42, 64 / 63   of 3000  72 / 57, 106 / 86
//                      128 of 300        25 / 25, 26 / 29   of 700    37 / 32, 45 / 43   of 1200  65 / 43, 81 / 63
//                      8 of 3000         46 / 39, 58 / 65   of 5000   71 / 54, 116 / 94
//                      1 of 5000         65 / 45, 43 / 71   of 16000  153 / 91, 355 / 177
//   rows of 512 bytes  32 pairs of 700   33 / 39, 39 / 55   of 1200   55 / 50, 67 / 74   of 2000  118 / 71, 123 / 108
//                      64 of 300         28 / 30, 30 / 38   of 700    49 / 43, 57 / 56   of 1200  73 / 58, 113 / 79
//                      8 of 2000         44 / 46, 59 / 73   of 5000   136 / 110, 201 / 158
static SimRoute similarity_route(const Plan& p) {
  const int64_t pairs = (int64_t)p.L * p.Hkv;
  if (p.dtype == MEDA_BF16) {
    if (pairs * ((p.T + kSimRows - 1) / kSimRows) <= kSimDirectGroups && p.T <= kSimDirectPositions) return kSimDirect;
    return resident_pays(p, pairs) ? kSimResident : kSimTiled;
  }
  const double positions = (double)pairs * p.T, kept = (double)p.B / ((double)p.L * p.T);
  const bool small = p.d == 64;
  const double from = small ? (kept < 0.2 ? 46000 : 64000) : (kept < 0.2 ? 24000 : 50000);
  const double longest = (pairs == 1 ? 4.1e4 : small ? 1.64e5 : 6.15e4) * kept;
  const bool split = positions >= from || (pairs <= 8 && positions >= 36000) || p.T > longest || p.T > 16384 ||
                     positions > (small ? 1.5e6 : 5e5) * kept;
  return split ? kSimSplit : kSimDirect;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Tiling of the two scoring passes for w query rows (the last w positions) of a sequence of t keys.  With
// `single_chunk` a pass-A workgroup walks all keys its rows see (the row-block mode, whose row blocks give that launch its
// workgroups).
static bool score_geometry(Plan* pl, int t, int w, int rows, bool single_chunk) {
  pl->Tb = t;
  pl->Wb = w;
  pl->RB = (w + 31) / 32;
  pl->Wp = pl->RB * 32;
  // Row blocks of one pass-A workgroup.  When every prompt row scores (single_chunk), pass A cuts the rows into its own
  // blocks: a workgroup of few (head, 32-row block) pairs walks the keys in a short chain and there are many of them, one
  // of many pairs re-reads the keys less often, which counts for long rows once the chip is full.
  pl->RBa = pl->RB;
  if (single_chunk) {
    const int have = (rows + 31) / 32;
    const int64_t all = pl->dtype == MEDA_BF16 && pl->d == 128 ? (int64_t)pl->L * pl->Hq * have : 0;
    int pairs = all <= kLargePairs ? 4 : (pl->Hkv % 8 == 0 || pl->G >= 7) ? 16 : 12;
    if (rows < t) pairs = all <= kLongWindowPairs[0] ? 4 : all <= kLongWindowPairs[1] ? 8 : 16;
    const int want = pl->G >= pairs ? 1 : pairs / pl->G;
    pl->RBa = want < have ? want : have;
  }
  pl->row_block_a = pl->RBa * 32;
  pl->n_blocks_a = single_chunk ? (rows + pl->row_block_a - 1) / pl->row_block_a : 1;
  const int combos = pl->G * pl->RBa;
  if (combos > 32 || pl->RB > 4) return false;
  // (head, row block) pairs a wave keeps in registers: four waves at work where they can be, which leaves two workgroups
  // per CU, one computing while the other waits at its barrier
  // (rows of 512 bytes do not fit the registers more than twice: G 8, 64 rows, 64 pairs of 3000 keys 335 us with two per wave
  // and eight waves, 530 with four and four)
  if (pl->d * pl->elt > 256)
    pl->NQ = combos <= 4 ? 1 : (combos <= 16 ? 2 : 4);
  else
    pl->NQ = combos <= 4 ? 1 : (combos <= 8 ? 2 : (combos <= 12 ? 3 : 4));
  pl->NCG = (combos + pl->NQ - 1) / pl->NQ;
  pl->CS = (pl->NCG <= 4) ? 4 / pl->NCG : 1;
  const int tiles = (t + kScoreTile - 1) / kScoreTile;
  pl->NT = tiles;
  const int64_t units = (int64_t)pl->L * pl->Hkv;
  int64_t nch = single_chunk ? 1 : (4096 + units - 1) / units;
  if (nch < 1) nch = 1;
  if (nch > tiles) nch = tiles;
  const int tiles_per_chunk = (int)((tiles + nch - 1) / nch);
  pl->CH = tiles_per_chunk * kScoreTile;
  pl->NCH = (t + pl->CH - 1) / pl->CH;
  pl->NPART = pl->NCH * pl->CS;
  return true;
}

meda_status make_plan(const meda_params* p, Plan* out) {
  if (!p) return MEDA_ERR_INVALID_ARG;
  if (p->n_layers < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1 || p->seq_len < 1 || p->window < 1)
    return MEDA_ERR_INVALID_ARG;
  if (p->n_q_heads % p->n_kv_heads != 0) return MEDA_ERR_INVALID_ARG;
  if (p->window > p->seq_len) return MEDA_ERR_INVALID_ARG;
  if (p->recent_den <= 0 || p->recent_num < 0 || p->recent_num > p->recent_den) return MEDA_ERR_INVALID_ARG;
  if (!(p->softmax_scale >= 0.0f) || !isfinite(p->softmax_scale)) return MEDA_ERR_INVALID_ARG;
  if (p->dtype != MEDA_F32 && p->dtype != MEDA_BF16) return MEDA_ERR_UNSUPPORTED;
  if (p->head_dim != 64 && p->head_dim != 128) return MEDA_ERR_UNSUPPORTED;
  if (p->n_seqs < 0) return MEDA_ERR_INVALID_ARG;
  const int n_seqs = p->n_seqs > 0 ? p->n_seqs : 1;
  const int64_t layers = (int64_t)n_seqs * p->n_layers;  // layers of the whole batch
  if (layers > kMaxLayers) return MEDA_ERR_UNSUPPORTED;
  if (layers * p->n_kv_heads * (int64_t)p->seq_len >= (1ll << 31)) return MEDA_ERR_UNSUPPORTED;
  {
    // row statistics are indexed with 32 bits over [layers][Hq][scoring rows, at least one padded window of 128];
    // offsets inside one (layer, head) of q, k, v are 32-bit byte counts
    const int64_t rows = (p->flags & MEDA_FLAG_FULL_PROMPT) ? p->seq_len : p->window;
    if (layers * p->n_q_heads * (rows > 128 ? rows : 128) >= (1ll << 31)) return MEDA_ERR_UNSUPPORTED;
    const int64_t elt = (p->dtype == MEDA_BF16) ? 2 : 4;
    if ((int64_t)p->seq_len * p->head_dim * elt >= (1ll << 31)) return MEDA_ERR_UNSUPPORTED;
  }
  {
    const int64_t lo1 = (int64_t)p->n_layers * (p->window < p->seq_len ? p->window : p->seq_len);
    if (p->total_budget < lo1 || p->total_budget > (int64_t)p->n_layers * p->seq_len) return MEDA_ERR_BUDGET;
  }

  Plan pl;
  pl.N = n_seqs; pl.Lseq = p->n_layers;
  pl.L = (int)layers; pl.Hq = p->n_q_heads; pl.Hkv = p->n_kv_heads; pl.G = pl.Hq / pl.Hkv;
  pl.d = p->head_dim; pl.T = p->seq_len; pl.W = p->window; pl.B = p->total_budget * n_seqs;
  pl.num = p->recent_num; pl.den = p->recent_den; pl.dtype = p->dtype; pl.flags = p->flags;
  pl.elt = (p->dtype == MEDA_BF16) ? 2 : 4;
  const int64_t lo = (int64_t)pl.L * (pl.W < pl.T ? pl.W : pl.T), hi = (int64_t)pl.L * pl.T;
  if (pl.B < lo || pl.B > hi) return MEDA_ERR_BUDGET;
  const double scale = (p->softmax_scale > 0.0f) ? (double)p->softmax_scale : 1.0 / sqrt((double)pl.d);
  pl.scale_log2 = (float)(scale * 1.4426950408889634074);

  const bool full_prompt = (pl.flags & MEDA_FLAG_FULL_PROMPT) != 0;
  pl.R = full_prompt ? pl.T : pl.W;
  // More than 128 scoring rows (a long observation window, or every prompt row), or more (head, 32-row block) pairs
  // per kv head than a workgroup of the window kernels holds: the rows are cut into row blocks counted from the end,
  // and one launch of each scoring kernel covers all of them.
  pl.blocks = (pl.R > kScoreRowBlock || pl.G * ((pl.R + 31) / 32) > 32) ? 1 : 0;
  pl.Tk = pl.T;
  pl.q_row0 = 0;
  pl.NTk = (pl.T + kScoreTile - 1) / kScoreTile;
  pl.accumulate = 0;
  const int w_score = (pl.blocks || pl.R > kScoreRowBlock) ? kScoreRowBlock : pl.R;
  if (!score_geometry(&pl, pl.T, w_score, pl.R, pl.blocks)) return MEDA_ERR_UNSUPPORTED;
  // Few column tiles over all layers: the kernels that cut the work finer (score_direct.hip).
  const bool direct_fits = !pl.blocks && pl.Hq * (pl.RB * 384 + 128) <= 130944;  // its LDS
  const bool many_heads = pl.Hq >= kDirectManyHeads && (pl.G == 1 || pl.d == 64 || pl.dtype == MEDA_F32);
  const int64_t seq_tiles = (int64_t)pl.NT * pl.Lseq, all_tiles = (int64_t)pl.NT * pl.L;
  const bool few = all_tiles <= kDirectTiles || (pl.N <= 4 && seq_tiles <= kDirectTiles);
  pl.direct = direct_fits && all_tiles <= kDirectTilesAll && (many_heads || few) ? 1 : 0;
  if (pl.direct) {
    const int tiles = (pl.T + 31) / 32;
    pl.NTk = tiles;
    // chunks of pass A: about 2048 waves for one sequence (the sums of a sequence then do not depend on the batch), at
    // most kDirParts partials per row
    const int64_t waves = (int64_t)pl.Lseq * pl.Hq * pl.RB;
    int64_t chunks = (2048 + waves - 1) / waves;
    if (chunks > kDirParts) chunks = kDirParts;
    if (chunks > tiles) chunks = tiles;
    pl.CH = (int)((tiles + chunks - 1) / chunks) * 32;
    pl.NCH = (pl.T + pl.CH - 1) / pl.CH;
    pl.NPART = pl.NCH;
  }
  pl.sim = similarity_route(pl);
  const size_t stats_rows = pl.blocks ? (size_t)pl.R : (size_t)pl.Wp;

  pl.n_less_total = (size_t)((int64_t)pl.L * pl.T - pl.B) * pl.Hkv;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes, 256); return at; };
  pl.off_stats_part = take((size_t)pl.L * pl.Hq * stats_rows * pl.NPART * 16);
  pl.off_stats = take((size_t)pl.L * pl.Hq * stats_rows * 16);
  pl.off_inv_norm = take((size_t)pl.L * pl.Hkv * pl.T * 4);
  pl.off_col_scores = take((size_t)pl.L * pl.Hkv * pl.T * 4);
  pl.off_ent_part = take((size_t)pl.L * pl.NTk * 2 * 8);
  pl.off_alloc = take((size_t)pl.L * 16);
  pl.off_layer_off = take((size_t)(pl.L + 1) * 8);
  pl.off_sel_idx = take((size_t)pl.B * pl.Hkv * 4);
  pl.off_sel_inv = take((size_t)pl.B * pl.Hkv * 4);
  pl.off_packed_k = take(pl.dtype == MEDA_BF16 ? (size_t)pl.B * pl.Hkv * pl.d * pl.elt : 0);  // no fp32 kernel reads packed keys
  const size_t less_bytes = pl.n_less_total * 4 + 16;
  pl.off_less_idx = take(less_bytes);
  pl.off_less_slot = take(less_bytes);
  pl.off_sort_a = take(less_bytes);
  pl.off_sort_b = take(less_bytes);
  pl.off_sort_c = take(less_bytes);
  pl.off_sort_d = take(less_bytes);
  pl.off_seg_beg = take((size_t)pl.B * pl.Hkv * 4);
  pl.off_seg_end = take((size_t)pl.B * pl.Hkv * 4);
  pl.total_bytes = o;
  *out = pl;
  return MEDA_OK;
}

// Kernels whose dynamic LDS limit has been raised, per device (a few dozen template instantiations at most).
hipError_t allow_dynamic_lds(const void* kernel, int bytes) {
  struct Entry { const void* fn; int bytes; unsigned long long devices; };
  static std::mutex mu;
  static std::vector<Entry> seen;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < 64;
  std::lock_guard<std::mutex> lk(mu);
  Entry* entry = nullptr;
  for (Entry& en : seen)
    if (en.fn == kernel && en.bytes >= bytes) entry = &en;
  if (entry && tracked && ((entry->devices >> dev) & 1ull)) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess || !tracked) return e;
  if (entry) entry->devices |= 1ull << dev;
  else seen.push_back(Entry{kernel, bytes, 1ull << dev});
  return hipSuccess;
}

// ------------------------------------------------------------------------------------- profiling
struct CallEvents {
  hipEvent_t ev[MEDA_N_PHASES + 1];
  int only;  // -1: every phase was bracketed; p: only phase p (events p and p+1)
};
static std::mutex g_mu;
static bool g_profile = false;
static int g_only = -1;
static std::vector<CallEvents> g_pending, g_pool;
static double g_ms[MEDA_N_PHASES] = {0};
static int g_calls = 0;
constexpr size_t kMaxPending = 4096;

static bool acquire_events(CallEvents* ce) {
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_profile || g_pending.size() >= kMaxPending) return false;
  if (!g_pool.empty()) {
    *ce = g_pool.back();
    g_pool.pop_back();
  } else {
    for (int i = 0; i <= MEDA_N_PHASES; ++i)
      if (hipEventCreate(&ce->ev[i]) != hipSuccess) return false;
  }
  ce->only = g_only;
  return true;
}

}  // namespace meda

using namespace meda;

extern "C" {

size_t meda_workspace_bytes(const meda_params* params) {
  Plan pl;
  if (make_plan(params, &pl) != MEDA_OK) return 0;
  return pl.total_bytes;
}

meda_status meda_workspace_region(const meda_params* params, int region, size_t* offset, size_t* bytes) {
  Plan pl;
  if (!offset || !bytes) return MEDA_ERR_INVALID_ARG;
  const meda_status st = make_plan(params, &pl);
  if (st != MEDA_OK) return st;
  switch (region) {
    case MEDA_REGION_COL_SCORES: *offset = pl.off_col_scores; *bytes = (size_t)pl.L * pl.Hkv * pl.T * 4; break;
    case MEDA_REGION_INV_NORM: *offset = pl.off_inv_norm; *bytes = (size_t)pl.L * pl.Hkv * pl.T * 4; break;
    case MEDA_REGION_ROW_STATS:
      *offset = pl.off_stats;
      *bytes = (size_t)pl.L * pl.Hq * (pl.blocks ? (size_t)pl.R : (size_t)pl.Wp) * 16;
      break;
    case MEDA_REGION_ALLOC: *offset = pl.off_alloc; *bytes = (size_t)pl.L * 16; break;
    case MEDA_REGION_LESS_IDX: *offset = pl.off_less_idx; *bytes = pl.n_less_total * 4; break;
    case MEDA_REGION_LESS_SLOT: *offset = pl.off_less_slot; *bytes = pl.n_less_total * 4; break;
    default: return MEDA_ERR_INVALID_ARG;
  }
  return MEDA_OK;
}

meda_status meda_compress(const meda_params* params, const void* q_win, const void* k, const void* v,
                          const uint8_t* modality, void* k_out, void* v_out, int32_t* layer_len,
                          int64_t* layer_off, double* entropy, int32_t* sel_idx, int32_t* merge_assign,
                          void* workspace, size_t workspace_bytes, void* hip_stream) {
  Plan pl;
  const meda_status st = make_plan(params, &pl);
  if (st != MEDA_OK) return st;
  if (!q_win || !k || !v || !modality || !k_out || !v_out || !layer_len || !layer_off) return MEDA_ERR_INVALID_ARG;
  if (!workspace || ((uintptr_t)workspace & 255u) != 0 || workspace_bytes < pl.total_bytes) return MEDA_ERR_WORKSPACE;
  const uintptr_t align_or = (uintptr_t)q_win | (uintptr_t)k | (uintptr_t)v | (uintptr_t)k_out | (uintptr_t)v_out;
  if (align_or & 15u) return MEDA_ERR_INVALID_ARG;  // rows are moved in 16-byte pieces

  Buffers b;
  b.q = q_win; b.k = k; b.v = v; b.mask = modality; b.k_out = k_out; b.v_out = v_out;
  b.layer_len = layer_len; b.layer_off = layer_off; b.entropy = entropy; b.sel_idx_user = sel_idx;
  b.merge_assign = merge_assign; b.ws = static_cast<char*>(workspace);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  CallEvents ce;
  const bool prof = acquire_events(&ce);
  typedef hipError_t (*Launcher)(const Plan&, const Buffers&, hipStream_t);
  const Launcher phases[MEDA_N_PHASES] = {launch_score_stats, launch_stats_combine, launch_score_accum,
                                          launch_allocate,    launch_select,        launch_similarity,
                                          launch_segment_sort, launch_merge_write};
  const bool no_merge = (pl.flags & MEDA_FLAG_NO_MERGE) || pl.B == (int64_t)pl.L * pl.T;
  hipError_t err = hipSuccess;
  if (prof && ce.only <= 0) err = hipEventRecord(ce.ev[0], s);
  for (int i = 0; i < MEDA_N_PHASES && err == hipSuccess; ++i) {
    const bool skip = no_merge && (i == 5 || i == 6);
    if (!skip) err = phases[i](pl, b, s);
    const bool rec = prof && (ce.only < 0 || i == ce.only || i + 1 == ce.only);
    if (rec && err == hipSuccess) err = hipEventRecord(ce.ev[i + 1], s);
  }
  if (prof) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (err == hipSuccess) g_pending.push_back(ce); else g_pool.push_back(ce);
  }
  return err == hipSuccess ? MEDA_OK : MEDA_ERR_HIP;
}

meda_status meda_profile_enable(int enable) {
  if (enable < 0 || enable > 1 + MEDA_N_PHASES) return MEDA_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(g_mu);
  g_profile = enable != 0;
  g_only = enable >= 2 ? enable - 2 : -1;
  return MEDA_OK;
}

meda_status meda_profile_read(double* phase_ms, int32_t* n_calls, int reset) {
  if (!phase_ms || !n_calls) return MEDA_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(g_mu);
  meda_status st = MEDA_OK;
  for (CallEvents& ce : g_pending) {
    const int last = ce.only < 0 ? MEDA_N_PHASES : ce.only + 1;
    if (hipEventSynchronize(ce.ev[last]) != hipSuccess) { st = MEDA_ERR_HIP; continue; }
    for (int i = 0; i < MEDA_N_PHASES; ++i) {
      if (ce.only >= 0 && i != ce.only) continue;
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, ce.ev[i], ce.ev[i + 1]) == hipSuccess) g_ms[i] += ms; else st = MEDA_ERR_HIP;
    }
    ++g_calls;
    g_pool.push_back(ce);
  }
  g_pending.clear();
  for (int i = 0; i < MEDA_N_PHASES; ++i) phase_ms[i] = g_ms[i];
  *n_calls = g_calls;
  if (reset) {
    for (int i = 0; i < MEDA_N_PHASES; ++i) g_ms[i] = 0.0;
    g_calls = 0;
  }
  return st;
}

const char* meda_phase_name(int phase) {
  static const char* names[MEDA_N_PHASES] = {"score_stats", "stats_combine", "score_accum", "allocate",
                                             "select",      "similarity",    "segment_sort", "merge_write"};
  return (phase >= 0 && phase < MEDA_N_PHASES) ? names[phase] : "?";
}

const char* meda_status_string(meda_status status) {
  switch (status) {
    case MEDA_OK: return "ok";
    case MEDA_ERR_INVALID_ARG: return "invalid argument";
    case MEDA_ERR_BUDGET: return "total budget outside [L*min(W,T), L*T]";
    case MEDA_ERR_UNSUPPORTED: return "unsupported head_dim, dtype, window or group size";
    case MEDA_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MEDA_ERR_HIP: return "HIP error";
    case MEDA_ERR_SCRATCH_LIMIT: return "the step needs more scratch than the no-allocation entry point's built-in array holds";
  }
  return "unknown status";
}

}  // extern "C"
