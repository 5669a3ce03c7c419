// Pass B of the scoring (Sections 3.2 and 3.3) for grouped query heads and observation windows of up to 96 rows: the
// sums of score_accum_kernel with another way of feeding it.  A workgroup walks over all query heads against one
// column tile of 128 keys; per head it needs the window's query rows and row statistics, per kv head the key tile.
// Here they come by asynchronous global-to-LDS copies (no staging registers, no LDS store instructions): the copies
// of head h+1 (and of the next kv head's key tile, when h+1 starts a new group) are issued when head h starts, so a
// head costs one wait and one barrier and no load is waited for where it is issued.
//
// The keys are operand A and the query rows operand B, so a lane owns one query row and 16 keys per block: the row's
// statistics are three registers of the lane (with a column per lane they were twelve 16-byte LDS reads per block of
// 32 x 32), and the column sums of a kv head are reduced over the lanes once per kv head.  Bound by the vector unit: a
// probability costs a multiply-add, an exponential and two multiply-adds.  32 layers of 16384 keys, 4 heads per kv head,
// 64 rows: 518 -> 423 us; 28 of 37376, 7 heads per kv head: 820 -> 679 us.
//
// One key tile buffer is enough with at least two query heads per kv head: every wave takes its key fragment out of
// the buffer in the first head of a group, and the next tile is requested in the last head of the group, at least one
// barrier later.  (With one query head per kv head score_accum_kernel stages the next tile through registers.)
//
// LDS tiles filled by the copies are unpadded and xor-swizzled (swizzle_of_row in device_utils.hpp).
// grid (NT, L) x 4 waves: wave cw owns the 32 key columns cw*32.. of the tile (a lane owns one column) and all RB
// 32-row blocks of the window.
#include "score_common.hpp"

namespace meda {

constexpr int kDmaWaves = 4;
constexpr int kDmaThreads = kDmaWaves * 64;

template <typename T, int D, int RB>
constexpr int dma_stage_bytes() {  // the window's query rows and the four planes of their statistics
  return RB * 32 * Tile<T, D>::kRowBytes + 4 * RB * 32 * (int)sizeof(float);
}

template <typename T, int D, int RB>
constexpr size_t dma_lds_bytes() {  // the key tile, two stages, the entropy reduction
  return (size_t)kScoreTile * Tile<T, D>::kRowBytes + 2 * (size_t)dma_stage_bytes<T, D, RB>() + kDmaWaves * 2 * sizeof(double);
}

template <typename T, int D, int RB>
__global__ void __launch_bounds__(kDmaThreads, 2) score_accum_dma_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  constexpr int RBt = TL::kRowBytes;
  constexpr int CPR = TL::kChunksPerRow;
  constexpr int NC = TL::kFragChunks;
  constexpr int RPI = 64 / CPR;                          // rows one copy instruction fills
  constexpr int PFK = kScoreTile / RPI / kDmaWaves;      // key copy instructions per wave and tile
  constexpr int QI = RB * 32 / RPI;                      // copy instructions of a window of query rows
  constexpr int PFQ = (QI + kDmaWaves - 1) / kDmaWaves;  // per wave (the last ones may be beyond QI)
  constexpr int Wp = RB * 32;
  constexpr int kTileBytes = kScoreTile * RBt;
  constexpr int kQBytes = Wp * RBt;
  constexpr int kStageBytes = dma_stage_bytes<T, D, RB>();
  static_assert(64 % CPR == 0 && kScoreTile % (RPI * kDmaWaves) == 0, "the copy instructions must tile a tile evenly");
  extern __shared__ __align__(16) char smem[];  // key tile, stage 0, stage 1, reduction
  double* red = reinterpret_cast<double*>(smem + kTileBytes + 2 * kStageBytes);  // [waves][2]

  // layers are walked in the opposite order of pass A, so the keys pass A touched last (still in the
  // memory-side cache) are the first ones read here
  const int tile = blockIdx.x, l = a.L - 1 - blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int cw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = tile * kScoreTile;
  const int jw = j0 + cw * 32;  // the wave's first key
  // rows past the window (W not a multiple of 32) repeat the last query row and have zero weights; the masked path
  // also drops their exponentials, which the plain path would multiply by zero (not safe if one overflowed)
  const bool full = j0 + kScoreTile - 1 <= a.T - a.W && a.W == Wp;

  // Key copy c of this wave fills the rows (cw * PFK + c) * RPI .. + RPI-1 of the tile, query copy c the rows
  // (cw * PFQ + c) * RPI .. of the window: this lane brings one 16-byte chunk.  Key rows past the end of the sequence
  // repeat the last key (their columns are masked), query rows past the window the last row.
  unsigned koff[PFK], qoff[PFQ];
#pragma unroll
  for (int c = 0; c < PFK; ++c) {
    const int r = (cw * PFK + c) * RPI + lane / CPR;
    koff[c] = (unsigned)min(j0 + r, a.Tk - 1) * RBt + (unsigned)(((lane % CPR) ^ swizzle_of_row<T, D>(r)) * 16);
  }
#pragma unroll
  for (int c = 0; c < PFQ; ++c) {
    const int r = (cw * PFQ + c) * RPI + lane / CPR;
    qoff[c] = (unsigned)(a.q_row0 + min(r, a.W - 1)) * RBt + (unsigned)(((lane % CPR) ^ swizzle_of_row<T, D>(r)) * 16);
  }
  const unsigned lds0 = (unsigned)(size_t)smem;
  const float* stats_f = reinterpret_cast<const float*>(a.stats);
  // the query rows and statistics of head h; with g >= 0 the key tile of kv head g too
  auto issue = [&](int h, int g) {
    const unsigned stage = lds0 + (unsigned)(kTileBytes + (h & 1) * kStageBytes);
    if (g >= 0) {
      const char* ksrc = uniform_ptr(a.k + (size_t)(l * a.Hkv + g) * a.Tk * RBt);
#pragma unroll
      for (int c = 0; c < PFK; ++c) async_copy16_to_lds_stream(ksrc, koff[c], lds0 + (unsigned)((cw * PFK + c) * 1024));
    }
    const char* qsrc = uniform_ptr(a.q + (size_t)(l * a.Hq + h) * a.q_rows * RBt);
#pragma unroll
    for (int c = 0; c < PFQ; ++c)
      if (cw * PFQ + c < QI) async_copy16_to_lds(qsrc, qoff[c], stage + (unsigned)((cw * PFQ + c) * 1024));
    // the 4 * Wp statistics of the head are contiguous: wave w brings the values w*64 .. w*64+63 of them
    const float* ssrc = uniform_ptr(stats_f + (size_t)(l * a.Hq + h) * 4 * Wp);
#pragma unroll
    for (int w0 = 0; w0 < 4 * Wp; w0 += kDmaThreads)
      if (w0 + cw * 64 < 4 * Wp)
        async_copy4_to_lds(ssrc, (unsigned)(w0 + cw * 64 + lane) * 4u,
                           stage + (unsigned)(kQBytes + (w0 + cw * 64) * 4));
  };

  // chunk c of this lane's fragment (chunk kg * NC + c of row n of a 32-row block) sits at (n * row bytes) +
  // 16 * ((kg * NC + c) ^ swz(n)) inside the block; the swizzle of a row does not depend on its block
  unsigned coff[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) coff[c] = (unsigned)(n * RBt + (((kg * NC + c) ^ swizzle_of_row<T, D>(n)) * 16));
  auto frag_from = [&](Frag<T, D>& f, const char* block) {
#pragma unroll
    for (int c = 0; c < NC; ++c) f.c[c] = *reinterpret_cast<const uint4*>(block + coff[c]);
  };

  float pbar[RB][16];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) pbar[rb][r] = 0.f;
  Frag<T, D> kf;
  float colsum[16];

  // The walk over the heads.  MASKED: the tile touches the causal diagonal or the end of the sequence, so every
  // probability is checked against its row; all other tiles take the plain walk.  (The two are separate loops: a branch
  // inside one loop made the compiler copy all accumulators around it, 48 moves beside the 64 instructions that a block
  // of 32 x 32 needs.)
  auto walk = [&](auto masked_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    int g = 0, hg = 0;
    for (int h = 0; h < a.Hq; ++h) {
      async_copy_wait<0>();  // this wave's pieces of the head have landed
      __syncthreads();       // every wave's have; and nobody reads the other stage (the previous head) any more
      if (h + 1 < a.Hq) issue(h + 1, hg + 1 == a.G ? g + 1 : -1);
      const char* stage = smem + kTileBytes + (h & 1) * kStageBytes;
      const float* st = reinterpret_cast<const float*>(stage + kQBytes);  // planes: maximum, 1/Z, the two cross-modal 1/Z
      if (hg == 0) {
        frag_from(kf, smem + cw * 32 * RBt);  // the key tile of this kv head
#pragma unroll
        for (int r = 0; r < 16; ++r) colsum[r] = 0.f;
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        Frag<T, D> qf;
        frag_from(qf, stage + rb * 32 * RBt);
        const float m = st[rb * 32 + n], rz = st[Wp + rb * 32 + n];
        // a row is of one modality, so one of its two weights is zero: the sum is its weight on the other modality's keys
        const float coef = st[2 * Wp + rb * 32 + n] + st[3 * Wp + rb * 32 + n];
        f32x16_t acc = acc_zero();
        mma<T, D>(acc, kf, qf);
        // The row sees the wave's key i iff i <= T - W + row - jw; rows past the window see none.  The bound is made
        // opaque so that the 16 comparisons per row block are redone per head instead of being kept in registers.
        int seen = rb * 32 + n < a.W ? a.T - a.W + rb * 32 + n - jw - kg * 4 : -1;
        if (MASKED) asm volatile("" : "+v"(seen));
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float e = fast_exp2(fmaf(acc[r], a.c, -m));
          if (MASKED) e = acc_row(r, 0) <= seen ? e : 0.f;
          colsum[r] = fmaf(e, rz, colsum[r]);
          pbar[rb][r] = fmaf(e, coef, pbar[rb][r]);
        }
      }
      if (++hg == a.G) {
        const float tot = reduce_lanes32(colsum, lane);  // of the key in register n / 2
        const int j = jw + acc_row(n >> 1, kg);
        if ((n & 1) == 0 && j < a.T) a.col_scores[(size_t)(l * a.Hkv + g) * a.Tk + j] = tot;  // one writer per column
        hg = 0;
        ++g;
      }
    }
  };
  issue(0, 0);
  if (full)
    walk(std::false_type{});
  else
    walk(std::true_type{});

  // Entropy terms of the head-averaged cross-modal probabilities: text rows on vision keys, vision rows on text keys
  // (the sums of a row over keys of its own modality are dropped here).
  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;
  const unsigned key_vision = (unsigned)__ballot(mask[min(jw + n, a.T - 1)] != 0);
  const float inv_heads = 1.0f / (float)a.Hq;
  float s_tv = 0.f, s_vt = 0.f;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const bool row_vision = mask[a.T - a.W + min(rb * 32 + n, a.W - 1)] != 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool vision = ((key_vision >> acc_row(r, kg)) & 1u) != 0;
      const float p = pbar[rb][r] * inv_heads;
      const float t = (p > 0.f && vision != row_vision) ? p * __logf(p) : 0.f;
      s_tv += vision ? t : 0.f;
      s_vt += vision ? 0.f : t;
    }
  }
  const double tv = wave_sum((double)s_tv), vt = wave_sum((double)s_vt);
  if (lane == 0) {
    red[cw * 2 + 0] = tv;
    red[cw * 2 + 1] = vt;
  }
  __syncthreads();
  if (tid < 2) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kDmaWaves; ++w) sum += red[w * 2 + tid];
    a.ent_part[((size_t)l * a.NTk + tile) * 2 + tid] = -sum;
  }
}

// ------------------------------------------------------------------------------------------ launch

template <typename T, int D, int RB>
static hipError_t launch_dma_k(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  constexpr size_t lds = dma_lds_bytes<T, D, RB>();
  auto kern = score_accum_dma_kernel<T, D, RB>;
  if (lds > 64 * 1024) {
    hipError_t e = allow_dynamic_lds(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(p.NT, p.L), dim3(kDmaThreads), lds, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_dma_t(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  switch (p.RB) {
    case 1: return launch_dma_k<T, D, 1>(p, a, s);
    case 2: return launch_dma_k<T, D, 2>(p, a, s);
    default: return launch_dma_k<T, D, 3>(p, a, s);
  }
}

// Grouped heads (one key tile buffer), windows of at most three 32-row blocks (four waves), rows of at most 256
// bytes (two stages fit twice per CU).
bool score_accum_dma_supported(const Plan& p) {
  return !p.blocks && p.accumulate == 0 && p.G >= 2 && p.RB <= 3 && p.d * p.elt <= 256;
}

hipError_t launch_score_accum_dma(const Plan& p, const Buffers& b, hipStream_t s) {
  const ScoreArgs a = make_args(p, b);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_dma_t<bf16_t, 128>(p, a, s) : launch_dma_t<bf16_t, 64>(p, a, s);
  return launch_dma_t<float, 64>(p, a, s);
}

}  // namespace meda
