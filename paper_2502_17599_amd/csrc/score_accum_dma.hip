// Pass B of the scoring (Sections 3.2 and 3.3) for grouped query heads and observation windows of up to 96 rows: the
// sums of score_accum_kernel with another way of feeding it.  A workgroup walks over all query heads against one
// column tile of 128 keys; per head it needs the window's query rows and row statistics, per kv head the key tile.
// Here the window comes by asynchronous global-to-LDS copies (no staging registers, no LDS store instructions), one wait
// and one barrier per head.
//
// A lane owns one key column (the query rows are operand A), as in score_accum_kernel, and every sum has that kernel's
// order.  The 1/Z and the cross-modal weight of the rows sit in two registers per row block, lane r of each 16 lanes
// holding those of the row of accumulator register r: the multiply-adds take them from there (DPP row broadcast) where
// score_accum_kernel reads LDS eight times per block of 32 x 32.  A row is of one modality and so has one weight: what it
// gathers over keys of its own modality is dropped when the entropy terms are taken.  Tiles below the causal diagonal have
// a loop of their own: a branch inside one loop made the compiler copy all accumulators around it, 48 moves beside the 64
// vector instructions that a block needs (a multiply-add, an exponential and two multiply-adds per probability), which is
// what bounds this kernel.  32 layers of 16384 keys, 4 heads per kv head, 64 rows: 518 -> 417 us; 28 of 37376, 7 heads per
// kv head: 830 -> 640 us.
//
// The query rows and statistics of head h+1 are requested when head h starts.  A wave's key rows are used by no other
// wave, so with much work per kv head they go straight to its registers; the next kv head's are requested when the last
// product with the present ones is done, before its probabilities are formed.  Without a key tile in LDS the workgroups
// of a CU are four (three with their registers) instead of two.  With little work per kv head (KEYS: one row block, or
// two and two heads) the stream of keys bounds the kernel, and fragment loads, which touch 64 lines each, and their late
// request cost more than the tile: there every wave has its key rows in LDS too, brought by copies of whole rows that
// start as soon as the present ones are in registers.  16 layers of 20000 keys, 2 kv heads, 32 rows, 2 / 4 / 8 heads per kv
// head: 54 / 65 / 87 us from registers, 41 / 55 / 83 from LDS; 64 rows, 2 heads: 66 and 63.
//
// LDS tiles filled by the copies are laid out as CopyTile (device_utils.hpp).
// grid (NT, L) x 4 waves: wave cw owns the 32 keys cw*32.. of the tile and all RB 32-row blocks of the window.
#include "score_common.hpp"

namespace meda {

constexpr int kDmaWaves = 4;
constexpr int kDmaThreads = kDmaWaves * 64;

template <typename T, int D, int RB>
constexpr int dma_stage_bytes() {  // the window's query rows and the four planes of their statistics
  return CopyTile<T, D>::bytes(RB * 32) + 4 * RB * 32 * (int)sizeof(float);
}

template <typename T, int D, int RB, bool KEYS>
constexpr size_t dma_lds_bytes() {  // two stages, the entropy reduction, the waves' key rows
  return 2 * (size_t)dma_stage_bytes<T, D, RB>() + kDmaWaves * 2 * sizeof(double) + (KEYS ? CopyTile<T, D>::bytes(kScoreTile) : 0);
}

template <typename T, int D, int RB, bool KEYS>
__global__ void __launch_bounds__(kDmaThreads, RB <= 2 ? 3 : 2) score_accum_dma_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  using CT = CopyTile<T, D>;
  constexpr int RBt = TL::kRowBytes;
  constexpr int CPR = TL::kChunksPerRow;
  constexpr int RPI = 64 / CPR;                          // rows one copy instruction fills
  constexpr int QI = RB * 32 / RPI;                      // copy instructions of a window of query rows
  constexpr int PFQ = (QI + kDmaWaves - 1) / kDmaWaves;  // per wave (the last ones may be beyond QI)
  constexpr int Wp = RB * 32;
  constexpr int kQBytes = CT::bytes(Wp);
  constexpr int kStageBytes = dma_stage_bytes<T, D, RB>();
  static_assert(RPI == CT::kRows && (RB * 32) % RPI == 0, "the copy instructions must tile the window evenly");
  constexpr int KI = 32 / RPI;                           // copy instructions of a wave's key rows
  extern __shared__ __align__(16) char smem[];  // stage 0, stage 1, reduction, key rows
  double* red = reinterpret_cast<double*>(smem + 2 * kStageBytes);  // [waves][2]

  // layers are walked in the opposite order of pass A, so the keys pass A touched last (still in the
  // memory-side cache) are the first ones read here
  const int tile = blockIdx.x, l = a.L - 1 - blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int cw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = tile * kScoreTile;
  const int j = j0 + cw * 32 + n;  // this lane's key column
  const bool col_ok = j < a.T;
  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;
  const bool col_is_vision = col_ok && mask[j] != 0;
  // Rows past the window (W not a multiple of 32) repeat the last query row and its maximum and have zero weights: their
  // exponentials are finite and add nothing.
  const bool full = j0 + kScoreTile - 1 <= a.T - a.W;

  // Query copy c of this wave fills the rows (cw * PFQ + c) * RPI .. of the window: this lane brings one 16-byte chunk.
  // Rows past the window repeat its last row; keys past the end of the sequence the last key (masked).
  unsigned qoff[PFQ];
#pragma unroll
  for (int c = 0; c < PFQ; ++c) {
    const int r = (cw * PFQ + c) * RPI + lane / CPR;
    qoff[c] = (unsigned)(a.q_row0 + min(r, a.W - 1)) * RBt + CT::source_chunk(lane);
  }
  const unsigned koff = (unsigned)min(j, a.Tk - 1) * RBt;  // this lane's key inside a (layer, kv head)
  char* key_rows = smem + 2 * kStageBytes + kDmaWaves * 2 * sizeof(double) + cw * CT::bytes(32);  // this wave's
  unsigned kcopy[KI];  // KEYS: the chunk this lane brings with copy c (keys past the end repeat the last one)
#pragma unroll
  for (int c = 0; c < KI; ++c)
    kcopy[c] = (unsigned)min(j0 + cw * 32 + c * RPI + lane / CPR, a.Tk - 1) * RBt + CT::source_chunk(lane);
  auto issue_keys = [&](int g) {
    const char* ksrc = uniform_ptr(a.k + (size_t)(l * a.Hkv + g) * a.Tk * RBt);
#pragma unroll
    for (int c = 0; c < KI; ++c) async_copy16_to_lds_stream(ksrc, kcopy[c], (unsigned)(size_t)key_rows + c * CT::kPiece);
  };
  // (the base straight from the kernel's arguments: through uniform_ptr it would lose its address space, and FLAT loads, which
  // count as LDS accesses too and come back in no order, cannot be waited for by number)
  auto load_keys = [&](Frag<T, D>& f, int g) { frag_load(f, a.k + (size_t)(l * a.Hkv + g) * a.Tk * RBt + koff, kg); };
  // this lane's value of the first kDmaThreads statistics (the plane of the maxima is among them)
  const unsigned soff = 4u * (unsigned)(tid < Wp ? min(tid, a.W - 1) : tid);
  const unsigned lds0 = (unsigned)(size_t)smem;
  const float* stats_f = reinterpret_cast<const float*>(a.stats);
  auto issue = [&](int h) {  // the query rows and statistics of head h
    const unsigned stage = lds0 + (unsigned)((h & 1) * kStageBytes);
    const char* qsrc = uniform_ptr(a.q + (size_t)(l * a.Hq + h) * a.q_rows * RBt);
#pragma unroll
    for (int c = 0; c < PFQ; ++c)
      if (cw * PFQ + c < QI) async_copy16_to_lds(qsrc, qoff[c], stage + (unsigned)((cw * PFQ + c) * CT::kPiece));
    // the 4 * Wp statistics of the head are contiguous: wave w brings the values w*64 .. w*64+63 of them
    const float* ssrc = uniform_ptr(stats_f + (size_t)(l * a.Hq + h) * 4 * Wp);
#pragma unroll
    for (int w0 = 0; w0 < 4 * Wp; w0 += kDmaThreads)
      if (w0 + cw * 64 < 4 * Wp)
        async_copy4_to_lds(ssrc, w0 == 0 ? soff : (unsigned)(w0 + cw * 64 + lane) * 4u,
                           stage + (unsigned)(kQBytes + (w0 + cw * 64) * 4));
  };

  const unsigned fbase = CT::frag_base(n, kg);

  issue(0);
  Frag<T, D> kf;
  if constexpr (KEYS)
    issue_keys(0);
  else
    load_keys(kf, 0);
  float pbar[RB][16];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) pbar[rb][r] = 0.f;
  float colsum = 0.f;

  // The walk over the heads.  MASKED: the tile touches the causal diagonal or the end of the sequence, so every
  // probability is checked against its row; all other tiles take the plain walk.
  auto walk = [&](auto masked_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    int g = 0, hg = 0;
    for (int h = 0; h < a.Hq; ++h) {
      // this wave's pieces of the head have landed (younger than them: the loads of its keys, at the start of a group, or
      // the copies of the next group's keys, which the first head of a group issues behind those of the second)
      if (!KEYS && hg == 0)
        async_copy_wait<TL::kFragChunks>();
      else if (KEYS && hg == 1 && g + 1 < a.Hkv)
        async_copy_wait<KI>();
      else
        async_copy_wait<0>();
      __syncthreads();  // every wave's have; and nobody reads the other stage (the previous head) any more
      const char* stage = smem + (h & 1) * kStageBytes;
      const float* st = reinterpret_cast<const float*>(stage + kQBytes);  // planes: maximum, 1/Z, the two cross-modal 1/Z
      if (KEYS && hg == 0) frag_from_tile(kf, key_rows, fbase);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        Frag<T, D> qf;
        frag_from_tile(qf, stage + CT::bytes(32) * rb, fbase);
        const int row = rb * 32 + acc_row(n & 15, kg);  // of register n % 16
        const float rz = st[Wp + row], coef = st[2 * Wp + row] + st[3 * Wp + row];
        f32x16_t acc = acc_zero();
        mma<T, D>(acc, qf, kf);
        // (behind the first product, so that the wait for the keys there does not wait for these copies)
        if (rb == 0 && h + 1 < a.Hq) issue(h + 1);
        if (KEYS && rb == 0 && hg == 0 && g + 1 < a.Hkv) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the present key rows have left LDS
          issue_keys(g + 1);
        }
        if (!KEYS && rb == RB - 1 && hg == a.G - 1)  // the next kv head's keys (past the last one: the same again)
          load_keys(kf, min(g + 1, a.Hkv - 1));
        // Row r (without the lane group's offset kg*4) counts for this lane's column iff row_min <= r < row_end: the row
        // exists and sees the column (j <= T - W + r + kg*4).  Opaque, so that the comparisons are redone per head instead
        // of being kept in registers.
        int row_min = col_ok ? j - (a.T - a.W) - kg * 4 : (1 << 30);
        int row_end = a.W - kg * 4;
        if (MASKED) asm volatile("" : "+v"(row_min), "+v"(row_end));
        static_for<4>([&](auto r4_tag) {
          constexpr int r4 = decltype(r4_tag)::value;
          const float4 m4 = *reinterpret_cast<const float4*>(st + rb * 32 + r4 * 8 + kg * 4);
          const float mm[4] = {m4.x, m4.y, m4.z, m4.w};
          float e[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            e[i] = fast_exp2(fmaf(acc[r4 * 4 + i], a.c, -mm[i]));
            if (MASKED) e[i] = (rb * 32 + r4 * 8 + i >= row_min && rb * 32 + r4 * 8 + i < row_end) ? e[i] : 0.f;
          }
          float* pb = &pbar[rb][r4 * 4];
          fma_rows4<r4 * 4>(colsum, pb[0], pb[1], pb[2], pb[3], rz, coef, e[0], e[1], e[2], e[3]);
        });
      }
      if (++hg == a.G) {
        const float tot = colsum + __shfl_xor(colsum, 32, kWave);
        if (kg == 0 && col_ok) a.col_scores[(size_t)(l * a.Hkv + g) * a.Tk + j] = tot;  // one writer per column
        colsum = 0.f;
        hg = 0;
        ++g;
      }
    }
  };
  if (full)
    walk(std::false_type{});
  else
    walk(std::true_type{});

  // Entropy terms of the head-averaged cross-modal probabilities: text rows on vision keys, vision rows on text keys.
  unsigned rows_vision[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) rows_vision[rb] = (unsigned)__ballot(mask[a.T - a.W + min(rb * 32 + n, a.W - 1)] != 0);
  const float inv_heads = 1.0f / (float)a.Hq;
  float s = 0.f;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool row_is_vision = ((rows_vision[rb] >> acc_row(r, kg)) & 1u) != 0;
      const float p = pbar[rb][r] * inv_heads;
      const float t = p * __logf(p);  // (no branch around the logarithm)
      s += ((p > 0.f) & (row_is_vision != col_is_vision)) ? t : 0.f;
    }
  const double tv = wave_sum(col_is_vision ? (double)s : 0.0);
  const double vt = wave_sum((col_ok && !col_is_vision) ? (double)s : 0.0);
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

template <typename T, int D, int RB, bool KEYS>
static hipError_t launch_dma_k(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  constexpr size_t lds = dma_lds_bytes<T, D, RB, KEYS>();
  auto kern = score_accum_dma_kernel<T, D, RB, KEYS>;
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
    case 1: return launch_dma_k<T, D, 1, true>(p, a, s);
    case 2: return p.G == 2 ? launch_dma_k<T, D, 2, true>(p, a, s) : launch_dma_k<T, D, 2, false>(p, a, s);
    default: return launch_dma_k<T, D, 3, false>(p, a, s);
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
