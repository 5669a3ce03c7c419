// Pass A of the scoring (Sections 3.2 and 3.3): row maxima and softmax normalisers of every scoring row, and
// 1/|k| of every key; then the merge of the per-chunk partials.  The layout of the pass is described in
// score_common.hpp.
#include "score_common.hpp"

namespace meda {

// ------------------------------------------------------------------------------------------ pass A
// grid (NCH, Hkv, L), or (Hkv * row blocks, 1, L) in the row-block mode (more than 128 scoring rows); NCG*CS waves.
// Wave (cg, cs) keeps NQ query fragments ((head of the group, row
// block) pairs cg*NQ .. cg*NQ+NQ-1) in registers and visits the 32-key blocks sb = cs, cs+CS, ... of
// every tile of its chunk.  The product is taken with the keys as operand A and the queries as
// operand B, so a lane owns one query row and 16 keys per block: the running (max, Z_vision, Z_text)
// of the row live in three registers per fragment and need no cross-lane traffic until the end.
//
// The next tile is fetched into registers while the current one is processed, and written to a padded LDS tile between
// two barriers.  Grouped heads and the row-block mode, with rows of at most 256 bytes, go to score_stats_dma.hip.
template <typename T, int D, int NQ, int NW, bool BLOCKS>
__global__ void __launch_bounds__(NW * 64, (NQ == 1 && NW == 4 && sizeof(T) == 2) ? 3 : 2) score_stats_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  constexpr int NC = TL::kFragChunks;
  extern __shared__ __align__(16) char smem[];
  char* ktile = smem;
  uint8_t* lmask = reinterpret_cast<uint8_t*>(smem + kScoreTile * TL::kStride);

  const int ch = BLOCKS ? 0 : blockIdx.x;
  int l = blockIdx.z, g = blockIdx.y, bi = 0;
  if (BLOCKS) {  // row-block mode (one chunk): this workgroup's row block, the largest ones first
    if ((a.Hkv & 7) == 0) {
      bi = blockIdx.x / a.Hkv;
      g = blockIdx.x - bi * a.Hkv;
    } else {  // row blocks by XCD in the order of the grid would give some XCDs all the long ones
      unsigned pair, rblock;
      pair_and_row_block(blockIdx.z * gridDim.x + blockIdx.x, (unsigned)(a.L * a.Hkv), gridDim.x / (unsigned)a.Hkv, pair, rblock);
      l = pair / (unsigned)a.Hkv;
      g = pair - (unsigned)(l * a.Hkv);
      bi = rblock;
    }
    select_row_block(a, bi);
  }
  constexpr int nthr = NW * 64;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: what derives from it stays in scalar registers
  const int lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int cgi = wave % a.NCG, cs = wave / a.NCG;
  const bool active = cs < a.CS;  // the workgroup is padded to 4 or 8 waves; spare waves only move data
  const int n_combos = a.G * a.RB;

  Frag<T, D> qf[NQ];
  float m[NQ], zv[NQ], zt[NQ];
  int qrow[NQ], qhead[NQ];
  int qlast[NQ];  // position of the last row of the fragment's 32-row block (uniform over the wave)
  int nvalid = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int cidx = cgi * NQ + q;
    m[q] = kNegBig;
    zv[q] = 0.f;
    zt[q] = 0.f;
    qrow[q] = 0;
    qhead[q] = 0;
    qlast[q] = -1;
    frag_zero(qf[q]);
    if (active && cidx < n_combos) {
      nvalid = q + 1;
      const int hg = cidx / a.RB, rb = cidx - hg * a.RB;
      qhead[q] = g * a.G + hg;
      qrow[q] = rb * 32 + n;
      qlast[q] = a.T - a.W + rb * 32 + 31;
      if (qrow[q] < a.W)
        frag_load(qf[q], a.q + ((size_t)(l * a.Hq + qhead[q]) * a.q_rows + a.q_row0 + qrow[q]) * TL::kRowBytes, kg);
    }
  }

  int wave_last = -1;
#pragma unroll
  for (int q = 0; q < NQ; ++q) wave_last = max(wave_last, qlast[q]);

  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;  // this layer's sequence
  const int jbeg = ch * a.CH;
  const int jend = min(a.T, jbeg + a.CH);
  const char* kbase = a.k + (size_t)(l * a.Hkv + g) * a.Tk * TL::kRowBytes;
  float* invn_out = a.inv_norm + (size_t)(l * a.Hkv + g) * a.Tk;

  TileStage<T, D, kScoreTile, nthr> stage;
  uint8_t mreg = 0;
  if (jbeg < jend) {
    stage.template fetch<true>(kbase + (size_t)jbeg * TL::kRowBytes, min(kScoreTile, a.T - jbeg), tid, nthr);
    if (tid < kScoreTile) mreg = (jbeg + tid < a.T) ? mask[jbeg + tid] : 0;
  }
  for (int j0 = jbeg; j0 < jend; j0 += kScoreTile) {
    const int rows_valid = min(kScoreTile, a.T - j0);
    __syncthreads();  // the previous tile is no longer read
    stage.commit(ktile, tid, nthr);
    if (tid < kScoreTile) lmask[tid] = mreg;
    __syncthreads();
    if (j0 + kScoreTile < jend) {  // next tile's loads are in flight while this one is processed
      const int jn = j0 + kScoreTile;
      stage.template fetch<true>(kbase + (size_t)jn * TL::kRowBytes, min(kScoreTile, a.T - jn), tid, nthr);
      if (tid < kScoreTile) mreg = (jn + tid < a.T) ? mask[jn + tid] : 0;
    }

    // 1/|k| of the tile's keys: two threads per row (the first row block sees every key; the others skip this)
    for (int row = tid >> 1; bi == 0 && row < kScoreTile; row += nthr >> 1) {
      float ss = 0.f;
      const uint4* p = reinterpret_cast<const uint4*>(ktile + row * TL::kStride + (tid & 1) * TL::kHalfBytes);
#pragma unroll
      for (int i = 0; i < NC; ++i) ss += chunk_sumsq<T>(p[i]);
      ss += __shfl_xor(ss, 1, kWave);
      if ((tid & 1) == 0 && row < rows_valid) invn_out[j0 + row] = 1.0f / fmaxf(sqrtf(ss), 1e-30f);
    }

    for (int sb = cs; active && sb < kScoreTile / 32; sb += a.CS) {
      const int jb = j0 + sb * 32;
      if (jb >= a.T || (BLOCKS && jb > wave_last)) break;  // past the sequence, or past every row of this wave
      Frag<T, D> kf;
      frag_load(kf, ktile + (sb * 32 + n) * TL::kStride, kg);
      const uint32_t mword = (uint32_t)__ballot(lmask[sb * 32 + n] != 0);
      const bool tail = jb + 31 >= a.T;  // the block runs past the end of the sequence
      const bool one_modality = mword == 0u || mword == 0xffffffffu;
      const bool full_all = jb + 31 <= a.T - a.W;  // every key of the block is visible to every row of the window
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        // A fragment's 32 rows sit at the positions qlast-31 .. qlast.  With row blocks of several hundred rows
        // (BLOCKS) the 32-key block is classified per fragment: keys after qlast are invisible to all of its rows
        // (nothing to add), keys up to qlast-31 are visible to all of them (no per-element test needed).
        if (q < nvalid && (!BLOCKS || jb <= qlast[q])) {
          const bool full = BLOCKS ? (!tail && jb + 31 <= qlast[q] - 31) : full_all;
          const bool uniform = full && one_modality;
          f32x16_t acc = acc_zero();
          mma<T, D>(acc, kf, qf[q]);
          if (full) {
            // every key of the block counts: the maximum is taken on the raw products (the scale is positive, so
            // it commutes with the maximum) and the scale is folded into the exponent's multiply-add
            float bm = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) bm = fmaxf(fmaxf(bm, acc[r]), acc[r + 1]);
            bm = fmaxf(bm, acc[15]);
            const float mn = fmaxf(m[q], bm * a.c);
            const float sc = fast_exp2(m[q] - mn);
            zv[q] *= sc;
            zt[q] *= sc;
            m[q] = mn;
            if (uniform) {
              float s = 0.f;
#pragma unroll
              for (int r = 0; r < 16; ++r) s += fast_exp2(fmaf(acc[r], a.c, -mn));
              if (mword)
                zv[q] += s;
              else
                zt[q] += s;
            } else {
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const float e = fast_exp2(fmaf(acc[r], a.c, -mn));
                const bool vis = (mword >> acc_row(r, kg)) & 1u;
                zv[q] += vis ? e : 0.f;
                zt[q] += vis ? 0.f : e;
              }
            }
          } else {
            float t[16];
            const int p = a.T - a.W + qrow[q];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int j = jb + acc_row(r, kg);
              t[r] = (j < a.T && j <= p) ? acc[r] * a.c : kNegBig;
            }
            float bm = t[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) bm = fmaxf(bm, t[r]);
            const float mn = fmaxf(m[q], bm);
            const float sc = fast_exp2(m[q] - mn);
            zv[q] *= sc;
            zt[q] *= sc;
            m[q] = mn;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              // the exponent in the form pass B uses (one rounding, as in the plain path above): the probability of
              // a row's largest logit is then the same number in both passes, and a nearly one-hot row keeps its
              // normaliser consistent with its probabilities
              const float e = (t[r] > 0.5f * kNegBig) ? fast_exp2(fmaf(acc[r], a.c, -mn)) : 0.f;
              const bool vis = (mword >> acc_row(r, kg)) & 1u;
              zv[q] += vis ? e : 0.f;
              zt[q] += vis ? 0.f : e;
            }
          }
        }
      }
    }
  }

  // the two lane groups hold disjoint keys of the same query row: merge them, then store the partial
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (q < nvalid) {
      const float mo = __shfl_xor(m[q], 32, kWave);
      const float zvo = __shfl_xor(zv[q], 32, kWave);
      const float zto = __shfl_xor(zt[q], 32, kWave);
      const float M = fmaxf(m[q], mo);
      const float f1 = fast_exp2(m[q] - M), f2 = fast_exp2(mo - M);
      if (kg == 0 && qrow[q] < a.W) {
        const size_t row_id = (size_t)(l * a.Hq + qhead[q]) * a.stats_rows + a.stats_row0 + qrow[q];
        a.stats_part[row_id * a.NPART + ch * a.CS + cs] =
            make_float4(M, zv[q] * f1 + zvo * f2, zt[q] * f1 + zto * f2, 0.f);
      }
    }
  }
}

// Merges the partials of every (layer, query head, row of the statistics arrays): one thread per row, which walks
// its partials in order.  STAGED: a workgroup takes `rows` rows and first copies all their partials (contiguous) into
// LDS, all loads in flight together: with one load after the other the memory latency of every partial bound the
// kernel (32 partials 11 -> 6 us, 37 partials 25 -> 17 us; at 12 and 16 partials the staging costs more than it saves,
// 7 and 8 us without it, 14 and 11 us with it).
constexpr int kCombineThreads = 256;
constexpr int kCombineDirect = 16;
constexpr int kCombineStaged = 2048;  // partials of a workgroup in LDS (each row padded by one: its lanes spread over the banks)

template <bool STAGED>
__global__ void __launch_bounds__(kCombineThreads) stats_combine_kernel(ScoreArgs a, int rows) {
  __shared__ float4 staged[STAGED ? kCombineStaged + kCombineThreads : 1];
  const int total = a.L * a.Hq * a.stats_rows;
  const int idx0 = blockIdx.x * rows, idx = idx0 + threadIdx.x;
  const int n_part = a.NPART, pad = (n_part & 1) ^ 1;  // an odd number of 16-byte pieces per row
  const int row = idx % a.stats_rows;
  // the row's position in the sequence (row-block mode: one chunk of keys per row block, every partial of the row
  // exists; else the rows from W on are padding)
  const int position = a.blocks ? a.Tk - a.q_rows + row : a.T - a.W + row;
  uint8_t row_mask = 0;
  if ((int)threadIdx.x < rows && idx < total && (a.blocks || row < a.W))
    row_mask = a.mask[(size_t)(idx / (a.Hq * a.stats_rows) / a.Lseq) * a.Tk + position];
  if (STAGED) {
    const float4* src = a.stats_part + (size_t)idx0 * n_part;
    const int n = min(rows, total - idx0) * n_part;
    float4 v[kCombineStaged / kCombineThreads];
#pragma unroll
    for (int i = 0; i < kCombineStaged / kCombineThreads; ++i)
      if (i * kCombineThreads < n) v[i] = src[min((int)threadIdx.x + i * kCombineThreads, n - 1)];
#pragma unroll
    for (int i = 0; i < kCombineStaged / kCombineThreads; ++i)
      if ((int)threadIdx.x + i * kCombineThreads < n) {
        const unsigned at = threadIdx.x + i * kCombineThreads;
        staged[at + at / (unsigned)n_part * (unsigned)pad] = v[i];
      }
    __syncthreads();
  }
  if ((int)threadIdx.x >= rows || idx >= total) return;
  if (!a.blocks && row >= a.W) {  // padding rows of the window: no weight
    float* plane = reinterpret_cast<float*>(a.stats) + (size_t)(idx / a.stats_rows) * 4 * a.stats_rows + row;
    plane[0] = plane[(size_t)a.stats_rows] = plane[2 * (size_t)a.stats_rows] = plane[3 * (size_t)a.stats_rows] = 0.f;
    return;
  }
  const float4* part = STAGED ? staged + threadIdx.x * (n_part + pad) : a.stats_part + (size_t)idx * n_part;
  float M = kNegBig;
  for (int i = 0; i < n_part; ++i) M = fmaxf(M, part[i].x);
  float zv = 0.f, zt = 0.f;
  for (int i = 0; i < n_part; ++i) {
    const float4 p = part[i];
    const float f = fast_exp2(p.x - M);
    zv = fmaf(p.y, f, zv);
    zt = fmaf(p.z, f, zt);
  }
  const bool row_is_vision = row_mask != 0;
  const float coef_v = (!row_is_vision && zv > 0.f) ? 1.0f / zv : 0.f;  // text row: attends to vision columns
  const float coef_t = (row_is_vision && zt > 0.f) ? 1.0f / zt : 0.f;   // vision row: attends to text columns
  if (a.blocks) {
    // The statistics are stored as four planes of stats_rows values per (layer, head), so that pass B can copy the
    // values of a row block and a plane as one contiguous piece.  Row-block mode: the planes hold the form the inner
    // loop of that mode wants.  The probability of key j is
    // exp2(c * (q.k_j + bias)) with bias = -(M + log2 Z) / c, which pass B puts into the accumulators before the
    // matrix products; the cross-modal probability is that times Z / Z_cross (0 for rows of the wrong modality or
    // without cross-modal mass).
    const float z = zv + zt;
    float* plane = reinterpret_cast<float*>(a.stats) + (size_t)(idx / a.stats_rows) * 4 * a.stats_rows + row;
    plane[0] = -(M + __log2f(z)) / a.c;
    plane[(size_t)a.stats_rows] = (!row_is_vision && zv > 1e-30f) ? z / zv : 0.f;     // weight on vision columns
    plane[2 * (size_t)a.stats_rows] = (row_is_vision && zt > 1e-30f) ? z / zt : 0.f;  // weight on text columns
    plane[3 * (size_t)a.stats_rows] = 0.f;
  } else {
    // the window: row maximum, 1/Z, and the cross-modal 1/Z as the weight on vision and on text columns
    float* plane = reinterpret_cast<float*>(a.stats) + (size_t)(idx / a.stats_rows) * 4 * a.stats_rows + row;
    plane[0] = M;
    plane[(size_t)a.stats_rows] = 1.0f / (zv + zt);
    plane[2 * (size_t)a.stats_rows] = coef_v;
    plane[3 * (size_t)a.stats_rows] = coef_t;
  }
}

// ------------------------------------------------------------------------------------------ launch

template <typename T, int D, int NQ, int NW, bool BLOCKS>
static hipError_t launch_stats_b(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  const size_t lds = (size_t)kScoreTile * Tile<T, D>::kStride + kScoreTile;
  auto kern = score_stats_kernel<T, D, NQ, NW, BLOCKS>;
  if (lds > 64 * 1024) {
    hipError_t e = allow_dynamic_lds(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  // (row blocks along x: the device promises 65536 workgroups along y)
  const dim3 grid = BLOCKS ? dim3(p.Hkv * p.n_blocks_a, 1, p.L) : dim3(p.NCH, p.Hkv, p.L), block(NW * 64);
  hipLaunchKernelGGL(kern, grid, block, lds, s, a);
  return hipGetLastError();
}

template <typename T, int D, int NQ, int NW>
static hipError_t launch_stats_w(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  return p.blocks ? launch_stats_b<T, D, NQ, NW, true>(p, a, s) : launch_stats_b<T, D, NQ, NW, false>(p, a, s);
}

// With one query head per kv head and a window the pass streams the keys at the rate a plain read reaches, and three
// workgroups per CU of the small register-staged form do that best (up to four pairs of one head and a row block: one per
// wave); rows of 512 bytes take it in every mode.
template <typename T, int D>
static hipError_t launch_stats_d(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  if constexpr (Tile<T, D>::kRowBytes <= 256) {
    return launch_stats_b<T, D, 1, 4, false>(p, a, s);
  } else {
    const bool four = p.NCG * p.CS <= 4;
    switch (p.NQ) {
      case 1: return launch_stats_w<T, D, 1, 4>(p, a, s);
      case 2: return four ? launch_stats_w<T, D, 2, 4>(p, a, s) : launch_stats_w<T, D, 2, 8>(p, a, s);
      default: return launch_stats_w<T, D, 4, 8>(p, a, s);
    }
  }
}

hipError_t launch_score_stats(const Plan& p, const Buffers& b, hipStream_t s) {
  if (p.direct) return launch_score_stats_direct(p, b, s);
  if (score_stats_dma_supported(p)) return launch_score_stats_dma(p, b, s);
  const ScoreArgs a = make_args(p, b, true);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_stats_d<bf16_t, 128>(p, a, s) : launch_stats_d<bf16_t, 64>(p, a, s);
  return p.d == 128 ? launch_stats_d<float, 128>(p, a, s) : launch_stats_d<float, 64>(p, a, s);
}

hipError_t launch_stats_combine(const Plan& p, const Buffers& b, hipStream_t s) {
  if (p.direct) return hipSuccess;  // pass B merges the partials itself
  const ScoreArgs a = make_args(p, b);
  const int total = p.L * p.Hq * (p.blocks ? p.R : p.Wp);
  if (a.NPART > kCombineDirect && a.NPART <= kCombineStaged) {
    const int fit = kCombineStaged / a.NPART, rows = fit < kCombineThreads ? fit : kCombineThreads;
    hipLaunchKernelGGL((stats_combine_kernel<true>), dim3((total + rows - 1) / rows), dim3(kCombineThreads), 0, s, a, rows);
  } else {
    hipLaunchKernelGGL((stats_combine_kernel<false>), dim3((total + kCombineThreads - 1) / kCombineThreads),
                       dim3(kCombineThreads), 0, s, a, kCombineThreads);
  }
  return hipGetLastError();
}

}  // namespace meda
