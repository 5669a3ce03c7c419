// Both scoring passes for observation windows over few keys: launches that would leave most CUs without a workgroup when
// a workgroup of pass B walks all query heads against 128 keys (2 layers, 56 heads, 1198 keys: 94 us in 20 workgroups).
// Here every operand comes straight from memory (L2) into the fragments, no LDS tile and no barrier in the loops, and
// the work is cut finer: pass A into waves of one (head, 32-row block) pair and a chunk of keys, pass B into workgroups of
// 32 keys whose waves share the query heads.  Bound by latency: a wave's chain is a few blocks of 32 x 32.
// A lane owns one query row, as in pass A of score_stats_dma.hip; here in pass B too, so that the statistics of a row are one
// value per lane.
#include "score_common.hpp"

namespace meda {

// ------------------------------------------------------------------------------------------ pass A
// grid (NCH, Hkv * ceil(pairs / 4), L), 4 waves: wave w takes the (head of the group, row block) pair 4 y + w.
constexpr int kDirWavesA = 4;

template <typename T, int D>
__global__ void __launch_bounds__(kDirWavesA * 64) score_stats_direct_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_pairs = a.G * a.RB, per_head = (n_pairs + kDirWavesA - 1) / kDirWavesA;
  const int ch = blockIdx.x, g = blockIdx.y / per_head, l = blockIdx.z;
  const int pair = (blockIdx.y - g * per_head) * kDirWavesA + wave;
  if (pair >= n_pairs) return;
  const int hg = pair / a.RB, rb = pair - hg * a.RB;
  const int row = rb * 32 + n, head = g * a.G + hg;
  const int jbeg = ch * a.CH, jend = min(a.T, jbeg + a.CH);
  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;
  const char* kbase = a.k + (size_t)(l * a.Hkv + g) * a.Tk * TL::kRowBytes;
  auto load_keys = [&](Frag<T, D>& f, int jb) { frag_load(f, kbase + (size_t)min(jb + n, a.T - 1) * TL::kRowBytes, kg); };

  Frag<T, D> qf, kf;
  load_keys(kf, jbeg);
  uint8_t mk = mask[min(jbeg + n, a.T - 1)];
  // rows past the window repeat its last one (their partials are not stored)
  frag_load(qf, a.q + ((size_t)(l * a.Hq + head) * a.q_rows + a.q_row0 + min(row, a.W - 1)) * TL::kRowBytes, kg);
  float m = kNegBig, zv = 0.f, zt = 0.f;
  const int first_row = a.T - a.W + rb * 32;  // its position
  for (int jb = jbeg; jb < jend; jb += 32) {
    const uint32_t mword = (uint32_t)__ballot(mk != 0);
    f32x16_t acc = acc_zero();
    mma<T, D>(acc, kf, qf);
    if (pair == 0) {  // 1/|k| of the block's keys, by one wave of the kv head
      const float inv = inverse_norm(kf);
      if (kg == 0 && jb + n < jend) a.inv_norm[(size_t)(l * a.Hkv + g) * a.Tk + jb + n] = inv;
    }
    load_keys(kf, jb + 32);
    mk = mask[min(jb + 32 + n, a.T - 1)];
    if (jb + 31 <= first_row)
      stats_add_plain(acc, a.c, mword, kg, m, zv, zt);
    else
      stats_add_masked(acc, a.c, mword, kg, min(a.T - 1, first_row + n) - jb, m, zv, zt);
  }
  const float4 part = stats_merge_halves(m, zv, zt);
  if (kg == 0 && row < a.W)
    a.stats_part[((size_t)(l * a.Hq + head) * a.stats_rows + row) * a.NPART + ch] = part;
}

// ------------------------------------------------------------------------------------------ pass B
// grid (ceil(T / 32), L).  The waves take contiguous shares of the query heads.  Prologue: a wave merges the statistics
// partials of its own heads' rows (at most kDirParts of them, all requested at once) into LDS; workgroup 0 of a layer
// also stores them as the row statistics.  Then one product per (head, row block), the next query fragment in flight.
// Epilogue: the waves' shares of the head-averaged probabilities are added up in LDS, one row block after the other, a
// thread per element or two, which then takes its entropy term.
constexpr int kDirWavesB = 8;
constexpr int kDirThreadsB = kDirWavesB * 64;

static size_t direct_lds_bytes(int Hq, int RB) {  // row statistics, column sums per head, shares of one row block, reduction
  return (size_t)Hq * RB * 32 * 3 * 4 + (size_t)Hq * 32 * 4 + (size_t)kDirWavesB * 16 * 64 * 4 + kDirWavesB * 2 * 8;
}

template <typename T, int D, int RB>
__global__ void __launch_bounds__(kDirThreadsB) score_accum_direct_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  constexpr int Wp = RB * 32;
  extern __shared__ __align__(16) char smem[];
  float* st = reinterpret_cast<float*>(smem);              // [Hq][RB][3][32]: maximum, 1/Z, cross-modal 1/Z
  float* col = st + (size_t)a.Hq * RB * 96;                // [Hq][32]
  float* shares = col + a.Hq * 32;                         // [waves][16][64]
  double* red = reinterpret_cast<double*>(shares + kDirWavesB * 16 * 64);  // [waves][2]

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jw = blockIdx.x * 32, l = blockIdx.y;
  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;
  const int h_beg = wave * a.Hq / kDirWavesB, h_end = (wave + 1) * a.Hq / kDirWavesB;
  const char* kbase = a.k + ((size_t)l * a.Hkv * a.Tk + min(jw + n, a.T - 1)) * TL::kRowBytes;  // this lane's key, kv head 0
  const size_t kv_stride = (size_t)a.Tk * TL::kRowBytes;
  auto load_rows = [&](Frag<T, D>& f, int h, int rb) {
    frag_load(f, a.q + ((size_t)(l * a.Hq + h) * a.q_rows + a.q_row0 + min(rb * 32 + n, a.W - 1)) * TL::kRowBytes, kg);
  };
  for (int i = tid; i < a.Hq * 32; i += kDirThreadsB) col[i] = 0.f;
  bool row_vision[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) row_vision[rb] = mask[a.T - a.W + min(rb * 32 + n, a.W - 1)] != 0;
  const unsigned key_vision = (unsigned)__ballot(mask[min(jw + n, a.T - 1)] != 0);

  Frag<T, D> kf, qn;
  if (h_beg < h_end) {
    frag_load(kf, kbase + (size_t)(h_beg / a.G) * kv_stride, kg);
    load_rows(qn, h_beg, 0);
  }
  // the two lane groups take every other partial of a row
  for (int h = h_beg; h < h_end; ++h) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int row = rb * 32 + n;
      const float4* part = a.stats_part + ((size_t)(l * a.Hq + h) * a.stats_rows + min(row, a.W - 1)) * a.NPART;
      float4 p[kDirParts / 2];
#pragma unroll
      for (int i = 0; i < kDirParts / 2; ++i) p[i] = part[min(2 * i + kg, a.NPART - 1)];
      float M = kNegBig, zv = 0.f, zt = 0.f;
#pragma unroll
      for (int i = 0; i < kDirParts / 2; ++i) M = fmaxf(M, p[i].x);
      M = fmaxf(M, __shfl_xor(M, 32, kWave));
#pragma unroll
      for (int i = 0; i < kDirParts / 2; ++i) {
        const float f = 2 * i + kg < a.NPART ? fast_exp2(p[i].x - M) : 0.f;
        zv = fmaf(p[i].y, f, zv);
        zt = fmaf(p[i].z, f, zt);
      }
      zv += __shfl_xor(zv, 32, kWave);
      zt += __shfl_xor(zt, 32, kWave);
      const bool exists = row < a.W;
      const float rz = exists ? 1.0f / (zv + zt) : 0.f;
      const float cv = exists && !row_vision[rb] && zv > 0.f ? 1.0f / zv : 0.f;  // text row: weight on vision keys
      const float ct = exists && row_vision[rb] && zt > 0.f ? 1.0f / zt : 0.f;   // vision row: weight on text keys
      if (kg == 0) {
        float* s = st + (h * RB + rb) * 96 + n;
        s[0] = M;
        s[32] = rz;
        s[64] = cv + ct;
        if (blockIdx.x == 0) {
          float* plane = reinterpret_cast<float*>(a.stats) + (size_t)(l * a.Hq + h) * 4 * Wp + row;
          plane[0] = exists ? M : 0.f;
          plane[Wp] = rz;
          plane[2 * Wp] = cv;
          plane[3 * Wp] = ct;
        }
      }
    }
  }
  __syncthreads();  // col is zero, the wave's own statistics are in LDS

  float pbar[RB][16], colsum[16];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) pbar[rb][r] = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) colsum[r] = 0.f;
  // row `row` sees the wave's key i iff i <= T - W + row - jw
  for (int h = h_beg; h < h_end; ++h) {
    const int g = h / a.G;
    const bool last_of_run = h + 1 == h_end || (h + 1) / a.G != g;  // of this kv head in this wave
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const Frag<T, D> qf = qn;
      if (rb + 1 < RB)
        load_rows(qn, h, rb + 1);
      else if (h + 1 < h_end)
        load_rows(qn, h + 1, 0);
      const float* s = st + (h * RB + rb) * 96 + n;
      const float m = s[0], rz = s[32], coef = s[64];
      f32x16_t acc = acc_zero();
      mma<T, D>(acc, kf, qf);
      if (rb == RB - 1 && last_of_run && h + 1 < h_end) frag_load(kf, kbase + (size_t)(g + 1) * kv_stride, kg);
      const int seen = rb * 32 + n < a.W ? min(a.T - 1, a.T - a.W + rb * 32 + n) - jw - kg * 4 : -1;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float e = fast_exp2(fmaf(acc[r], a.c, -m));
        e = acc_row(r, 0) <= seen ? e : 0.f;
        colsum[r] = fmaf(e, rz, colsum[r]);
        pbar[rb][r] = fmaf(e, coef, pbar[rb][r]);
      }
    }
    if (last_of_run) {
      const float tot = reduce_lanes32(colsum, lane);  // of the key in register n / 2
      if ((n & 1) == 0) col[h * 32 + acc_row(n >> 1, kg)] = tot;
#pragma unroll
      for (int r = 0; r < 16; ++r) colsum[r] = 0.f;
    }
  }

  // Entropy terms of the head-averaged cross-modal probabilities: text rows on vision keys, vision rows on text keys.
  const float inv_heads = 1.0f / (float)a.Hq;
  float s_tv = 0.f, s_vt = 0.f;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (rb > 0) __syncthreads();  // the previous row block's shares are no longer read
#pragma unroll
    for (int r = 0; r < 16; ++r) shares[(wave * 16 + r) * 64 + lane] = pbar[rb][r];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16 / kDirWavesB; ++i) {
      const int r = wave * (16 / kDirWavesB) + i;  // this wave's registers; the lane is the shares' lane
      float p = 0.f;
#pragma unroll
      for (int w = 0; w < kDirWavesB; ++w) p += shares[(w * 16 + r) * 64 + lane];
      p *= inv_heads;
      const bool vision = ((key_vision >> acc_row(r, kg)) & 1u) != 0;
      const float t = (p > 0.f && vision != row_vision[rb]) ? p * __logf(p) : 0.f;
      s_tv += vision ? t : 0.f;
      s_vt += vision ? 0.f : t;
    }
  }
  const double tv = wave_sum((double)s_tv), vt = wave_sum((double)s_vt);
  if (lane == 0) {
    red[wave * 2 + 0] = tv;
    red[wave * 2 + 1] = vt;
  }
  __syncthreads();
  for (int i = tid; i < a.Hkv * 32; i += kDirThreadsB) {  // column scores: the runs of a kv head in head order
    const int g = i >> 5, c = i & 31;
    float sum = 0.f;
    for (int hg = 0; hg < a.G; ++hg) sum += col[(g * a.G + hg) * 32 + c];
    if (jw + c < a.T) a.col_scores[(size_t)(l * a.Hkv + g) * a.Tk + jw + c] = sum;
  }
  if (tid < 2) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kDirWavesB; ++w) sum += red[w * 2 + tid];
    a.ent_part[((size_t)l * a.NTk + blockIdx.x) * 2 + tid] = -sum;
  }
}

// ------------------------------------------------------------------------------------------ launch

template <typename T, int D>
static hipError_t launch_stats_t(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  const int groups = (p.G * p.RB + kDirWavesA - 1) / kDirWavesA;
  hipLaunchKernelGGL((score_stats_direct_kernel<T, D>), dim3(p.NCH, p.Hkv * groups, p.L), dim3(kDirWavesA * 64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_score_stats_direct(const Plan& p, const Buffers& b, hipStream_t s) {
  const ScoreArgs a = make_args(p, b, true);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_stats_t<bf16_t, 128>(p, a, s) : launch_stats_t<bf16_t, 64>(p, a, s);
  return p.d == 128 ? launch_stats_t<float, 128>(p, a, s) : launch_stats_t<float, 64>(p, a, s);
}

template <typename T, int D, int RB>
static hipError_t launch_accum_k(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  const size_t lds = direct_lds_bytes(p.Hq, RB);
  auto kern = score_accum_direct_kernel<T, D, RB>;
  if (lds > 64 * 1024) {
    hipError_t e = allow_dynamic_lds(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(p.NTk, p.L), dim3(kDirThreadsB), lds, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_accum_t(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  switch (p.RB) {
    case 1: return launch_accum_k<T, D, 1>(p, a, s);
    case 2: return launch_accum_k<T, D, 2>(p, a, s);
    case 3: return launch_accum_k<T, D, 3>(p, a, s);
    default: return launch_accum_k<T, D, 4>(p, a, s);
  }
}

hipError_t launch_score_accum_direct(const Plan& p, const Buffers& b, hipStream_t s) {
  const ScoreArgs a = make_args(p, b);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_accum_t<bf16_t, 128>(p, a, s) : launch_accum_t<bf16_t, 64>(p, a, s);
  return p.d == 128 ? launch_accum_t<float, 128>(p, a, s) : launch_accum_t<float, 64>(p, a, s);
}

}  // namespace meda
