// Layer budgets from the cross-modal entropies (Section 3.2 allocation equation, Appendix A.3,
// Section 4.3 for the recent : important split) and per-head token selection (Section 3.3: text
// prior, recent window, Top-N).
#include "device_utils.hpp"
#include "plan.hpp"

namespace meda {

// ------------------------------------------------------------------------------------ allocation
struct AllocArgs {
  const double* ent_part;  // [L][NT][2]: minus sum p log p over text rows / vision rows, per column tile
  const uint8_t* mask;
  int32_t* alloc;          // [L][4]: S, M, N, 0
  int64_t* off;            // [L+1]
  int32_t* layer_len;      // user outputs
  int64_t* layer_off;
  double* entropy;         // may be null
  int L, NT, T, W, R, num, den, flags;   // L layers and budget B of ONE sequence; W: recent window; R: scoring rows
  int N;                                 // sequences (one workgroup each)
  long long B;
};

__device__ __forceinline__ double clampd(double v, double lo, double hi) { return fmin(fmax(v, lo), hi); }

// One workgroup per sequence.  S_l = B * softmax_l(E_CM) when no bound is active; shares are kept inside
// [min(W,T), T] by water-filling (x_l = clamp(lambda * w_l), sum x_l = B) and rounded by largest
// remainder, so that sum_l S_l = B exactly.  All real arithmetic is double precision.
__global__ void __launch_bounds__(1024) allocate_kernel(AllocArgs a) {
  __shared__ double E[kMaxLayers], w[kMaxLayers], frac[kMaxLayers];
  __shared__ double kink[2 * kMaxLayers], filled[2 * kMaxLayers];
  __shared__ int S[kMaxLayers], order[kMaxLayers];
  __shared__ double s_lambda;
  const int tid = threadIdx.x, lane = tid & 63, L = a.L;
  const double lo = (double)min(a.W, a.T), hi = (double)a.T, B = (double)a.B;
  // sequence n: its layers are the layers n*L .. n*L + L-1 of the batch, its output rows start at n*B
  const int n = blockIdx.x;
  a.ent_part += (size_t)n * L * a.NT * 2;
  a.mask += (size_t)n * a.T;
  if (a.entropy) a.entropy += (size_t)n * L;

  // scoring rows of each modality (the denominators of the two entropy means)
  int n_vis = 0;
  for (int r0 = 0; r0 < a.R; r0 += blockDim.x)
    n_vis += __syncthreads_count(r0 + tid < a.R && a.mask[a.T - a.R + r0 + tid] != 0);
  const int n_text = a.R - n_vis;
  // per-tile entropy partials of a layer are summed by one wave (lanes stride over the tiles)
  for (int l = tid >> 6; l < L; l += blockDim.x >> 6) {
    const double2* p = reinterpret_cast<const double2*>(a.ent_part + (size_t)l * a.NT * 2);
    double tv = 0.0, vt = 0.0;
#pragma unroll 4
    for (int t = lane; t < a.NT; t += 64) {
      const double2 v = p[t];
      tv += v.x;
      vt += v.y;
    }
    tv = wave_sum(tv);
    vt = wave_sum(vt);
    if (lane == 0) {
      const double e = (n_text ? tv / n_text : 0.0) + (n_vis ? vt / n_vis : 0.0);
      E[l] = e;
      if (a.entropy) a.entropy[l] = e;
    }
  }
  __syncthreads();

  // From here on the kernel is a chain of short steps over L values, bound by the latency of LDS and of the fp64
  // operations: everything that can be is done by a wave (reductions over the lanes) or by a thread per value (32
  // layers: 22 -> 11 us against one thread walking the kinks and the remainders).
  const bool uniform = (a.flags & MEDA_FLAG_UNIFORM_BUDGET) != 0;
  if (tid < L) {
    double emax = E[0];
#pragma unroll 8
    for (int i = 1; i < L; ++i) emax = fmax(emax, E[i]);
    w[tid] = uniform ? 1.0 : exp(E[tid] - emax);
  }
  __syncthreads();
  // the filled amount sum_l clamp(lambda w_l) is piecewise linear in lambda with kinks at lo/w and hi/w
  for (int i = tid; i < 2 * L; i += blockDim.x) {
    const double b = (i < L) ? lo / w[i] : hi / w[i - L];
    double f = 0.0;
#pragma unroll 8
    for (int j = 0; j < L; ++j) f += clampd(b * w[j], lo, hi);
    kink[i] = b;
    filled[i] = f;
  }
  __syncthreads();
  if (tid < 64) {  // first kink at or above the budget, last one below it
    double upper = INFINITY, lower = 0.0;
    for (int i = lane; i < 2 * L; i += 64) {
      const double k = kink[i];
      if (filled[i] >= B) upper = fmin(upper, k);
      else lower = fmax(lower, k);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      upper = fmin(upper, __shfl_xor(upper, o, kWave));
      lower = fmax(lower, __shfl_xor(lower, o, kWave));
    }
    if (upper == INFINITY) upper = -1.0;
    const double mid = 0.5 * (lower + upper);
    double wsum = 0.0;
    int n_lo = 0, n_hi = 0;
    for (int j = lane; j < L; j += 64) {
      const double v = mid * w[j];
      if (v <= lo) ++n_lo;
      else if (v >= hi) ++n_hi;
      else wsum += w[j];
    }
    wsum = wave_sum(wsum);
    n_lo = wave_sum(n_lo);
    n_hi = wave_sum(n_hi);
    if (lane == 0) s_lambda = (wsum > 0.0) ? (B - lo * n_lo - hi * n_hi) / wsum : upper;
  }
  __syncthreads();
  if (tid < L) {
    double xv = clampd(s_lambda * w[tid], lo, hi);
    if (a.B == (long long)L * a.T) xv = hi;
    if (a.B == (long long)L * min(a.W, a.T)) xv = lo;
    const double fl = floor(xv);
    frac[tid] = xv - fl;
    S[tid] = (int)clampd(fl, lo, hi);
  }
  __syncthreads();
  if (tid < L) {
    int rank = 0;
    const double f = frac[tid];
#pragma unroll 8
    for (int j = 0; j < L; ++j) rank += (frac[j] > f || (frac[j] == f && j < tid)) ? 1 : 0;
    order[rank] = tid;  // decreasing fractional part, ties towards the lower layer
  }
  __syncthreads();
  if (tid < 64) {
    long long sum = 0;
    bool full = false;  // a layer that cannot take another slot
    for (int j = lane; j < L; j += 64) {
      sum += S[j];
      full = full || S[j] >= a.T;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    long long rest = a.B - sum;
    if (rest >= 0 && rest <= L && __ballot(full) == 0ull) {
      // the usual case: the first `rest` layers of the order take one slot each
      for (int r = lane; r < (int)rest; r += 64) ++S[order[r]];
    } else if (lane == 0) {
      for (int round = 0; round < 4 && rest > 0; ++round)
        for (int r = 0; r < L && rest > 0; ++r) {
          const int lyr = order[r];
          if (S[lyr] < a.T) { ++S[lyr]; --rest; }
        }
      for (int round = 0; round < 4 && rest < 0; ++round)  // only reachable through rounding fuzz
        for (int r = L - 1; r >= 0 && rest < 0; --r) {
          const int lyr = order[r];
          if (S[lyr] > min(a.W, a.T)) { --S[lyr]; ++rest; }
        }
    }
  }
  __syncthreads();
  if (tid < L) {
    const int s = S[tid];
    const int m = max(min(a.W, s), (int)(((long long)s * a.num) / a.den));
    long long o = (long long)n * a.B;
    // layers ranked by decreasing budget (ties: lower layer first), for kernels that launch the
    // longest workgroups first; in a batch the ranks of the sequences are interleaved (rank r of
    // sequence n is entry r*N + n), which keeps the order of one sequence and is decreasing on average
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < L; ++j) {
      const int sj = S[j];
      o += j < tid ? sj : 0;
      rank += (sj > s || (sj == s && j < tid)) ? 1 : 0;
    }
    const int lv = n * L + tid;  // layer of the batch
    a.alloc[4 * lv + 0] = s;
    a.alloc[4 * lv + 1] = m;
    a.alloc[4 * lv + 2] = s - m;
    a.alloc[4 * (rank * a.N + n) + 3] = lv;
    a.off[lv] = o;
    a.layer_len[lv] = s;
    a.layer_off[(size_t)n * (L + 1) + tid] = o;
    if (tid == L - 1) {
      if (n == a.N - 1) a.off[(size_t)a.N * L] = o + s;
      a.layer_off[(size_t)n * (L + 1) + L] = o + s;
    }
  }
}

// ------------------------------------------------------------------------------------- selection
struct SelectArgs {
  const float* col_scores;  // [L][Hkv][T]
  const uint8_t* mask;
  const int32_t* alloc;
  const int64_t* off;
  int32_t* sel_idx;         // ragged [B*Hkv]: row ids (l*Hkv+g)*T + position
  float* sel_inv_norm;      // ragged [B*Hkv]: 1/|k| of every conserved key
  const float* inv_norm;    // [L][Hkv][T]
  int32_t* sel_idx_user;    // may be null
  int32_t* less_idx;        // ragged [(L*T-B)*Hkv]: row ids
  int32_t* merge_assign;    // may be null, [L][Hkv][T]
  int L, Hkv, T, no_merge;
  int Lseq;                 // layers per sequence (the mask is per sequence)
  const char* k;            // the keys, row_bytes each (COPIES)
  int row_bytes;
};

constexpr int kSelMaxThreads = 1024;
constexpr int kSelMaxWaves = kSelMaxThreads / 64;

template <int BITS>
struct SelectShared {
  int hist[2][1 << BITS];     // text, vision (the later digits use the first half)
  int wsum[2][kSelMaxWaves];
  int bin, rest;
};

// Copies of a key (COPIES, fp32 keys that are to be merged): of the conserved keys that are equal bit for bit the lowest
// slot stands for all in the similarity search, the 1/|k| of the others becomes kNoSlot.  They are found by their equal
// 1/|k|: an entry of the table holds the smallest (bits of 1/|k|, position) that falls on it.  A copy is missed where a key
// with a smaller 1/|k| falls on its entry and where a workgroup finds more than kMaxCopies candidates; the search then
// decides that tie by itself, which costs time and nothing else.
constexpr int kCopyEntries = 2048, kMaxCopies = 512;
struct CopyShared {
  unsigned long long first[kCopyEntries];
  int at[kMaxCopies], of[kMaxCopies], slot[kMaxCopies];  // positions of a candidate and of its first, its slot
  int n;
};
__device__ __forceinline__ unsigned copy_entry(unsigned inv_bits) { return inv_bits * 2654435769u >> 21; }
static_assert(kCopyEntries == 1 << (32 - 21), "the shift leaves the bits of an entry");

// The digit of the `want`-th largest key of a histogram (want >= 1, at most the histogram's total) and how many of
// that digit's keys are still wanted.  Every thread takes the same number of adjacent bins, from the top.
template <int BITS>
__device__ __forceinline__ void find_digit(SelectShared<BITS>& sh, const int* hist, int want) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
  const int per = (1 << BITS) / (int)blockDim.x, top = (1 << BITS) - 1 - tid * per;
  int own = 0;
  for (int b = 0; b < per; ++b) own += hist[top - b];
  int inc = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += t;
  }
  if (lane == 63) sh.wsum[0][wave] = inc;
  __syncthreads();
  int before = inc - own;
  for (int w = 0; w < n_waves; ++w) before += w < wave ? sh.wsum[0][w] : 0;
  if (before < want && before + own >= want) {
    int bin = top;
    while (before + hist[bin] < want) before += hist[bin--];
    sh.bin = bin;
    sh.rest = want - before;
  }
  __syncthreads();
}

// grid (Hkv, L).  Adding max(A_s) to every text score puts all text candidates above all vision
// candidates and keeps the order inside each modality, so the Top-N of the boosted scores is:
// all text candidates plus the best vision ones if N exceeds the number of text candidates, else
// the best N text candidates.  The order inside one modality is found exactly on the unboosted
// fp32 scores (no bits are lost to the addition) with a radix select over their bit patterns, 11 + 11 + 10 bits or four
// times 8 for short prompts (scores are >= 0, so the unsigned order of the bits is the order of the values); equal scores go to the smaller
// position.  The first sweep counts both modalities, so the number of text candidates needs no sweep of its own.
//
// Bound by the latency of its sweeps and, before, by histogram atomics: with 8-bit digits the first one (two octaves
// of score per bin) put nearly all of a wave's adds on one or two addresses.  A wave takes ITEMS x 64 consecutive
// positions per iteration, lane by lane (loads and stores coalesced, ranks from ballots).  Up to ITEMS positions per
// thread (SINGLE) the scores are read once and stay in registers.  One barrier per iteration of the output sweep:
// the positions a tie may take before p are min(ties before p, ties taken), so one prefix over (certain, tied)
// counts places everything.  Before and now, in us: 256 (layer, head) pairs of 131072 positions 370 / 233, 112 of 37376
// 92 / 64, 256 of 16384 45 / 32, 1024 of 4096 31 / 29, 360 of 3001 23 / 16.5, 256 of 300 and of 100 11 / 10 and 10 / 9.4.
template <int ITEMS, bool SINGLE, int BITS, bool COPIES>
__global__ void __launch_bounds__(kSelMaxThreads) select_kernel(SelectArgs a) {
  constexpr int kBins = 1 << BITS;
  __shared__ SelectShared<BITS> sh;
  struct Nothing {};
  __shared__ std::conditional_t<COPIES, CopyShared, Nothing> copies;
  const int g = blockIdx.x, l = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_thr = blockDim.x, n_waves = n_thr >> 6;
  const int T = a.T;
  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * T;  // this layer's sequence
  const int S = a.alloc[4 * l + 0], M = a.alloc[4 * l + 1], N = a.alloc[4 * l + 2];
  const int ncand = T - M;
  const long long off_l = a.off[l];
  const int head_row0 = (l * a.Hkv + g) * T;  // row id of position 0 of this (layer, head)
  const float* scores = a.col_scores + (size_t)head_row0;
  const size_t c_base = (size_t)off_l * a.Hkv + (size_t)g * S;
  const size_t less_base = ((size_t)l * T - (size_t)off_l) * a.Hkv + (size_t)g * (T - S);

  const int span = ITEMS * n_thr;           // positions per iteration of the workgroup
  const int w0 = wave * ITEMS * 64 + lane;  // this lane's first position of an iteration
  unsigned key[ITEMS];
  uint8_t mk[ITEMS];
  auto load = [&](int base) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = min(base + w0 + i * 64, T - 1);
      mk[i] = mask[j];
      key[i] = __float_as_uint(scores[j]);
    }
  };
  // f(position, key, class) for every candidate
  auto sweep = [&](auto f) {
    for (int base = 0; base < ncand; base += span) {
      if (!SINGLE) load(base);
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (base + w0 + i * 64 < ncand) f(key[i], mk[i] != 0 ? 1 : 0);
    }
  };
  if (SINGLE) load(0);

  if constexpr (COPIES) {  // published by the barriers of the sweeps
    for (int b = tid; b < kCopyEntries; b += n_thr) copies.first[b] = ~0ull;
    if (tid == 0) copies.n = 0;
  }
  for (int b = tid; b < 2 * kBins; b += n_thr) (&sh.hist[0][0])[b] = 0;
  __syncthreads();
  sweep([&](unsigned k, int c) { atomicAdd(&sh.hist[c][k >> (32 - BITS)], 1); });
  __syncthreads();
  int n_text = 0;
  for (int b = tid; b < kBins; b += n_thr) n_text += sh.hist[0][b];
  n_text = wave_sum(n_text);
  if (lane == 0) sh.wsum[1][wave] = n_text;
  __syncthreads();
  n_text = 0;
  for (int w = 0; w < n_waves; ++w) n_text += sh.wsum[1][w];

  const bool pick_text = N <= n_text;            // class in which the cut falls
  const int K = pick_text ? N : N - n_text;      // how many of that class are taken
  const bool other_taken = !pick_text;           // vision cut: every text candidate is taken
  const int cls = pick_text ? 0 : 1;

  unsigned threshold = 0xffffffffu;
  int ties_taken = 0;
  if (K > 0) {
    find_digit(sh, sh.hist[cls], K);
    unsigned prefix = (unsigned)sh.bin;
    int want = sh.rest;
#pragma unroll
    for (int left = 32 - BITS; left > 0; left -= BITS) {
      const int bits = left < BITS ? left : BITS, shift = left - bits;
      for (int b = tid; b < kBins; b += n_thr) sh.hist[0][b] = 0;
      __syncthreads();
      sweep([&](unsigned k, int c) {
        if (c == cls && (k >> (shift + bits)) == prefix) atomicAdd(&sh.hist[0][(k >> shift) & ((1u << bits) - 1u)], 1);
      });
      __syncthreads();
      find_digit(sh, sh.hist[0], want);
      prefix = (prefix << bits) | (unsigned)sh.bin;
      want = sh.rest;
    }
    threshold = prefix;
    ties_taken = want;
  }

  // ordered output: conserved positions ascending, the rest ascending
  int run_sure = 0, run_tie = 0;  // certain and tied positions before this iteration
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  float inv[ITEMS];
  auto load_inv = [&](int base) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) inv[i] = a.inv_norm[head_row0 + min(base + w0 + i * 64, T - 1)];
  };
  int buf = 0;
  for (int base = 0; base < T; base += span, buf ^= 1) {
    if (!SINGLE) load(base);
    load_inv(base);
    unsigned long long sure[ITEMS], tie[ITEMS];  // uniform over the wave
    int n_sure = 0, n_tie = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = base + w0 + i * 64;
      const bool cand = j < ncand, in_cls = (mk[i] != 0 ? 1 : 0) == cls;
      sure[i] = __ballot(j < T && (!cand || (in_cls ? key[i] > threshold : other_taken)));
      tie[i] = __ballot(cand && in_cls && key[i] == threshold);
      n_sure += __popcll(sure[i]);
      n_tie += __popcll(tie[i]);
    }
    if (lane == 0) sh.wsum[buf][wave] = n_sure | (n_tie << 16);  // at most 16384 positions per iteration
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < n_waves; ++w) {
      const int v = sh.wsum[buf][w];
      before += w < wave ? v : 0;
      total += v;
    }
    int sure_b = run_sure + (before & 0xffff), tie_b = run_tie + (before >> 16);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = base + w0 + i * 64;
      const int my_tie = tie_b + __popcll(tie[i] & lt_mask);
      const int pos_c = sure_b + __popcll(sure[i] & lt_mask) + min(my_tie, ties_taken);  // conserved positions before j
      const bool sel = ((sure[i] >> lane) & 1ull) || (((tie[i] >> lane) & 1ull) && my_tie < ties_taken);
      if (sel) {
        a.sel_idx[c_base + pos_c] = head_row0 + j;
        a.sel_inv_norm[c_base + pos_c] = inv[i];
        if constexpr (COPIES) {
          const unsigned bits = __float_as_uint(inv[i]);
          atomicMin(&copies.first[copy_entry(bits)], (unsigned long long)bits << 32 | (unsigned)j);
        }
        if (a.sel_idx_user) a.sel_idx_user[c_base + pos_c] = j;
        if (a.merge_assign) a.merge_assign[head_row0 + j] = pos_c;
      } else if (j < T) {
        a.less_idx[less_base + (j - pos_c)] = head_row0 + j;
        if (a.merge_assign && a.no_merge) a.merge_assign[head_row0 + j] = -1;
      }
      sure_b += __popcll(sure[i]);
      tie_b += __popcll(tie[i]);
    }
    run_sure += total & 0xffff;
    run_tie += total >> 16;
  }
  if constexpr (COPIES) {
    __syncthreads();  // the table and this workgroup's sel_idx, sel_inv_norm are complete
    for (int slot = tid; slot < S; slot += n_thr) {
      const unsigned bits = __float_as_uint(a.sel_inv_norm[c_base + slot]);
      const int j = a.sel_idx[c_base + slot] - head_row0;
      const unsigned long long first = copies.first[copy_entry(bits)];
      if ((unsigned)(first >> 32) != bits || (int)(unsigned)first == j) continue;
      const int n = atomicAdd(&copies.n, 1);
      if (n >= kMaxCopies) break;
      copies.at[n] = j;
      copies.of[n] = (int)(unsigned)first;
      copies.slot[n] = slot;
    }
    __syncthreads();
    const int pieces = a.row_bytes / 16, piece = tid % pieces;  // 16 or 32 adjacent lanes compare two keys
    const char* keys = a.k + (size_t)head_row0 * a.row_bytes + piece * 16;
    const int n_copies = min(copies.n, kMaxCopies);
    for (int i = tid / pieces; i < n_copies; i += n_thr / pieces) {
      const uint4 x = *reinterpret_cast<const uint4*>(keys + (size_t)copies.at[i] * a.row_bytes);
      const uint4 y = *reinterpret_cast<const uint4*>(keys + (size_t)copies.of[i] * a.row_bytes);
      unsigned differ = (x.x ^ y.x) | (x.y ^ y.y) | (x.z ^ y.z) | (x.w ^ y.w);
      for (int o = pieces / 2; o > 0; o >>= 1) differ |= __shfl_xor((int)differ, o, kWave);
      if (piece == 0 && differ == 0) a.sel_inv_norm[c_base + copies.slot[i]] = __uint_as_float(kNoSlot);
    }
  }
}

// ------------------------------------------------------------------------------------------ launch

hipError_t launch_allocate(const Plan& p, const Buffers& b, hipStream_t s) {
  AllocArgs a;
  a.ent_part = reinterpret_cast<const double*>(b.ws + p.off_ent_part);
  a.mask = b.mask;
  a.alloc = reinterpret_cast<int32_t*>(b.ws + p.off_alloc);
  a.off = reinterpret_cast<int64_t*>(b.ws + p.off_layer_off);
  a.layer_len = b.layer_len;
  a.layer_off = b.layer_off;
  a.entropy = b.entropy;
  a.L = p.Lseq; a.NT = p.NTk; a.T = p.T; a.W = p.W; a.R = p.R; a.num = p.num; a.den = p.den; a.flags = p.flags;
  a.N = p.N;
  a.B = p.B / p.N;
  hipLaunchKernelGGL(allocate_kernel, dim3(p.N), dim3(1024), 0, s, a);  // 16 waves share the per-layer sums of the entropy partials
  return hipGetLastError();
}

hipError_t launch_select(const Plan& p, const Buffers& b, hipStream_t s) {
  SelectArgs a;
  a.col_scores = reinterpret_cast<const float*>(b.ws + p.off_col_scores);
  a.mask = b.mask;
  a.alloc = reinterpret_cast<const int32_t*>(b.ws + p.off_alloc);
  a.off = reinterpret_cast<const int64_t*>(b.ws + p.off_layer_off);
  a.sel_idx = reinterpret_cast<int32_t*>(b.ws + p.off_sel_idx);
  a.sel_inv_norm = reinterpret_cast<float*>(b.ws + p.off_sel_inv);
  a.inv_norm = reinterpret_cast<const float*>(b.ws + p.off_inv_norm);
  a.sel_idx_user = b.sel_idx_user;
  a.less_idx = reinterpret_cast<int32_t*>(b.ws + p.off_less_idx);
  a.merge_assign = b.merge_assign;
  a.L = p.L; a.Hkv = p.Hkv; a.T = p.T; a.no_merge = (p.flags & MEDA_FLAG_NO_MERGE) ? 1 : 0;
  a.Lseq = p.Lseq;
  a.k = static_cast<const char*>(b.k);
  a.row_bytes = p.d * p.elt;
  const dim3 grid(p.Hkv, p.L);
  // Short prompts: one sweep costs less than clearing and searching 2048 bins, so 8-bit digits and as few positions per
  // thread as cover the prompt (256 pairs of 300 positions 12.1 -> 10.1 us, 1024 pairs 16.4 -> 12.1).  Longer ones: the
  // workgroup is as large as the CUs can hold for the number of pairs (of 1024 threads a CU holds one): 1024 pairs of
  // 4100 positions 57 us with 1024 threads, 37 with 512, 34 with 256, but 256 pairs 18.4, 18.7 and 22 us.  From 8192
  // positions on the scores are read again in every sweep (8 registers of them per thread hide the loads as well).
  const int pairs = p.L * p.Hkv;
  auto launch = [&](auto copies_tag) {
    constexpr bool C = decltype(copies_tag)::value;
    if (p.T <= 256) hipLaunchKernelGGL((select_kernel<1, true, 8, C>), grid, dim3(256), 0, s, a);
    else if (p.T <= 512) hipLaunchKernelGGL((select_kernel<2, true, 8, C>), grid, dim3(256), 0, s, a);
    else if (p.T <= 1024) hipLaunchKernelGGL((select_kernel<4, true, 8, C>), grid, dim3(256), 0, s, a);
    else if (p.T <= 2048 && pairs <= 512) hipLaunchKernelGGL((select_kernel<4, true, 11, C>), grid, dim3(512), 0, s, a);
    else if (p.T <= 2048) hipLaunchKernelGGL((select_kernel<8, true, 11, C>), grid, dim3(256), 0, s, a);
    else if (p.T <= 4096) hipLaunchKernelGGL((select_kernel<8, true, 11, C>), grid, dim3(512), 0, s, a);
    else if (p.T <= 8192 && pairs <= 256) hipLaunchKernelGGL((select_kernel<8, true, 11, C>), grid, dim3(1024), 0, s, a);
    else {
      const int n_thr = pairs <= 256 ? (p.T < 16384 ? 512 : 1024) : (pairs > 512 && p.T <= 16384 ? 256 : 512);
      hipLaunchKernelGGL((select_kernel<8, false, 11, C>), grid, dim3(n_thr), 0, s, a);
    }
  };
  if (p.sim == kSimSplit && !a.no_merge) launch(std::true_type{});
  else launch(std::false_type{});
  return hipGetLastError();
}

}  // namespace meda
