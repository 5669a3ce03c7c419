// One decoding step over the ragged compressed cache: out = Softmax(q K^T / sqrt(d)) V per layer and
// query head (Section 3.1, "Decoding with Multimodal KV Cache"), the cache being the rows the
// compression pass kept for the layer (S_l per kv head, Section 3.2) followed by the rows appended
// since (K = [K, k_t], V = [V, v_t]).
//
// The step reads every cached key and value once and does 4*G*d flops per (key, value) pair, so it is bound by HBM
// as long as the instructions per byte stay few: fp32 caches take a plain streaming kernel on the vector unit, bf16
// and 8-bit caches put both products on the matrix unit.  The rows of every (layer, kv head) are cut into chunks of
// about the same size over all layers (budgets differ by more than a factor of ten between layers); one workgroup
// takes one chunk for all G query heads of the group (flash-decoding style: a running maximum, normaliser and
// weighted value sum per head), a second small kernel merges the chunks.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "../../include/meda.h"
#include "device_utils.hpp"
#include "fp8.hpp"

namespace meda {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
// Rows per chunk: the rows of the whole cache over kDecTargetGroups workgroups (256 CUs, three workgroups each, two
// rounds), between one step of a workgroup's four waves and a size that bounds the unevenness.  Measured over 524288
// bf16 rows (one head per kv head) with 1024 / 1536 / 2048 / 3072 workgroups: 52 / 48 / 52 / 52 us; over 838856 8-bit
// rows: 53 / 50 / 51 / 53 us.
constexpr int kDecTargetGroups = 1536;
constexpr int kDecMinRows = 128, kDecMaxRows = 2048;
// So many appended rows ride with the layer's last chunk instead of chunks of their own.  fp32 rows take longer: 32 layers
// of 64 rows, one kv head and eight query heads, 128 appended rows: bf16 16 us either way, fp32 21.8 with the last chunk
// and 17.9 as chunks of their own; 32 appended rows 16 us either way, after longer chunks 7 % less with the last one.
constexpr int kDecInlineNew = 128, kDecInlineNewF32 = 32;
constexpr int kDecMaxSplit = 64;  // average number of chunks per layer, at most

struct DecodeArgs {
  const char* q;            // [L][Hq][d]
  const char* k_cache;      // ragged, layer l at row off[l]*Hkv: [Hkv][S_l][d]
  const char* v_cache;
  const int32_t* layer_len; // [L]   S_l
  const int64_t* layer_off; // [L+1]
  const char* k_new;        // [L][Hkv][n_new][d] or null
  const char* v_new;
  char* out;                // [L][Hq][d]
  float* part;              // [NC + L*NSN][Hq][d + 2]: weighted value sum, maximum (base-2 logits), normaliser
  int L, Hq, Hkv, G, n_new;
  unsigned R, R_inv;        // rows per chunk aimed at, floor(2^32 / R)
  int NC, NSN;              // chunk ids of the cached rows (at most), chunks of a layer's appended rows
  float scale_log2;
  // 8-bit cache (FP8 instantiation): k_cache / v_cache hold E4M3 codes, one scale per row
  const float* k_scale;     // [B*Hkv]
  const float* v_scale;
};

// The chunks of the cached rows are numbered layer after layer: layer l has ceil(S_l / R) of them, at least one.  The host sizes
// the launch for NC ids, at least floor(B / R) + L in general, which bounds their number for S_1 + .. + S_L <= B; should
// the lengths exceed B, R is doubled until they fit (every workgroup computes the same R).  Evaluated by every wave on its own.
struct LayerChunks {
  int layer;      // the layer asked for, or the one that owns the chunk id asked for (-1: id past the last chunk)
  int first;      // id of its first chunk
  int n;          // its number of chunks
  int rows;       // S_l
  long long off;  // layer_off[layer]
};
// Inclusive sum over the lanes of the wave (data-parallel primitives, no LDS traffic).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8: inside the rows of 16
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // lane 15 of rows 0, 2 to rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2, 3
  return v;
}
// max(1, ceil(s / R)), inv = floor(2^32 / R): the estimate is the quotient or one less.  (A division here was most of
// what the search cost with many layers: every workgroup of both kernels walks them all.)
__device__ __forceinline__ int chunks_of(int s, unsigned R, unsigned inv) {
  const unsigned x = (unsigned)s + R - 1u, q = __umulhi(x, inv);
  return max(1, (int)(q + (x - q * R >= R ? 1u : 0u)));
}
// by_layer >= 0: the chunks of that layer; otherwise the owner of chunk `id`.  A lane holds one layer of 64; with more
// layers the lengths of kDecScan x 64 are loaded together and the offset only of the layer found.
constexpr int kDecScan = 4;
__device__ __forceinline__ LayerChunks find_chunks(const DecodeArgs& a, int by_layer, int id) {
  const int lane = threadIdx.x & 63;
  LayerChunks out{-1, 0, 0, 0, 0};
  unsigned R = a.R, inv = a.R_inv;
  while (true) {
    int total = 0;
    // the layers base .. base + 63, of which this lane has one of s rows
    auto search = [&](int base, int s) {
      const int n = base + lane < a.L ? chunks_of(s, R, inv) : 0;
      const int inc = wave_inclusive_sum(n);
      const int first = total + inc - n;
      const unsigned long long b = __ballot(by_layer >= 0 ? base + lane == by_layer : (id >= first && id < first + n));
      total += __builtin_amdgcn_readlane(inc, 63);
      if (b == 0ull) return -1;
      const int src = __ffsll((unsigned long long)b) - 1;
      out.layer = base + src;
      out.first = __builtin_amdgcn_readlane(first, src);
      out.n = __builtin_amdgcn_readlane(n, src);
      out.rows = __builtin_amdgcn_readlane(s, src);
      return src;
    };
    if (a.L <= 64) {
      const int lc = min(lane, a.L - 1);
      const int s = a.layer_len[lc];
      const long long off = a.layer_off[lc];
      const int src = search(0, s);
      if (src >= 0)
        out.off = (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(off >> 32), src) << 32) |
                              (unsigned)__builtin_amdgcn_readlane((int)off, src));
    } else {
      for (int base = 0; base < a.L; base += 64 * kDecScan) {
        int s[kDecScan];
#pragma unroll
        for (int j = 0; j < kDecScan; ++j) s[j] = a.layer_len[min(base + 64 * j + lane, a.L - 1)];
#pragma unroll
        for (int j = 0; j < kDecScan; ++j)
          if (base + 64 * j < a.L) search(base + 64 * j, s[j]);
      }
    }
    if (total <= a.NC || R == 1u << 31) break;
    out.layer = -1;
    inv = R < (1u << 30) ? inv >> 1 : 2u;
    R = R < (1u << 30) ? 2u * R : 1u << 31;  // 2^31: one chunk per layer, which always fits
  }
  if (a.L > 64 && out.layer >= 0) out.off = a.layer_off[out.layer];
  return out;
}

// The same for a workgroup: with more layers than a wave holds at once its first wave searches for all.  512 and 2000
// layers of 64 rows, one kv head and eight query heads: 19 and 109 us with every wave searching and dividing, 16 and 73
// now; an equal number of chunks per layer (no search) 15 and 32, but with lengths of 100 to 1800 rows 57 and 214
// against 44 and 207.
__device__ __forceinline__ LayerChunks find_chunks_of_group(const DecodeArgs& a, int by_layer, int id) {
  if (a.L <= 64) return find_chunks(a, by_layer, id);
  __shared__ LayerChunks found;
  if (threadIdx.x < 64) {
    const LayerChunks lc = find_chunks(a, by_layer, id);
    if (threadIdx.x == 0) found = lc;
  }
  __syncthreads();
  LayerChunks out;
  out.layer = __builtin_amdgcn_readfirstlane(found.layer);
  out.first = __builtin_amdgcn_readfirstlane(found.first);
  out.n = __builtin_amdgcn_readfirstlane(found.n);
  out.rows = __builtin_amdgcn_readfirstlane(found.rows);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)found.off);
  out.off = (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(found.off >> 32)) << 32) | lo);
  return out;
}

// What one workgroup works on.
struct DecodeChunk {
  int l;         // layer
  size_t row0;   // first row of the chunk, of head 0 (cached or appended rows) ...
  size_t head;   // ... and rows from one head to the next
  int rows;      // its length
  bool fresh;    // appended rows
  bool last;     // last chunk of the layer's cached rows: the appended rows follow it when they have no chunks (NSN = 0)
};
__device__ __forceinline__ bool chunk_of_group(const DecodeArgs& a, int id, DecodeChunk& c) {
  if (id >= a.NC) {
    const int k = id - a.NC, s = k % a.NSN;  // (NSN > 0: the launch has ids past NC)
    const int rows = (a.n_new + a.NSN - 1) / a.NSN;
    const int beg = min(s * rows, a.n_new);
    c.l = k / a.NSN;
    c.rows = min(a.n_new - beg, rows);
    c.row0 = (size_t)c.l * a.Hkv * a.n_new + beg;
    c.head = a.n_new;
    c.fresh = true;
    c.last = false;
    return true;
  }
  const LayerChunks lc = find_chunks_of_group(a, -1, id);
  if (lc.layer < 0) return false;
  const int per = (lc.rows + lc.n - 1) / lc.n;
  const int rows = (per + 31) & ~31;  // whole steps of a wave
  const int beg = min((id - lc.first) * rows, lc.rows);
  c.l = lc.layer;
  c.rows = min(lc.rows - beg, rows);
  c.row0 = (size_t)lc.off * a.Hkv + beg;
  c.head = lc.rows;
  c.fresh = false;
  c.last = id - lc.first == lc.n - 1;
  return true;
}

// 8-byte load of data that is read once (see load16_stream)
__device__ __forceinline__ uint2 load8_stream(const void* p) {
  typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
  const u32x2_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
  return make_uint2(t.x, t.y);
}

__device__ __forceinline__ void store_elem(char* dst, float x, bf16_t) {
  *reinterpret_cast<uint16_t*>(dst) = (uint16_t)float_to_bf16_rne(x);
}
__device__ __forceinline__ void store_elem(char* dst, float x, float) { *reinterpret_cast<float*>(dst) = x; }

__device__ __forceinline__ void unpack4(const uint4& v, float (&f)[4]) {
  f[0] = __uint_as_float(v.x);
  f[1] = __uint_as_float(v.y);
  f[2] = __uint_as_float(v.z);
  f[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ float dot4(const uint4& a, const uint4& b) {
  float d = __uint_as_float(a.x) * __uint_as_float(b.x);
  d = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), d);
  d = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), d);
  return fmaf(__uint_as_float(a.w), __uint_as_float(b.w), d);
}

// Chunk `id` of head h of a workgroup: the waves' results (red_*) merged and written.
template <int H, int D>
__device__ __forceinline__ void write_partial(const DecodeArgs& a, int id, int l, int g, const float (&red_o)[kDecWaves][H][D],
                                              const float (&red_m)[kDecWaves][H], const float (&red_z)[kDecWaves][H]) {
  for (int i = threadIdx.x; i < a.G * D; i += kDecThreads) {
    const int h = i / D, j = i - h * D;
    float mn = red_m[0][h];
#pragma unroll
    for (int w = 1; w < kDecWaves; ++w) mn = fmaxf(mn, red_m[w][h]);
    float zs = 0.f, os = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float c = __builtin_amdgcn_exp2f(red_m[w][h] - mn);
      zs = fmaf(red_z[w][h], c, zs);
      os = fmaf(red_o[w][h][j], c, os);
    }
    float* dst = a.part + ((size_t)id * a.Hq + g * a.G + h) * (D + 2);
    dst[j] = os;
    if (j == 0) {
      dst[D] = mn;
      dst[D + 1] = zs;
    }
  }
}

// Value of a partner lane whose lane-index bit X differs (X = 1, 2, 4, 8 inside a row of 16 lanes: data-parallel
// primitives, no LDS traffic; the partners of 4 and 8 are the mirrored lanes of the half row / row, which differ
// in the lower bits too; X = 16: the lane 16 away).
template <int X>
__device__ __forceinline__ float lane_partner(float v) {
  const int i = __float_as_int(v);
  if constexpr (X == 1) return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0xB1, 0xF, 0xF, true));        // quad_perm 1,0,3,2
  else if constexpr (X == 2) return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x4E, 0xF, 0xF, true));   // quad_perm 2,3,0,1
  else if constexpr (X == 4) return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x141, 0xF, 0xF, true));  // row_half_mirror
  else if constexpr (X == 8) return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x140, 0xF, 0xF, true));  // row_mirror
  else return __shfl_xor(v, X, kWave);
}

// The LPR lanes that read one row each hold, for every query head of the group, a partial dot product.
// RowReduceScatter sums them over the lanes and leaves in v[0] the total of ONE head per lane (the head
// row_head() names: the upper lane-index bits choose it), at GP + log2(LPR) - 1 exchanges instead of
// GP * log2(LPR); RowAllGather is the inverse: from one value per lane for that lane's head to all GP
// values in every lane.  N: values still held, X: bit in which the partner differs.  All array indices
// are compile-time constants (the arrays live in registers).
template <int GP, int N, int X>
struct RowReduceScatter {
  static __device__ __forceinline__ void run(float (&v)[GP], int cc) {
    if constexpr (X >= 1) {
      if constexpr (N > 1) {
        const bool up = (cc & X) != 0;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
          const float keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
          v[i] = keep + lane_partner<X>(send);
        }
        RowReduceScatter<GP, N / 2, X / 2>::run(v, cc);
      } else {
        v[0] += lane_partner<X>(v[0]);
        RowReduceScatter<GP, 1, X / 2>::run(v, cc);
      }
    }
  }
};
template <int GP, int LPR>
__device__ __forceinline__ int row_head(int cc) {
  int h = 0, n = GP;
#pragma unroll
  for (int x = LPR / 2; x >= 1; x >>= 1) {
    if (n > 1) {
      n >>= 1;
      h += (cc & x) ? n : 0;
    }
  }
  return h;
}
// N: values held so far (w[0..N)), X: partner bit of this step; the steps run from the last halving
// distance of the reduce-scatter back up to LPR / 2.
template <int GP, int N, int X>
struct RowAllGather {
  static __device__ __forceinline__ void run(float (&w)[GP], int cc) {
    if constexpr (N < GP) {
      const bool up = (cc & X) != 0;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float other = lane_partner<X>(w[i]);
        w[i + N] = up ? w[i] : other;
        w[i] = up ? other : w[i];
      }
      RowAllGather<GP, 2 * N, 2 * X>::run(w, cc);
    }
  }
};
template <int GP, int LPR>
__device__ __forceinline__ void row_reduce_scatter(float (&v)[GP], int cc) {
  RowReduceScatter<GP, GP, LPR / 2>::run(v, cc);
}
template <int GP, int LPR>
__device__ __forceinline__ void row_all_gather(float mine, float (&w)[GP], int cc) {
  w[0] = mine;
  RowAllGather<GP, 1, LPR / GP>::run(w, cc);   // the last halving step of the reduce-scatter had distance LPR / GP
}

// fp32 cache.  grid (NC + L*NSN, Hkv), 256 threads.  A row is read by LPR = row bytes / 16 lanes (16 bytes each), so
// a wave takes 64 / LPR rows per step; every lane group keeps, per query head of the group, the running maximum, the
// normaliser and its piece of the weighted value sum over the rows it has seen.  GP is the group size rounded up to a
// power of two (heads past G repeat head 0 and are not stored).
template <int D, int GP>
__global__ void __launch_bounds__(kDecThreads, 2) decode_partial_kernel(DecodeArgs a) {
  using TL = Tile<float, D>;
  constexpr int LPR = TL::kChunksPerRow;
  constexpr int MS = 64 / LPR;
  constexpr int E = 4;
  constexpr int U = 2;  // steps whose loads are issued together
  __shared__ float red_o[kDecWaves][GP][D];
  __shared__ float red_m[kDecWaves][GP], red_z[kDecWaves][GP];

  const int id = blockIdx.x, g = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = lane / LPR, cc = lane - sub * LPR;

  DecodeChunk ch;
  if (!chunk_of_group(a, id, ch)) return;
  const int l = ch.l;

  // this lane's piece of the G queries, kept packed
  uint4 qp[GP];
#pragma unroll
  for (int h = 0; h < GP; ++h) {
    const int hq = g * a.G + (h < a.G ? h : 0);
    qp[h] = *reinterpret_cast<const uint4*>(a.q + ((size_t)(l * a.Hq + hq)) * TL::kRowBytes + cc * 16);
  }
  // running maximum and normaliser of the ONE head this lane evaluates (row_head), weighted value sums of all
  float m1 = kNegBig, z1 = 0.f, o[GP][E];
#pragma unroll
  for (int h = 0; h < GP; ++h)
#pragma unroll
    for (int e = 0; e < E; ++e) o[h][e] = 0.f;

  auto walk = [&](const char* k, const char* v, size_t row0, int r_end) {
    const char *kb = k + row0 * TL::kRowBytes + cc * 16, *vb = v + row0 * TL::kRowBytes + cc * 16;
    // TAIL: some of the rows lie past the end.  They repeat the last one with weight zero, and their values, among
    // which an infinity can be, count as zeros.
    auto step = [&](int r0, auto tail) {
      constexpr bool TAIL = decltype(tail)::value;
      uint4 kv[U], vv[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * kDecWaves * MS + sub;
        ok[u] = !TAIL || r < r_end;
        const size_t ro = (size_t)(TAIL ? min(r, r_end - 1) : r) * TL::kRowBytes;
        kv[u] = load16_stream(kb + ro);
        vv[u] = load16_stream(vb + ro);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float s[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) s[h] = dot4(qp[h], kv[u]);
        row_reduce_scatter<GP, LPR>(s, cc);
        const float s1 = ok[u] ? s[0] * a.scale_log2 : kNegBig;
        // a new maximum of some head in some lane group: rescale what that head has so far (rare after
        // the first rows)
        if (__ballot(s1 > m1) != 0ull) {
          const float mn = fmaxf(m1, s1);
          const float c1 = __builtin_amdgcn_exp2f(m1 - mn);
          z1 *= c1;
          m1 = mn;
          float c[GP];
          row_all_gather<GP, LPR>(c1, c, cc);
#pragma unroll
          for (int h = 0; h < GP; ++h)
#pragma unroll
            for (int e = 0; e < E; ++e) o[h][e] *= c[h];
        }
        const float p1 = ok[u] ? __builtin_amdgcn_exp2f(s1 - m1) : 0.f;
        z1 += p1;
        float p[GP], vf[E];
        row_all_gather<GP, LPR>(p1, p, cc);
        unpack4(vv[u], vf);
#pragma unroll
        for (int e = 0; e < E; ++e) vf[e] = ok[u] ? vf[e] : 0.f;
#pragma unroll
        for (int h = 0; h < GP; ++h)
#pragma unroll
          for (int e = 0; e < E; ++e) o[h][e] = fmaf(p[h], vf[e], o[h][e]);
      }
    };
    int r0 = wave * MS;
    for (; r0 + ((U - 1) * kDecWaves + 1) * MS <= r_end; r0 += U * kDecWaves * MS) step(r0, std::false_type());
    if (r0 < r_end) step(r0, std::true_type());
  };
  if (ch.fresh) {
    walk(a.k_new, a.v_new, ch.row0 + g * ch.head, ch.rows);
  } else {
    walk(a.k_cache, a.v_cache, ch.row0 + g * ch.head, ch.rows);
    if (ch.last && a.n_new > 0 && a.NSN == 0) walk(a.k_new, a.v_new, (size_t)(l * a.Hkv + g) * a.n_new, a.n_new);
  }
  float m[GP], z[GP];
  row_all_gather<GP, LPR>(m1, m, cc);
  row_all_gather<GP, LPR>(z1, z, cc);

  // merge the lane groups of the wave (they saw different rows), then the waves through LDS
#pragma unroll
  for (int x = LPR; x < 64; x <<= 1) {
#pragma unroll
    for (int h = 0; h < GP; ++h) {
      const float mo = __shfl_xor(m[h], x, kWave), zo = __shfl_xor(z[h], x, kWave);
      const float mn = fmaxf(m[h], mo);
      const float c0 = __builtin_amdgcn_exp2f(m[h] - mn), c1 = __builtin_amdgcn_exp2f(mo - mn);
      z[h] = z[h] * c0 + zo * c1;
#pragma unroll
      for (int e = 0; e < E; ++e) o[h][e] = o[h][e] * c0 + __shfl_xor(o[h][e], x, kWave) * c1;
      m[h] = mn;
    }
  }
  if (sub == 0) {
#pragma unroll
    for (int h = 0; h < GP; ++h) {
#pragma unroll
      for (int e = 0; e < E; ++e) red_o[wave][h][cc * E + e] = o[h][e];
      if (cc == 0) {
        red_m[wave][h] = m[h];
        red_z[wave][h] = z[h];
      }
    }
  }
  __syncthreads();
  write_partial<GP, D>(a, id, l, g, red_o, red_m, red_z);
}

// bf16 and 8-bit caches, on the matrix unit.  grid (NC + L*NSN, Hkv), 4 waves, each taking every fourth step of 32
// rows (keys) of the chunk.
//   logits  D[key][col] = sum_d K[key][d] Q[col][d]     2 x d/32 x v_mfma_f32_16x16x32_bf16 (exact products, fp32 sums)
//   output  O[row][col] += sum_key P[row][key] V[key][col]   d/16 x v_mfma_f32_16x16x32_bf16
// The softmax weights are not rounded: a weight p in fp32 is the exact sum of three bf16 numbers (8 significant bits
// each), and the second product takes the three parts as rows of its own, which
// the 16 rows of the instruction have room for: column c of the first product is query head c % GP, so lane column c
// holds the weights of that head and passes on part c / GP (GP heads, rounded up to a power of two).  Groups of 5 to
// 8 heads fill the 16 rows with two parts and take a second instruction for the third, half of it in each.
// Infinite values: the parts of a weight that is not zero are none of them zero (0 * inf would be NaN, see
// weight_part) and rows past the end count as zeros, so a value of +-inf under a nonzero weight gives +-inf, as the
// definition does.
//
// Lane (c, g) = (l % 16, l / 16).  First product: it holds, for every k-step, 8 elements of key c (and 16 + c) and the
// same 8 of query head c % GP (any assignment of elements to (lane group, step) gives the same sum: step k takes
// the elements 32 k + 8 g .. + 7, or 64 (k / 2) + 16 g + 8 (k % 2) .. + 7 with FP8, so that a load brings 16 bytes of a
// row in either case), and receives that head's logits for the keys 4 g + i and 16 + 4 g + i, i = 0..3.  The second
// product contracts over keys, in the order (lane group, register): its weight operand is then exactly what the lane
// has (no movement between lanes), and its value operand the same 8 keys at one column: the lane loads piece c (d/16
// elements) of these 8 rows and transposes them in registers (one byte permutation per two elements; unpacking to
// fp32 would cost one instruction per element).
// FP8: the cached rows are E4M3 codes with one scale per row, converted to packed bf16 on arrival (exact); the key's
// scale multiplies the logit and the value's scale the weight.  The appended rows of a step are bf16 in either case.
//
// Bound by HBM.  Whole steps (both launches) over caches not read before: 524288 bf16 rows, one head per kv head, 50 us
// (5.3 TB/s); 650000 rows, seven heads, 67 us (5.0 TB/s); 838856 8-bit rows, four heads, 51 us (4.5 TB/s).  With the
// kernels this one replaced 52, 86 and 90 us: they spent about 160 vector instructions per 16 rows and wave (up to four
// heads) or 32 fp32 matrix instructions of 32 clocks (five to eight), and cut every layer into the same number of chunks,
// so that the layer with the largest budget had the longest ones.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// out[i] = the value of lane FIRST + i of this lane's row of 16 lanes, i = 0..7 (0x150 + n: broadcast of lane n)
template <int FIRST>
__device__ __forceinline__ void row_broadcast(float v, float (&out)[8]) {
  const int i = __float_as_int(v);
  out[0] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 0, 0xF, 0xF, true));
  out[1] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 1, 0xF, 0xF, true));
  out[2] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 2, 0xF, 0xF, true));
  out[3] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 3, 0xF, 0xF, true));
  out[4] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 4, 0xF, 0xF, true));
  out[5] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 5, 0xF, 0xF, true));
  out[6] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 6, 0xF, 0xF, true));
  out[7] = __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x150 + FIRST + 7, 0xF, 0xF, true));
}

__device__ __forceinline__ float group_max(float v) {  // over the four lane groups of 16
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The upper part of a positive weight: the largest bf16 number BELOW it (0 for 0).  What remains is then exact and
// never zero: after two parts it has 8 significant bits or less.
__device__ __forceinline__ float weight_part(float w) {
  return __uint_as_float(__builtin_elementwise_sub_sat(__float_as_uint(w), 1u) & 0xffff0000u);
}

// N bytes of a row that is read once, as dwords (see load16_stream)
template <int N>
__device__ __forceinline__ void load_piece(const char* p, uint32_t (&w)[N / 4]) {
  if constexpr (N == 16) {
    const uint4 v = load16_stream(p);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else if constexpr (N == 8) {
    const uint2 v = load8_stream(p);
    w[0] = v.x; w[1] = v.y;
  } else {
    w[0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
  }
}

// State of a wave while it walks its rows.
template <int D>
struct DecodeState {
  float m_run, z_run;   // of head c % GP; m_run is the same in the four lane groups
  f32x4_t acc[D / 16];  // acc[j][r]: output column (d/16) c + j, row 4 g + r
};

// The r_end rows of one chunk.  kb, vb (ksc, vsc): its first row.  LEAN: keys and values are never held together
// (fewer registers, more waiting).
template <int D, int GP, bool FP8, bool LEAN>
__device__ __forceinline__ void decode_rows(DecodeState<D>& st, const uint4 (&qp)[D / 32], const char* kb, const char* vb,
                                            const float* ksc, const float* vsc, int r_end, float scale_log2) {
  constexpr int KS = D / 32;                  // k-steps of the first product
  constexpr int PE = D / 16;                  // elements of a value piece = instructions of the second product
  constexpr int kEl = FP8 ? 1 : 2;            // bytes per element
  constexpr int kRowBytes = D * kEl;
  constexpr int kStep = 32, kStride = kDecWaves * kStep;
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = c / GP;

  constexpr int KL = D * kEl / 64;            // 16-byte loads per key and lane
  // One step's rows.
  struct Rows {
    uint32_t k[2][KL][4], v[8][PE * kEl / 4];
    float scale;
  };
  const float* sc = c < 8 ? ksc : vsc;
  // A step's first row has a 64-bit offset (a chunk can be longer than 4 GiB), the same for the wave; inside a step the
  // offsets are 32-bit.  Rows past the end repeat the last one (their weights are zero).
  auto load_keys = [&](Rows& t, int r0) {
    const char* base = kb + (size_t)r0 * kRowBytes;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      // No streaming hint here: a load instruction takes half a cache line of every row (with the hint the line was
      // fetched again for the other half: 5.3 instead of 5.6 TB/s)
      const unsigned ro = (unsigned)(min(16 * b + c, r_end - 1 - r0) * kRowBytes + 16 * g);
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const uint4 x = *reinterpret_cast<const uint4*>(base + ro + 64 * k);
        t.k[b][k][0] = x.x; t.k[b][k][1] = x.y; t.k[b][k][2] = x.z; t.k[b][k][3] = x.w;
      }
    }
  };
  auto load_values = [&](Rows& t, int r0, auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    const char* base = vb + (size_t)r0 * kRowBytes;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int row = 16 * (e >> 2) + 4 * g + (e & 3);
      const unsigned ro = (unsigned)((TAIL ? min(row, r_end - 1 - r0) : row) * kRowBytes + c * PE * kEl);
      load_piece<PE * kEl>(base + ro, t.v[e]);
    }
    // the scales of the 8 keys this row of 16 lanes has logits and weights for: lanes 0..7 the keys', 8..15 the
    // values', handed to the other lanes of the row by broadcasts
    const int row = r0 + 16 * ((c >> 2) & 1) + 4 * g + (c & 3);
    if constexpr (FP8) t.scale = sc[TAIL ? min(row, r_end - 1) : row];
  };
  auto logits = [&](const Rows& rows, float (&t)[8]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      f32x4_t s4 = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        uint4 kp;
        if constexpr (FP8) kp = e4m3x8_to_bf16x8(make_uint2(rows.k[b][k / 2][2 * (k & 1)], rows.k[b][k / 2][2 * (k & 1) + 1]));
        else kp = make_uint4(rows.k[b][k][0], rows.k[b][k][1], rows.k[b][k][2], rows.k[b][k][3]);
        s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kp), __builtin_bit_cast(bf16x8_t, qp[k]), s4, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) t[4 * b + i] = s4[i];
    }
  };
  // TAIL: some of the step's rows lie past the end
  auto finish = [&](Rows& rows, int r0, float (&t)[8], auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    float bm = kNegBig;
    float sk[8], sv[8];
    if constexpr (FP8) {
      row_broadcast<0>(rows.scale * scale_log2, sk);
      row_broadcast<8>(rows.scale, sv);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] *= FP8 ? sk[e] : scale_log2;
    if constexpr (TAIL) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool in = r0 + 16 * (e >> 2) + 4 * g + (e & 3) < r_end;
        t[e] = in ? t[e] : kNegBig;
#pragma unroll
        for (uint32_t& x : rows.v[e]) x = in ? x : 0u;  // the last row, which they repeat, may hold an infinity
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) bm = fmaxf(bm, t[e]);
    bm = group_max(bm);
    if (__ballot(bm > st.m_run) != 0ull) {  // a new maximum of some head: rescale what that head has so far (rare)
      const float mn = fmaxf(st.m_run, bm);
      const float c1 = __builtin_amdgcn_exp2f(st.m_run - mn);
      st.z_run *= c1;
      st.m_run = mn;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float cr = __shfl(c1, 4 * g + r, kWave);  // row 4 g + r belongs to the head of lane column 4 g + r
#pragma unroll
        for (int j = 0; j < PE; ++j) st.acc[j][r] *= cr;
      }
    }
    // the weights, their parts as packed bf16 (rows past the third part repeat it and are dropped)
    uint32_t pa[4], pl[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      uint32_t x[2], y[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float p = __builtin_amdgcn_exp2f(t[e + u] - st.m_run);
        float w = FP8 ? fmaf(p, sv[e + u], 0.f) : p;  // the sum takes the sign of a zero
        if constexpr (TAIL) {
          const bool in = r0 + 16 * ((e + u) >> 2) + 4 * g + ((e + u) & 3) < r_end;
          p = in ? p : 0.f;
          w = in ? w : 0.f;
        }
        st.z_run += p;
        const float hi = weight_part(w), r1 = w - hi;
        const float mid = weight_part(r1), lo = r1 - mid;
        if constexpr (GP == 8) {
          x[u] = __float_as_uint(part == 0 ? hi : mid);
          y[u] = __float_as_uint(0.5f * lo);
        } else {
          x[u] = __float_as_uint(part == 0 ? hi : (part == 1 ? mid : lo));
          y[u] = 0u;
        }
      }
      pa[e / 2] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302u);
      pl[e / 2] = __builtin_amdgcn_perm(y[1], y[0], 0x07060302u);
    }
    const bf16x8_t wa = __builtin_bit_cast(bf16x8_t, make_uint4(pa[0], pa[1], pa[2], pa[3]));
    const bf16x8_t wl = __builtin_bit_cast(bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
#pragma unroll
    for (int j2 = 0; j2 < PE / 2; ++j2) {  // two columns at a time: one dword of every row
      uint32_t d[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (FP8) d[e] = e4m3x2_to_bf16x2(rows.v[e][j2 / 2], (j2 & 1) != 0);
        else d[e] = rows.v[e][j2];
      }
      uint32_t lo[4], hi[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        lo[u] = __builtin_amdgcn_perm(d[2 * u + 1], d[2 * u], 0x05040100u);
        hi[u] = __builtin_amdgcn_perm(d[2 * u + 1], d[2 * u], 0x07060302u);
      }
      const bf16x8_t v0 = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
      const bf16x8_t v1 = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
      st.acc[2 * j2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, v0, st.acc[2 * j2], 0, 0, 0);
      st.acc[2 * j2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, v1, st.acc[2 * j2 + 1], 0, 0, 0);
      if constexpr (GP == 8) {
        st.acc[2 * j2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, v0, st.acc[2 * j2], 0, 0, 0);
        st.acc[2 * j2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, v1, st.acc[2 * j2 + 1], 0, 0, 0);
      }
    }
  };

  int r0 = wave * kStep;
  if (r0 >= r_end) return;
  float t[8];
  Rows rows;
  if constexpr (!LEAN) load_keys(rows, r0);
  auto step = [&](auto tail) {
    if constexpr (LEAN) {
      load_keys(rows, r0);
      logits(rows, t);
      load_values(rows, r0, tail);
    } else {
      load_values(rows, r0, tail);
      logits(rows, t);
      if (r0 + kStride < r_end) load_keys(rows, r0 + kStride);  // in flight while this step is finished
    }
    finish(rows, r0, t, tail);
  };
  for (; r0 + kStep <= r_end; r0 += kStride) step(std::false_type());
  if (r0 < r_end) step(std::true_type());
}

// Three waves per SIMD (138 to 152 registers with rows of 256 bytes; four spill, and took twice the time).
template <int D, int GP, bool FP8>
__global__ void __launch_bounds__(kDecThreads, 3) decode_matrix_kernel(DecodeArgs a) {
  constexpr int PE = D / 16;
  __shared__ float red_o[kDecWaves][GP][D];
  __shared__ float red_m[kDecWaves][GP], red_z[kDecWaves][GP];

  const int id = blockIdx.x, g = blockIdx.y;
  const int lane = threadIdx.x & 63, c = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  DecodeChunk ch;
  if (!chunk_of_group(a, id, ch)) return;
  const int l = ch.l;

  // query head c % GP of the group (heads past G: zeros, their rows are dropped)
  uint4 qp[D / 32];
  auto load_queries = [&](bool codes) {
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      qp[k] = make_uint4(0u, 0u, 0u, 0u);
      const int e0 = codes ? 64 * (k / 2) + 16 * grp + 8 * (k & 1) : 32 * k + 8 * grp;
      if (c % GP < a.G) qp[k] = *reinterpret_cast<const uint4*>(a.q + ((size_t)(l * a.Hq + g * a.G + c % GP) * D + e0) * 2);
    }
  };
  load_queries(FP8 && !ch.fresh);
  DecodeState<D> st;
  st.m_run = kNegBig;
  st.z_run = 0.f;
#pragma unroll
  for (int j = 0; j < PE; ++j) st.acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  if (!ch.fresh) {
    const size_t row0 = ch.row0 + g * ch.head;
    if constexpr (FP8)
      decode_rows<D, GP, true, false>(st, qp, a.k_cache + row0 * D, a.v_cache + row0 * D, a.k_scale + row0, a.v_scale + row0,
                                      ch.rows, a.scale_log2);
    else
      decode_rows<D, GP, false, false>(st, qp, a.k_cache + row0 * (D * 2), a.v_cache + row0 * (D * 2), nullptr, nullptr,
                                       ch.rows, a.scale_log2);
  }
  if (ch.fresh || (ch.last && a.n_new > 0 && a.NSN == 0)) {
    const size_t row0 = ch.fresh ? ch.row0 + g * ch.head : (size_t)(l * a.Hkv + g) * a.n_new;
    if (FP8 && !ch.fresh) load_queries(false);
    decode_rows<D, GP, false, true>(st, qp, a.k_new + row0 * (D * 2), a.v_new + row0 * (D * 2), nullptr, nullptr,
                                    ch.fresh ? ch.rows : a.n_new, a.scale_log2);
  }

  // the four lane groups saw different keys of the same head: one normaliser
  const float z = group_sum(st.z_run);
  if (lane < GP) {
    red_m[wave][lane] = st.m_run;
    red_z[wave][lane] = z;
  }
  // row R = 4 grp + r is part R / GP of head R % GP: the parts are summed
#pragma unroll
  for (int j = 0; j < PE; ++j) {
    float* dst = &red_o[wave][0][PE * c + j];
    if constexpr (GP == 8) {  // rows 0..7: first part and half of the third, rows 8..15: second part and the other half
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(st.acc[j][r]), __float_as_uint(st.acc[j][r]), false, false);
        if (grp < 2) dst[(4 * grp + r) * D] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
      }
    } else if constexpr (GP == 4) {  // lane groups 0, 1, 2: the three parts; 3: dropped
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float s = group_sum(grp < 3 ? st.acc[j][r] : 0.f);
        if (grp == 0) dst[r * D] = s;
      }
    } else if constexpr (GP == 2) {  // rows 0, 1 | 2, 3 in group 0, rows 4, 5 in group 1
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float s = group_sum(grp == 0 ? st.acc[j][h] + st.acc[j][2 + h] : (grp == 1 ? st.acc[j][h] : 0.f));
        if (grp == 0) dst[h * D] = s;
      }
    } else {  // rows 0, 1, 2 in group 0
      const float s = st.acc[j][0] + st.acc[j][1] + st.acc[j][2];
      if (grp == 0) dst[0] = s;
    }
  }
  __syncthreads();
  write_partial<GP, D>(a, id, l, g, red_o, red_m, red_z);
}

// grid (Hq / H, L), H * D threads: merges the chunks of H query heads, one per D threads, and writes their output rows.
// Four chunks are in flight together.  H = 4 with more than 64 layers: one search for four heads.
constexpr int kDecCombineHeads = 4;
template <typename T, int D>
__global__ void __launch_bounds__(kDecCombineHeads * D) decode_combine_kernel(DecodeArgs a) {
  const int h = blockIdx.x * (blockDim.x / D) + threadIdx.x / D, l = blockIdx.y, j = threadIdx.x % D;
  const LayerChunks lc = find_chunks_of_group(a, l, 0);
  if (h >= a.Hq) return;
  const int n = lc.n + a.NSN;
  constexpr int U = 4;
  float mn = kNegBig, zs = 0.f, os = 0.f;
  for (int s0 = 0; s0 < n; s0 += U) {
    float m[U], z[U], o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = min(s0 + u, n - 1);
      const int id = s < lc.n ? lc.first + s : a.NC + l * a.NSN + (s - lc.n);
      const float* p = a.part + ((size_t)id * a.Hq + h) * (D + 2);
      m[u] = (s0 + u < n) ? p[D] : kNegBig;
      z[u] = (s0 + u < n) ? p[D + 1] : 0.f;
      o[u] = p[j];  // always: a load under a condition would wait for itself
    }
    float top = mn;
#pragma unroll
    for (int u = 0; u < U; ++u) top = fmaxf(top, m[u]);
    const float c0 = __builtin_amdgcn_exp2f(mn - top);
    zs *= c0;
    os *= c0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float c = __builtin_amdgcn_exp2f(m[u] - top);
      zs = fmaf(z[u], c, zs);
      os = s0 + u < n ? fmaf(o[u], c, os) : os;
    }
    mn = top;
  }
  store_elem(a.out + ((size_t)(l * a.Hq + h) * D + j) * sizeof(T), os / zs, T{});
}

struct DecodePlan {
  int L, Hq, Hkv, G, GP, d, dtype, n_new, R, NC, NSN;
  float scale_log2;
  size_t ws_bytes;
};

static meda_status make_decode_plan(const meda_decode_params* p, DecodePlan* pl) {
  if (!p) return MEDA_ERR_INVALID_ARG;
  if (p->n_layers < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1 || p->n_new < 0) return MEDA_ERR_INVALID_ARG;
  if (p->n_q_heads % p->n_kv_heads != 0) return MEDA_ERR_INVALID_ARG;
  if (p->total_budget < p->n_layers) return MEDA_ERR_BUDGET;  // every layer keeps at least one row
  if (!(p->softmax_scale >= 0.0f) || !isfinite(p->softmax_scale)) return MEDA_ERR_INVALID_ARG;
  if (p->dtype != MEDA_F32 && p->dtype != MEDA_BF16) return MEDA_ERR_UNSUPPORTED;
  if (p->head_dim != 64 && p->head_dim != 128) return MEDA_ERR_UNSUPPORTED;
  const int G = p->n_q_heads / p->n_kv_heads;
  if (G > 8 || p->n_layers > 65535 || p->n_kv_heads > 65535) return MEDA_ERR_UNSUPPORTED;
  if ((int64_t)p->n_layers * p->n_q_heads >= (1ll << 24)) return MEDA_ERR_UNSUPPORTED;  // (layer, head) ids are ints
  pl->L = p->n_layers; pl->Hq = p->n_q_heads; pl->Hkv = p->n_kv_heads; pl->G = G; pl->d = p->head_dim;
  pl->GP = G <= 1 ? 1 : (G <= 2 ? 2 : (G <= 4 ? 4 : 8));
  pl->dtype = p->dtype; pl->n_new = p->n_new;
  // lengths are 32-bit, so a larger budget bounds nothing more
  const int64_t L = pl->L, most = L * INT32_MAX, B = p->total_budget < most ? p->total_budget : most;
  int64_t rows = (B * pl->Hkv + kDecTargetGroups - 1) / kDecTargetGroups;
  rows = (rows + 127) / 128 * 128;
  rows = rows < kDecMinRows ? kDecMinRows : (rows > kDecMaxRows ? kDecMaxRows : rows);
  // at most kDecMaxSplit chunks per layer on average (the chunk partials are workspace)
  const int64_t least = B / ((kDecMaxSplit - 1) * L) + 1;
  if (rows < least) rows = least;
  // The workspace is sized so that one for a larger budget and more appended rows always serves a smaller step: for
  // `extra` chunks beyond one per layer, the most that any budget up to B is cut into, and for the appended rows in
  // chunks of the least size.
  const int64_t extra_small = B / kDecMinRows, extra_mid = kDecTargetGroups / pl->Hkv, extra_large = B / kDecMaxRows;
  int64_t extra = extra_small < extra_mid ? extra_small : extra_mid;
  extra = extra > extra_large ? extra : extra_large;
  extra = extra < (kDecMaxSplit - 1) * L ? extra : (kDecMaxSplit - 1) * L;
  const bool own = p->n_new > (pl->dtype == MEDA_F32 ? kDecInlineNewF32 : kDecInlineNew);  // appended rows have chunks of their own
  int64_t new_chunks = own ? ((int64_t)p->n_new + kDecMinRows - 1) / kDecMinRows : 0;
  new_chunks = new_chunks < kDecMaxSplit ? new_chunks : kDecMaxSplit;
  // Where every layer cut into equally many chunks of 128 rows per query head of the group (up to 4) at the average
  // length fits the built-in scratch array, the chunks are made long enough to fit it too.
  const int even_rows = kDecMinRows * (pl->GP < 4 ? pl->GP : 4);
  int64_t even = (B / L + even_rows - 1) / even_rows;
  even = even < kDecMaxSplit ? even : kDecMaxSplit;
  const int64_t partial_bytes = (int64_t)pl->Hq * (pl->d + 2) * (int64_t)sizeof(float);
  const int64_t room = (int64_t)MEDA_DECODE_NOALLOC_MAX_BYTES / partial_bytes, least_chunks = L * (1 + new_chunks);
  if (L * (even + new_chunks) <= room && least_chunks + extra > room) {
    extra = room - least_chunks;
    if (rows < B / (extra + 1) + 1) rows = B / (extra + 1) + 1;
  }
  if (rows > 1 << 30) rows = 1 << 30;  // find_chunks goes on from there
  pl->R = (int)rows;
  pl->NC = (int)(L + (B / rows < extra ? B / rows : extra));
  const int64_t nsn = own ? ((int64_t)p->n_new + rows - 1) / rows : 0;
  pl->NSN = (int)(nsn < kDecMaxSplit ? nsn : kDecMaxSplit);
  pl->ws_bytes = (size_t)(((least_chunks + extra) * partial_bytes + 255) / 256 * 256);
  const double scale = p->softmax_scale > 0.0f ? (double)p->softmax_scale : 1.0 / sqrt((double)p->head_dim);
  pl->scale_log2 = (float)(scale * 1.4426950408889634074);
  return MEDA_OK;
}

template <typename T, int D, int GP>
static hipError_t launch_decode_g(const DecodePlan& pl, const DecodeArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)(pl.NC + pl.L * pl.NSN), pl.Hkv), block(kDecThreads);
  if constexpr (sizeof(T) == 2) {
    if (a.k_scale) hipLaunchKernelGGL((decode_matrix_kernel<D, GP, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((decode_matrix_kernel<D, GP, false>), grid, block, 0, s, a);
  } else {
    hipLaunchKernelGGL((decode_partial_kernel<D, GP>), grid, block, 0, s, a);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int heads = pl.L > 64 ? kDecCombineHeads : 1;
  hipLaunchKernelGGL((decode_combine_kernel<T, D>), dim3((pl.Hq + heads - 1) / heads, pl.L), dim3(heads * D), 0, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_decode_t(const DecodePlan& pl, const DecodeArgs& a, hipStream_t s) {
  switch (pl.GP) {
    case 1: return launch_decode_g<T, D, 1>(pl, a, s);
    case 2: return launch_decode_g<T, D, 2>(pl, a, s);
    case 4: return launch_decode_g<T, D, 4>(pl, a, s);
    default: return launch_decode_g<T, D, 8>(pl, a, s);
  }
}

// Scratch of the entry point that allocates nothing: the chunk partials of one decoding step live in this
// file-scope device array instead of a caller-provided workspace.  Every GPU holds its own copy at its own
// address; the name below is only the host-side handle of the symbol, the address a kernel can use is looked
// up once per device (scratch_of_current_device) and kept.
constexpr size_t kDecodeScratchBytes = (size_t)MEDA_DECODE_NOALLOC_MAX_BYTES;
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kDecodeScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on the current device, or null (with *err set) if a HIP call failed.
static void* scratch_of_current_device(hipError_t* err) {
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDevices) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    *err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (*err != hipSuccess || !ptr) {
      if (*err == hipSuccess) *err = hipErrorInvalidSymbol;
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

}  // namespace meda

extern "C" {

size_t meda_decode_workspace_bytes(const meda_decode_params* params) {
  meda::DecodePlan pl;
  return meda::make_decode_plan(params, &pl) == MEDA_OK ? pl.ws_bytes : 0;
}

static meda_status decode_common(const meda_decode_params* params, const void* q, const void* k_cache,
                                 const void* v_cache, const float* k_scale, const float* v_scale, bool fp8,
                                 const int32_t* layer_len, const int64_t* layer_off, const void* k_new,
                                 const void* v_new, void* out, void* workspace, size_t workspace_bytes,
                                 void* hip_stream) {
  using namespace meda;
  DecodePlan pl;
  const meda_status st = make_decode_plan(params, &pl);
  if (st != MEDA_OK) return st;
  if (fp8 && pl.dtype != MEDA_BF16) return MEDA_ERR_UNSUPPORTED;
  if (!q || !k_cache || !v_cache || !layer_len || !layer_off || !out) return MEDA_ERR_INVALID_ARG;
  if (fp8 && (!k_scale || !v_scale || (((uintptr_t)k_scale | (uintptr_t)v_scale) & 3u))) return MEDA_ERR_INVALID_ARG;
  if (pl.n_new > 0 && (!k_new || !v_new)) return MEDA_ERR_INVALID_ARG;
  const uintptr_t al = (uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)k_new | (uintptr_t)v_new;
  if (al & 15u) return MEDA_ERR_INVALID_ARG;  // rows are moved in 16-byte pieces
  if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < pl.ws_bytes) return MEDA_ERR_WORKSPACE;

  DecodeArgs a;
  a.q = static_cast<const char*>(q);
  a.k_cache = static_cast<const char*>(k_cache);
  a.v_cache = static_cast<const char*>(v_cache);
  a.layer_len = layer_len;
  a.layer_off = layer_off;
  a.k_new = static_cast<const char*>(k_new);
  a.v_new = static_cast<const char*>(v_new);
  a.out = static_cast<char*>(out);
  a.part = static_cast<float*>(workspace);
  a.L = pl.L; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.G = pl.G; a.n_new = pl.n_new;
  a.R = (unsigned)pl.R; a.R_inv = (unsigned)((1ull << 32) / (unsigned)pl.R); a.NC = pl.NC; a.NSN = pl.NSN;
  a.scale_log2 = pl.scale_log2;
  a.k_scale = fp8 ? k_scale : nullptr;
  a.v_scale = fp8 ? v_scale : nullptr;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  hipError_t e;
  if (pl.dtype == MEDA_BF16) e = pl.d == 128 ? launch_decode_t<bf16_t, 128>(pl, a, s) : launch_decode_t<bf16_t, 64>(pl, a, s);
  else e = pl.d == 128 ? launch_decode_t<float, 128>(pl, a, s) : launch_decode_t<float, 64>(pl, a, s);
  return e == hipSuccess ? MEDA_OK : MEDA_ERR_HIP;
}

meda_status meda_decode_attention(const meda_decode_params* params, const void* q, const void* k_cache,
                                  const void* v_cache, const int32_t* layer_len, const int64_t* layer_off,
                                  const void* k_new, const void* v_new, void* out, void* workspace,
                                  size_t workspace_bytes, void* hip_stream) {
  return decode_common(params, q, k_cache, v_cache, nullptr, nullptr, false, layer_len, layer_off, k_new, v_new, out,
                       workspace, workspace_bytes, hip_stream);
}

meda_status meda_decode_attention_noalloc(const meda_decode_params* params, const void* q, const void* k_cache,
                                          const void* v_cache, const int32_t* layer_len, const int64_t* layer_off,
                                          const void* k_new, const void* v_new, void* out, void* hip_stream) {
  meda::DecodePlan pl;
  const meda_status st = meda::make_decode_plan(params, &pl);
  if (st != MEDA_OK) return st;
  if (pl.ws_bytes > meda::kDecodeScratchBytes) return MEDA_ERR_SCRATCH_LIMIT;
  hipError_t err = hipSuccess;
  void* ptr = meda::scratch_of_current_device(&err);
  if (!ptr) return MEDA_ERR_HIP;
  // every chunk partial the combine kernel reads is written by the kernel before it in the same call (also for
  // chunks without rows), so nothing in the array has to be cleared between calls
  return decode_common(params, q, k_cache, v_cache, nullptr, nullptr, false, layer_len, layer_off, k_new, v_new, out,
                       ptr, meda::kDecodeScratchBytes, hip_stream);
}

meda_status meda_decode_attention_fp8(const meda_decode_params* params, const void* q, const uint8_t* k_codes,
                                      const uint8_t* v_codes, const float* k_scales, const float* v_scales,
                                      const int32_t* layer_len, const int64_t* layer_off, const void* k_new,
                                      const void* v_new, void* out, void* workspace, size_t workspace_bytes,
                                      void* hip_stream) {
  return decode_common(params, q, k_codes, v_codes, k_scales, v_scales, true, layer_len, layer_off, k_new, v_new, out,
                       workspace, workspace_bytes, hip_stream);
}

}  // extern "C"
