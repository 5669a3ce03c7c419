// Merging phases (Section 3.3, "Multimodal KV Pair Merging"): cosine similarity between every
// less-important key and every conserved key with a fused row argmax, a stable sort of the
// less-important positions by the slot they merge into, and the average merge of keys and values
// written straight into the ragged output.
#include "device_utils.hpp"
#include "plan.hpp"

namespace meda {

struct MergeArgs {
  const char* k;
  const char* v;
  char* k_out;
  char* v_out;
  const float* inv_norm;    // [L][Hkv][T]
  const int32_t* alloc;     // [L][4]
  const int64_t* off;       // [L+1]
  const int32_t* sel_idx;   // ragged [B*Hkv]: row id (l*Hkv+g)*T + position of every conserved key
  const float* sel_inv_norm;  // ragged: 1/|k| of the conserved keys
  char* packed_k;           // ragged [B*Hkv][d]: the conserved keys, copied once so that tiles of them are contiguous
  const int32_t* less_idx;  // ragged: row ids of the less-important keys (ascending)
  int32_t* less_slot;       // ragged: slot each of them merges into
  int32_t* sort_key[2];     // ping-pong buffers of the segment sort
  int32_t* sort_val[2];
  int32_t* seg_beg;         // [B*Hkv]: members of output row w are sort_val[0][seg_beg[w] .. seg_end[w])
  int32_t* seg_end;
  int32_t* merge_assign;    // may be null
  int L, Hkv, T, flags;
  int merge_members;        // 0: every output row is a plain copy (no merge requested or nothing to merge)
  long long total_slots;    // B * Hkv
  int merge_rows;           // output rows a wave of the merge walks
  int use_resident;         // layers whose conserved set fits into LDS go to the resident-set kernel
  int adjacent_order;       // layers whose conserved set fits into LDS sum their products in adjacent order
  int n_members;            // keys that are not conserved, all layers and heads: (L * T - B) * Hkv
};

__device__ __forceinline__ size_t less_base_of(int l, int g, int T, int Hkv, long long off_l, int S) {
  return ((size_t)l * T - (size_t)off_l) * Hkv + (size_t)g * (T - S);
}

// ------------------------------------------------------------------------ similarity + argmax
// Small problems go to the direct kernel, larger ones with fp32 keys to the split kernel, with bf16 keys to the tiled
// kernel; layers whose conserved set fits into LDS may go to the resident-set kernel (one workgroup of 8 waves per (layer,
// head) part, all 160 KB of LDS): then both are launched and every workgroup looks up its layer's budget.  The rules that
// choose (Plan::sim) stand beside the plan.
constexpr int kResWaves = 8;
constexpr int kResThreads = kResWaves * 64;
constexpr int kResLdsBytes = 160 * 1024;
constexpr int kResSplit = 1;  // 2 and 3 parts per pair (more, shorter workgroups) measured slower; so did giving this
                             // kernel only as many layers as fill whole rounds of one workgroup per CU

// conserved keys (a multiple of 32) that fit: one padded row and one 1/|k| each
template <typename T, int D>
constexpr int resident_capacity() {
  return kResLdsBytes / (Tile<T, D>::kStride + 4) / 32 * 32;
}

// Order of the k-steps of a product.  Halves: step i takes the bytes [16 i, + 16) of each half of a row, the lane groups one
// half each.  Adjacent: step i takes the bytes [32 i, + 32), the lane groups 16 of them each, so that a load instruction
// touches 32 cache lines instead of 64; the resident-set kernel, which loads rows all the time, works that way.  The two
// round differently and decide near ties differently (1e-6 to 1e-5 of the rows of clustered keys), so the order is a
// property of the problem and the layer, not of the kernel that a rule of speed picks for them: adjacent for a set that
// fits into LDS among at least kAdjacentPairs (layer, head) pairs, halves for every other one.
constexpr unsigned kAdjacentPairs = 256;
static_assert(kSimDirectGroups < kAdjacentPairs && kAdjacentPairs <= kResidentPairs, "each kernel with one order keeps to it");
template <typename T, int D>
__device__ __forceinline__ void frag_load_adjacent(Frag<T, D>& f, const char* row_ptr, int kg) {
#pragma unroll
  for (int i = 0; i < Tile<T, D>::kFragChunks; ++i) f.c[i] = *reinterpret_cast<const uint4*>(row_ptr + i * 32 + kg * 16);
}

// u_ij = (k_i . k_j)/(|k_i| |k_j|): the raw keys are multiplied (bf16 products are exact in the fp32
// accumulator), the factor 1/|k_j| of the conserved key is applied to the accumulator, and the positive
// factor 1/|k_i| of the row is dropped because it cannot change the argmax over j.  Ties go to the lower slot.
//
// A wave keeps 64 less-important rows as two B-operand fragments in registers and takes the conserved keys of
// its (layer, head) from LDS as A operands, 32 slots (one block) at a time.  With the conserved keys as
// operand A, a lane owns ONE row and sees 16 candidate slots per block in its 16 accumulator registers: the
// running best of the row is one value per lane and the block maximum is a max3 tree.
//
// Running best of one row (one lane) over the blocks it has seen: the best value, the first slot of
// the block that produced it and that block's 16 scaled products.  Keeping the products postpones the
// search for the winning register to the end of the kernel: per block only the maximum is formed
// (max3 tree), and the 16 products are copied in blocks where some lane of the wave improved.
struct RowBest {
  float best;
  int slot0;
  float u[16];
};

__device__ __forceinline__ void row_best_init(RowBest& rb) {
  rb.best = -INFINITY;
  rb.slot0 = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) rb.u[r] = -INFINITY;
}

// The 1/|k_j| of this lane's 16 slots of a block (iv_lds points at the block's entries of this lane group: slot
// r4*8 + i of the group sits at iv_lds[r4*8 + i]).
__device__ __forceinline__ void load_inv(float (&iv)[16], const float* iv_lds) {
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    const float4 v = *reinterpret_cast<const float4*>(iv_lds + r4 * 8);
    iv[r4 * 4 + 0] = v.x;
    iv[r4 * 4 + 1] = v.y;
    iv[r4 * 4 + 2] = v.z;
    iv[r4 * 4 + 3] = v.w;
  }
}

// Scales the 16 products of this lane by the 1/|k_j| of their slots and returns their maximum.
__device__ __forceinline__ float scale_max(f32x16_t& p, const float (&iv)[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) p[r] *= iv[r];
  float bm = fmaxf(fmaxf(p[0], p[1]), p[2]);
#pragma unroll
  for (int r = 3; r < 15; r += 2) bm = fmaxf(fmaxf(bm, p[r]), p[r + 1]);
  return fmaxf(bm, p[15]);
}

__device__ __forceinline__ void keep_if_improved(const f32x16_t& u, float bm, int slot0, RowBest& rb) {
  const bool improved = bm > rb.best;  // strict: an equal value in a later block does not replace
  if (__ballot(improved) != 0ull) {
#pragma unroll
    for (int r = 0; r < 16; ++r) rb.u[r] = improved ? u[r] : rb.u[r];
    rb.best = improved ? bm : rb.best;
    rb.slot0 = improved ? slot0 : rb.slot0;
  }
}

// Slot of the row's best: the lowest register of the saved block that holds the maximum.  `best` is the maximum of
// exactly these 16 values (the max3 tree of keep_if_improved's caller), so one of them compares equal to it; walking
// down from register 15 leaves the lowest such register.  (Not a search for the smallest best - u[r] through a packed
// integer key: a key of 32 bits has no room for all 31 bits of a non-negative float beside the 4 bits of r, and
// whichever float bits are dropped, some nonzero difference then packs to the same key as the zero of the maximum.)
__device__ __forceinline__ int row_best_slot(const RowBest& rb, int kg) {
  int ridx = 15;
#pragma unroll
  for (int r = 14; r >= 0; --r) ridx = (rb.u[r] == rb.best) ? r : ridx;
  return rb.slot0 + (ridx >> 2) * 8 + kg * 4 + (ridx & 3);
}

// The two lane groups of a wave saw disjoint slots of the same row: the better one, ties -> lower slot.
__device__ __forceinline__ int row_best_merge(const RowBest& rb, int kg) {
  const int mine = row_best_slot(rb, kg);
  const float ov = __shfl_xor(rb.best, 32, kWave);
  const int oi = __shfl_xor(mine, 32, kWave);
  const bool take = ov > rb.best || (ov == rb.best && oi < mine);
  return take ? oi : mine;
}

// One block of 32 conserved slots against the wave's two row fragments: fragment and 1/|k_j| from LDS, both
// products (the two accumulator chains alternate), then scaling, maxima and the copy of an improved block.
// With two waves per SIMD one wave's vector phase runs beside the other's matrix phase.  (Variants that
// interleave the vector work of the previous block with the matrix instructions inside one wave, by hand or
// through the scheduler, measured the same or slower on every workload: under random operands the chip is
// limited by power, its clock drops to about 1.5 GHz in this kernel, and what counts is the number of
// instructions and LDS bytes per block, not their order.)
// The last tile of a (layer, head) is padded with copies of the last conserved key: a copy ties with the
// original and the tie rules (strict improvement, lowest register, lower slot between the lane groups)
// always prefer the original, so no slot needs masking and there is a single code path.
template <typename T, int D>
__device__ __forceinline__ void sim_block_products(const char* block, const unsigned (&coff)[Tile<T, D>::kFragChunks],
                                                   const Frag<T, D> (&lf)[2], f32x16_t (&acc)[2]) {
  Frag<T, D> cf;
#pragma unroll
  for (int c = 0; c < Tile<T, D>::kFragChunks; ++c) cf.c[c] = *reinterpret_cast<const uint4*>(block + coff[c]);
  acc[0] = acc_zero();
  acc[1] = acc_zero();
  mma<T, D>(acc[0], cf, lf[0]);
  mma<T, D>(acc[1], cf, lf[1]);
}

template <typename T, int D>
__device__ __forceinline__ void sim_block_simple(const char* block, const unsigned (&coff)[Tile<T, D>::kFragChunks],
                                                 const Frag<T, D> (&lf)[2], const float* iv_lds, int slot0, RowBest (&rb)[2]) {
  float iv[16];
  load_inv(iv, iv_lds);
  f32x16_t acc[2];
  sim_block_products<T, D>(block, coff, lf, acc);
  const float bm0 = scale_max(acc[0], iv), bm1 = scale_max(acc[1], iv);
  keep_if_improved(acc[0], bm0, slot0, rb[0]);
  keep_if_improved(acc[1], bm1, slot0, rb[1]);
}

// Tiled kernel: grid over (row block of 256, kv head, layer); 4 waves x 64 less-important rows.  The conserved
// keys stream through a ring of four LDS tiles of 64 slots, filled by asynchronous copies that go from global
// memory straight into LDS (no registers, no LDS store instructions): while tile t is multiplied, tile t+1 has
// landed, tile t+2 is landing and the copies of tile t+3 have just been issued, which gives every copy two tile
// times to arrive; one wait and one barrier per tile.
//
// LDS layout of a tile: 64 rows, unpadded, 16-byte chunk c of row r at position c ^ swz(r) of the row.  A copy
// instruction writes lane i's 16 bytes at (instruction base) + 16 i, so the rows cannot be padded; which global
// chunk a lane fetches is free, and the xor spreads the 16 rows a fragment load touches in one pass over all
// banks (rows of 256 bytes start at the same bank: swz(r) = r mod 16; two rows of 128 bytes share a bank
// line: swz(r) = (r / 2) mod 8).
// The 1/|k_j| of a tile are copied the same way (4 bytes per lane); every wave keeps its own copy, so all waves
// issue the same number of copies per tile and wait for the same count.
constexpr int kSimRing = 4;
constexpr int kSimInvRing = 8;

template <typename T, int D>
constexpr int sim_tiled_lds_bytes() {
  return kSimRing * kSimSlotTile * Tile<T, D>::kRowBytes + kSimInvRing * kSimWaves * kSimSlotTile * (int)sizeof(float);
}

template <typename T, int D>
__global__ void __launch_bounds__(kSimWaves * 64, 2) similarity_argmax_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  constexpr int CPR = TL::kChunksPerRow;
  constexpr int NC = TL::kFragChunks;
  constexpr int RPI = 64 / CPR;                        // rows one copy instruction fills
  constexpr int PF = kSimSlotTile / RPI / kSimWaves;   // key copy instructions per wave and tile
  constexpr int NB = kSimSlotTile / 32;                // blocks per tile
  constexpr int KPT = PF + 1;                          // copies per wave and tile (keys and 1/|k|)
  constexpr int kTileBytes = kSimSlotTile * TL::kRowBytes;
  static_assert(kSimSlotTile % (RPI * kSimWaves) == 0, "the copy instructions must tile the rows of a tile evenly");
  extern __shared__ __align__(16) char smem[];
  char* ctile = smem;                                                       // [kSimRing][64 rows]
  float* cinv = reinterpret_cast<float*>(smem + kSimRing * kTileBytes);     // [kSimInvRing][waves][64]

  unsigned pair, rblock;
  pair_and_row_block(blockIdx.x, (unsigned)(a.L * a.Hkv), (a.T + kSimRows - 1) / kSimRows, pair, rblock);
  const int l = a.alloc[4 * (pair / a.Hkv) + 3], g = pair % a.Hkv;  // layers by decreasing budget
  const int S = a.alloc[4 * l];
  const bool fits = S <= resident_capacity<T, D>();
  if (a.use_resident && fits) return;  // the resident-set kernel below takes this layer
  const bool adjacent = a.adjacent_order && fits;
  const int n_less = a.T - S;
  const int row_base = rblock * kSimRows;
  if (row_base >= n_less) return;

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long off_l = a.off[l];
  const size_t cbase = (size_t)off_l * a.Hkv + (size_t)g * S;
  // the bases of the asynchronous copies below must sit in scalar registers: said explicitly, not left to what the
  // compiler can prove about the address arithmetic
  const float* sinv = uniform_ptr(a.sel_inv_norm + cbase);
  const char* pk = uniform_ptr(a.packed_k + cbase * TL::kRowBytes);  // this pair's conserved keys, contiguous
  const size_t lbase = less_base_of(l, g, a.T, a.Hkv, off_l, S);
  const int32_t* less = a.less_idx + lbase;
  const char* kbase = a.k;  // positions are stored as row ids over all layers and heads

  // first the row ids this wave needs (its own rows; rows past the end repeat the last one and are
  // never stored), so that all index loads of the prologue are in flight before any row load
  const int r0 = row_base + wave * kSimRowsPerWave;
  int lrow[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) lrow[s] = less[min(r0 + s * 32 + n, n_less - 1)];
  RowBest rb[2];
  row_best_init(rb[0]);
  row_best_init(rb[1]);
  Frag<T, D> lf[2];
  if (adjacent) {
#pragma unroll
    for (int s = 0; s < 2; ++s) frag_load_adjacent(lf[s], kbase + (size_t)lrow[s] * TL::kRowBytes, kg);
  } else {
#pragma unroll
    for (int s = 0; s < 2; ++s) frag_load(lf[s], kbase + (size_t)lrow[s] * TL::kRowBytes, kg);
  }

  // Copy instruction j of this wave fills the rows (wave * PF + j) * RPI .. + RPI-1 of a tile: this lane brings
  // one 16-byte chunk of row crow_r + j * RPI.  Slots past the end of the set repeat the last conserved key (see
  // sim_block_simple).  Tiles past the last one repeat it too (they are never read; issuing them keeps the number
  // of copies in flight the same in every iteration).
  const int ntiles = (S + kSimSlotTile - 1) / kSimSlotTile;
  const int crow_r = wave * PF * RPI + lane / CPR;
  const unsigned lds_ring = (unsigned)(size_t)ctile, lds_inv = (unsigned)(size_t)cinv;
  auto issue_tile = [&](int t, int ring_slot) {  // tile t of the stream into slot ring_slot of the rings
    const int tc = min(t, ntiles - 1);
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int r = crow_r + j * RPI;   // row of the tile; its swizzle does not depend on the tile
      const int slot = min(tc * kSimSlotTile + r, S - 1);
      const unsigned goff = (unsigned)(slot * TL::kRowBytes + (((lane % CPR) ^ swizzle_of_row<T, D>(r)) * 16));
      async_copy16_to_lds(pk, goff, lds_ring + (unsigned)((ring_slot % kSimRing) * kTileBytes + (wave * PF + j) * 1024));
    }
    const unsigned goff4 = (unsigned)(min(tc * kSimSlotTile + lane, S - 1) * 4);
    const unsigned loff4 = (unsigned)((((ring_slot % kSimInvRing) * kSimWaves + wave) * kSimSlotTile) * 4);
    async_copy4_to_lds(sinv, goff4, lds_inv + loff4);
  };
  issue_tile(0, 0);
  issue_tile(1, 1);
  issue_tile(2, 2);

  // chunk x of row n of a block sits at (n * row bytes) + 16 * (x ^ swz(n)) inside a block of 32 rows; step c takes the chunk
  // kg * NC + c, or 2 c + kg in adjacent order: no bits in common, so the step goes in by another xor
  const unsigned coff0 = (unsigned)(n * TL::kRowBytes + (((adjacent ? kg : kg * NC) ^ swizzle_of_row<T, D>(n)) * 16));
  const unsigned step = adjacent ? 32u : 16u;
  unsigned coff[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) coff[c] = coff0 ^ (c * step);
  // block cb of the tile in ring slot rs: its rows and where its 1/|k_j| start in this wave's copy
  auto block_rows = [&](int rs, int cb) { return ctile + (rs % kSimRing) * kTileBytes + cb * 32 * TL::kRowBytes; };
  auto inv_index = [&](int rs, int cb) { return ((rs % kSimInvRing) * kSimWaves + wave) * kSimSlotTile + cb * 32; };

  async_copy_wait<KPT>();  // tiles 0 and 1 have landed (this wave's part)
  __syncthreads();         // every wave's part has
  issue_tile(3, 3);
  for (int t = 0; t < ntiles; ++t) {
    if (t > 0) {
      async_copy_wait<KPT>();    // this wave's part of tile t+1 has landed; tile t+2 may still be in flight
      __syncthreads();           // every wave's part has; and nobody reads tile t-1 any more
      issue_tile(t + 3, t + 3);  // into the buffer of tile t-1
    }
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
      sim_block_simple<T, D>(block_rows(t, cb), coff, lf, cinv + inv_index(t, cb) + kg * 4, (t * NB + cb) * 32, rb);
  }
  async_copy_wait<0>();  // nothing of this wave is still on its way into LDS when it ends

#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int bi = row_best_merge(rb[s], kg);
    const int ri = r0 + s * 32 + n;
    if (kg == 0 && ri < n_less) {
      a.less_slot[lbase + ri] = bi;
      if (a.merge_assign) a.merge_assign[less[ri]] = bi;
    }
  }
}

// Variant for layers whose conserved set fits into LDS: one workgroup keeps ALL conserved keys of its
// (layer, head) resident and every wave streams chunks of 64 less-important rows through registers.
// After the prologue there is no barrier: the waves run independently and the keys are read from HBM once.
// grid (kResSplit * L * Hkv): part p of a pair takes the chunks p*8 + wave, then steps of 8*kResSplit.
// Layers above the capacity are left to the tiled kernel above (and skipped there when they fit).
template <typename T, int D>
__global__ void __launch_bounds__(kResThreads, 2) similarity_resident_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  constexpr int CPR = TL::kChunksPerRow;
  extern __shared__ __align__(16) char smem[];

  // workgroups are launched in the order of decreasing budget (longest first: the last ones to start
  // are the shortest), alloc[4 * rank + 3] is the layer of that rank
  const int pair = blockIdx.x / kResSplit, part = blockIdx.x % kResSplit;
  const int l = a.alloc[4 * (pair / a.Hkv) + 3], g = pair % a.Hkv;
  const int S = a.alloc[4 * l];
  const int n_less = a.T - S;
  if (S > resident_capacity<T, D>() || n_less == 0) return;
  const int n_chunks = (n_less + kSimRowsPerWave - 1) / kSimRowsPerWave;
  if (part * kResWaves >= n_chunks) return;

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long off_l = a.off[l];
  const size_t cbase = (size_t)off_l * a.Hkv + (size_t)g * S;
  const float* sinv = a.sel_inv_norm + cbase;
  const int32_t* sel = a.sel_idx + cbase;
  const size_t lbase = less_base_of(l, g, a.T, a.Hkv, off_l, S);
  const int32_t* less = a.less_idx + lbase;
  const char* kbase = a.k;  // positions are stored as row ids over all layers and heads

  // the wave's first rows are requested before the conserved set, so they arrive during the prologue
  int c = part * kResWaves + wave;
  constexpr int kChunkStep = kResWaves * kResSplit;
  auto chunk_rows = [&](int chunk, int (&rows)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) rows[s] = less[min(chunk * kSimRowsPerWave + s * 32 + n, n_less - 1)];
  };
  int lrow[2], nrow[2];
  chunk_rows(c, lrow);
  chunk_rows(c + kChunkStep, nrow);
  // adjacent order: this kernel loads 64 rows per wave and chunk, all the time
  auto row_frag = [&](Frag<T, D>& f, const char* row_ptr) { frag_load_adjacent(f, row_ptr, kg); };
  Frag<T, D> lf[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) row_frag(lf[s], kbase + (size_t)lrow[s] * TL::kRowBytes);

  // Prologue: the conserved keys into LDS.  The set is padded to a multiple of 32 slots with
  // copies of the last key (a copy can never win a tie against the original, see sim_block_simple).
  const int S_pad = (S + 31) & ~31;
  char* ckeys = smem;
  float* cinv = reinterpret_cast<float*>(smem + (size_t)S_pad * TL::kStride);
  // All row ids, then all pieces of the set are requested before the first one is stored (two memory latencies for the
  // whole set; at most kMaxPieces 16-byte pieces per thread; the bounds are the same for every thread of the workgroup, so the
  // tests are scalar branches).  The batch is an array of a native vector type: as an array of uint4 the compiler
  // kept it in scratch memory.
  constexpr int kMaxPieces = (resident_capacity<T, D>() * CPR + kResThreads - 1) / kResThreads;
  const int n_pieces = S_pad * CPR;
  {
    typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
    u32x4_t v[kMaxPieces];
    int id[kMaxPieces];
#pragma unroll
    for (int i = 0; i < kMaxPieces; ++i)
      if (i * kResThreads < n_pieces) id[i] = sel[min(min(tid + i * kResThreads, n_pieces - 1) / CPR, S - 1)];
#pragma unroll
    for (int i = 0; i < kMaxPieces; ++i) {
      if (i * kResThreads < n_pieces) {
        const int p = min(tid + i * kResThreads, n_pieces - 1);
        v[i] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)id[i] * TL::kRowBytes + (p % CPR) * 16);
      }
    }
#pragma unroll
    for (int i = 0; i < kMaxPieces; ++i) {
      if (i * kResThreads < n_pieces) {
        const int p = min(tid + i * kResThreads, n_pieces - 1);  // a repeated piece: the same bytes to the same place
        *reinterpret_cast<u32x4_t*>(ckeys + (p / CPR) * TL::kStride + (p % CPR) * 16) = v[i];
      }
    }
  }
  for (int sl = tid; sl < S_pad; sl += kResThreads) cinv[sl] = sinv[min(sl, S - 1)];
  __syncthreads();

  const int nblocks = S_pad / 32;
  unsigned coff[TL::kFragChunks];   // chunk c of this lane's fragment inside a block of 32 padded rows
#pragma unroll
  for (int c = 0; c < TL::kFragChunks; ++c) coff[c] = (unsigned)(n * TL::kStride + c * 32 + kg * 16);
  auto block_base = [&](int b) { return ckeys + b * 32 * TL::kStride; };
  auto block_inv = [&](int b) { return cinv + b * 32 + kg * 4; };
  while (c < n_chunks) {
    // the rows of the wave's next chunk and the row ids of the one after it are in flight while
    // this chunk is multiplied (past the last chunk they repeat the last row and are dropped)
    const int r0 = c * kSimRowsPerWave;
    Frag<T, D> lfn[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) row_frag(lfn[s], kbase + (size_t)nrow[s] * TL::kRowBytes);
    int nnrow[2];
    chunk_rows(c + 2 * kChunkStep, nnrow);
    RowBest rb[2];
    row_best_init(rb[0]);
    row_best_init(rb[1]);
    for (int b = 0; b < nblocks; ++b) sim_block_simple<T, D>(block_base(b), coff, lf, block_inv(b), b * 32, rb);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int bi = row_best_merge(rb[s], kg);
      const int ri = r0 + s * 32 + n;
      if (kg == 0 && ri < n_less) {
        a.less_slot[lbase + ri] = bi;
        if (a.merge_assign) a.merge_assign[lrow[s]] = bi;
      }
    }
    c += kChunkStep;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      lrow[s] = nrow[s];
      nrow[s] = nnrow[s];
      lf[s] = lfn[s];
    }
  }
}

// Direct kernel: no conserved set in LDS, no packed copy.  grid over (row block of 32 F, kv head, layer), XCD-aware
// as the tiled kernel; the NW waves of a workgroup take the same 32 F rows and every NW-th block of 32 conserved keys,
// whose fragments come from the key cache itself (L2), one block ahead; the waves' bests are merged at the end.
// For problems that leave CUs empty with 256 rows per workgroup, where the serial chain of one wave bounds the kernel.
// Every 32 rows read the whole set again, eight times as often as in the tiled kernel, so with the chip full it loses:
// see similarity_route.
template <typename T, int D, int F, int NW>
__global__ void __launch_bounds__(NW * 64, 2) similarity_direct_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  constexpr int kRows = 32 * F;
  __shared__ __align__(16) float inv_lds[NW][2][32];
  __shared__ float best_v[NW][kRows];
  __shared__ int best_s[NW][kRows];

  unsigned pair, rblock;
  pair_and_row_block(blockIdx.x, (unsigned)(a.L * a.Hkv), (a.T + kRows - 1) / kRows, pair, rblock);
  const int l = a.alloc[4 * (pair / a.Hkv) + 3], g = pair % a.Hkv;  // layers by decreasing budget
  const int S = a.alloc[4 * l];
  const int n_less = a.T - S;
  const int row_base = rblock * kRows;
  if (row_base >= n_less) return;

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long off_l = a.off[l];
  const size_t cbase = (size_t)off_l * a.Hkv + (size_t)g * S;
  const int32_t* sel = a.sel_idx + cbase;
  const float* sinv = a.sel_inv_norm + cbase;
  const size_t lbase = less_base_of(l, g, a.T, a.Hkv, off_l, S);
  const int32_t* less = a.less_idx + lbase;

  const int nblocks = (S + 31) / 32;
  // slots past the end repeat the last conserved key (see sim_block_products)
  auto slot_of = [&](int b) { return min(b * 32 + n, S - 1); };
  int lrow[F];
#pragma unroll
  for (int s = 0; s < F; ++s) lrow[s] = less[min(row_base + s * 32 + n, n_less - 1)];
  int id = sel[slot_of(wave)], id1 = sel[slot_of(wave + NW)];
  float iv0 = sinv[slot_of(wave)], iv1 = sinv[slot_of(wave + NW)];
  Frag<T, D> lf[F], cf;
#pragma unroll
  for (int s = 0; s < F; ++s) frag_load(lf[s], a.k + (size_t)lrow[s] * TL::kRowBytes, kg);
  frag_load(cf, a.k + (size_t)id * TL::kRowBytes, kg);
  RowBest rb[F];
#pragma unroll
  for (int s = 0; s < F; ++s) row_best_init(rb[s]);

  int par = 0;
  for (int b = wave; b < nblocks; b += NW, par ^= 1) {
    Frag<T, D> cn;
    frag_load(cn, a.k + (size_t)id1 * TL::kRowBytes, kg);
    const int id2 = sel[slot_of(b + 2 * NW)];
    const float iv2 = sinv[slot_of(b + 2 * NW)];
    // This wave's own copy: its LDS operations stay in order in hardware, and the fences (no instructions at this scope)
    // keep the compiler from moving the loads, which other lanes' stores feed, before them.
    if (kg == 0) inv_lds[wave][par][n] = iv0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float iv[16];
    load_inv(iv, &inv_lds[wave][par][kg * 4]);
    f32x16_t acc[F];
#pragma unroll
    for (int s = 0; s < F; ++s) {
      acc[s] = acc_zero();
      mma<T, D>(acc[s], cf, lf[s]);
    }
#pragma unroll
    for (int s = 0; s < F; ++s) keep_if_improved(acc[s], scale_max(acc[s], iv), b * 32, rb[s]);
    cf = cn;
    id1 = id2;
    iv0 = iv1;
    iv1 = iv2;
  }
#pragma unroll
  for (int s = 0; s < F; ++s) {
    const int bi = row_best_merge(rb[s], kg);
    const float bv = fmaxf(rb[s].best, __shfl_xor(rb[s].best, 32, kWave));
    if (kg == 0) {
      best_v[wave][s * 32 + n] = bv;
      best_s[wave][s * 32 + n] = bi;
    }
  }
  __syncthreads();
  if (tid < kRows && row_base + tid < n_less) {
    float v = best_v[0][tid];
    int slot = best_s[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float ov = best_v[w][tid];
      const int os = best_s[w][tid];
      const bool take = ov > v || (ov == v && os < slot);
      v = take ? ov : v;
      slot = take ? os : slot;
    }
    a.less_slot[lbase + row_base + tid] = slot;
    if (a.merge_assign) a.merge_assign[less[row_base + tid]] = slot;
  }
}

// ------------------------------------------------------------------------ fp32 keys in three bf16 parts
// x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m, each rounded to nearest: 8 + 8 + 8 significant bits hold
// all 24 of x, and every subtraction is exact (for finite x whose h does not overflow).  Two elements per call.
__device__ __forceinline__ void split2(float x, float y, unsigned& h, unsigned& m, unsigned& l) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  auto pack = [](float p, float q) { return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2_t){p, q}, bf16x2_t)); };
  h = pack(x, y);
  x -= __uint_as_float(h << 16);
  y -= __uint_as_float(h & 0xffff0000u);
  m = pack(x, y);
  x -= __uint_as_float(m << 16);
  y -= __uint_as_float(m & 0xffff0000u);
  l = pack(x, y);
}
// 8 consecutive elements: one 16-byte chunk of each part.
__device__ __forceinline__ void split8(const uint4& a, const uint4& b, uint4 (&part)[3]) {
  const unsigned x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  unsigned h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split2(__uint_as_float(x[2 * i]), __uint_as_float(x[2 * i + 1]), h[i], m[i], l[i]);
  part[0] = make_uint4(h[0], h[1], h[2], h[3]);
  part[1] = make_uint4(m[0], m[1], m[2], m[3]);
  part[2] = make_uint4(l[0], l[1], l[2], l[3]);
}

// Twice what the two sums of a product may lie apart, as a share of the lengths of both keys (which bound every partial
// sum): D fused multiply-adds of the fp32 instruction and at most D additions of the leading bf16 products, each rounded to
// 2^-24 of what it returns, and below 8 + D / 16 of that unit for the smaller products, those left out, 1/|k| and scaling.
template <int D>
constexpr float split_margin() {
  return 5 * D * 5.9604645e-8f;
}
// 1/|k| of a key of length 2^-40 to 2^60: its parts exist and no product or sum leaves the normal range.
__device__ __forceinline__ bool splits(float inv_norm) { return inv_norm >= 8.6736174e-19f && inv_norm <= 1.0995116e12f; }

// Split kernel: fp32 keys on the bf16 matrix instructions.  A product of two keys is h h' + (h m' + m h') + (m m' + h l' +
// l h') of their parts, added from the smallest terms to the largest in the fp32 accumulator; the three products left out
// are below 2^-23 of the keys' lengths (2^-26 as a rule).  6 x 32 matrix clocks per 32 x 32 x 16 products instead of 512.
//
// These sums find the slots that can win, those of the fp32 instruction decide: a row with more than one slot within
// split_margin of its best takes the products of the blocks they are in once more, with the fp32 instruction, so that near
// ties fall as they do with that instruction alone.  For that a lane keeps, beside the best block, two others that came
// within the margin of it, and the maximum of all further ones; where that is inside the margin too, its wave goes over
// its whole share of the set.  One row in two thousand of clustered keys needs it, with two blocks as a rule.  Copies of
// a lower slot's key, which would tie in both sums, have been taken out by the selection: their 1/|k| is a NaN, which no
// maximum takes.  A workgroup with a key that splits() excludes goes over everything with the fp32 instruction.
//
// grid over (row block of 32 NW, kv head, layer); a wave keeps a fragment of 32 less-important rows split in registers;
// the conserved keys come from the key cache in tiles of 64: a thread loads its pieces of the next tile before it multiplies
// the present one, splits them after it and stores the parts into the other of two LDS tiles (one barrier per tile).
// Bound by the bf16 matrix instructions (1.9 PFLOP/s of them where the sets are long) and, in short launches, by the waves
// that take their blocks again, 3 to 10 us.  Selection and similarity together, against the direct and tiled kernels, in
// us, three tenths kept: rows of 256 bytes 256 pairs of 700 69 -> 50, of 2000 290 -> 163, 32 of 8000 456 -> 279; rows of 512
// bytes 116 -> 81, 593 -> 333, 886 -> 503.
template <int D>
struct SplitTile {
  static constexpr int kSlots = 64;
  static constexpr int kPart = D * 2;             // bytes of one part of a key
  static constexpr int kStride = 3 * kPart + 16;  // three parts and padding: bank pattern as Tile<bf16_t, D>::kStride
  static constexpr int kTileBytes = kSlots * kStride;
  static constexpr int kLdsBytes = 2 * kTileBytes + 2 * kSlots * (int)sizeof(float) + 16;
};

template <int D, int NW>
__global__ void __launch_bounds__(NW * 64, 2) similarity_split_kernel(MergeArgs a) {
  using TF = Tile<float, D>;
  using ST = SplitTile<D>;
  constexpr int kSplitSlots = ST::kSlots;
  constexpr int kRows = 32 * NW;
  constexpr int NT = NW * 64;
  constexpr int NC = D / 16;                     // chunks per lane and part
  constexpr int GPR = D / 8;                     // pieces of 8 elements per key
  constexpr int NG = kSplitSlots * GPR / NT;     // pieces per thread and tile
  static_assert(NG * NT == kSplitSlots * GPR, "the pieces of a tile must come out even");
  extern __shared__ __align__(16) char smem[];
  float* inv_lds = reinterpret_cast<float*>(smem + 2 * ST::kTileBytes);  // [2][kSplitSlots]
  int* bad_lds = reinterpret_cast<int*>(inv_lds + 2 * kSplitSlots);

  unsigned pair, rblock;
  pair_and_row_block(blockIdx.x, (unsigned)(a.L * a.Hkv), (a.T + kRows - 1) / kRows, pair, rblock);
  const int l = a.alloc[4 * (pair / a.Hkv) + 3], g = pair % a.Hkv;  // layers by decreasing budget
  const int S = a.alloc[4 * l];
  const int n_less = a.T - S;
  const int row_base = rblock * kRows;
  if (row_base >= n_less) return;

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long off_l = a.off[l];
  const size_t cbase = (size_t)off_l * a.Hkv + (size_t)g * S;
  const int32_t* sel = a.sel_idx + cbase;
  const float* sinv = a.sel_inv_norm + cbase;
  const size_t lbase = less_base_of(l, g, a.T, a.Hkv, off_l, S);
  const int32_t* less = a.less_idx + lbase;

  // slots past the end repeat the last conserved key, and their 1/|k| is a NaN as well
  const int ntiles = (S + kSplitSlots - 1) / kSplitSlots, nblocks = (S + 31) / 32;
  auto load_ids = [&](int t, int (&id)[NG]) {
#pragma unroll
    for (int i = 0; i < NG; ++i) id[i] = sel[min(t * kSplitSlots + (tid + i * NT) / GPR, S - 1)];
  };
  uint4 piece[NG][2];
  float piece_inv = 0.f;
  auto load_tile = [&](int t, const int (&id)[NG]) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint4* src = reinterpret_cast<const uint4*>(a.k + (size_t)id[i] * TF::kRowBytes + (tid + i * NT) % GPR * 32);
      piece[i][0] = src[0];
      piece[i][1] = src[1];
    }
    if (tid < kSplitSlots) {
      const int s = t * kSplitSlots + tid;
      piece_inv = sinv[min(s, S - 1)];
      piece_inv = s < S ? piece_inv : __uint_as_float(kNoSlot);
    }
  };
  bool bad = false;  // a key that splits() excludes has been seen
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      uint4 part[3];
      split8(piece[i][0], piece[i][1], part);
      char* dst = smem + buf * ST::kTileBytes + (tid + i * NT) / GPR * ST::kStride + (tid + i * NT) % GPR * 16;
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(dst + p * ST::kPart) = part[p];
    }
    if (tid < kSplitSlots) {
      inv_lds[buf * kSplitSlots + tid] = piece_inv;
      bad |= piece_inv == piece_inv && !splits(piece_inv);
    }
  };

  // rows past the end repeat the last one and are never stored
  const int r0 = row_base + wave * 32;
  int id[NG];
  load_ids(0, id);
  const int lrow = less[min(r0 + n, n_less - 1)];
  load_tile(0, id);
  load_ids(1, id);
  const float row_inv = a.inv_norm[lrow];
  bad |= !splits(row_inv);
  uint4 rows[3][NC];
  {
    const uint4* src = reinterpret_cast<const uint4*>(a.k + (size_t)lrow * TF::kRowBytes + kg * TF::kHalfBytes);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      uint4 part[3];
      split8(src[2 * c], src[2 * c + 1], part);
#pragma unroll
      for (int p = 0; p < 3; ++p) rows[p][c] = part[p];
    }
  }
  if (tid == 0) *bad_lds = 0;
  store_tile(0);
  RowBest rb;
  row_best_init(rb);
  // Blocks beside the best one that came within the margin of it: the best two of them and the maximum of all others.
  float second = -INFINITY, third = -INFINITY, further = -INFINITY;
  int second_slot0 = 0, third_slot0 = 0;
  const float margin = split_margin<D>() / row_inv;
  __syncthreads();

  for (int t = 0; t < ntiles; ++t) {
    const bool more = t + 1 < ntiles;
    if (more) {
      load_tile(t + 1, id);
      load_ids(t + 2, id);
    }
#pragma unroll
    for (int cb = 0; cb < kSplitSlots / 32; ++cb) {
      const int b = t * (kSplitSlots / 32) + cb;
      if (b >= nblocks) break;
      const char* src = smem + (t & 1) * ST::kTileBytes + (cb * 32 + n) * ST::kStride + kg * (ST::kPart / 2);
      uint4 keys[3][NC];
#pragma unroll
      for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int c = 0; c < NC; ++c) keys[p][c] = *reinterpret_cast<const uint4*>(src + p * ST::kPart + c * 16);
      f32x16_t acc = acc_zero();
      auto product = [&](int pk, int pr) {
#pragma unroll
        for (int c = 0; c < NC; ++c) mma_chunk<bf16_t>(acc, keys[pk][c], rows[pr][c]);
      };
      product(2, 0);
      product(1, 1);
      product(0, 2);
      product(1, 0);
      product(0, 1);
      product(0, 0);
      float iv[16];
      load_inv(iv, inv_lds + (t & 1) * kSplitSlots + cb * 32 + kg * 4);
      const float bm = scale_max(acc, iv);
      // (one that is further behind the best so far, or is left further behind, cannot hold the nearest slot)
      const bool close = fabsf(bm - rb.best) <= margin;
      if (__ballot(close) != 0ull) {
        const float lower = close ? fminf(bm, rb.best) : -INFINITY;
        const int lower_slot0 = bm > rb.best ? rb.slot0 : b * 32;
        const bool is_second = lower > second, is_third = lower > third;
        further = fmaxf(further, is_third ? third : lower);
        third = is_second ? second : is_third ? lower : third;
        third_slot0 = is_second ? second_slot0 : is_third ? lower_slot0 : third_slot0;
        second = is_second ? lower : second;
        second_slot0 = is_second ? lower_slot0 : second_slot0;
      }
      keep_if_improved(acc, bm, b * 32, rb);
    }
    if (more) store_tile((t + 1) & 1);
    __syncthreads();
  }

  if (bad) *bad_lds = 1;
  __syncthreads();
  const bool all_fp32 = *bad_lds != 0;

  // The best slot by these sums.  The two lane groups saw disjoint slots of the same row: the better one, ties -> lower slot.
  float best = rb.best;
  int slot = row_best_slot(rb, kg);
  auto keep_better = [&](float ov, int os) {
    const bool take = ov > best || (ov == best && os < slot);
    best = take ? ov : best;
    slot = take ? os : slot;
  };
  auto merge_lane_groups = [&]() {
    const float ov = __shfl_xor(best, 32, kWave);
    const int os = __shfl_xor(slot, 32, kWave);
    keep_better(ov, os);
  };
  merge_lane_groups();

  // Which rows have another slot within the margin.
  const float limit = best - margin;
  int undecided = all_fp32 || second >= limit ? 1 : 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) undecided |= rb.u[r] >= limit && rb.slot0 + acc_row(r, kg) != slot ? 1 : 0;
  undecided |= __shfl_xor(undecided, 32, kWave);
  if (__ballot(undecided) != 0ull) {
    // The fp32 instruction, operands straight from the key cache: the blocks that hold a slot within the margin, or all
    // blocks.  (More blocks than a row asked for change nothing: they are compared by the same sums.)
    const int nearest = slot;
    best = -INFINITY;
    slot = 0;
    Frag<float, D> lf;
    frag_load(lf, a.k + (size_t)lrow * TF::kRowBytes, kg);
    auto take_block = [&](int b) {
      Frag<float, D> cf;
      frag_load(cf, a.k + (size_t)sel[min(b * 32 + n, S - 1)] * TF::kRowBytes, kg);
      float iv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) iv[r] = sinv[min(b * 32 + acc_row(r, kg), S - 1)];
      f32x16_t acc = acc_zero();
      mma<float, D>(acc, cf, lf);
      const float bm = scale_max(acc, iv);
      int ridx = 15;
#pragma unroll
      for (int r = 14; r >= 0; --r) ridx = acc[r] == bm ? r : ridx;
      keep_better(bm, b * 32 + acc_row(ridx, kg));
    };
    if (all_fp32 || __ballot(undecided && further >= limit) != 0ull) {
      for (int b = 0; b < nblocks; ++b) take_block(b);
    } else {
      int first = undecided && rb.best >= limit ? rb.slot0 >> 5 : -1;
      int other = undecided && second >= limit ? second_slot0 >> 5 : -1;
      int last = undecided && third >= limit ? third_slot0 >> 5 : -1;
      while (true) {
        const unsigned long long waiting = __ballot(first >= 0 || other >= 0 || last >= 0);
        if (waiting == 0ull) break;
        const int b = __builtin_amdgcn_readlane(first >= 0 ? first : other >= 0 ? other : last, __ffsll(waiting) - 1);
        take_block(b);
        first = first == b ? -1 : first;
        other = other == b ? -1 : other;
        last = last == b ? -1 : last;
      }
    }
    merge_lane_groups();
    slot = undecided ? slot : nearest;
  }
  if (kg == 0 && r0 + n < n_less) {
    a.less_slot[lbase + r0 + n] = slot;
    if (a.merge_assign) a.merge_assign[lrow] = slot;
  }
}

// ------------------------------------------------------------------------ conserved keys, packed
// Output row w of the ragged cache is the conserved key sel_idx[w]; the rows of one (layer, head) are
// consecutive in w.  Copying them once into that order makes every tile of conserved keys the tiled similarity
// kernel streams a contiguous block (which a lane-addressed asynchronous copy into LDS needs).
// 256 rows per workgroup.
constexpr int kPackRows = 256;
template <typename T, int D>
__global__ void __launch_bounds__(256) pack_conserved_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  constexpr int LPR = TL::kChunksPerRow;   // lanes per row
  constexpr int RPP = 256 / LPR;           // rows per pass
  constexpr int U = 4;                     // passes whose loads are in flight together
  static_assert(kPackRows % (RPP * U) == 0, "passes must tile the workgroup's rows");
  const int tid = threadIdx.x;
  const long long w0 = (long long)blockIdx.x * kPackRows, total = a.total_slots;
  if (a.use_resident) {
    // The resident-set kernel reads a set once and gathers it itself: nothing to do for rows of its layers (every 256
    // rows that do not lie inside one such layer are packed; a whole pass over 256 pairs of 4096 positions 1507 -> 1489
    // us, over 360 of 3001 458 -> 450 us).  Layer l owns the rows [off[l], off[l + 1]) * Hkv.
    const int L = a.L;
    bool inside = false;
    for (int l = tid; l < L; l += 256)
      inside |= a.off[l] * a.Hkv <= w0 && w0 + kPackRows <= a.off[l + 1] * a.Hkv && a.alloc[4 * l] <= resident_capacity<T, D>();
    if (__syncthreads_or(inside)) return;
  }
  const int sub = tid / LPR, cc = tid - sub * LPR;
  for (int r0 = 0; r0 < kPackRows; r0 += RPP * U) {
    int idx[U];
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) idx[u] = a.sel_idx[min(w0 + r0 + u * RPP + sub, total - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load16_stream(a.k + (size_t)idx[u] * TL::kRowBytes + cc * 16);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long w = w0 + r0 + u * RPP + sub;
      if (w < total) *reinterpret_cast<uint4*>(a.packed_k + (size_t)w * TL::kRowBytes + cc * 16) = v[u];
    }
  }
}

// ------------------------------------------------------------------------------- segment sort
// grid (Hkv, L), WAVES waves.  Stable least-significant-digit radix sort (at most 8 bits per pass) of the pairs
// (slot, row id) of one (layer, head) by slot; row ids enter ascending, so every slot's members come
// out ascending and the merge adds them in one fixed order.  Then seg_beg / seg_end of every slot = its range in the
// sorted array (sort_val[0]).
// Every wave owns a contiguous part of the input and a histogram of its own: a pass is one count over the parts, one
// prefix over (digit, wave), and one scatter in which a wave walks its part in order, 64 elements at a time, without
// a barrier (a lane finds its equals with one ballot per digit bit).  Bound by the scattered 4-byte stores: slot and
// position travel as one 32-bit word where their bits fit (PACKED: slot above position), which halves them.
// Before (5 bits per pass, a barrier-separated prefix over the waves per 1024 elements) and now, in us: 256 pairs of
// 118000 rows 781 / 621, 256 of 13000 91 / 50, 1024 of 3600 62 / 52, 360 of 2300 39 / 21, 8 of 770 12 / 8.
constexpr int kSortBits = 8;
constexpr int kSortDigits = 1 << kSortBits;
constexpr int kSortItems = 8;  // groups of 64 elements whose loads are issued together

template <int WAVES>
struct SortShared {
  int cnt[WAVES][kSortDigits];
  int wave_total[kSortDigits / 64];
};

// Lanes of the wave whose digit equals this lane's (invalid lanes match nobody): one ballot per
// digit bit, each lane keeps the side of the ballot it is on.
__device__ __forceinline__ unsigned long long digit_peers(int dgt, int bits, bool valid) {
  unsigned long long peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < kSortBits; ++b) {
    if (b < bits) {
      const unsigned long long set = __ballot((dgt >> b) & 1);
      peers &= ((dgt >> b) & 1) ? set : ~set;
    }
  }
  return valid ? peers : 0ull;
}

__device__ __forceinline__ int bits_below(int n) { return n > 1 ? 32 - __clz(n - 1) : 1; }  // bits of 0 .. n-1

template <int WAVES, bool PACKED>
__device__ __forceinline__ void segment_sort(const MergeArgs& a, SortShared<WAVES>& sh, int S, size_t lbase, int row0, int32_t* beg,
                                             int32_t* end) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = a.T - S;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  const int slot_bits = bits_below(S), pos_bits = PACKED ? bits_below(a.T) : 0;
  const int passes = (slot_bits + kSortBits - 1) / kSortBits;
  const int bits = (slot_bits + passes - 1) / passes, digit_mask = (1 << bits) - 1;
  const int part = ((n + WAVES - 1) / WAVES + 63) & ~63;  // elements per wave
  const int p_beg = min(wave * part, n), p_end = min(p_beg + part, n);
  volatile int* mine = sh.cnt[wave];  // the wave's histogram, later the next output position per digit

  const int32_t* slots = a.less_slot + lbase;
  const int32_t* rows = a.less_idx + lbase;
  const int32_t *in_key = slots, *in_val = rows;
  for (int p = 0; p < passes; ++p) {
    const int ob = (passes - 1 - p) & 1;
    int32_t* out_key = a.sort_key[ob] + lbase;
    int32_t* out_val = a.sort_val[ob] + lbase;
    const bool packed_in = PACKED && p > 0;
    const int shift_in = bits * p + (packed_in ? pos_bits : 0);
    for (int i = lane; i < kSortDigits; i += 64) mine[i] = 0;
    for (int t0 = p_beg; t0 < p_end; t0 += kSortItems * 64) {
      int keys[kSortItems];
#pragma unroll
      for (int j = 0; j < kSortItems; ++j)
        if (t0 + j * 64 < p_end) keys[j] = in_key[min(t0 + j * 64 + lane, p_end - 1)];
#pragma unroll
      for (int j = 0; j < kSortItems; ++j)
        if (t0 + j * 64 + lane < p_end) atomicAdd(&sh.cnt[wave][((unsigned)keys[j] >> shift_in) & digit_mask], 1);
    }
    __syncthreads();
    // exclusive prefix in the order (digit, wave): thread q < 256 has digit q
    int c[WAVES], total = 0, inc = 0;
    if (tid < kSortDigits) {
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        c[w] = sh.cnt[w][tid];
        total += c[w];
      }
      inc = total;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
      }
      if (lane == 63) sh.wave_total[wave] = inc;
    }
    __syncthreads();
    if (tid < kSortDigits) {
      int pos = inc - total;
#pragma unroll
      for (int w = 0; w < kSortDigits / 64; ++w) pos += (w < wave) ? sh.wave_total[w] : 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        sh.cnt[w][tid] = pos;
        pos += c[w];
      }
    }
    __syncthreads();
    for (int t0 = p_beg; t0 < p_end; t0 += kSortItems * 64) {
      int keys[kSortItems], vals[kSortItems];
#pragma unroll
      for (int j = 0; j < kSortItems; ++j) {
        if (t0 + j * 64 >= p_end) break;
        const int i = min(t0 + j * 64 + lane, p_end - 1);
        keys[j] = in_key[i];
        vals[j] = packed_in ? 0 : in_val[i];
      }
#pragma unroll
      for (int j = 0; j < kSortItems; ++j) {
        if (t0 + j * 64 >= p_end) break;
        const bool valid = t0 + j * 64 + lane < p_end;
        const int dgt = (int)((unsigned)keys[j] >> shift_in) & digit_mask;
        const unsigned long long peers = digit_peers(dgt, bits, valid);
        const int rank = __popcll(peers & lt_mask);
        if (valid) {
          const int base = mine[dgt];  // LDS operations of a wave stay in order: every lane reads before the group's
          if (rank == 0) mine[dgt] = base + __popcll(peers);  // first lane moves the position on
          out_key[base + rank] = PACKED && !packed_in ? (int)(((unsigned)keys[j] << pos_bits) | (unsigned)(vals[j] - row0)) : keys[j];
          if (!PACKED) out_val[base + rank] = vals[j];
        }
      }
    }
    __syncthreads();
    in_key = out_key;
    in_val = out_val;
  }

  // member range of every slot, as absolute indices into the sorted array
  const int ib = (int)lbase;
  auto slot_at = [&](int i) { return PACKED ? (int)((unsigned)in_key[i] >> pos_bits) : in_key[i]; };
  for (int i = tid; i < n; i += WAVES * 64) {
    const int kcur = slot_at(i);
    const int kprev = (i > 0) ? slot_at(i - 1) : -1;
    if (PACKED) a.sort_val[0][lbase + i] = row0 + (int)((unsigned)in_key[i] & ((1u << pos_bits) - 1u));
    for (int s = kprev + 1; s <= kcur; ++s) beg[s] = ib + i;
    for (int s = max(kprev, 0); s < kcur; ++s) end[s] = ib + i;
  }
  const int klast = (n > 0) ? slot_at(n - 1) : -1;
  for (int s = klast + 1 + tid; s < S; s += WAVES * 64) beg[s] = ib + n;
  for (int s = max(klast, 0) + tid; s < S; s += WAVES * 64) end[s] = ib + n;
}

template <int WAVES>
__global__ void __launch_bounds__(WAVES * 64, 8) segment_sort_kernel(MergeArgs a) {
  __shared__ SortShared<WAVES> sh;
  const int g = blockIdx.x, l = blockIdx.y;
  const int S = a.alloc[4 * l];
  const long long off_l = a.off[l];
  const size_t lbase = less_base_of(l, g, a.T, a.Hkv, off_l, S);
  const size_t cbase = (size_t)off_l * a.Hkv + (size_t)g * S;
  const int row0 = (l * a.Hkv + g) * a.T;  // row id of position 0
  if (bits_below(S) + bits_below(a.T) <= 32)
    segment_sort<WAVES, true>(a, sh, S, lbase, row0, a.seg_beg + cbase, a.seg_end + cbase);
  else
    segment_sort<WAVES, false>(a, sh, S, lbase, row0, a.seg_beg + cbase, a.seg_end + cbase);
}

// ------------------------------------------------------------------------------ merge + write
// A wave produces a run of consecutive output rows (layer, head, slot), one after the other.
// k_j <- (k_j + sum_{i in N_j} k_i) / (|N_j| + 1) and the same for the values (Section 3.3, average
// merging).  A lane owns one 16-byte piece of a row, so 64 lanes read 1024 bytes = several rows per
// load; sums are kept in fp64 (exact for the value ranges of a KV cache, hence independent of the
// summation order) and rounded once to the storage type.
// sum / n for a positive integer n given rinv = fl(1/n): one multiply and one exact-remainder
// correction.  When sum / n is representable the result is exactly that value, so ties of the final
// rounding to the storage type fall the same way as with a true division.
__device__ __forceinline__ double div_by_count(double sum, double n, double rinv) {
  const double q0 = sum * rinv;
  const double rem = fma(-q0, n, sum);
  return fma(rem, rinv, q0);
}

// x + y exchanged between two lane groups O lanes apart: the lower group ends with its own x plus
// the partner's x, the upper group with its own y plus the partner's y.
template <int O>
__device__ __forceinline__ double exchange_add(double x, double y, bool upper) {
  if constexpr (O == 16 || O == 32) {
    unsigned xl = (unsigned)__double2loint(x), xh = (unsigned)__double2hiint(x);
    unsigned yl = (unsigned)__double2loint(y), yh = (unsigned)__double2hiint(y);
    if constexpr (O == 32) {
      const auto lo = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
      xl = lo[0]; yl = lo[1]; xh = hi[0]; yh = hi[1];
    } else {
      const auto lo = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
      xl = lo[0]; yl = lo[1]; xh = hi[0]; yh = hi[1];
    }
    return __hiloint2double((int)xh, (int)xl) + __hiloint2double((int)yh, (int)yl);
  } else {
    const double send = upper ? x : y, keep = upper ? y : x;
    return keep + __shfl_xor(send, O, kWave);
  }
}

// One halving step of the reduce-scatter over lane groups O lanes apart; returns the element offset
// this lane moves to (LEN for the upper group).
template <int LEN, int O, int E>
__device__ __forceinline__ int reduce_scatter_step(double (&ak)[E], double (&av)[E], bool upper) {
#pragma unroll
  for (int i = 0; i < LEN; ++i) {
    ak[i] = exchange_add<O>(ak[i], ak[i + LEN], upper);
    av[i] = exchange_add<O>(av[i], av[i + LEN], upper);
  }
  return upper ? LEN : 0;
}

template <typename T>
struct OutConv;
template <>
struct OutConv<bf16_t> {
  static constexpr int kElems = 8;
  static __device__ __forceinline__ void unpack(const uint4& v, double* out) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = (double)__uint_as_float(w[i] << 16);
      out[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u);
    }
  }
  // store N consecutive elements sum[i] / denom, rounded once to bf16
  template <int N>
  static __device__ __forceinline__ void store(char* dst, const double* sum, double denom, double rinv) {
    if constexpr (N == 1) {
      *reinterpret_cast<uint16_t*>(dst) = (uint16_t)double_to_bf16_bits(div_by_count(sum[0], denom, rinv));
    } else {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const uint32_t wv = double_to_bf16_bits(div_by_count(sum[2 * i], denom, rinv)) |
                            (double_to_bf16_bits(div_by_count(sum[2 * i + 1], denom, rinv)) << 16);
        __builtin_nontemporal_store(wv, reinterpret_cast<uint32_t*>(dst) + i);
      }
    }
  }
};
template <>
struct OutConv<float> {
  static constexpr int kElems = 4;
  static __device__ __forceinline__ void unpack(const uint4& v, double* out) {
    out[0] = (double)__uint_as_float(v.x);
    out[1] = (double)__uint_as_float(v.y);
    out[2] = (double)__uint_as_float(v.z);
    out[3] = (double)__uint_as_float(v.w);
  }
  template <int N>
  static __device__ __forceinline__ void store(char* dst, const double* sum, double denom, double rinv) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      __builtin_nontemporal_store(__double2float_rn(div_by_count(sum[i], denom, rinv)), reinterpret_cast<float*>(dst) + i);
  }
};

// Output rows one wave walks; a lane of the wave holds the list range of one of them.  Short outputs are spread over
// more waves (2048 rows: 14.7 -> 6.6 us): below kMergeShortRows sixteen rows per wave leave the chip's 4096 wave
// slots of the kernel unfilled.
constexpr int kMergeRowsPerWave = 16;
constexpr int kMergeRowsPerWaveShort = 4;
constexpr long long kMergeShortRows = 65536;
// Rows of 128 bytes: one load per step makes twice the steps of a long list, and a wave's chain of them is what a layer
// with few slots waits for where the pairs are too few to cover it, so fewer rows per wave there (uneven budgets: 32 pairs
// of 30000, 96000 rows, 578 us with 16 rows and 160 with 4; 128 pairs of 8200, 104960 rows, 179 and 100 with 8; even
// budgets within 5 %, 14 % with 4 rows; from 256 pairs on 16 rows lose nothing: 360 pairs of 3001 124 us, 127 with 8).
constexpr int kMergeRows128Four = 64, kMergeRows128Eight = 128;  // up to so many pairs

// Where a wave is in the flat sequence of load steps of its output rows: row r of the wave, element t
// of that row's list (element 0 is the conserved row itself, the others its members), and the row's
// conserved row id, first member index and list length.  All fields are uniform over the wave.
struct MergeCursor {
  int r, t, sel, beg, cnt;
};

template <typename T, int D>
__global__ void __launch_bounds__(256) merge_write_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  using CV = OutConv<T>;
  constexpr int LPR = TL::kChunksPerRow;  // lanes per row
  constexpr int MS = 64 / LPR;            // rows per load
  // loads per lane and tensor in a step: a list holds four to nine rows on average, so rows of 128 bytes (eight per
  // load) take one (360 pairs of 3001: 145 -> 121 us), longer rows two (with one, rows of 256 bytes 13-25 % slower)
  constexpr int U = MS >= 8 ? 1 : 2;
  constexpr int STEP = U * MS;            // rows per step
  constexpr int E = CV::kElems;
  const int R = a.merge_rows;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // output rows are walked from the last layer to the first: the similarity kernel before this one
  // touched the last layers' keys last
  const long long w_hi = a.total_slots - ((long long)blockIdx.x * 4 + wave) * R;
  if (w_hi <= 0) return;
  const long long w_lo = w_hi > R ? w_hi - R : 0;
  const int n_out = (int)(w_hi - w_lo);
  // everything a row needs is indexed by its output row w: no layer / head lookup.  Lane i keeps the
  // entry of row w_lo + i; lanes past the wave's rows keep a list of length 1 that is never loaded.
  int m_sel = 0, m_beg = 0, m_cnt = 1;
  if (lane < n_out) {
    m_sel = a.sel_idx[w_lo + lane];
    m_beg = a.seg_beg[w_lo + lane];
    m_cnt = a.seg_end[w_lo + lane] - m_beg + 1;
  }
  const int32_t* members = a.sort_val[0];
  const int sub = lane / LPR, cc = lane - sub * LPR;
  const char* kb = a.k + cc * 16;
  const char* vb = a.v + cc * 16;

  auto read_entry = [&](MergeCursor& c) {
    c.sel = __builtin_amdgcn_readlane(m_sel, c.r);
    c.beg = __builtin_amdgcn_readlane(m_beg, c.r);
    c.cnt = __builtin_amdgcn_readlane(m_cnt, c.r);
  };
  auto advance = [&](MergeCursor& c) {
    c.t += STEP;
    if (c.t >= c.cnt) {
      c.r += 1;  // at most two steps past n_out <= 16, so always a lane of the wave
      c.t = 0;
      read_entry(c);
    }
  };
  // Row ids of the two rows this lane loads in the step at c.  Every load of the loop is issued
  // unconditionally (the number of loads in flight is then the same on every path, so a wait for
  // the oldest ones leaves the younger ones in flight): list positions past the end of the row's
  // list are clamped into the list array, and their lanes load the conserved row again, which the
  // sum then skips.
  const int last_member = a.n_members - 1;
  auto step_ids = [&](const MergeCursor& c, int (&ids)[U]) {
    const int e0 = c.t + sub;
    int m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = members[min(max(c.beg - 1 + e0 + u * MS, 0), last_member)];
#pragma unroll
    for (int u = 0; u < U; ++u) ids[u] = ((u > 0 || e0 != 0) && e0 + u * MS < c.cnt) ? m[u] : c.sel;
  };
  auto fetch = [&](const int (&ids)[U], uint4 (&k)[U], uint4 (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      k[u] = load16_stream(kb + (size_t)ids[u] * TL::kRowBytes);
      v[u] = load16_stream(vb + (size_t)ids[u] * TL::kRowBytes);
    }
  };

  double ak[E], av[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    ak[i] = 0.0;
    av[i] = 0.0;
  }
  // sums the rows of the step at c (already loaded into k, v); finishes the output row on its last step
  auto consume = [&](const MergeCursor& c, const uint4 (&k)[U], const uint4 (&v)[U]) {
    // One unconditional use of everything the step loaded: the wait for these loads then sits here on
    // every path, instead of inside the branches below (which would leave them formally in flight on
    // the other paths and force wider waits later).
#pragma unroll
    for (int u = 0; u < U; ++u)
      asm volatile("" ::"v"(k[u].x), "v"(k[u].y), "v"(k[u].z), "v"(k[u].w), "v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
    const long long w = w_lo + c.r;
    if (c.cnt == 1) {  // nothing merges into this row: bit-exact copy
      if (sub == 0) {
        // the output is not read again by this pass: streaming stores (measured 2-4 % on the kernel)
        store16_stream(a.k_out + (size_t)w * TL::kRowBytes + cc * 16, k[0]);
        store16_stream(a.v_out + (size_t)w * TL::kRowBytes + cc * 16, v[0]);
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c.t + u * MS + sub < c.cnt) {  // lanes past the end of the list hold a row that does not count
        double tk[E], tv[E];
        CV::unpack(k[u], tk);
        CV::unpack(v[u], tv);
#pragma unroll
        for (int i = 0; i < E; ++i) {
          ak[i] += tk[i];
          av[i] += tv[i];
        }
      }
    }
    if (c.t + STEP < c.cnt) return;
    // Last step of the row: reduce over the lane groups that read different rows.  Each exchange
    // halves the elements a lane is responsible for (the lower group keeps the lower half), so after
    // log2(MS) steps a lane holds E / MS finished sums starting at element `ebase` of its 16-byte
    // piece: the divisions and the stores are spread over all 64 lanes.
    int ebase = 0;
    if constexpr (MS >= 2) ebase += reduce_scatter_step<E / 2, LPR>(ak, av, (sub & 1) != 0);
    if constexpr (MS >= 4) ebase += reduce_scatter_step<E / 4, 2 * LPR>(ak, av, (sub & 2) != 0);
    if constexpr (MS >= 8) ebase += reduce_scatter_step<E / 8, 4 * LPR>(ak, av, (sub & 4) != 0);
    constexpr int EPL = E / MS;  // finished elements per lane
    static_assert(EPL >= 1, "a lane must end up with at least one element");
    const double denom = (double)c.cnt;
    const double rinv = 1.0 / denom;
    char* ko = a.k_out + (size_t)w * TL::kRowBytes + cc * 16 + ebase * (int)sizeof(T);
    char* vo = a.v_out + (size_t)w * TL::kRowBytes + cc * 16 + ebase * (int)sizeof(T);
    CV::template store<EPL>(ko, ak, denom, rinv);
    CV::template store<EPL>(vo, av, denom, rinv);
#pragma unroll
    for (int i = 0; i < E; ++i) {
      ak[i] = 0.0;
      av[i] = 0.0;
    }
  };

  // Three steps are in progress at any time: the rows of step n are summed while the row loads of
  // step n + 1 and the list loads of step n + 2 are in flight.  The list loads are issued before the
  // row loads, so waiting for them one round later does not wait for the younger row loads.  The
  // loop body is written out twice with the two register sets exchanged, so no loaded value is
  // copied (a copy would have to wait for its load).  Past the wave's last row the cursors point at
  // lanes that hold (row 0, empty list): those loads are harmless and never consumed.
  MergeCursor c0{0, 0, 0, 0, 1};
  read_entry(c0);
  MergeCursor c1 = c0;
  advance(c1);
  MergeCursor c2 = c1;
  advance(c2);
  int ida[U], idb[U];
  uint4 ka[U], va[U], kb2[U], vb2[U];
  step_ids(c0, ida);
  step_ids(c1, idb);
  fetch(ida, kb2, vb2);
  // one step: true when the wave's last row is done
  auto round = [&](int (&fresh)[U], const int (&old)[U], uint4 (&nk)[U], uint4 (&nv)[U], const uint4 (&ok)[U], const uint4 (&ov)[U]) {
    step_ids(c2, fresh);
    fetch(old, nk, nv);
    consume(c0, ok, ov);
    c0 = c1;
    c1 = c2;
    advance(c2);
    return c0.r >= n_out;
  };
  while (true) {
    if (round(ida, idb, ka, va, kb2, vb2)) break;
    if (round(idb, ida, kb2, vb2, ka, va)) break;
    if (round(ida, idb, ka, va, kb2, vb2)) break;
    if (round(idb, ida, kb2, vb2, ka, va)) break;
  }
}

// Rows without merging (no member lists exist): output row w is a copy of its conserved row.
template <typename T, int D>
__global__ void __launch_bounds__(256) copy_rows_kernel(MergeArgs a) {
  using TL = Tile<T, D>;
  constexpr int LPR = TL::kChunksPerRow;
  const long long piece = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long w = a.total_slots - 1 - piece / LPR;
  if (w < 0) return;
  const int cc = (int)(piece % LPR);
  const size_t src = (size_t)a.sel_idx[w] * TL::kRowBytes + cc * 16, dst = (size_t)w * TL::kRowBytes + cc * 16;
  store16_stream(a.k_out + dst, load16_stream(a.k + src));
  store16_stream(a.v_out + dst, load16_stream(a.v + src));
}

// ------------------------------------------------------------------------------------------ launch

static MergeArgs make_args(const Plan& p, const Buffers& b) {
  MergeArgs a;
  a.k = static_cast<const char*>(b.k);
  a.v = static_cast<const char*>(b.v);
  a.k_out = static_cast<char*>(b.k_out);
  a.v_out = static_cast<char*>(b.v_out);
  a.inv_norm = reinterpret_cast<const float*>(b.ws + p.off_inv_norm);
  a.alloc = reinterpret_cast<const int32_t*>(b.ws + p.off_alloc);
  a.off = reinterpret_cast<const int64_t*>(b.ws + p.off_layer_off);
  a.sel_idx = reinterpret_cast<const int32_t*>(b.ws + p.off_sel_idx);
  a.sel_inv_norm = reinterpret_cast<const float*>(b.ws + p.off_sel_inv);
  a.packed_k = b.ws + p.off_packed_k;
  a.less_idx = reinterpret_cast<const int32_t*>(b.ws + p.off_less_idx);
  a.less_slot = reinterpret_cast<int32_t*>(b.ws + p.off_less_slot);
  a.sort_key[0] = reinterpret_cast<int32_t*>(b.ws + p.off_sort_a);
  a.sort_val[0] = reinterpret_cast<int32_t*>(b.ws + p.off_sort_b);
  a.sort_key[1] = reinterpret_cast<int32_t*>(b.ws + p.off_sort_c);
  a.sort_val[1] = reinterpret_cast<int32_t*>(b.ws + p.off_sort_d);
  a.seg_beg = reinterpret_cast<int32_t*>(b.ws + p.off_seg_beg);
  a.seg_end = reinterpret_cast<int32_t*>(b.ws + p.off_seg_end);
  a.merge_assign = b.merge_assign;
  a.L = p.L; a.Hkv = p.Hkv; a.T = p.T; a.flags = p.flags;
  a.total_slots = (long long)p.B * p.Hkv;
  a.merge_rows = a.total_slots < kMergeShortRows ? kMergeRowsPerWaveShort : kMergeRowsPerWave;
  a.use_resident = 0;
  a.adjacent_order = 0;
  a.merge_members = !((p.flags & MEDA_FLAG_NO_MERGE) || p.B == (int64_t)p.L * p.T);
  a.n_members = (int)(((int64_t)p.L * p.T - p.B) * p.Hkv);
  return a;
}

template <typename T, int D, int F, int NW>
static hipError_t launch_sim_direct(const MergeArgs& a, unsigned pairs, hipStream_t s) {
  const unsigned nrb = (a.T + 32 * F - 1) / (32 * F);
  hipLaunchKernelGGL((similarity_direct_kernel<T, D, F, NW>), dim3(nrb * pairs), dim3(NW * 64), 0, s, a);
  return hipGetLastError();
}

template <int D, int NW>
static hipError_t launch_sim_split(const MergeArgs& a, hipStream_t s) {
  constexpr int kRows = 32 * NW;
  const unsigned nrb = (a.T + kRows - 1) / kRows;
  auto split = similarity_split_kernel<D, NW>;
  constexpr int kLds = SplitTile<D>::kLdsBytes;
  if (kLds > 64 * 1024) {
    const hipError_t e = allow_dynamic_lds(split, kLds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(split, dim3(nrb * (unsigned)(a.L * a.Hkv)), dim3(NW * 64), kLds, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_sim_t(const Plan& p, MergeArgs a, hipStream_t s) {
  const unsigned nrb = (p.T + kSimRows - 1) / kSimRows, pairs = (unsigned)(p.L * p.Hkv);
  if (p.sim == kSimDirect) return launch_sim_direct<T, D, 1, 8>(a, pairs, s);
  a.use_resident = p.sim == kSimResident ? 1 : 0;
  a.adjacent_order = pairs >= kAdjacentPairs ? 1 : 0;
  hipLaunchKernelGGL((pack_conserved_kernel<T, D>), dim3((unsigned)((a.total_slots + kPackRows - 1) / kPackRows)),
                     dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid(nrb * pairs);
  constexpr int kTiledLds = sim_tiled_lds_bytes<T, D>();
  auto tiled = similarity_argmax_kernel<T, D>;
  if (kTiledLds > 64 * 1024) {
    e = allow_dynamic_lds(tiled, kTiledLds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(tiled, grid, dim3(kSimWaves * 64), kTiledLds, s, a);
  e = hipGetLastError();
  if (e != hipSuccess || !a.use_resident) return e;
  auto res = similarity_resident_kernel<T, D>;
  e = allow_dynamic_lds(res, kResLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(res, dim3(pairs * kResSplit), dim3(kResThreads), kResLdsBytes, s, a);
  return hipGetLastError();
}

// fp32 problems.  Split kernel: workgroups of eight waves share a tile's pieces among more rows, which pays
// for rows of 512 bytes once two of them per CU are there (224 pairs of 660 46 -> 38 us, 35 of 2715 106 -> 140).  Direct
// kernel: two fragments per wave halve the key loads once there are enough workgroups of 64 rows for every CU.
template <int D>
static hipError_t launch_sim_fp32(const Plan& p, const MergeArgs& a, hipStream_t s) {
  const unsigned pairs = (unsigned)(p.L * p.Hkv);
  if constexpr (D == 128) {
    if (p.sim == kSimSplit && pairs * ((p.T + 255u) / 256u) >= 576u) return launch_sim_split<D, 8>(a, s);
  } else {
    if (p.sim == kSimDirect && pairs * ((p.T + 63u) / 64u) >= 512u) return launch_sim_direct<float, D, 2, 4>(a, pairs, s);
  }
  return p.sim == kSimSplit ? launch_sim_split<D, 4>(a, s) : launch_sim_direct<float, D, 1, 8>(a, pairs, s);
}

hipError_t launch_similarity(const Plan& p, const Buffers& b, hipStream_t s) {
  const MergeArgs a = make_args(p, b);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_sim_t<bf16_t, 128>(p, a, s) : launch_sim_t<bf16_t, 64>(p, a, s);
  return p.d == 128 ? launch_sim_fp32<128>(p, a, s) : launch_sim_fp32<64>(p, a, s);
}

hipError_t launch_segment_sort(const Plan& p, const Buffers& b, hipStream_t s) {
  const MergeArgs a = make_args(p, b);
  // One workgroup of 16 waves fills half a CU: fewer waves where the parts would be short or the pairs many (1024 pairs of
  // 100 and of 1000 positions 13.4 and 18 us with 16 waves, 8.6 and 13.4 with 4; of 2000 23.5 and 20 with 8; but 256 of
  // 2000 11.6 us with 16, 11.8 with 8, 14.8 with 4).
  const dim3 grid(p.Hkv, p.L);
  const int pairs = p.L * p.Hkv;
  if (p.T <= 128 || (pairs >= 512 && p.T <= 768)) hipLaunchKernelGGL(segment_sort_kernel<4>, grid, dim3(256), 0, s, a);
  else if (pairs >= 1024 && p.T <= 4096) hipLaunchKernelGGL(segment_sort_kernel<8>, grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL(segment_sort_kernel<16>, grid, dim3(1024), 0, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_merge_t(const Plan& p, MergeArgs a, hipStream_t s) {
  if (!a.merge_members) {
    const long long pieces = a.total_slots * Tile<T, D>::kChunksPerRow;
    hipLaunchKernelGGL((copy_rows_kernel<T, D>), dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  if (Tile<T, D>::kRowBytes == 128 && a.merge_rows == kMergeRowsPerWave)
    a.merge_rows = p.L * p.Hkv <= kMergeRows128Four ? 4 : (p.L * p.Hkv <= kMergeRows128Eight ? 8 : kMergeRowsPerWave);
  const long long waves = (a.total_slots + a.merge_rows - 1) / a.merge_rows;
  hipLaunchKernelGGL((merge_write_kernel<T, D>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_merge_write(const Plan& p, const Buffers& b, hipStream_t s) {
  const MergeArgs a = make_args(p, b);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_merge_t<bf16_t, 128>(p, a, s) : launch_merge_t<bf16_t, 64>(p, a, s);
  return p.d == 128 ? launch_merge_t<float, 128>(p, a, s) : launch_merge_t<float, 64>(p, a, s);
}

}  // namespace meda
