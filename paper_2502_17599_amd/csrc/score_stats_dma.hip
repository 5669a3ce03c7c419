// Pass A of the scoring (Sections 3.2 and 3.3) for grouped query heads and for the row-block mode: row maxima and softmax
// normalisers of the scoring rows, and 1/|k| of every key, with the key tiles brought into LDS by asynchronous copies.
//
// grid (NCH, Hkv, L), or (Hkv * row blocks, 1, L) in the row-block mode; NCG * CS waves at work.  Wave (cg, cs) keeps NQ
// query fragments ((head of the group, row block) pairs cg*NQ .. cg*NQ+NQ-1) in registers and visits the 32-key blocks
// sb = cs, cs+CS, ... of every tile of its chunk.  The keys are operand A, the queries operand B, so a lane owns one
// query row and 16 keys per block: the running (max, Z_vision, Z_text) of the row are three registers per fragment and
// need no cross-lane traffic until the end.
//
// Two LDS tiles of 128 keys (CopyTile in device_utils.hpp): the copies of tile t+1 are issued when tile t starts, one wait
// and one barrier per tile, no staging registers; the modality bits of a tile are a ballot of one byte per lane that
// every wave loads for itself one tile ahead.  Tiles whose keys every row of the workgroup sees have a loop of their own.
// Bound by the vector unit (a probability costs a multiply-add, an exponential, an addition and half a maximum) and by the
// barriers: up to 16 pairs per kv head go to four waves (of up to four fragments each), so that two workgroups fit on a CU
// and one computes while the other waits.  14 pairs (28 layers of 37376, 7 heads per kv head, 64 rows) with eight waves of
// two fragments 759 us, with four of four 613; row blocks of 16 pairs (32 layers, 32 heads, 4096 positions) 2950 -> 2760;
// 8 pairs (four waves of two in both): 400 -> 370 with the separate loops.
#include "score_common.hpp"

namespace meda {

constexpr int kStatTile = 128;  // keys per tile

template <typename T, int D, int NQ, int NW, bool BLOCKS>
__global__ void __launch_bounds__(NW * 64, 2) score_stats_dma_kernel(ScoreArgs a) {
  using TL = Tile<T, D>;
  using CT = CopyTile<T, D>;
  constexpr int RBt = TL::kRowBytes;
  constexpr int CPR = TL::kChunksPerRow;
  constexpr int RPI = CT::kRows;
  constexpr int kTileBytes = CT::bytes(kStatTile);
  constexpr int NI = kStatTile / RPI;              // copy instructions of a tile
  constexpr int PF = (NI + NW - 1) / NW;           // per wave
  static_assert(NI % NW == 0, "the copy instructions must tile a tile evenly");
  extern __shared__ __align__(16) char smem[];  // two tiles

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
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, n = lane & 31, kg = lane >> 5;
  const int cgi = wave % a.NCG, cs = wave / a.NCG;
  const bool active = cs < a.CS;  // the workgroup is padded to 4 or 8 waves; spare waves only move data
  const int n_combos = a.G * a.RB;

  Frag<T, D> qf[NQ];
  float m[NQ], zv[NQ], zt[NQ];
  int qlast[NQ];  // position of the last row of the fragment's 32-row block (uniform over the wave)
  int nvalid = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int cidx = cgi * NQ + q;
    m[q] = kNegBig;
    zv[q] = 0.f;
    zt[q] = 0.f;
    qlast[q] = -1;
    frag_zero(qf[q]);
    if (active && cidx < n_combos) {
      nvalid = q + 1;
      const int hg = cidx / a.RB, rb = cidx - hg * a.RB;
      qlast[q] = a.T - a.W + rb * 32 + 31;
      if (rb * 32 + n < a.W)
        frag_load(qf[q], a.q + ((size_t)(l * a.Hq + g * a.G + hg) * a.q_rows + a.q_row0 + rb * 32 + n) * TL::kRowBytes, kg);
    }
  }

  const uint8_t* mask = a.mask + (size_t)(l / a.Lseq) * a.Tk;  // this layer's sequence
  const int jbeg = ch * a.CH;
  const int jend = min(a.T, jbeg + a.CH);
  const char* kbase = uniform_ptr(a.k + (size_t)(l * a.Hkv + g) * a.Tk * TL::kRowBytes);
  float* invn_out = a.inv_norm + (size_t)(l * a.Hkv + g) * a.Tk;

  // Copy instruction c of this wave fills the rows (wave * PF + c) * RPI .. + RPI-1 of a tile, this lane brings one 16-byte
  // chunk; rows past the end of the sequence repeat the last key (their columns are masked below).
  const int crow = wave * PF * RPI + lane / CPR;
  const unsigned chunk = CT::source_chunk(lane);
  const unsigned fbase = CT::frag_base(n, kg);
  const unsigned lds0 = (unsigned)(size_t)smem;
  uint8_t mk0 = 0, mk1 = 0;  // modality bytes of the keys lane and 64 + lane of the next tile
  auto issue = [&](int jt, int slot) {
#pragma unroll
    for (int c = 0; c < PF; ++c)
      async_copy16_to_lds_stream(kbase, (unsigned)min(jt + crow + c * RPI, a.T - 1) * RBt + chunk,
                                 lds0 + (unsigned)(slot * kTileBytes + (wave * PF + c) * CT::kPiece));
    mk0 = mask[min(jt + lane, a.T - 1)];
    mk1 = mask[min(jt + 64 + lane, a.T - 1)];
  };

  int slot = 0;
  // The tiles from j_from on, up to j_to.  MASKED: some key of a tile is not seen by some row of the workgroup.
  auto walk = [&](int j_from, int j_to, auto masked_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    for (int j0 = j_from; j0 < j_to; j0 += kStatTile, slot ^= 1) {
      async_copy_wait<0>();  // this wave's pieces of the tile have landed
      __syncthreads();       // every wave's have; and nobody reads the other tile (the previous one) any more
      const unsigned long long vis0 = __ballot(mk0 != 0), vis1 = __ballot(mk1 != 0);
      if (j0 + kStatTile < jend) issue(j0 + kStatTile, slot ^ 1);
      const char* tile = smem + slot * kTileBytes;
      for (int sb = cs; active && sb < kStatTile / 32; sb += a.CS) {
        const int jb = j0 + sb * 32;
        if (MASKED && jb >= a.T) break;
        Frag<T, D> kf;
        frag_from_tile(kf, tile + CT::bytes(32) * sb, fbase);
        // 1/|k| of the block's keys, by one of the waves that have them; the first row block sees every key
        if (bi == 0 && (jb >> 5) % a.NCG == cgi) {
          const float inv = inverse_norm(kf);
          if (kg == 0 && (!MASKED || jb + n < a.T)) invn_out[jb + n] = inv;
        }
        const uint32_t mword = (uint32_t)((sb & 2 ? vis1 : vis0) >> ((sb & 1) * 32));
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          // A fragment's 32 rows sit at the positions qlast-31 .. qlast: keys after qlast are invisible to all of them
          // (nothing to add), keys up to qlast-31 are visible to all of them (no per-element test needed).
          if (q >= nvalid || (MASKED && jb > qlast[q])) continue;
          f32x16_t acc = acc_zero();
          mma<T, D>(acc, kf, qf[q]);
          if (!MASKED || jb + 31 <= qlast[q] - 31)
            stats_add_plain(acc, a.c, mword, kg, m[q], zv[q], zt[q]);
          else
            stats_add_masked(acc, a.c, mword, kg, min(a.T - 1, qlast[q] - 31 + n) - jb, m[q], zv[q], zt[q]);
        }
      }
    }
  };
  if (jbeg < jend) issue(jbeg, 0);
  // plain tiles: their last key is not past the first row of the workgroup
  const int n_plain = max(0, min(jend, a.T - a.W + 1) - jbeg) / kStatTile;
  walk(jbeg, jbeg + n_plain * kStatTile, std::false_type{});
  walk(jbeg + n_plain * kStatTile, jend, std::true_type{});

  // the partial of every row over this workgroup's keys
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (q < nvalid) {
      const float4 part = stats_merge_halves(m[q], zv[q], zt[q]);
      const int hg = (cgi * NQ + q) / a.RB, row = (cgi * NQ + q - hg * a.RB) * 32 + n;
      if (kg == 0 && row < a.W) {
        const size_t row_id = (size_t)(l * a.Hq + g * a.G + hg) * a.stats_rows + a.stats_row0 + row;
        a.stats_part[row_id * a.NPART + ch * a.CS + cs] = part;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------ launch

template <typename T, int D, int NQ, int NW>
static hipError_t launch_dma_w(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  constexpr int kLds = 2 * CopyTile<T, D>::bytes(kStatTile);
  // (row blocks along x: the device promises 65536 workgroups along y)
  const dim3 grid = p.blocks ? dim3(p.Hkv * p.n_blocks_a, 1, p.L) : dim3(p.NCH, p.Hkv, p.L), block(NW * 64);
  auto kern = p.blocks ? score_stats_dma_kernel<T, D, NQ, NW, true> : score_stats_dma_kernel<T, D, NQ, NW, false>;
  if (kLds > 64 * 1024) {
    hipError_t e = allow_dynamic_lds(kern, kLds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, grid, block, kLds, s, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_dma_d(const Plan& p, const ScoreArgs& a, hipStream_t s) {
  const bool four = p.NCG * p.CS <= 4;  // (always up to 16 pairs)
  switch (p.NQ) {
    case 1: return launch_dma_w<T, D, 1, 4>(p, a, s);
    case 2: return launch_dma_w<T, D, 2, 4>(p, a, s);
    case 3: return launch_dma_w<T, D, 3, 4>(p, a, s);
    default: return four ? launch_dma_w<T, D, 4, 4>(p, a, s) : launch_dma_w<T, D, 4, 8>(p, a, s);
  }
}

// Grouped heads and the row-block mode: bound by the vector unit, not by the stream of the keys.
bool score_stats_dma_supported(const Plan& p) { return p.d * p.elt <= 256 && (p.blocks || p.G >= 2); }

hipError_t launch_score_stats_dma(const Plan& p, const Buffers& b, hipStream_t s) {
  const ScoreArgs a = make_args(p, b, true);
  if (p.dtype == MEDA_BF16) return p.d == 128 ? launch_dma_d<bf16_t, 128>(p, a, s) : launch_dma_d<bf16_t, 64>(p, a, s);
  return launch_dma_d<float, 64>(p, a, s);
}

}  // namespace meda
