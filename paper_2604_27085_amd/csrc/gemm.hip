// bf16 GEMM on the gfx950 matrix cores: C = A*B with fp32 accumulation, v_mfma_f32_32x32x16_bf16.
//
// Every wave owns a 128x64 block of C (4x2 MFMA tiles, 128 accumulator registers); a workgroup is a WGM x WGN grid of
// such waves.  Two waves per SIMD keep the matrix pipeline fed: while one wave waits at a barrier, on LDS or on HBM,
// the other one issues MFMAs.
//
//   256x256 (2x4 waves, K tile 64, the whole LDS of a CU), 256x128 with two groups of 2x2 waves (K tile 64)
//
// The smaller tiles are in gemm_mid.hip; which one a product takes is decided by the cost model of choose() below.
//
// Operands are staged through registers (16-byte buffer loads; rows outside the matrix read as zero through the
// descriptor, so the loop has no branch) and LDS is double buffered.  The K loop is written slot by slot -- one MFMA
// followed by that slot's share of memory instructions, pinned with scheduling barriers: the fragments of the next
// 16-deep step are read at the start of a step; every 16-byte staging chunk rotates on its own (stored to LDS, then
// reloaded with the tile after next), so that global loads and LDS stores arrive evenly instead of in bursts that
// stall MFMA issue behind a full memory queue, and every load has a whole tile of time to return; the workgroup
// barrier sits before the last four MFMAs of a tile and the first fragments of the next tile are read under them.
// Measured on MI355X the 256x256 tile asks L2 for one byte per 128 FLOP; the matrix pipe is busy 75-79 % of the kernel's
// cycles and the chip runs power-limited near 1.65 GHz under it.  Tried and dropped here: touching lines two tiles
// ahead to pull them into L2, touching the first lines of the workgroup's successor tile before the epilogue,
// staggered K-loop starts, a reduction split merged by the last workgroup to arrive.  Most products on 256x256 tiles run
// on a kernel of their own (gemm_dtl.hip: four waves of 128x128, one per SIMD, operands loaded straight into LDS); the eight-wave 256x256
// kernel here is for short reductions and skinny outputs, and the reference that one is tested against bit for bit.
// Outputs too small to fill the chip with 256x256 tiles use a 256x128 tile worked
// on by two wave groups that split every K tile (merged through LDS) or the small tiles; products that would still leave
// CUs idle are split along the reduction: the slices write partial products to scratch memory and a
// second kernel adds them in slice order (reproducible run to run).  A variant keeps the B operand out of LDS (BD).
//
// Operands whose reduction index is not contiguous in memory (the weight in an activation-gradient GEMM, both operands
// of a weight-gradient GEMM) keep their memory layout in LDS and are read with the transposing LDS load, so all
// three layouts run the same code.  The epilogue stages each wave's block through LDS (16-byte global accesses).
#include "gemm_device.hpp"
#include <stdlib.h>
#include <type_traits>

using namespace gemm_dev;

namespace {

// Copies a tile of one operand from HBM to LDS through registers, NREG 16-byte chunks per thread.
template <int BX, int BK, int NTHR, bool TR>
struct TileLoader {
  using S = TileShape<BX, BK, TR>;
  static constexpr int NREG = S::ROWS * S::CH / NTHR;
  static constexpr int RSTEP = NTHR / S::CH;               // tile rows between a thread's consecutive chunks
  static_assert((S::ROWS * S::CH) % NTHR == 0 && NTHR % S::CH == 0, "tile does not divide over the threads");
  uint32_t voff[NREG];
  uint32_t kstep;
  int row0, ch;

  // fold_half (only !TR): the tile's rows are the two halves of a folded index range -- rows [0, BX/2) are x0/2 + row,
  // rows [BX/2, BX) are fold_half + x0/2 + row - BX/2 (the gate and up rows of one SwiGLU column block).
  // row_map (only !TR): row gx is read from row row_map[gx] of the buffer.
  RP_DEV void init(long ld, int x0, int Xdim, int tid, int fold_half = 0, const int* row_map = nullptr) {
    row0 = tid / S::CH;
    ch = tid % S::CH;
    kstep = TR ? (uint32_t)ld * 2u : 2u;
#pragma unroll
    for (int it = 0; it < NREG; ++it) {
      const int row = row0 + it * RSTEP;
      if constexpr (!TR) {
        const int gl = fold_half ? (x0 >> 1) + (row < BX / 2 ? row : row - BX / 2) : x0 + row;
        const int gx = fold_half && row >= BX / 2 ? fold_half + gl : gl;
        const bool in = gl < (fold_half ? fold_half : Xdim);
        const long src = (row_map && in) ? row_map[gx] : gx;
        voff[it] = in ? (uint32_t)(src * ld + ch * 8) * 2u : OOB;
      } else {
        const int gx = x0 + ch * 8;
        voff[it] = gx < Xdim ? (uint32_t)((long)row * ld + gx) * 2u : OOB;
      }
    }
  }

  // Loads the tile whose reduction range starts at k0; chunks past Klim read as zero.
  RP_DEV void load(uint4 (&r)[NREG], rsrc_t rs, int k0, int Klim) const {
    const uint32_t soff = (uint32_t)k0 * kstep;
#pragma unroll
    for (int it = 0; it < NREG; ++it) {
      const bool kok = TR ? (k0 + row0 + it * RSTEP) < Klim : (k0 + ch * 8) < Klim;
      r[it] = buf_load16(rs, kok ? voff[it] : OOB, soff);
    }
  }

  RP_DEV void store(const uint4 (&r)[NREG], bf16* Sm) const {
#pragma unroll
    for (int it = 0; it < NREG; ++it) *reinterpret_cast<uint4*>(Sm + (row0 + it * RSTEP) * S::LDROW + ch * 8) = r[it];
  }

  // One chunk at a time, for the steady state of the K loop; `other` is the loader of the second operand pair (same
  // thread -> chunk mapping), selected without a branch when second is set.
  RP_DEV uint4 load_one(int it, const TileLoader& other, bool second, rsrc_t rs, int k0, int Klim) const {
    const uint32_t vo = second ? other.voff[it] : voff[it];
    const uint32_t kst = second ? other.kstep : kstep;
    const bool kok = TR ? (k0 + row0 + it * RSTEP) < Klim : (k0 + ch * 8) < Klim;
    return buf_load16(rs, kok ? vo : OOB, (uint32_t)k0 * kst);
  }
  RP_DEV void store_one(int it, const uint4& r, bf16* Sm) const {
    *reinterpret_cast<uint4*>(Sm + (row0 + it * RSTEP) * S::LDROW + ch * 8) = r;
  }
};

// KG wave groups share one output tile: group g runs the 16-deep steps [g*KS/KG, (g+1)*KS/KG) of every K tile, and the
// groups' accumulators are added through LDS before the epilogue.  With KG = 2 a 256x128 tile is worked on by eight
// waves of 128x64 each, which fills the chip with half as many output elements as the 256x256 tile needs.
template <int WGM, int WGN, int BK, bool TA, bool TB, int KG = 1>
struct Cfg {
  static constexpr int BM = WGM * WAVE_M, BN = WGN * WAVE_N, NWT = WGM * WGN, NW = NWT * KG, NTHR = NW * 64;
  static_assert((BK / 16) % KG == 0, "the K tile does not divide over the wave groups");
  static_assert(KG == 1 || NW * (TM * 16 * 64 * 4) <= 160 * 1024, "accumulator exchange does not fit in LDS");
  using LA = TileLoader<BM, BK, NTHR, TA>;
  using LB = TileLoader<BN, BK, NTHR, TB>;
  static constexpr int MAIN_BYTES = 2 * (LA::S::ELEMS + LB::S::ELEMS) * 2;
  static constexpr int XCH_BYTES = KG > 1 ? NW * (TM * 16 * 64 * 4) : 0;   // every wave hands over one column of MFMA tiles
  static constexpr int SMEM0 = MAIN_BYTES > NW * STG_BYTES ? MAIN_BYTES : NW * STG_BYTES;   // every wave stages
  static constexpr int SMEM = SMEM0 > XCH_BYTES ? SMEM0 : XCH_BYTES;
  // waves per SIMD the register budget is set for
  static constexpr int WPS = (NW == 8) ? 2 : (SMEM * 2 <= 160 * 1024 ? 2 : 1);
};

// GATED: the conditional instance (a name of its own in profiles): returns at once unless *p.run_flag is set.
// BD: the B operand does not pass through LDS.  p.B (and p.B2) point at copies in MFMA fragment order (gemm_arrange):
// every wave streams the fragments of its 64 columns straight into registers, 1 KB per load instruction, through a ring
// that holds one K tile and is refilled fragment by fragment right after a fragment's last MFMA -- a whole K tile of
// latency per load.  Half of the LDS stores and a third of the LDS reads of the staged kernel go away.
//
// GRP: grouped mode.  Tile rows are the entries of the table.
template <int WGM, int WGN, int BK, bool TA, bool TB, int KG, bool GATED, bool BD, bool GRP>
__global__ void __launch_bounds__(WGM* WGN* KG * 64)
    __attribute__((amdgpu_waves_per_eu(Cfg<WGM, WGN, BK, TA, TB, KG>::WPS, Cfg<WGM, WGN, BK, TA, TB, KG>::WPS)))
    gemm_kernel(const GemmArgs p) {
  using C = Cfg<WGM, WGN, BK, TA, TB, KG>;
  using LA = typename C::LA;
  using LB = typename C::LB;
  constexpr int BM = C::BM, BN = C::BN, KS = BK / 16, KSL = KS / KG;
  constexpr int LDA = LA::S::LDROW, LDB = LB::S::LDROW;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16* const sA0 = reinterpret_cast<bf16*>(smem);
  bf16* const sB0 = sA0 + LA::S::ELEMS;
  bf16* const sA1 = sB0 + LB::S::ELEMS;
  bf16* const sB1 = sA1 + LA::S::ELEMS;

  if constexpr (GATED) {
    if (*p.run_flag == 0) return;                      // uniform over the grid
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int kg = wave / C::NWT, wmn = wave % C::NWT;   // wave group, wave within the output tile
  const int wm = wmn / WGN, wn = wmn % WGN;
  const int ks0 = kg * KSL;

  int tile_m, tile_n, m0, Mlim = p.M;
  const bf16* Bbase = static_cast<const bf16*>(p.B);
  const int* row_map = nullptr;
  if constexpr (GRP) {
    static_assert(!TA && KG == 1 && !GATED && !BD && BM == 256, "grouped mode");
    const int tiles_n = (p.N + BN - 1) / BN;
    tile_m = (int)blockIdx.x / tiles_n;
    tile_n = (int)blockIdx.x % tiles_n;
    if (tile_m >= *p.grp_ntiles) return;
    const int4 g = p.grp_tab[tile_m];
    m0 = g.y;
    Mlim = g.y + g.z;
    Bbase += (long)g.x * p.grp_strideB;
    row_map = p.row_map;
  } else {
    tile_of_block(p.M, p.N, BM, BN, tile_m, tile_n);
    m0 = tile_m * BM;
  }
  const int n0 = tile_n * BN;
  const int nk1 = (p.K + BK - 1) / BK;
  const int nk_all = nk1 + (p.K2 + BK - 1) / BK;
  // split along the reduction: slice blockIdx.y takes K tiles [kt0, kt0 + nk)
  const int per_split = (nk_all + (int)gridDim.y - 1) / (int)gridDim.y;
  const int kt0 = (int)blockIdx.y * per_split;
  const int nk = (nk_all - kt0) < per_split ? (nk_all - kt0 > 0 ? nk_all - kt0 : 0) : per_split;

  LA la, la2;
  LB lb, lb2;
  la.init(p.lda, m0, Mlim, tid, 0, row_map);
  const int fold = (!TB && p.epi == EPI_SWIGLU_FWD) ? p.N >> 1 : 0;   // uniform
  lb.init(p.ldb, n0, p.N, tid, fold);
  const rsrc_t rsA = make_rsrc(p.A, p.bytesA), rsB = make_rsrc(Bbase, p.bytesB);
  rsrc_t rsA2 = rsA, rsB2 = rsB;
  la2 = la;
  lb2 = lb;
  if (p.K2 > 0) {
    la2.init(p.lda2, m0, p.M, tid);
    lb2.init(p.ldb2, n0, p.N, tid, fold);
    rsA2 = make_rsrc(p.A2, p.bytesA2);
    rsB2 = make_rsrc(p.B2, p.bytesB2);
  }
  // Staging registers: chunk r < LA::NREG belongs to the A tile, the others to the B tile.  In the steady state
  // every chunk rotates on its own: at its slot of K tile kt it is stored to LDS (it holds tile kt+1, loaded one
  // tile earlier) and immediately reloaded with tile kt+2, so global loads and LDS stores are spread evenly over
  // the MFMAs of a tile instead of arriving in bursts, and every load has a full tile of time to return.
  static_assert(!BD || (KG == 1 && BK == 64), "the direct B path is built for one wave group and K tiles of 64");
  constexpr int NLD = LA::NREG + (BD ? 0 : LB::NREG);
  static_assert(NLD % KSL == 0, "staging chunks do not divide over the steps of a K tile");
  uint4 rg[NLD];
  struct Seg { bool second; int k0, Klim; };
  auto seg_of = [&](int kt_local) {
    const int kt = kt0 + kt_local;
    const bool second = kt >= nk1;
    return Seg{second, (second ? kt - nk1 : kt) * BK, second ? p.K2 : p.K};
  };
  auto load_chunk = [&](int r, const Seg& sg) {
    if (r < LA::NREG) rg[r] = la.load_one(r, la2, sg.second, sg.second ? rsA2 : rsA, sg.k0, sg.Klim);
    else rg[r] = lb.load_one(r - LA::NREG, lb2, sg.second, sg.second ? rsB2 : rsB, sg.k0, sg.Klim);
  };
  auto store_chunk = [&](int r, bf16* sa, bf16* sb) {
    if (r < LA::NREG) la.store_one(r, rg[r], sa);
    else lb.store_one(r - LA::NREG, rg[r], sb);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // direct B path: fragment (ks, j) of K tile t of the wave's 64-column block blk lies at
  // (((blk * tiles_in_segment + t) * KS + ks) * TN + j) KB of the arranged copy, 16 bytes per lane
  [[maybe_unused]] uint4 bq[KS][TN];
  [[maybe_unused]] const uint32_t bd_blk = (uint32_t)(n0 / WAVE_N + wn);
  [[maybe_unused]] const uint32_t bd_nk2 = (uint32_t)((p.K2 + BK - 1) / BK);
  [[maybe_unused]] auto bd_load = [&](int ks, int j, const Seg& sg) {
    const uint32_t t = bd_blk * (sg.second ? bd_nk2 : (uint32_t)nk1) + (uint32_t)(sg.k0 / BK);
    return buf_load16(sg.second ? rsB2 : rsB, ((t * KS + ks) * TN + j) * 1024u + (uint32_t)lane * 16u, 0u);
  };

  if (nk > 0) {
    const Seg s0 = seg_of(0);
    if constexpr (BD) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int j = 0; j < TN; ++j) bq[ks][j] = bd_load(ks, j, s0);
    }
#pragma unroll
    for (int r = 0; r < NLD; ++r) load_chunk(r, s0);
#pragma unroll
    for (int r = 0; r < NLD; ++r) store_chunk(r, sA0, sB0);
    if (nk > 1) {
      const Seg s1 = seg_of(1);
#pragma unroll
      for (int r = 0; r < NLD; ++r) load_chunk(r, s1);
    }
  }
  __syncthreads();

  const int offA = frag_base<LDA, TA>(lane, wm * WAVE_M);
  const int offB = frag_base<LDB, TB>(lane, wn * WAVE_N);
  uint4 af[2][TM], bfr[2][TN];
  auto load_frags = [&](int buf, const bf16* pa, const bf16* pb, int ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) af[buf][i] = read_frag<LDA, TA>(pa, i * 32, ks);
    if constexpr (!BD) {
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[buf][j] = read_frag<LDB, TB>(pb, j * 32, ks);
    }
  };
  // One K tile.  STORE: tile kt+1 exists (its chunks are in the staging registers); LOAD: tile kt+2 exists.
  // The tile is a flat sequence of S = KSL * NM slots, one MFMA each, followed by that slot's share of the memory
  // instructions, with a scheduling barrier so that the compiler keeps the order:
  //   - the fragments of the next 16-deep step, one read per slot at the start of a step;
  //   - the chunk rotations, spread evenly over slots 0 .. S-5;
  //   - before slot S-4 the workgroup barrier: by then every wave has stored its chunks of tile kt+1 and has all its
  //     fragments of tile kt in registers, so the first fragments of tile kt+1 are read under the last four MFMAs
  //     and the next tile may overwrite this tile's buffer.
  constexpr int NM = TM * TN, NF = TM + (BD ? 0 : TN), S = KSL * NM, TAIL = 4;
  static_assert(NF <= NM && KSL % 2 == 0 && NLD <= S - TAIL, "slot plan does not fit");
  load_frags(0, sA0 + offA, sB0 + offB, ks0);
  auto tile = [&](int kt, auto store_tag, auto load_tag) {
    constexpr bool STORE = decltype(store_tag)::value, LOAD = decltype(load_tag)::value;
    const bf16* pa = ((kt & 1) ? sA1 : sA0) + offA;
    const bf16* pb = ((kt & 1) ? sB1 : sB0) + offB;
    bf16* const na = (kt & 1) ? sA0 : sA1;
    bf16* const nb = (kt & 1) ? sB0 : sB1;
    const Seg sg = seg_of(kt + 2);
    [[maybe_unused]] const Seg sg1 = seg_of(kt + 1);
#pragma unroll
    for (int sl = 0; sl < S; ++sl) {
      const int ks = sl / NM, I = sl % NM, cur = ks & 1;
      if (STORE && sl == S - TAIL) __syncthreads();
      if constexpr (BD) acc[I / TN][I % TN] = mfma32(af[cur][I / TN], bq[ks][I % TN], acc[I / TN][I % TN]);
      else acc[I / TN][I % TN] = mfma32(af[cur][I / TN], bfr[cur][I % TN], acc[I / TN][I % TN]);
      if (ks + 1 < KSL && I < NF) {
        if (I < TM) af[cur ^ 1][I] = read_frag<LDA, TA>(pa, I * 32, ks0 + ks + 1);
        else if constexpr (!BD) bfr[cur ^ 1][I - TM] = read_frag<LDB, TB>(pb, (I - TM) * 32, ks0 + ks + 1);
      }
      if (STORE && sl >= S - TAIL) {   // first step of tile kt+1, from the other buffer, into the idle fragment set
#pragma unroll
        for (int f = ((sl - (S - TAIL)) * NF) / TAIL; f < ((sl - (S - TAIL) + 1) * NF) / TAIL; ++f) {
          if (f < TM) af[0][f] = read_frag<LDA, TA>(na + offA, f * 32, ks0);
          else if constexpr (!BD) bfr[0][f - TM] = read_frag<LDB, TB>(nb + offB, (f - TM) * 32, ks0);
        }
      }
      if constexpr (BD && STORE) {   // this was the last MFMA of the tile that reads fragment (ks, j): refill it for tile kt+1
        if (I >= NM - TN) bq[ks][I - (NM - TN)] = bd_load(ks, I - (NM - TN), sg1);
      }
#pragma unroll
      for (int q = 0; q < NLD; ++q)
        if (((q + 1) * (S - TAIL)) / NLD - 1 == sl) {
          if constexpr (STORE) store_chunk(q, na, nb);
          if constexpr (LOAD) load_chunk(q, sg);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int kt = 0; kt + 2 < nk; ++kt) tile(kt, std::true_type{}, std::true_type{});
  if (nk > 1) tile(nk - 2, std::true_type{}, std::false_type{});
  if (nk > 0) tile(nk - 1, std::false_type{}, std::false_type{});
  __syncthreads();   // every wave is done with the operand tiles: the epilogue reuses the LDS

  if constexpr (KG > 1) {
    static_assert(KG == 2 && TN == 2, "the exchange pairs two wave groups with the two column halves of a block");
    // The K loop ended with a barrier, so the operand tiles are dead.  The two groups hold partial sums of the same
    // blocks: group 1 hands its left half (tile column 0) to group 0 and takes group 0's right half, in one exchange
    // ([group][wave][register][lane], conflict-free), and each group finishes and writes its own half.
    float* const mine = reinterpret_cast<float*>(smem) + (kg * C::NWT + wmn) * (TM * 16 * 64) + lane;
    float* const theirs = reinterpret_cast<float*>(smem) + ((kg ^ 1) * C::NWT + wmn) * (TM * 16 * 64) + lane;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (j == kg) continue;   // wave-uniform: the half this wave gives away is j = 1 - kg
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) mine[(i * 16 + v) * 64] = acc[i][j][v];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (j != kg) continue;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] += theirs[(i * 16 + v) * 64];
    }
    __syncthreads();   // the staging of the epilogue overwrites the exchange area
    epilogue(p, p.M, acc, smem, wave, lane, m0 + wm * WAVE_M, n0 + wn * WAVE_N, p.part_row0 + tile_m * WGM + wm, kg, kg + 1);
    return;
  }
  // a folded tile's wave columns: waves 0, 1 of a row hold gate columns, waves 2, 3 the up columns that go with them
  const int wcol = fold ? (n0 >> 1) + (wn & 1) * WAVE_N + (wn >> 1) * fold : n0 + wn * WAVE_N;
  epilogue(p, Mlim, acc, smem, wmn, lane, m0 + wm * WAVE_M, wcol, p.part_row0 + tile_m * WGM + wm);
}

template <int WGM, int WGN, int BK, bool TA, bool TB, int KG = 1, bool GATED = false, bool BD = false, bool GRP = false>
hipError_t launch_one(hipStream_t st, const GemmArgs& a) {
  using C = Cfg<WGM, WGN, BK, TA, TB, KG>;
  static bool attr_done = false;
  auto kern = gemm_kernel<WGM, WGN, BK, TA, TB, KG, GATED, BD, GRP>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int tiles = (GRP ? a.grp_max_tiles : (a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN);
  RP_LAUNCH(kern, dim3(tiles, a.splits > 0 ? a.splits : 1), dim3(C::NTHR), C::SMEM, st, a);
  return hipGetLastError();
}

template <bool TA, bool TB>
hipError_t launch_tile(hipStream_t st, const GemmArgs& a, int tile) {
  if (a.run_flag) {   // only the frozen head's conditional logits product: NT, 256x256 (checked by gemm_launch)
    if constexpr (!TA && !TB) return launch_one<2, 4, 64, false, false, 1, true>(st, a);
    return hipErrorInvalidValue;
  }
  if (a.b_direct) {   // B in fragment order: its memory layout no longer matters, one instance serves NT and NN
    if constexpr (!TA) return launch_one<2, 4, 64, false, false, 1, false, true>(st, a);
    return hipErrorInvalidValue;
  }
  if (a.grp_tab) {
    if constexpr (!TA) return launch_one<2, 4, 64, TA, TB, 1, false, false, true>(st, a);
    return hipErrorInvalidValue;
  }
  switch (tile) {
    case 1: return launch_one<2, 4, 64, TA, TB>(st, a);
    case 5: return launch_one<2, 2, 64, TA, TB, 2>(st, a);
    default: return gemm_mid_launch(st, a, TA ? GEMM_TN : TB ? GEMM_NN : GEMM_NT, tile);
  }
}

// Merge of a reduction split: C (+)= sum over the slices, added in slice order (one thread per four columns); a bf16
// result takes the residual R (optional) here.
template <bool OUT_BF16>
__global__ void __launch_bounds__(256) splitk_merge_kernel(const float* __restrict__ ws, int splits, long slice_stride,
                                                           void* Cout, long ldc, int M, int N, int beta,
                                                           const bf16* R, long ldr) {
  const int n4 = N >> 2;
  const long total = (long)M * n4;
  for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
    const long row = idx / n4;
    const int c = (int)(idx - row * n4) * 4;
    const float* src = ws + row * N + c;
    float4 acc = *reinterpret_cast<const float4*>(src);
    for (int s = 1; s < splits; ++s) {
      const float4 v = *reinterpret_cast<const float4*>(src + (long)s * slice_stride);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if constexpr (OUT_BF16) {
      if (R) {
        const uint2 r = *reinterpret_cast<const uint2*>(R + row * ldr + c);
        acc.x += bf16_lo(r.x); acc.y += bf16_hi(r.x); acc.z += bf16_lo(r.y); acc.w += bf16_hi(r.y);
      }
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16*>(Cout) + row * ldc + c) = make_uint2(pack_bf16x2(acc.x, acc.y), pack_bf16x2(acc.z, acc.w));
    } else {
      float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float*>(Cout) + row * ldc + c);
      if (beta) { const float4 o = *dst; acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w; }
      *dst = acc;
    }
  }
}

// The merges of a group's split products in one launch: 256 quads of columns per workgroup.
struct MergeOne { const float* ws; void* C; const bf16* R; long stride, ldc, ldr; int splits, M, N, beta, out_bf16, first; };
struct MergeArgs { int n; MergeOne m[GEMM_GROUP_MAX]; };
__global__ void __launch_bounds__(256) group_merge_kernel(const MergeArgs a) {
  int i = 0;
  while (i + 1 < a.n && (int)blockIdx.x >= a.m[i + 1].first) ++i;
  i = __builtin_amdgcn_readfirstlane(i);
  const MergeOne& q = a.m[i];
  const int n4 = q.N >> 2;
  const long idx = (long)((int)blockIdx.x - q.first) * 256 + threadIdx.x;
  if (idx >= (long)q.M * n4) return;
  const long row = idx / n4;
  const int c = (int)(idx - row * n4) * 4;
  const float* src = q.ws + row * q.N + c;
  float4 acc = *reinterpret_cast<const float4*>(src);
  for (int s = 1; s < q.splits; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(src + (long)s * q.stride);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  if (q.out_bf16) {
    if (q.R) {
      const uint2 r = *reinterpret_cast<const uint2*>(q.R + row * q.ldr + c);
      acc.x += bf16_lo(r.x); acc.y += bf16_hi(r.x); acc.z += bf16_lo(r.y); acc.w += bf16_hi(r.y);
    }
    *reinterpret_cast<uint2*>(reinterpret_cast<bf16*>(q.C) + row * q.ldc + c) = make_uint2(pack_bf16x2(acc.x, acc.y), pack_bf16x2(acc.z, acc.w));
  } else {
    float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float*>(q.C) + row * q.ldc + c);
    if (q.beta) { const float4 o = *dst; acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w; }
    *dst = acc;
  }
}

// One 16-byte chunk of the fragment order per thread (see gemm_arranged_bytes).
__global__ void __launch_bounds__(256) gemm_arrange_kernel(const bf16* __restrict__ B, long ldb, int N, int K, int transposed,
                                                           uint4* __restrict__ out, long chunks, int nkt) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= chunks) return;
  const int lane = (int)(idx & 63);
  const long f = idx >> 6;
  const int j = (int)(f & 1), ks = (int)((f >> 1) & 3);
  const long t = f >> 3;
  const int kt = (int)(t % nkt);
  const int blk = (int)(t / nkt);
  const int n = blk * 64 + j * 32 + (lane & 31), k = kt * 64 + ks * 16 + (lane >> 5) * 8;
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (n < N && k < K) {   // K is a multiple of 8: the eight indices are in range together
    if (!transposed) {
      v = *reinterpret_cast<const uint4*>(B + (long)n * ldb + k);
    } else {
      const unsigned short* src = reinterpret_cast<const unsigned short*>(B) + (long)k * ldb + n;
      unsigned short e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = src[(long)i * ldb];
      v = make_uint4(e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16), e[4] | ((uint32_t)e[5] << 16), e[6] | ((uint32_t)e[7] << 16));
    }
  }
  out[idx] = v;
}

// Modelled cost of a product on one tile, in microseconds.  Elapsed time = launch + rounds * (K tiles * time per K tile +
// epilogue), rounds = workgroups on the busiest CU.  The constants are fits to measured times (K = 128 to 24576, 16 to 1500
// workgroups, weights coming from HBM; within 10 % of the measurement on most shapes):
//   - the 256x256 and 256x128 tiles are bound by the matrix pipe and the power it draws: their K tile takes longer the more
//     of the chip is busy;
//   - the small tiles are bound by what a CU can fetch -- 50 bytes/ns of data that comes from HBM, however many loads are
//     in flight (80 from the Infinity Cache, 150 from L2) -- so their K tile costs its operand bytes.
// A split into `splits` slices adds the merge kernel and its traffic.  For accumulating outputs the part of it beyond 64 MB counts as chip
// time as well; where that changes the choice it is fewer slices of a head's input gradient (K = 151936), which cost nothing on one
// stream and leave more to the others.  Whole frozen head, us, one stream | three, without that term and with it: 3000 x 2048 in eight slices
// or five 3302 | 3299 -> 3302 | 3290, 2040 x 2880 eight or five 3156 | 3066 -> 3155 | 3027, 1504 x 4096 eight or five 3122 | 3087 -> 3114 | 3050,
// 2504 x 4096 eight or three 5170 | 5098 -> 5151 | 5058, 2040 x 5120 eight or three 5090 | 5077 -> 5080 | 4992.  The 64 MB are a bound drawn
// between these (250 MB and more in eight slices) and the weight gradients and bf16 results of short batches, which are 2-3 % slower
// with fewer slices; nothing was measured in between.  Added to the elapsed time is the chip time the
// workgroups use up (their summed time over 256 CUs): what is left over belongs to other streams, so a small tile has to buy
// enough latency for the extra operand traffic it causes.  A worker runs its calls on one stream, so the weight is one at which none of them is
// slower there.  Whole stage calls, us, weight 1.3 | 0.7 | 0.35 | 0, on one stream and with three calls at once: forward of 1000 tokens at
// h = 2048 178 | 173 | 165 | 165 and 161 | 158 | 159 | 163; LoRA backward of 392 at h = 4096 710 | 688 | 689 | 688 and 580 | 569 | 578 | 577, of
// 2 x 508 1069 | 1067 | 1070 | 1082 and 957 | 961 | 961 | 978; backward of a full fine-tune of 4096 at h = 2048 1593 | 1595 | 1600 | 1622 and
// 1584 | 1582 | 1584 | 1617.
constexpr double CHIP_WEIGHT = 0.7;
struct TileModel { int bm, bn; double tau, tau_fill, epi; };
// by tile number; 256x256 tiles are 1 on the eight-wave kernel, 7 on the four-wave one
constexpr TileModel TILE_MODEL[9] = {{},
                                     {256, 256, 0.95, 0.60, 6.0}, {256, 128, 0.60, 0.35, 4.0}, {128, 128, 0.55, 0.0, 3.5},
                                     {128, 64, 0.36, 0.0, 3.5},   {256, 128, 0.53, 0.40, 5.0}, {}, {256, 256, 0.78, 0.58, 4.5}, {64, 64, 0.31, 0.0, 3.5}};

double tile_cost(int tile, int splits, int M, int N, int k_tiles, int epi) {
  TileModel t = TILE_MODEL[tile];
  // SwiGLU epilogues: what they read and write beside the product, per 256x256 tile on a full chip
  t.epi += (epi == EPI_SWIGLU_BWD ? 18.0 : epi == EPI_SWIGLU_FWD ? 6.0 : 0.0) * (t.bm * t.bn) / 65536.0;
  const long wg = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * splits;
  const double rounds = (double)((wg + 255) / 256), fill = wg < 256 ? wg / 256.0 : 1.0;
  double tau = t.tau + t.tau_fill * fill;
  if (t.tau_fill == 0.0) {   // rows and columns past the end of a skinny output are not fetched
    const double part = (double)((M < t.bm ? M : t.bm) + (N < t.bn ? N : t.bn)) / (t.bm + t.bn);
    tau *= part > 0.6 ? part : 0.6;
  }
  const int per = (k_tiles + splits - 1) / splits;
  double us = 3.0 + rounds * (per * tau + t.epi) + CHIP_WEIGHT * wg / 256.0 * (per * (tau + t.tau_fill * (1.0 - fill)) + t.epi);
  if (splits > 1) {
    const double bytes = (double)M * N * (8.0 * splits + (epi != EPI_BF16 ? 8.0 : 2.0)), beyond = bytes > 64.0e6 ? bytes - 64.0e6 : 0.0;
    us += 4.0 + (bytes + (epi != EPI_BF16 ? CHIP_WEIGHT * beyond : 0.0)) / 4.0e6;
  }
  return us;
}

struct Choice { int tile, splits; };

long big_tiles(const GemmArgs& a, int splits) { return (long)((a.M + 255) / 256) * ((a.N + 255) / 256) * splits; }

// Which kernel a product on 256x256 tiles runs: the four-wave one that loads its operands straight into LDS (gemm_dtl.hip), unless a kernel
// is asked for by name (hint 1: eight waves, hint 7: four), the variant has no counterpart there, or the reduction of a slice is short.  Its
// 16x16x32 instructions are ahead per K tile where the power binds, that is with most of the chip busy; its start and its one wave per SIMD cost
// more.  So the line lies by the share of the CUs that have a tile, over all rounds.  Eight waves | four, us, bf16 NT, K = 512, 1024, 1536, 2048:
//   144 tiles (0.56) 17.1 | 19.3, 25.9 | 26.9, 35.0 | 36.3, 44.5 | 44.3     288 (0.56) 33.4 | 34.8, 52.3 | 53.1, 73.7 | 75.5, 95.3 | 92.1
//   160 (0.63) 18.1 | 19.2, 26.7 | 27.9, 39.4 | 36.7, 47.2 | 45.6           192 (0.75) 19.0 | 19.5, 29.5 | 28.7, 39.4 | 39.2, 49.6 | 47.0
//   224 (0.88) 20.7 | 20.7, 32.8 | 31.2, 45.0 | 40.5, 56.6 | 52.6           256 22.3 | 21.6, 34.0 | 31.1, 47.2 | 42.1, 60.7 | 53.2
//   1024 84.7 | 81.7, 132 | 120 at 1024;  384 (0.75) 34.4 | 36.0, 58.2 | 57.6;  fp32 176 (0.69) 21.7 | 23.6, 31.0 | 32.2, -, 50.5 | 49.0
// A residual and the SwiGLU epilogues are shorter from its registers: with a residual, 144 tiles 25.4 | 21.5, 33.3 | 29.0, 41.8 | 38.3, 50.6 | 46.7,
// 288 53 | 41 and 113 | 98 at both ends; SwiGLU forward, 144 tiles 28.4 | 27.8, 38.3 | 36.4, 45.8 | 44.0, 55.6 | 54.4; backward, 192 tiles 43.7 |
// 38.9, 58.4 | 62.1 (K = 1024, the one that loses), -, 83.0 | 79.0.  Outputs that accumulate, TN, K = 512, 768, 1024: 512 tiles 70.8 | 65.8, 83.5 | 77.3,
// 95.8 | 86.6; 640 85.8 | 87.4, 101.8 | 101.2, 118 | 115; 1024 144 | 147, 169 | 166, 191 | 186 (but 2048 tiles with rows of 64 KB 415 | 425 at 1024, 500 |
// 504 at 1536, 595 | 585 at 2048).
// Cross-entropy epilogues that stage their tile are longer in four waves: with them from 40 K tiles on.  The probabilities (EPI_CE_P) go out
// from the registers: trainable head of 151936 x 2048, 4096 tokens, 6437 us with eight waves, 6246 with four.  Skinny outputs (the LoRA
// products, bound by reading the other operand once) stay on the eight-wave kernel: +14 %.
bool four_waves(const GemmArgs& a, int splits, int tile_hint) {
  if (tile_hint == 1 || a.run_flag || a.b_direct) return false;
  if (tile_hint == 7) return true;
  if (a.M <= 64 || a.N <= 64) return false;
  const bool ce = a.epi == EPI_CE_STATS || a.epi == EPI_CE_DZ || a.epi == EPI_F32_COLMAX;
  const long n = big_tiles(a, splits);
  const double busy = n / (256.0 * ((n + 255) / 256));
  int min_k = busy > 0.8 ? 512 : busy > 0.7 ? 1024 : busy > 0.6 ? 1536 : 2048;
  if (splits == 1) {      // (slices write plain fp32)
    if (n > 128 && (a.R || a.epi == EPI_CE_P)) min_k = 512;     // R: the residual, or gate and up of a SwiGLU backward
    if (n > 128 && a.epi == EPI_SWIGLU_FWD) min_k = 512;
    if (a.epi == EPI_F32 && a.beta && min_k < 768) min_k = 768;
  }
  return a.K + a.K2 >= (ce ? 2560 : splits * min_k);
}

// The four-wave kernel addresses the 256 rows of an output tile with 31-bit byte offsets: others run elsewhere, whoever launches.
bool near_rows(const GemmArgs& a) { return a.ldc < 1L << 21 && a.ldr < 1L << 21 && a.ldc2 < 1L << 21; }

// tile_cost of the kernel that would be launched
double product_cost(const GemmArgs& a, int tile, int splits, int tile_hint) {
  return tile_cost(tile == 1 && four_waves(a, splits, tile_hint) ? 7 : tile, splits, a.M, a.N, (a.K + 63) / 64 + (a.K2 + 63) / 64, a.epi);
}

// Bytes spanned by a [rows, cols] bf16 view with row stride ld; 0 for an empty view, ~0 when it does not fit 31 bits.
unsigned extent_bytes(long rows, long cols, long ld) {
  if (rows <= 0 || cols <= 0) return 0;
  const long b = ((rows - 1) * ld + cols) * 2;
  return b < (1L << 31) ? (unsigned)b : ~0u;
}

}  // namespace

void gemm_zero_args(GemmArgs& a) {
  a = GemmArgs{};
  a.alpha = 1.f;
}

int gemm_ce_stats_partials(int M) { return 2 * ((M + 255) / 256); }

size_t gemm_arranged_bytes(int N, int K) { return (size_t)((N + 63) / 64) * (size_t)((K + 63) / 64) * 8192; }

hipError_t gemm_arrange(hipStream_t st, const void* B, long ldb, int N, int K, int transposed, void* out) {
  if (N <= 0 || K <= 0) return hipSuccess;
  if (!B || !out || K % 8 || ldb % 8 || (transposed && N % 8)) return hipErrorInvalidValue;
  const long chunks = (long)(gemm_arranged_bytes(N, K) / 16);
  RP_LAUNCH(gemm_arrange_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st, (const bf16*)B, ldb, N, K, transposed,
            (uint4*)out, chunks, (K + 63) / 64);
  return hipGetLastError();
}

// Tile and reduction slices of a product, the cheapest by the model above.  Cross-entropy epilogues are written for the
// 256x256 tile: the partial rows of three of them are numbered by it, and EPI_CE_DZ, which has none, is faster there even where
// tokens fill a corner of it (second sweep over 32768 vocabulary rows of 2048 for 8 | 64 tokens: 128x64 tiles 84 | 87 us,
// 256x256 47 | 49; 32000 rows of 5120: 191 | 205 and 103 | 107).  SwiGLU epilogues are not part of the 256x128 two-group tile.
// Only plain outputs can be summed from slices, a bf16 one only while its 256x128 tiles leave CUs idle: from 256 of them on a
// split gains nothing (4096 x 2048 x 12288 NN in two slices 187 -> 180 us with its merge, but the product behind it 217 -> 224
// and the backward stage of 4096 tokens 1864 -> 1873).  A slice keeps at least four K tiles of a small tile, sixteen of a large
// one (four for a skinny output, which is bound by reading the other operand).
// Up to 128 tiles of 256x256 leave half of the chip idle: the 256x128 tiles are ahead there at any reduction.  256x256 (the faster of its two kernels) |
// 256x128 by two groups | by eight waves (gemm_mid.hip), us, K = 512, 1024, 2048, 4096, 6144: 4096 x 2048 NT 17.4 | 14.7 | 15.9, 25.6 | 22.1 | 22.7,
// 42.4 | 37.3 | 35.7, 76.4 | 65.4 | 63.9, 110 | 94 | 91; NN 110 | 99 | 92 and fp32 accumulating TN 118 | 104 | 98 at 6144; 2048 x 3072 NT (96 tiles) 16.2 |
// 12.9 | 14.0, 24.9 | 18.8 | 19.8, 42.3 | 31.2 | 32.1, 76.4 | 55.6 | 57.8, 110 | 85 | 85.  From 144 tiles on it is the other way round: 3072 x 3072 NT
// 17.1 | 23.9 | 24.9 at 512, 77.9 | 104 | 101 at 4096.  (Three such calls at once fill the chip with 256x256 tiles and are faster with them: backward of
// a full fine-tune of 4096 tokens at h = 2048 1519 us against 1582; but on one stream it takes 1663 against 1595.)
static Choice choose(const GemmArgs& a, int tile_hint) {
  if (a.grp_tab) return {1, 1};      // the table's entries are rows of 256-row tiles
  if (a.b_direct || a.epi == EPI_CE_STATS || a.epi == EPI_CE_DZ || a.epi == EPI_F32_COLMAX || a.epi == EPI_CE_P) return {1, 1};
  const bool swiglu = a.epi == EPI_SWIGLU_FWD || a.epi == EPI_SWIGLU_BWD;
  const bool may_split = a.split_ws && a.run_flag == nullptr &&
                         ((a.epi == EPI_BF16 && (long)((a.M + 255) / 256) * ((a.N + 127) / 128) < 256) || a.epi == EPI_F32);
  const int k_tiles = (a.K + 63) / 64 + (a.K2 + 63) / 64;
  const bool skinny = a.N <= 64 || a.M <= 64;
  Choice best{1, 1};
  double best_cost = 1e300;
  // (the eight-wave 256x128 tile of gemm_mid.hip stands in for the two-group one under a SwiGLU epilogue: 1000 x 6144 x 2048
  // backward 57 us on 256x256, 37)
  const int order[5] = {1, swiglu ? 2 : 5, 3, 4, 8};
  for (int i = 0; i < 5; ++i) {
    const int t = tile_hint ? (tile_hint == 7 ? 1 : tile_hint) : order[i];
    const int min_per = (t == 1 || t == 5) && !skinny ? 16 : 4;
    for (int sp = 1; sp <= (may_split ? 16 : 1); ++sp) {
      if (sp > 1 && (k_tiles / sp < min_per || (size_t)sp * a.M * a.N * 4 > a.split_ws_bytes)) break;
      if (t == 1 && !tile_hint && !skinny && big_tiles(a, sp) <= 128) continue;
      const double c = product_cost(a, t, sp, tile_hint);
      if (c < best_cost) { best_cost = c; best = {t, sp}; }
    }
    if (tile_hint) break;
  }
  return best;
}

int gemm_pick_tile(const GemmArgs& a, int tile_hint) { return choose(a, tile_hint).tile; }

// Argument checks and the derived fields (byte extents, the form of a bf16 result that may be summed from slices).
static hipError_t prepare(int layout, GemmArgs& a) {
  // 16-byte accesses everywhere: the output width and every leading dimension must keep rows aligned
  const bool out_f32 = a.epi == EPI_F32 || a.epi == EPI_F32_ATOMIC || a.epi == EPI_F32_COLMAX;
  if (a.epi == EPI_F32_COLMAX && (a.beta || !a.part || !a.labels || !a.zlab)) return hipErrorInvalidValue;
  if (a.run_flag && (a.epi != EPI_F32_COLMAX || layout != GEMM_NT)) return hipErrorInvalidValue;
  if (a.epi == EPI_CE_P && (!a.part || !a.labels || !a.zlab || !a.lse)) return hipErrorInvalidValue;
  if (a.N % 8 || a.K % 8 || a.lda % 8 || (!a.b_direct && a.ldb % 8)) return hipErrorInvalidValue;
  if (a.epi != EPI_CE_STATS && a.ldc % (out_f32 ? 4 : 8)) return hipErrorInvalidValue;
  if (a.R && a.ldr % 4) return hipErrorInvalidValue;
  if (a.epi == EPI_SWIGLU_FWD && (layout != GEMM_NT || !a.C2 || a.R || a.b_direct || a.N % 16 || a.ldc2 % 8 || a.alpha != 1.f))
    return hipErrorInvalidValue;
  if (a.epi == EPI_SWIGLU_BWD && (!a.R || a.ldr % 8 || a.ldc % 8 || a.grp_tab)) return hipErrorInvalidValue;
  const bool ta = layout == GEMM_TN, tb = layout != GEMM_NT;
  if (ta && a.M % 8) return hipErrorInvalidValue;
  if (!a.A2 || !a.B2) a.K2 = 0;
  if (a.K2 && (a.K2 % 8 || a.lda2 % 8 || (!a.b_direct && a.ldb2 % 8))) return hipErrorInvalidValue;
  a.bytesA = ta ? extent_bytes(a.K, a.M, a.lda) : extent_bytes(a.M, a.K, a.lda);
  a.bytesB = tb ? extent_bytes(a.K, a.N, a.ldb) : extent_bytes(a.N, a.K, a.ldb);
  a.bytesA2 = ta ? extent_bytes(a.K2, a.M, a.lda2) : extent_bytes(a.M, a.K2, a.lda2);
  a.bytesB2 = tb ? extent_bytes(a.K2, a.N, a.ldb2) : extent_bytes(a.N, a.K2, a.ldb2);
  if (a.b_direct) {
    if (ta || a.grp_tab || a.run_flag) return hipErrorInvalidValue;
    const size_t b1 = gemm_arranged_bytes(a.N, a.K), b2 = a.K2 ? gemm_arranged_bytes(a.N, a.K2) : 0;
    if (b1 >= ((size_t)1 << 31) || b2 >= ((size_t)1 << 31)) return hipErrorInvalidValue;
    a.bytesB = (unsigned)b1;
    a.bytesB2 = (unsigned)b2;
  }
  // operands are addressed with 32-bit byte offsets
  if (a.bytesA == ~0u || a.bytesB == ~0u || a.bytesA2 == ~0u || a.bytesB2 == ~0u) return hipErrorInvalidValue;
  if (a.split_out_bf16) {   // a bf16 result that may be summed from slices
    if (a.epi != EPI_F32 || !a.split_ws || a.ldc % 4 || (size_t)a.M * a.N * 4 > a.split_ws_bytes) return hipErrorInvalidValue;
    a.epi = EPI_BF16;
  }
  return hipSuccess;
}

// Grouped: 256-row tiles as in the table, rows of A are tile rows, one operand pair.
static hipError_t prepare_grouped(int layout, GemmArgs& a) {
  if (layout == GEMM_TN || a.K2 || !a.grp_ntiles || a.grp_max_tiles <= 0 || (a.epi != EPI_BF16 && a.epi != EPI_F32 && a.epi != EPI_SWIGLU_FWD)) return hipErrorInvalidValue;
  if (a.row_map) {
    a.bytesA = extent_bytes(a.row_map_rows, a.K, a.lda);
    if (a.bytesA == ~0u || a.row_map_rows <= 0) return hipErrorInvalidValue;
  }
  return hipSuccess;
}

hipError_t gemm_launch(hipStream_t st, int layout, const GemmArgs& a_in, int tile_hint) {
  if (a_in.M <= 0 || a_in.N <= 0) return hipSuccess;
  if (layout < GEMM_NT || layout > GEMM_TN) return hipErrorInvalidValue;
  GemmArgs a = a_in;
  hipError_t e = prepare(layout, a);
  if (e != hipSuccess) return e;
  const Choice ch = choose(a, tile_hint);
  const int tile = ch.tile;
  const bool four = four_waves(a, ch.splits, tile_hint);
  if (a.grp_tab) {
    e = prepare_grouped(layout, a);
    if (e != hipSuccess) return e;
  }
  // Reduction split: the slices' partial products go to scratch memory and a second kernel adds them in a fixed order, so
  // results are reproducible run to run.
  a.splits = ch.splits;
  a.c_slice_stride = 0;
  const bool out_bf16 = a.epi == EPI_BF16;
  void* const C_final = a.C;
  const long ldc_final = a.ldc;
  const int beta_final = a.beta;
  const bool merged = a.splits > 1;
  if (merged) {   // the slices write fp32 partials [slice][M][N]
    a.C = a.split_ws; a.ldc = a.N; a.beta = 0; a.c_slice_stride = (long)a.M * a.N;
    a.epi = EPI_F32; a.R = nullptr;
  }
  // Grouped products run the four-wave kernel (it spares a tile's empty rows their matrix instructions), but for reductions of up to 16 K tiles over
  // weights that the caches hold (grp_cached): these are bound by that fixed cost, and by fetching the larger code.  Forward
  // of a layer, us, eight waves | four: 8 experts of 256 x 96, 136 tokens 71 | 79 (a product 11 | 16), 1064 92 | 100; of 512 x 512, 136 | 4096 tokens
  // 83 | 87, 151 | 161; of 768 x 3072, 16384 tokens 1004 | 1039; 32 of 512 x 1024, 4096 tokens 220 | 233.  With weights from
  // memory the four waves are ahead: 64 of 1024 x 512 (201 MB), 4096 | 16384 tokens 276 | 268, 857 | 833; 128 of 2048 x 768, 16384 2521 | 2468.
  const bool short_grp = a.grp_tab && a.grp_cached && !a.grp_once && a.K <= 1024;
  const bool dtl = near_rows(a) && (a.grp_tab ? !short_grp : tile == 1 && four);
  if (dtl) {
    e = gemm_dtl_launch(st, a, layout);
  } else {
    switch (layout) {
      case GEMM_NT: e = launch_tile<false, false>(st, a, tile); break;
      case GEMM_NN: e = launch_tile<false, true>(st, a, tile); break;
      default: e = launch_tile<true, true>(st, a, tile); break;
    }
  }
  if (e != hipSuccess || !merged) return e;
  const long quads = (long)a.M * (a.N / 4);
  const int grid = (int)((quads + 255) / 256 < 4096 ? (quads + 255) / 256 : 4096);
  if (out_bf16)
    RP_LAUNCH(splitk_merge_kernel<true>, dim3(grid), dim3(256), 0, st, a.split_ws, a.splits, a.c_slice_stride, C_final, ldc_final, a.M, a.N, 0,
              (const bf16*)a_in.R, a_in.ldr);
  else
    RP_LAUNCH(splitk_merge_kernel<false>, dim3(grid), dim3(256), 0, st, a.split_ws, a.splits, a.c_slice_stride, C_final, ldc_final, a.M, a.N, beta_final,
              (const bf16*)nullptr, 0L);
  return hipGetLastError();
}

// Skinny products (the adapters') and outputs of at most 128 tiles of 64x64: neither fills the chip, and a launch of its own
// is most of what either costs.
bool gemm_groupable(const GemmArgs& a) {
  if (a.M <= 0 || a.N <= 0 || a.grp_tab || a.b_direct || a.run_flag) return false;
  if (a.epi != EPI_BF16 && a.epi != EPI_F32 && a.epi != EPI_SWIGLU_BWD) return false;
  return a.M <= 64 || a.N <= 64 || (long)((a.M + 63) / 64) * ((a.N + 63) / 64) <= 128;
}

hipError_t gemm_group_launch(hipStream_t st, int n, const int* layouts, const GemmArgs* g) {
  if (n < 0 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
  GemmArgs q[GEMM_GROUP_MAX];
  int lay[GEMM_GROUP_MAX], cnt = 0;
  for (int i = 0; i < n; ++i)
    if (gemm_groupable(g[i])) { q[cnt] = g[i]; lay[cnt++] = layouts[i]; }
  for (int i = 0; i < n; ++i) {
    if (cnt > 1 && gemm_groupable(g[i])) continue;
    const hipError_t e = gemm_launch(st, layouts[i], g[i]);
    if (e != hipSuccess) return e;
  }
  if (cnt <= 1) return hipSuccess;
  // Slices: every workgroup gets about the same share of the group's K tiles (weighted by what a tile fetches), with some 320
  // workgroups in all and at least six K tiles each; the partial products share the scratch.
  double total = 0.0, weight[GEMM_GROUP_MAX];
  for (int i = 0; i < cnt; ++i) {
    const hipError_t e = prepare(lay[i], q[i]);
    if (e != hipSuccess) return e;
    const double w = ((q[i].M < 64 ? q[i].M : 64) + (q[i].N < 64 ? q[i].N : 64)) / 128.0;
    weight[i] = w > 0.6 ? w : 0.6;
    total += weight[i] * ((q[i].M + 63) / 64) * ((q[i].N + 63) / 64) * (double)((q[i].K + 63) / 64 + (q[i].K2 + 63) / 64);
  }
  const double per = total / 320.0 > 6.0 ? total / 320.0 : 6.0;
  MergeArgs ma{};
  size_t used = 0;
  int merge_blocks = 0;
  float* const ws = g[0].split_ws;
  for (int i = 0; i < cnt; ++i) {
    GemmArgs& a = q[i];
    const int nk = (a.K + 63) / 64 + (a.K2 + 63) / 64;
    const bool may = ws && a.split_ws == ws && (a.epi == EPI_BF16 || (a.epi == EPI_F32 && a.beta));
    int sp = may ? (int)(nk * weight[i] / per + 0.999) : 1;
    if (sp > 16) sp = 16;
    while (sp > 1 && (nk / sp < 4 || used + (size_t)sp * a.M * a.N * 4 > a.split_ws_bytes)) --sp;
    if (sp < 1) sp = 1;
    a.splits = sp;
    a.c_slice_stride = 0;
    if (sp > 1) {
      MergeOne& m = ma.m[ma.n++];
      m = {ws + used / 4, a.C, (const bf16*)a.R, (long)a.M * a.N, a.ldc, a.ldr, sp, a.M, a.N, a.beta, a.epi == EPI_BF16, merge_blocks};
      merge_blocks += (int)(((long)a.M * (a.N / 4) + 255) / 256);
      a.C = ws + used / 4; a.ldc = a.N; a.beta = 0; a.R = nullptr; a.epi = EPI_F32; a.c_slice_stride = (long)a.M * a.N;
      used += (size_t)sp * m.M * m.N * 4;
    }
  }
  hipError_t e = gemm_multi_run(st, cnt, lay, q);
  if (e != hipSuccess || ma.n == 0) return e;
  RP_LAUNCH(group_merge_kernel, dim3(merge_blocks), dim3(256), 0, st, ma);
  return hipGetLastError();
}

bool gemm_wgrad_joined(int n, const GemmArgs* g) {
  if (n < 2 || n > GEMM_WGRAD_MAX) return false;
  double apart = 0.0;
  long tiles = 0;
  for (int i = 0; i < n; ++i) {
    GemmArgs q = g[i];
    if (prepare(GEMM_TN, q) != hipSuccess || !near_rows(q)) return false;
    const Choice ch = choose(q, 0);
    apart += product_cost(q, ch.tile, ch.splits, 0);
    tiles += (long)((q.M + 255) / 256) * ((q.N + 255) / 256);
  }
  return tile_cost(7, 1, (int)(256 * tiles), 256, (g[0].K + 63) / 64, EPI_F32) < apart;
}

hipError_t gemm_wgrad_launch(hipStream_t st, int n, const GemmArgs* g) {
  if (n < 1 || n > GEMM_WGRAD_MAX) return hipErrorInvalidValue;
  GemmArgs q[GEMM_WGRAD_MAX];
  for (int i = 0; i < n; ++i) {
    q[i] = g[i];
    const hipError_t e = prepare(GEMM_TN, q[i]);
    if (e != hipSuccess) return e;
    if (!near_rows(q[i])) return hipErrorInvalidValue;
  }
  return gemm_wgrad_run(st, n, q);
}

hipError_t gemm_pair_launch(hipStream_t st, const GemmArgs& nt, const GemmArgs& nn) {
  GemmArgs a = nt, b = nn;
  if (a.M <= 0 || a.N <= 0 || b.N <= 0) return hipErrorInvalidValue;
  if (!a.grp_tab || a.grp_tab != b.grp_tab || a.grp_ntiles != b.grp_ntiles || a.grp_max_tiles != b.grp_max_tiles || a.epi != EPI_BF16 || b.epi != EPI_BF16 ||
      a.R || b.R || a.alpha != 1.f || b.alpha != 1.f || !near_rows(a) || !near_rows(b))
    return hipErrorInvalidValue;
  hipError_t e = prepare(GEMM_NT, a);
  if (e == hipSuccess) e = prepare_grouped(GEMM_NT, a);
  if (e == hipSuccess) e = prepare(GEMM_NN, b);
  if (e == hipSuccess) e = prepare_grouped(GEMM_NN, b);
  return e == hipSuccess ? gemm_pair_run(st, a, b) : e;
}
