// bf16 GEMM for outputs that leave the chip idle on 256x256 tiles: small tiles, operands loaded straight into LDS, every
// wave a 64x64 block of C (2x2 tiles of v_mfma_f32_32x32x16_bf16, 64 accumulator registers).
//
// A workgroup is KG wave groups of WGM x WGN blocks of 64x64.  The groups work on the same output tile and take the K tiles of
// the reduction in turn (group g: tiles g, g + KG, ...), each from operand tiles of its own in LDS, so a small tile still keeps
// four or eight waves busy.  Inside a group KI waves (one, or two in the 128x128 tile) share a block and take 4 / KI of the four
// 16-deep steps of every K tile.  A wave has 16 / KI MFMAs between two barriers: sixteen, or eight in the 128x128 tile.  The sums
// of the groups and of the waves of a block are added through LDS in a fixed order before the epilogue.
//
//   LDS       a ring of NST stages; a stage holds, per group, one K tile (64 deep) of A and of B in the layout of
//             gemm_dtl.hip: [rows][128 bytes] with the 16-byte chunk c of row r at c ^ ((r >> 1) & 7) for an operand whose
//             reduction index is contiguous; [64 reduction rows][columns] with 64-byte segments swizzled by the row for a
//             strided one, read with the transposing LDS load.
//   loop      one stage per trip, S = 16 / KI slots of one MFMA each.  Slots 0..S-5 issue the loads of the stage NST - 1 ahead
//             into the ring slot that the barrier of the previous trip freed; at slot S-4 the wave has all its fragments, waits
//             for its loads of the next stage, and after the barrier reads that stage's first fragments under the last step.
//             Stages past the end are loaded through offsets outside the descriptor: the number of loads in flight, and
//             with it every s_waitcnt immediate, is the same in every trip.
//   epilogue  the accumulators go to LDS as fp32, and the workgroup writes the tile row by row, 8 columns per thread.
//
// What bounds it: a CU has about 64 KB of loads in flight whatever the ring depth (three, four and five stages measure the
// same, two are 1.6x slower), i.e. 50 bytes/ns of operands that come from HBM, 80 from the Infinity Cache; the products
// without their loads take 0.38 us per 128x128 K tile against 0.55 with them.  Measured on MI355X, weights from HBM, against
// the tiles that served these shapes before (256x128 by eight waves, or one or two waves per workgroup), us per product:
//   1000 x 2048 x 6144 NT 79.8 -> 43.6 (128x64);   1016 x 4096 x 4096 NT 52.4 -> 41.5 (128x128);
//   512 x 2048 x 2048 NT 26.0 -> 14.7;   256 x 4096 x 24576 NN 298 -> 148;   2048 x 2048 x 2040 TN 29.9 -> 22.6
#include "gemm_device.hpp"
#include <type_traits>
#include <utility>

using namespace gemm_dev;

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int V>
using IC = std::integral_constant<int, V>;
template <class F, int... S>
RP_DEV void for_seq(F&& f, std::integer_sequence<int, S...>) {
  (f(IC<S>{}), ...);
}

constexpr int BK = 64;
constexpr int ST_LD = 68;                 // epilogue staging row stride in floats
constexpr int ST_BLOCK = 64 * ST_LD;      // one wave's 64x64 block

RP_DEV void load_to_lds(uint32_t lds, uint32_t voff, i32x4 rs, uint32_t soff) {   // see gemm_dtl.hip
  // (a scalar write of M0 has to be one wait state old when a load to LDS reads it)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" : : "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory");
}

RP_DEV i32x4 raw_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r.x = (int)(uint32_t)b;
  r.y = (int)((uint32_t)(b >> 32) & 0xffffu);
  r.z = (int)bytes;
  r.w = 0x00020000;
  return r;
}

// One operand's unit: X = 64 * (waves along it) rows or columns of one K tile, loaded by NWT waves with NL instructions each.
template <int X, int NWT, bool TR>
struct Unit {
  static constexpr int BYTES = X * BK * 2;
  static constexpr int NL = X / 8 / NWT;                     // 1 KB load instructions per wave
  static constexpr int ROWB = TR ? X * 2 : 128;              // bytes of a row
  static constexpr int RPI = 1024 / ROWB;                    // rows per instruction
  static constexpr int CPR = ROWB / 16;                      // 16-byte chunks per row
  static_assert(X / 8 % NWT == 0, "the unit does not divide over the waves");
  // swizzle of the 64-byte segments of a transposed unit: the four reduction rows that a transposing read touches at once
  // fall into the four 64-byte quarters of the banks
  static RP_DEV int seg_swz(int kr) { return X == 64 ? (kr >> 1) & 1 : kr & 3; }

  int kidx[TR ? NL : 2];      // the lane's reduction index inside the K tile, per instruction (TR) or its parity
  // byte offsets of the lane's chunks at reduction offset 0; xof(r): operand row of tile row r, or -1 past the end
  template <class F>
  RP_DEV void offsets(uint32_t (&vo)[NL], int w, int lane, long ld, F&& xof) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = (w * NL + i) * RPI + lane / CPR, pos = lane % CPR;
      if constexpr (!TR) {
        const int ch = pos ^ ((row >> 1) & 7);
        kidx[i & 1] = ch * 8;
        const long x = xof(row);
        vo[i] = x >= 0 ? (uint32_t)(x * ld + ch * 8) * 2u : OOB;
      } else {
        kidx[i] = row;
        const long x = xof((((pos >> 2) ^ seg_swz(row)) * 32) + (pos & 3) * 8);
        vo[i] = x >= 0 ? (uint32_t)((long)row * ld + x) * 2u : OOB;
      }
    }
  }
  // the same for a unit that is one 16 KB block of dS (128 columns, see attention.hip)
  RP_DEV void offsets_ds(uint32_t (&vo)[NL], int w, int lane) {
    static_assert(TR && X == 128, "the layout of dS");
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = (w * NL + i) * RPI + lane / CPR, pos = lane % CPR;
      const int q = ((pos >> 2) ^ seg_swz(row)) * 32 + (pos & 3) * 8;
      kidx[i] = row;
      vo[i] = (uint32_t)(((row >> 5) * 8 + (q >> 4)) * 1024 + ((q >> 3) & 1) * 512 + (row & 31) * 16);
    }
  }
  RP_DEV int k_of(int i) const { return kidx[TR ? i : (i & 1)]; }
};

template <int WGM, int WGN, int KG, int KI, int NST, bool TA, bool TB>
struct MidCfg {
  static constexpr int NWT = WGM * WGN * KI, NW = NWT * KG, BM = 64 * WGM, BN = 64 * WGN;
  using UA = Unit<BM, NWT, TA>;
  using UB = Unit<BN, NWT, TB>;
  static constexpr int SUB = UA::BYTES + UB::BYTES, STAGE = SUB * KG;
  static constexpr int MAIN = STAGE * NST, EPI = NW * ST_BLOCK * 4;
  static constexpr int SMEM = MAIN > EPI ? MAIN : EPI;
  static constexpr int WPS = NW == 8 ? 2 : (SMEM * 2 <= 160 * 1024 ? 2 : 1);     // waves per SIMD
  static_assert(SMEM <= 160 * 1024, "LDS");
};

// One workgroup's tile of one product: tile number `blk` of the product's `tiles`, reduction slice `slice` of `nslices`.
// ADS: A is a row of blocks of dS.
template <int WGM, int WGN, int KG, int KI, int NST, bool TA, bool TB, bool ADS = false>
RP_DEV void mid_block(const GemmArgs& p, int blk, int slice, int nslices) {
  using C = MidCfg<WGM, WGN, KG, KI, NST, TA, TB>;
  using UA = typename C::UA;
  using UB = typename C::UB;
  constexpr int BM = C::BM, BN = C::BN, NWT = C::NWT, LPT = UA::NL + UB::NL;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NWT, wg = wave % NWT;                     // group, wave within it (loads)
  const int ki = wg / (WGM * WGN), wm = wg % (WGM * WGN) / WGN, wn = wg % WGN;
  const int lr = lane & 31, lk = lane >> 5;

  int tile_m, tile_n;
  tile_of_block(p.M, p.N, BM, BN, tile_m, tile_n, 8, blk);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk1 = (p.K + BK - 1) / BK;
  const int nk_all = nk1 + (p.K2 + BK - 1) / BK;
  const int per_split = (nk_all + nslices - 1) / nslices;
  const int kt0 = slice * per_split;
  const int nk = (nk_all - kt0) < per_split ? (nk_all - kt0 > 0 ? nk_all - kt0 : 0) : per_split;
  const int niter = (nk + KG - 1) / KG;
  // SwiGLU forward: the tile is BN/2 gate columns and the BN/2 up columns that go with them
  const int fold = (!TB && p.epi == EPI_SWIGLU_FWD) ? p.N >> 1 : 0;

  UA ua;
  UB ub;
  uint32_t va[UA::NL], vb[UB::NL];
  auto a_row = [&](int r) -> long { return m0 + r < p.M ? m0 + r : -1; };
  auto b_row = [&](int r) -> long {
    if (!fold) return n0 + r < p.N ? n0 + r : -1;
    const int gl = (n0 >> 1) + (r < BN / 2 ? r : r - BN / 2);
    return gl < fold ? (r < BN / 2 ? gl : fold + gl) : -1;
  };
  if constexpr (ADS) ua.offsets_ds(va, wg, lane);
  else ua.offsets(va, wg, lane, p.lda, a_row);
  ub.offsets(vb, wg, lane, p.ldb, b_row);
  i32x4 rsA = raw_rsrc(p.A, p.bytesA), rsB = raw_rsrc(p.B, p.bytesB);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)kg * C::SUB;

  // the stage being loaded: reduction indices left from its K tile on (0 or less: past the end), byte offsets of the tile,
  // ring slot
  bool second = false;
  int lim = 0;
  uint32_t soffA = 0, soffB = 0, stepA = 0, stepB = 0, atA = 0, atB = 0, lds_ring = 0, ldsA = 0, ldsB = 0;
  auto start = [&](int kt, int kend, long lda, long ldb) {
    lim = kend - kt * BK;
    stepA = (TA ? (uint32_t)lda * 2u : 2u) * BK;
    stepB = (TB ? (uint32_t)ldb * 2u : 2u) * BK;
    atA = (uint32_t)kt * stepA;
    atB = (uint32_t)kt * stepB;
  };
  int kt = kt0 + kg;                                             // K tile of the stage, over both operand pairs
  const int kt_end = kt0 + nk;
  start(kt, kt_end < nk1 ? kt_end * BK : p.K, p.lda, p.ldb);
  auto prep = [&]() {
    if (lim <= 0 && !second && kt >= nk1 && kt < kt_end) {       // uniform over the wave, once: on to the second operand pair
      asm volatile("" ::: "memory");
      second = true;
      ua.offsets(va, wg, lane, p.lda2, a_row);
      ub.offsets(vb, wg, lane, p.ldb2, b_row);
      rsA = raw_rsrc(p.A2, p.bytesA2);
      rsB = raw_rsrc(p.B2, p.bytesB2);
      start(kt - nk1, kt_end - nk1 < (p.K2 + BK - 1) / BK ? (kt_end - nk1) * BK : p.K2, p.lda2, p.ldb2);
    }
    soffA = lim > 0 ? atA : 0u;
    soffB = lim > 0 ? atB : 0u;
    ldsA = lds0 + lds_ring + (uint32_t)(wg * UA::NL * 1024);
    ldsB = lds0 + lds_ring + UA::BYTES + (uint32_t)(wg * UB::NL * 1024);
    lds_ring = lds_ring + C::STAGE == (uint32_t)C::MAIN ? 0u : lds_ring + C::STAGE;
  };
  auto advance = [&]() {
    kt += KG;
    lim -= KG * BK;
    atA += KG * stepA;
    atB += KG * stepB;
  };
  auto issue = [&](auto qtag) __attribute__((always_inline)) {
    constexpr int q = decltype(qtag)::value;
    if constexpr (q < UA::NL) load_to_lds(ldsA + q * 1024, ua.k_of(q) < lim ? va[q] : OOB, rsA, soffA);
    else load_to_lds(ldsB + (q - UA::NL) * 1024, ub.k_of(q - UA::NL) < lim ? vb[q - UA::NL] : OOB, rsB, soffB);
  };

  // fragment reads: byte offsets inside a stage
  const int l16 = lane & 15, g16 = lane >> 4, c2 = l16 >> 2, s7 = (lr >> 1) & 7;
  uint32_t fA[4], fB[4], fAt[2], fBt[2];
  const uint32_t baseA = (uint32_t)kg * C::SUB, baseB = baseA + UA::BYTES;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    fA[ks] = baseA + (uint32_t)((wm * 64 + lr) * 128 + ((2 * ks + lk) ^ s7) * 16);
    fB[ks] = baseB + (uint32_t)((wn * 64 + lr) * 128 + ((2 * ks + lk) ^ s7) * 16);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    fAt[i] = baseA + (uint32_t)((8 * lk + c2) * UA::ROWB + ((wm * 2 + i) ^ UA::seg_swz(c2)) * 64 + 32 * (g16 & 1) + 8 * (l16 & 3));
    fBt[i] = baseB + (uint32_t)((8 * lk + c2) * UB::ROWB + ((wn * 2 + i) ^ UB::seg_swz(c2)) * 64 + 32 * (g16 & 1) + 8 * (l16 & 3));
  }
  uint4 af[2][2], bfr[2][2];
  auto read_tr = [&](uint32_t off, int rowb) -> uint4 {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(smem + off)));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(smem + off + 4 * rowb)));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // vmcnt encoding of s_waitcnt: bits 3:0 and 15:14; lgkmcnt bits 11:8, expcnt 6:4
  constexpr int VM = (NST - 2) * LPT, VMBITS = (VM & 15) | ((VM >> 4) << 14);
  static_assert(VM < 64 && NST >= 2 && KI <= 2, "loads in flight");
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) {
    prep();
    for_seq(issue, std::make_integer_sequence<int, LPT>{});
    advance();
  }
  __builtin_amdgcn_s_waitcnt(0x0f70 | VMBITS);
  __syncthreads();
  // this wave's steps of a K tile: SP from ks0 on
  constexpr int SP = 4 / KI, S = 4 * SP;
  uint32_t fa[SP], fb[SP];
#pragma unroll
  for (int q = 0; q < SP; ++q) {
    fa[q] = ki == 0 ? fA[q] : fA[(SP + q) & 3];
    fb[q] = ki == 0 ? fB[q] : fB[(SP + q) & 3];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) { fAt[i] += ki * SP * 16 * UA::ROWB; fBt[i] += ki * SP * 16 * UB::ROWB; }
  auto read_a = [&](int set, uint32_t ring, auto qtag, int i) __attribute__((always_inline)) {
    constexpr int q = decltype(qtag)::value;
    if constexpr (!TA) af[set][i] = *reinterpret_cast<const uint4*>(smem + ring + fa[q] + i * 4096);
    else af[set][i] = read_tr(ring + fAt[i] + q * 16 * UA::ROWB, UA::ROWB);
  };
  auto read_b = [&](int set, uint32_t ring, auto qtag, int j) __attribute__((always_inline)) {
    constexpr int q = decltype(qtag)::value;
    if constexpr (!TB) bfr[set][j] = *reinterpret_cast<const uint4*>(smem + ring + fb[q] + j * 4096);
    else bfr[set][j] = read_tr(ring + fBt[j] + q * 16 * UB::ROWB, UB::ROWB);
  };
  read_a(0, 0, IC<0>{}, 0); read_b(0, 0, IC<0>{}, 0); read_b(0, 0, IC<0>{}, 1); read_a(0, 0, IC<0>{}, 1);

  uint32_t ring = 0;
  for (int it = 0; it < niter; ++it) {
    prep();
    const uint32_t nring = ring + C::STAGE == (uint32_t)C::MAIN ? 0u : ring + C::STAGE;
    auto slot = [&](auto sltag) __attribute__((always_inline)) {
      constexpr int sl = decltype(sltag)::value;
      constexpr int q = sl >> 2, I = sl & 3, i = I >> 1, j = I & 1, set = SP == 1 ? 0 : q & 1;
      if constexpr (sl == S - 4) {
        __builtin_amdgcn_s_waitcnt(0x0070 | VMBITS);    // this stage's fragments, the loads of the next stage
        __syncthreads();
      }
      acc[i][j] = mfma32(af[set][i], bfr[set][j], acc[i][j]);
      constexpr int nset = SP == 1 ? 0 : q + 1 < SP ? set ^ 1 : 0;
      const uint32_t rd = q + 1 < SP ? ring : nring;
      using NQ = IC<(q + 1 < SP ? q + 1 : 0)>;
      if constexpr (I == 0) { read_a(nset, rd, NQ{}, 0); read_b(nset, rd, NQ{}, 0); }
      if constexpr (I == 1) { read_b(nset, rd, NQ{}, 1); read_a(nset, rd, NQ{}, 1); }
      for_seq([&](auto ltag) __attribute__((always_inline)) {
        constexpr int l = decltype(ltag)::value;
        if constexpr (l * (S - 4) / LPT == sl) issue(ltag);
      }, std::make_integer_sequence<int, LPT>{});
      if constexpr (sl == S - 2) advance();
      __builtin_amdgcn_sched_barrier(0);
    };
    for_seq(slot, std::make_integer_sequence<int, S>{});
    ring = nring;
  }
  __builtin_amdgcn_s_waitcnt(0x0070);    // the empty loads past the end write LDS too
  __syncthreads();

  float* const stg = reinterpret_cast<float*>(smem);
  {
    float* const d = stg + wave * ST_BLOCK + 4 * lk * ST_LD + lr;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) d[AccMap<false>::acc_row(i, v) * ST_LD + j * 32] = acc[i][j][v];
  }
  __syncthreads();

  // eight columns of a row of the tile, the groups' parts added in order, times alpha
  auto take = [&](int row, int col, float (&o)[8]) {
    const float* s = stg + ((row >> 6) * WGN + (col >> 6)) * ST_BLOCK + (row & 63) * ST_LD + (col & 63);
    float4 x = *reinterpret_cast<const float4*>(s), y = *reinterpret_cast<const float4*>(s + 4);
#pragma unroll
    for (int g = 1; g < KG * KI; ++g) {
      const float4 x2 = *reinterpret_cast<const float4*>(s + g * WGM * WGN * ST_BLOCK), y2 = *reinterpret_cast<const float4*>(s + g * WGM * WGN * ST_BLOCK + 4);
      x.x += x2.x; x.y += x2.y; x.z += x2.z; x.w += x2.w;
      y.x += y2.x; y.y += y2.y; y.z += y2.z; y.w += y2.w;
    }
    o[0] = p.alpha * x.x; o[1] = p.alpha * x.y; o[2] = p.alpha * x.z; o[3] = p.alpha * x.w;
    o[4] = p.alpha * y.x; o[5] = p.alpha * y.y; o[6] = p.alpha * y.z; o[7] = p.alpha * y.w;
  };
  auto pack = [](const float (&o)[8]) {
    return make_uint4(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7]));
  };
  auto unpack = [](const uint4& u, float (&f)[8]) {
    f[0] = bf16_lo(u.x); f[1] = bf16_hi(u.x); f[2] = bf16_lo(u.y); f[3] = bf16_hi(u.y);
    f[4] = bf16_lo(u.z); f[5] = bf16_hi(u.z); f[6] = bf16_lo(u.w); f[7] = bf16_hi(u.w);
  };
  constexpr int NTH = C::NW * 64;
  bf16* const Cp = reinterpret_cast<bf16*>(p.C);
  if (fold) {
    constexpr int CW = BN / 16, NIT = (BM * CW + NTH - 1) / NTH;
    bf16* const Ap = reinterpret_cast<bf16*>(p.C2);
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
      const int c = t * NTH + tid, row = c / CW, col = c % CW * 8, grow = m0 + row, gcol = (n0 >> 1) + col;
      if (BM * CW % NTH && row >= BM) break;
      float g[8], u[8], a[8];
      take(row, col, g);
      take(row, col + BN / 2, u);
      if (grow < p.M && gcol < fold) {
        const uint4 gp = pack(g), up = pack(u);
        *reinterpret_cast<uint4*>(Cp + (long)grow * p.ldc + gcol) = gp;
        *reinterpret_cast<uint4*>(Cp + (long)grow * p.ldc + fold + gcol) = up;
        unpack(gp, g);      // the activation is that of the rounded values, as a kernel reading them back computes it
        unpack(up, u);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = silu_f32(g[e]) * u[e];
        *reinterpret_cast<uint4*>(Ap + (long)grow * p.ldc2 + gcol) = pack(a);
      }
    }
    return;
  }
  constexpr int CW = BN / 8, NIT = BM * CW / NTH, NB = NIT < 4 ? NIT : 4;
  static_assert(NIT % NB == 0, "epilogue batches");
  const bf16* const Rp = reinterpret_cast<const bf16*>(p.R);
  float* const Cf = reinterpret_cast<float*>(p.C) + (long)slice * p.c_slice_stride;
  // what is added from memory is loaded for NB chunks before any is stored (see gemm_device.hpp)
#pragma unroll
  for (int t0 = 0; t0 < NIT; t0 += NB) {
    uint4 r0[NB], r1[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int c = (t0 + u) * NTH + tid, row = c / CW, col = c % CW * 8, grow = m0 + row, gcol = n0 + col;
      r0[u] = make_uint4(0u, 0u, 0u, 0u);
      r1[u] = r0[u];
      if (grow < p.M && gcol < p.N) {
        if (p.epi == EPI_SWIGLU_BWD) {
          r0[u] = *reinterpret_cast<const uint4*>(Rp + (long)grow * p.ldr + gcol);
          r1[u] = *reinterpret_cast<const uint4*>(Rp + (long)grow * p.ldr + p.N + gcol);
        } else if (p.epi == EPI_F32) {
          if (p.beta) {
            r0[u] = *reinterpret_cast<const uint4*>(Cf + (long)grow * p.ldc + gcol);
            r1[u] = *reinterpret_cast<const uint4*>(Cf + (long)grow * p.ldc + gcol + 4);
          }
        } else if (p.epi == EPI_BF16 && p.R) {   // ldr is a multiple of 4 only
          const uint2 lo = *reinterpret_cast<const uint2*>(Rp + (long)grow * p.ldr + gcol), hi = *reinterpret_cast<const uint2*>(Rp + (long)grow * p.ldr + gcol + 4);
          r0[u] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int c = (t0 + u) * NTH + tid, row = c / CW, col = c % CW * 8, grow = m0 + row, gcol = n0 + col;
      float o[8];
      take(row, col, o);
      if (grow >= p.M || gcol >= p.N) continue;
      if (p.epi == EPI_SWIGLU_BWD) {
        float d[8], g[8], up[8], dg[8], du[8];
        unpack(pack(o), d);      // the product is rounded as if it had been stored
        unpack(r0[u], g);
        unpack(r1[u], up);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float sg = sigmoid_f32(g[e]);
          dg[e] = d[e] * up[e] * sg * (1.f + g[e] * (1.f - sg));
          du[e] = d[e] * g[e] * sg;
        }
        *reinterpret_cast<uint4*>(Cp + (long)grow * p.ldc + gcol) = pack(dg);
        *reinterpret_cast<uint4*>(Cp + (long)grow * p.ldc + p.N + gcol) = pack(du);
      } else if (p.epi == EPI_F32) {
        const float4 x = __builtin_bit_cast(float4, r0[u]), y = __builtin_bit_cast(float4, r1[u]);
        float4* const dst = reinterpret_cast<float4*>(Cf + (long)grow * p.ldc + gcol);
        dst[0] = make_float4(o[0] + x.x, o[1] + x.y, o[2] + x.z, o[3] + x.w);
        dst[1] = make_float4(o[4] + y.x, o[5] + y.y, o[6] + y.z, o[7] + y.w);
      } else if (p.epi == EPI_F32_ATOMIC) {
#pragma unroll
        for (int e = 0; e < 8; ++e) atomicAdd(reinterpret_cast<float*>(p.C) + (long)grow * p.ldc + gcol + e, o[e]);
      } else {
        float r[8];
        unpack(r0[u], r);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += r[e];
        *reinterpret_cast<uint4*>(Cp + (long)grow * p.ldc + gcol) = pack(o);
      }
    }
  }
}

template <int WGM, int WGN, int KG, int KI, int NST, bool TA, bool TB>
__global__ void __launch_bounds__(64 * WGM * WGN * KG * KI)
    __attribute__((amdgpu_waves_per_eu(MidCfg<WGM, WGN, KG, KI, NST, TA, TB>::WPS, MidCfg<WGM, WGN, KG, KI, NST, TA, TB>::WPS)))
    gemm_mid_kernel(const GemmArgs p) {
  mid_block<WGM, WGN, KG, KI, NST, TA, TB>(p, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.y);
}

// Several independent products in one launch, on 64x64 tiles: workgroups [first, first + tiles * slices) work on a product.
// A product that needs a few of the 256 CUs for a few microseconds spends most of its 8 to 12 us on being launched and on
// filling its pipeline; the adapters' products of one projection and the weight gradients of short sequences are four to seven
// of them.  Measured (one stream): fused toy step of 128 tokens 479 -> 395 us, backward stage of 2 x 508 tokens at h = 4096
// with seven adapters 1264 -> 1195 us, of 176 tokens at h = 5120 1080 -> 964 us, of 8192 tokens at h = 4096 8525 -> 8407 us.
// (the fields a product of a group has: the kernel arguments are copied at every launch)
struct MultiOne {
  const void *A, *B, *A2, *B2, *R;
  void* C;
  long lda, ldb, lda2, ldb2, ldr, ldc, c_slice_stride;
  unsigned bytesA, bytesB, bytesA2, bytesB2;
  int M, N, K, K2, beta, epi, splits, layout, first, tiles;
  float alpha;
};
struct MultiArgs { int n; MultiOne g[GEMM_GROUP_MAX]; };

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_multi_kernel(const MultiArgs a) {
  int i = 0;
  while (i + 1 < a.n && (int)blockIdx.x >= a.g[i + 1].first) ++i;
  const MultiOne& q = a.g[__builtin_amdgcn_readfirstlane(i)];
  const int local = (int)blockIdx.x - q.first;
  const int slice = local / q.tiles, blk = local - slice * q.tiles;
  GemmArgs g{};
  g.A = q.A; g.B = q.B; g.A2 = q.A2; g.B2 = q.B2; g.R = q.R; g.C = q.C;
  g.lda = q.lda; g.ldb = q.ldb; g.lda2 = q.lda2; g.ldb2 = q.ldb2; g.ldr = q.ldr; g.ldc = q.ldc; g.c_slice_stride = q.c_slice_stride;
  g.bytesA = q.bytesA; g.bytesB = q.bytesB; g.bytesA2 = q.bytesA2; g.bytesB2 = q.bytesB2;
  g.M = q.M; g.N = q.N; g.K = q.K; g.K2 = q.K2; g.beta = q.beta; g.epi = q.epi; g.alpha = q.alpha;
  if (q.layout == GEMM_NT) mid_block<1, 1, 4, 1, 2, false, false>(g, blk, slice, q.splits);
  else if (q.layout == GEMM_NN) mid_block<1, 1, 4, 1, 2, false, true>(g, blk, slice, q.splits);
  else mid_block<1, 1, 4, 1, 2, true, true>(g, blk, slice, q.splits);
}

// dQ of causal attention from the dS that the dK/dV kernel left: per head and 128-query tile t a product of a [64 (2t + 2), 128]
// matrix (blocks of dS) with the head's K, reduction over the keys up to the tile's last query.  Heaviest
// tiles first; an XCD works on neighbouring heads, i.e. on few K/V heads.  Bound by reading dS:
// 8192 tokens, 32 heads 2.2 GB in 506 us (4.3 TB/s), where the kernel that recomputes the scores takes 726.
struct AttnDqArgs { const bf16 *ds, *k; bf16* dq; size_t head; long ldk, lddq; int batch, seq, a, kh; float scale; };
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) attn_dq_from_ds_kernel(const AttnDqArgs p) {
  const int nt = (p.seq + 127) / 128, nhb = p.a * p.batch;
  const int t = nt - 1 - (int)blockIdx.x / nhb, i = (int)blockIdx.x % nhb;
  const int hb = (nhb & 7) ? i : (i & 7) * (nhb >> 3) + (i >> 3);
  const int hq = hb % p.a, b = hb / p.a;
  const long tok0 = (long)b * p.seq;
  GemmArgs g{};
  g.M = p.seq - 128 * t < 128 ? p.seq - 128 * t : 128;
  g.N = 128;
  g.K = 128 * t + g.M;                       // the keys up to the tile's last query
  g.A = p.ds + (size_t)hb * p.head + (size_t)(t * (t + 1)) * 8192;
  g.lda = 128;
  g.bytesA = (unsigned)(2 * t + 2) * 16384u;
  g.B = p.k + tok0 * p.ldk + hq / (p.a / p.kh) * 128;
  g.ldb = p.ldk;
  g.bytesB = (unsigned)(((long)(g.K - 1) * p.ldk + 128) * 2);
  g.C = p.dq + (tok0 + 128 * t) * p.lddq + hq * 128;
  g.ldc = p.lddq;
  g.alpha = p.scale;
  g.epi = EPI_BF16;
  mid_block<2, 2, 1, 2, 4, true, true, true>(g, 0, 0, 1);
}

template <int WGM, int WGN, int KG, int KI, int NST, bool TA, bool TB>
hipError_t mid_launch_one(hipStream_t st, const GemmArgs& a) {
  using C = MidCfg<WGM, WGN, KG, KI, NST, TA, TB>;
  static bool attr_done = false;
  auto kern = gemm_mid_kernel<WGM, WGN, KG, KI, NST, TA, TB>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int tiles = ((a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN);
  RP_LAUNCH(kern, dim3(tiles, a.splits > 0 ? a.splits : 1), dim3(64 * C::NW), C::SMEM, st, a);
  return hipGetLastError();
}

template <int WGM, int WGN, int KG, int KI, int NST>
hipError_t mid_launch_layout(hipStream_t st, const GemmArgs& a, int layout) {
  switch (layout) {
    case GEMM_NT: return mid_launch_one<WGM, WGN, KG, KI, NST, false, false>(st, a);
    case GEMM_NN: return mid_launch_one<WGM, WGN, KG, KI, NST, false, true>(st, a);
    default: return mid_launch_one<WGM, WGN, KG, KI, NST, true, true>(st, a);
  }
}

}  // namespace

hipError_t gemm_mid_launch(hipStream_t st, const GemmArgs& a, int layout, int tile) {
  switch (tile) {
    case 2: return mid_launch_layout<4, 2, 1, 1, 3>(st, a, layout);   // 256x128, eight waves
    case 3: return mid_launch_layout<2, 2, 1, 2, 4>(st, a, layout);   // 128x128, eight waves (two per block, half of the steps each)
    case 4: return mid_launch_layout<2, 1, 2, 1, 3>(st, a, layout);   // 128x64, four waves in two groups
    case 8: return mid_launch_layout<1, 1, 4, 1, 2>(st, a, layout);   // 64x64, four waves in four groups
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_attn_dq(hipStream_t st, const void* ds, size_t head_bytes, const void* k, long ldk, void* dq, long lddq, int batch, int seq,
                        int a, int kh, int d, float scale) {
  constexpr int SMEM = MidCfg<2, 2, 1, 2, 4, true, true>::SMEM;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_dq_from_ds_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if (d != 128 || ldk % 8 || lddq % 8 || (long)seq * ldk >= (1L << 30)) return hipErrorInvalidValue;
  const AttnDqArgs p{(const bf16*)ds, (const bf16*)k, (bf16*)dq, head_bytes / 2, ldk, lddq, batch, seq, a, kh, scale};
  RP_LAUNCH(attn_dq_from_ds_kernel, dim3((unsigned)((seq + 127) / 128 * a * batch)), dim3(512), SMEM, st, p);
  return hipGetLastError();
}

hipError_t gemm_multi_run(hipStream_t st, int n, const int* layouts, const GemmArgs* g) {
  constexpr int SMEM = MidCfg<1, 1, 4, 1, 2, false, false>::SMEM;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_multi_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if (n < 1 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
  MultiArgs a{};
  a.n = n;
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& p = g[i];
    const int tiles = ((p.M + 63) / 64) * ((p.N + 63) / 64);
    a.g[i] = {p.A, p.B, p.A2, p.B2, p.R, p.C, p.lda, p.ldb, p.lda2, p.ldb2, p.ldr, p.ldc, p.c_slice_stride, p.bytesA, p.bytesB, p.bytesA2,
              p.bytesB2, p.M, p.N, p.K, p.K2, p.beta, p.epi, p.splits, layouts[i], blocks, tiles, p.alpha};
    blocks += tiles * p.splits;
  }
  RP_LAUNCH(gemm_multi_kernel, dim3(blocks), dim3(256), SMEM, st, a);
  return hipGetLastError();
}
