// bf16 GEMM C = A * B^T (NT: both operands reduction-contiguous), C = A * B (NN: B is [K, N]) or C = A^T * B (TN: A is
// [K, M] as well), 256x256 output tile, operands loaded from HBM straight into LDS (no staging registers, no LDS store instructions) and four waves of 128x128
// each -- one wave per SIMD, 256 accumulator registers per lane (the AGPR half of the register file).
//
// Against the eight-wave kernel of gemm.hip a K tile of the same output tile costs a third fewer fragment reads (every
// fragment feeds eight MFMAs), no LDS stores and hardly any vector or scalar arithmetic: the loop is 128 MFMAs, 32
// fragment reads (TN: 64 half ones), 16 loads and a barrier.  What bounds it is the power that the matrix pipe draws: the chip clocks
// down until it fits, so what an instruction costs in energy counts before what it costs in slots.  v_mfma_f32_16x16x32_bf16 moves half
// the accumulators of the 32x32x16 instruction per FLOP and gives the same bits (mfma16 in common.hpp).  Measured on MI355X (8192 x 8192 x
// 2048 | 4096 | 8192 | 16384, same box, 32x32x16 -> 16x16x32, us): NT 223 | 405 | 781 | 1562 -> 194 | 361 | 709 | 1436 (1.38 -> 1.55
// PFLOP/s at 8192), NN 222 | 404 | 779 | 1559 -> 197 | 367 | 714 | 1445, TN 222 | 404 | 783 | 1569 -> 200 | 370 | 721 | 1453.
// Where the reads, the loads and the barrier stand among the MFMAs no longer matters (four plans within 0.5 %).
//
//   LDS       a ring of five 32 KB units; a unit is one operand of one K tile of 64: 256 rows of 128 bytes -- a load
//             fetches whole 128-byte lines (rows of 64 bytes, as a K tile of 32 would have, double the requests to L2:
//             measured, and slower than the staged kernel).  The 16-byte chunk c of row r sits at chunk position
//             c ^ ((r >> 1) & 7): fragment reads meet no bank conflict, and since a load instruction fills 1 KB of LDS
//             with consecutive lanes while the 16 bytes a lane fetches are free to choose, the swizzle costs nothing.
//             Units are used in the order B(0), A(0), B(1), A(1), ...: unit u lives in ring slot u mod 5.
//   loads     eight per wave and unit, in slots of their own.  B(t+2) is issued in the first half of tile t (into the slot of A(t-1),
//             free since the barrier of tile t-1), A(t+2) behind the barrier of tile t (into the slot of B(t)).
//   barrier   one per K tile, at slot 74 of 128: by then the wave has all its fragments of tile t.  Before it the wave
//             waits for its own loads of tile t+1 (s_waitcnt vmcnt(8): B(t+2) may be in flight); after it tile t+1 is
//             complete in LDS and its first fragments are read under the last step of tile t.
//   tail      tiles past the end are "loaded" with an offset outside the descriptor (no memory traffic), which keeps
//             the number of loads in flight -- and with it the s_waitcnt immediates -- the same to the end.
//
// The loads are inline assembly: the compiler orders a buffer-load-to-LDS builtin against every later LDS read with
// s_waitcnt vmcnt(0), which would serialise the pipeline; here the counts are kept by hand, and no compiler-visible
// memory instruction may be pending when the loop is entered (see the rare paths of the load state).
//   NN        B's units keep the operand's [K, N] layout (64 rows of 512 bytes; the 32-byte segment of MFMA tile column s of row k at
//             segment s ^ seg_swizzle(k)), its fragments are two transposing reads (ds_read_b64_tr_b16) each.
//   TN        the same for A.
// Second operand pair, row map, reduction slices and every epilogue as in gemm.hip; results are bit-identical to its 256x256 tile (the same
// order of the reduction).  Most grouped products (GRP below) run here, and of the others those that gemm_launch sends (all but short
// reductions and skinny outputs).
#include "gemm_device.hpp"
#include <type_traits>
#include <utility>

using namespace gemm_dev;

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int V>
using IC = std::integral_constant<int, V>;
// f(IC<0>), f(IC<1>), ... in order: a loop whose index is a constant expression in its body
template <class F, int... S>
RP_DEV void for_seq(F&& f, std::integer_sequence<int, S...>) {
  (f(IC<S>{}), ...);
}

constexpr int BK = 64;                            // reduction indices per K tile: a row of a tile is one 128-byte line
constexpr int UNIT_BYTES = 256 * BK * 2;          // one operand of one K tile: 256 rows of 128 bytes, 32 KB
constexpr int NUNIT = 5;
constexpr int DTL_SMEM = NUNIT * UNIT_BYTES;      // 160 KB: the whole LDS of a CU; the epilogue's four staging areas (72 KB) reuse it
static_assert(DTL_SMEM >= 4 * STG_BYTES, "epilogue staging does not fit");

// [K, X] units: 64 rows of 512 bytes, sixteen 32-byte segments = the columns of one 16x16 tile each; segment s of row k lies at
// s ^ seg_swizzle(k).  A transposing read touches the rows 8 g + c (c < 4) of the tile's segment for four lane groups g: eight rows at a
// time (two groups), which then lie in eight different places of the banks.
RP_DEV int seg_swizzle(int k) { return ((k & 3) << 1) | ((k >> 3) & 1); }

// acc += a b in the accumulator's own registers of the AGPR half.  (Written with the builtin the compiler moves the 64 accumulators of the
// loop around: 100 to 400 copies per K tile.)  The hazards are the loop's to keep: fragments come from LDS reads, for which the compiler
// waits, an accumulator is next used 64 instructions later, and nothing reads one before the wait behind the loop.
RP_DEV void mfma16_in_place(f32x4& acc, const uint4& a, const uint4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(__builtin_bit_cast(bf16x8, a)), "v"(__builtin_bit_cast(bf16x8, b)));
}

// Where the reads and loads of a K tile go (see the slot plan in dtl_block): RB reads of B's and RA of A's fragments per step.
template <int RB, int RA>
struct SlotPlan {
  static constexpr int BAR = 74, N = RB + RA;
  static constexpr int first(int s) { return s == 0 ? 2 : 76; }
  static constexpr int span(int s) { return s == 0 ? 56 : 52; }
  static constexpr int at(int s, int n) { return first(s) + n * span(s) / N; }      // slot of read n of the coming step
  // number of the read in slot sl, B's first; -1: none
  static constexpr int read(int sl) {
    const int s = sl >= 76 ? 1 : 0;
    for (int n = 0; n < N; ++n)
      if (at(s, n) == sl) return n;
    return -1;
  }
  // A's tiles in the order 6, 7, 0, 1, .. 5
  static constexpr int a_read(int n) { return (n + RA / 8 * 6) % RA; }
  // number of the load in slot sl: 0..7 B's, 8..15 A's; each in the first slot without a read from its place on
  static constexpr int load_slot(int n) {
    int sl = 0;
    for (int q = 0; q <= n; ++q) {
      const int want = q < 8 ? 4 + 7 * q : 77 + 4 * (q - 8);
      sl = want > sl + 1 ? want : sl + 1;
      while (read(sl) >= 0) ++sl;
    }
    return sl;
  }
  static constexpr int load(int sl) {
    for (int n = 0; n < 16; ++n)
      if (load_slot(n) == sl) return n;
    return -1;
  }
  static constexpr bool sound() {
    for (int n = 0; n < N; ++n)
      if (n > 0 && (at(0, n) == at(0, n - 1) || at(1, n) == at(1, n - 1))) return false;
    // A's tiles 0 .. 5 are read again behind their last MFMA; B's loads are out before the barrier, A's before the state moves on
    for (int n = 2 * (RA / 8); n < RA; ++n) {
      const int tile = a_read(n) / (RA / 8);
      if (at(0, RB + n) < 8 * tile + 8 || at(1, RB + n) - 64 < 8 * tile + 8) return false;
    }
    return load_slot(7) < BAR && load_slot(8) > BAR && load_slot(15) < 120 && at(0, N - 1) < 60 && at(1, N - 1) < 128;
  }
};
static_assert(SlotPlan<8, 8>::sound() && SlotPlan<16, 8>::sound() && SlotPlan<16, 16>::sound(), "slot plan");

// 64 lanes x 16 bytes from the buffer (per-lane byte offset voff, wave-uniform soff) to LDS bytes [lds + IMM,
// lds + IMM + 1024) of the workgroup, lane l at + 16 l.  Lanes whose offset lies outside the descriptor deliver zeros.
// The LDS address travels in M0; a scalar write of M0 has to be one wait state old when the load reads it (the no-op costs
// nothing: 8192^3 within 0.2 % on all layouts).
// NT: marked non-temporal, for what no other workgroup reads.
template <int IMM, bool NT = false>
RP_DEV void load_to_lds(uint32_t lds, uint32_t voff, i32x4 rs, uint32_t soff) {
  if constexpr (NT)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %4 offen nt lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rs), "n"(IMM), "s"(soff)
                 : "memory", "scc");
  else
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %4 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rs), "n"(IMM), "s"(soff)
                 : "memory", "scc");
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

// What a kernel makes of its tile.  OUT_ROWS: bf16 (plus residual), fp32 (accumulating), SwiGLU forward; OUT_SWIGLU_BWD, OUT_CE_P: those
// epilogues; all on transposed accumulators, straight from the registers.  OUT_COLS: the other cross-entropy epilogues, in which a lane owns
// columns, and the rare ones, through LDS (gemm_device.hpp).
enum { OUT_ROWS = 0, OUT_SWIGLU_BWD = 1, OUT_COLS = 2, OUT_CE_P = 3 };

RP_DEV float acc_read(const f32x4& a, int e) {
  float x;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(a[e]));
  return x;
}
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
RP_DEV void buf_store16(rsrc_t r, uint32_t off, const uint4& v) {
  __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.x, v.y, v.z, v.w}, r, (int)off, 0, 0);
}

// A transposed accumulator gives lane group g (lane / 16) columns 4 g .. 4 g + 3 of the row lane % 16 of a 16x16 tile.  Of two tiles side by
// side, after an exchange between neighbouring groups, it holds eight consecutive columns from pair_column(g) of the 32 on.
RP_DEV int pair_column(int g) { return ((g & 1) << 4) | ((g >> 1) << 3); }
RP_DEV uint4 join_pair(const uint2& l, const uint2& r) {
  const auto x = __builtin_amdgcn_permlane16_swap(l.x, r.x, false, false), y = __builtin_amdgcn_permlane16_swap(l.y, r.y, false, false);
  return make_uint4(x[0], y[0], x[1], y[1]);
}
// Two 16-byte chunks of every row of a row tile, l on the left of r (four lanes hold 64 bytes of a row each) -> 128 bytes of rows 0 .. 7 (a) and of
// rows 8 .. 15 (b), in order, after an exchange between the lanes of rows eight apart; hi: the lane's row is one of the latter.
RP_DEV uint32_t from_row8(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false); }    // row_ror:8
RP_DEV void word_to_lines(bool hi, uint32_t l, uint32_t r, uint32_t& a, uint32_t& b) {
  const uint32_t t = from_row8(hi ? l : r);
  a = hi ? t : l;
  b = hi ? r : t;
}
RP_DEV void to_lines(bool hi, const uint4& l, const uint4& r, uint4& a, uint4& b) {
  word_to_lines(hi, l.x, r.x, a.x, b.x);
  word_to_lines(hi, l.y, r.y, a.y, b.y);
  word_to_lines(hi, l.z, r.z, a.z, b.z);
  word_to_lines(hi, l.w, r.w, a.w, b.w);
}
RP_DEV void unpack8(const uint4& u, float (&f)[8]) {
  f[0] = bf16_lo(u.x); f[1] = bf16_hi(u.x); f[2] = bf16_lo(u.y); f[3] = bf16_hi(u.y);
  f[4] = bf16_lo(u.z); f[5] = bf16_hi(u.z); f[6] = bf16_lo(u.w); f[7] = bf16_hi(u.w);
}
RP_DEV uint4 pack8(const float (&f)[8]) {
  return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}

// The wave's 128x128 block of transposed tiles to memory, from the registers: no LDS, no barrier.  Whatever goes in or out does so as whole
// 128-byte lines, eight rows an instruction (64 bytes of sixteen rows are as good for stores alone, but loads of half lines cost more).
// Rows and columns past the end fall outside the descriptors.  A tile is bound by what it moves while the CU's matrix pipe stands still, and
// more of it in flight is not better: columns outermost, a step's loads ahead, of as few rows as cover the latency.  Against staging each
// half of the block through LDS, same box, us: 8192 x 8192 x 2048 NT 205 -> 191, with a residual 234 -> 221 (4 | 8 row tiles a step 226 | 230, all
// at once 224), fp32 accumulating TN 285 -> 278 (rows outermost, two | four row tiles ahead 296 | 308); 8192 x 24576 x 4096 with SwiGLU forward
// 1220 -> 1173; 8192 x 12288 x 4096 with SwiGLU backward 737 -> 697 (2 | 4 row tiles a step 701 | 714).
template <bool GRP, bool SWB>
RP_DEV void store_rows(const GemmArgs& p, f32x4 (&acc)[8][8], int m0, int Mlim, int n0, int wm, int wn, int lane, int fold) {
  const int r16 = lane & 15, g = lane >> 4;
  const bool hi = r16 & 8;
  const int rows = Mlim - m0 < 256 ? Mlim - m0 : 256;                 // of the tile, from m0 on
  // descriptor of the tile's rows of a matrix with `cols` columns of es bytes and row stride ld
  auto tile_rsrc = [&](const void* base, long ld, int es, int cols) {
    return make_rsrc(static_cast<const char*>(base) + (long)m0 * ld * es, (uint32_t)(((long)(rows - 1) * ld + cols) * es));
  };
  // byte offset of the lane's 16 bytes in row tile i, 128 bytes of a row from column c on; d = 0, 8: its upper, lower rows
  auto at = [&](int i, int d, int c, int lim, long ld, int es) __attribute__((always_inline)) {
    const int col = c + (hi ? 64 / es : 0) + (es == 2 ? pair_column(g) : 4 * g);
    const int row = (GRP ? (i >> 1) * 64 + wm * 32 + (i & 1) * 16 : wm * 128 + i * 16) + (r16 & 7) + d;
    return col < lim ? ((uint32_t)row * (uint32_t)ld + (uint32_t)col) * (uint32_t)es : OOB;
  };
  if (p.alpha != 1.f) {       // uniform, rare
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = p.alpha * acc_read(acc[i][j], e);
          float y;
          asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(y) : "v"(x));
          acc[i][j][e] = y;
        }
    asm volatile("s_nop 7");
  }
  // tiles j, j + 1 as bf16, eight columns a lane
  auto pair = [&](int i, int j) __attribute__((always_inline)) {
    uint2 t[2];
#pragma unroll
    for (int w = 0; w < 2; ++w)
      t[w] = make_uint2(pack_bf16x2(acc_read(acc[i][j + w], 0), acc_read(acc[i][j + w], 1)), pack_bf16x2(acc_read(acc[i][j + w], 2), acc_read(acc[i][j + w], 3)));
    return join_pair(t[0], t[1]);
  };
  if constexpr (!SWB) {
    if (fold) {
      // gate | up, and silu(gate) * up from the rounded values (what a SwiGLU kernel would read back); tiles j and j + 4 go together
      const int c0 = (n0 >> 1) + wn * 64;                             // gate column of the wave
      const rsrc_t rg = tile_rsrc(p.C, p.ldc, 2, fold), ru = tile_rsrc(static_cast<const bf16*>(p.C) + fold, p.ldc, 2, fold), ra = tile_rsrc(p.C2, p.ldc2, 2, fold);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint4 gv[2], uv[2];
        to_lines(hi, pair(i, 0), pair(i, 2), gv[0], gv[1]);
        to_lines(hi, pair(i, 4), pair(i, 6), uv[0], uv[1]);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          const uint32_t o = at(i, 8 * w, c0, fold, p.ldc, 2);
          buf_store16(rg, o, gv[w]);
          buf_store16(ru, o, uv[w]);
          float gf[8], uf[8];
          unpack8(gv[w], gf);
          unpack8(uv[w], uf);
#pragma unroll
          for (int e = 0; e < 8; ++e) gf[e] = silu_f32(gf[e]) * uf[e];
          buf_store16(ra, at(i, 8 * w, c0, fold, p.ldc2, 2), pack8(gf));
        }
      }
      return;
    }
  }
  const int c0 = n0 + wn * 128;
  if constexpr (SWB) {
    const rsrc_t rg = tile_rsrc(p.R, p.ldr, 2, p.N), ru = tile_rsrc(static_cast<const bf16*>(p.R) + p.N, p.ldr, 2, p.N),
                 sg = tile_rsrc(p.C, p.ldc, 2, p.N), su = tile_rsrc(static_cast<const bf16*>(p.C) + p.N, p.ldc, 2, p.N);
    constexpr int RT = 1, NS = 16 / RT;      // step n: 64 columns (n / (NS / 2)), RT row tiles
    uint4 gv[2][2 * RT], uv[2][2 * RT];
    auto load_gu = [&](int n) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2 * RT; ++u) {
        const uint32_t o = at(RT * (n % (NS / 2)) + (u >> 1), 8 * (u & 1), c0 + 64 * (n / (NS / 2)), p.N, p.ldr, 2);
        gv[n & 1][u] = buf_load16(rg, o, 0);
        uv[n & 1][u] = buf_load16(ru, o, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    load_gu(0);
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      if (n + 1 < NS) load_gu(n + 1);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int i = RT * (n % (NS / 2)) + t, q = n / (NS / 2);
        uint4 d[2];
        to_lines(hi, pair(i, 4 * q), pair(i, 4 * q + 2), d[0], d[1]);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          uint4 dg, du;
          swiglu_bwd8(d[w], gv[n & 1][2 * t + w], uv[n & 1][2 * t + w], dg, du);
          const uint32_t o = at(i, 8 * w, c0 + 64 * q, p.N, p.ldc, 2);
          buf_store16(sg, o, dg);
          buf_store16(su, o, du);
        }
      }
    }
    return;
  }
  if (p.epi == EPI_BF16) {
    const rsrc_t rc = tile_rsrc(p.C, p.ldc, 2, p.N);
    if (!p.R) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          uint4 v[2];
          to_lines(hi, pair(i, 4 * q), pair(i, 4 * q + 2), v[0], v[1]);
#pragma unroll
          for (int w = 0; w < 2; ++w) buf_store16(rc, at(i, 8 * w, c0 + 64 * q, p.N, p.ldc, 2), v[w]);
        }
      return;
    }
    const rsrc_t rr = tile_rsrc(p.R, p.ldr, 2, p.N);
    constexpr int RT = 2, NS = 16 / RT;      // step n: 64 columns (n / (NS / 2)), RT row tiles
    uint4 rv[2][2 * RT];
    auto load_r = [&](int n) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2 * RT; ++u) rv[n & 1][u] = buf_load16(rr, at(RT * (n % (NS / 2)) + (u >> 1), 8 * (u & 1), c0 + 64 * (n / (NS / 2)), p.N, p.ldr, 2), 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    load_r(0);
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      if (n + 1 < NS) load_r(n + 1);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int i = RT * (n % (NS / 2)) + t, q = n / (NS / 2);
        uint4 x[2][2];      // [left, right chunk][columns 0 .. 3, 4 .. 7] in fp32
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          uint32_t f[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc_read(acc[i][4 * q + 2 * c], e)), __float_as_uint(acc_read(acc[i][4 * q + 2 * c + 1], e)), false, false);
            f[e] = y[0];
            f[4 + e] = y[1];
          }
          x[c][0] = make_uint4(f[0], f[1], f[2], f[3]);
          x[c][1] = make_uint4(f[4], f[5], f[6], f[7]);
        }
        uint4 v[2][2];      // [upper, lower rows][columns]
#pragma unroll
        for (int e = 0; e < 2; ++e) to_lines(hi, x[0][e], x[1][e], v[0][e], v[1][e]);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          float r[8];
          unpack8(rv[n & 1][2 * t + w], r);
          const uint32_t f[8] = {v[w][0].x, v[w][0].y, v[w][0].z, v[w][0].w, v[w][1].x, v[w][1].y, v[w][1].z, v[w][1].w};
#pragma unroll
          for (int e = 0; e < 8; ++e) r[e] += __uint_as_float(f[e]);
          buf_store16(rc, at(i, 8 * w, c0 + 64 * q, p.N, p.ldc, 2), pack8(r));
        }
      }
    }
    return;
  }
  // fp32, plus the old output where it accumulates; blockIdx.y: slice of a reduction split
  const rsrc_t rc = tile_rsrc(reinterpret_cast<float*>(p.C) + (long)blockIdx.y * p.c_slice_stride, p.ldc, 4, p.N);
  auto raw = [&](int i, int j) __attribute__((always_inline)) {
    return make_uint4(__float_as_uint(acc_read(acc[i][j], 0)), __float_as_uint(acc_read(acc[i][j], 1)), __float_as_uint(acc_read(acc[i][j], 2)), __float_as_uint(acc_read(acc[i][j], 3)));
  };
  if (!p.beta) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint4 v[2];
        to_lines(hi, raw(i, 2 * q), raw(i, 2 * q + 1), v[0], v[1]);
#pragma unroll
        for (int w = 0; w < 2; ++w) buf_store16(rc, at(i, 8 * w, c0 + 32 * q, p.N, p.ldc, 4), v[w]);
      }
    return;
  }
  constexpr int RT = 4, NS = 32 / RT;      // step n: 32 columns (n / (NS / 4)), RT row tiles
  uint4 ov[2][2 * RT];
  auto load_o = [&](int n) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2 * RT; ++u) ov[n & 1][u] = buf_load16(rc, at(RT * (n % (NS / 4)) + (u >> 1), 8 * (u & 1), c0 + 32 * (n / (NS / 4)), p.N, p.ldc, 4), 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  load_o(0);
#pragma unroll
  for (int n = 0; n < NS; ++n) {
    if (n + 1 < NS) load_o(n + 1);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int i = RT * (n % (NS / 4)) + t, q = n / (NS / 4);
      uint4 v[2];
      to_lines(hi, raw(i, 2 * q), raw(i, 2 * q + 1), v[0], v[1]);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const uint4 o = ov[n & 1][2 * t + w];
        buf_store16(rc, at(i, 8 * w, c0 + 32 * q, p.N, p.ldc, 4),
                    make_uint4(__float_as_uint(__uint_as_float(v[w].x) + __uint_as_float(o.x)), __float_as_uint(__uint_as_float(v[w].y) + __uint_as_float(o.y)),
                               __float_as_uint(__uint_as_float(v[w].z) + __uint_as_float(o.z)), __float_as_uint(__uint_as_float(v[w].w) + __uint_as_float(o.w))));
      }
    }
  }
}

// 16 numbers a lane, one per column, reduced over the sixteen lanes r of its row: the lane ends with the result of column r.  Each step halves the
// columns a lane keeps (by bits 3, 2, 1, 0 of r) in an exchange with the lane that differs in that bit (and, in the second step, the lower ones).
template <class Op>
RP_DEV float reduce_columns(float (&v)[16], int r, Op op) {
  auto step = [&](auto ntag, auto dtag, bool up) __attribute__((always_inline)) {
    constexpr int n = decltype(ntag)::value, dpp = decltype(dtag)::value;
#pragma unroll
    for (int k = 0; k < n; ++k) {
      const float give = up ? v[k] : v[k + n];
      v[k] = op(up ? v[k + n] : v[k], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), dpp, 0xf, 0xf, false)));
    }
  };
  step(IC<8>{}, IC<0x128>{}, r & 8);      // row_ror:8
  step(IC<4>{}, IC<0x141>{}, r & 4);      // row_half_mirror
  step(IC<2>{}, IC<0x4e>{}, r & 2);       // quad_perm [2, 3, 0, 1]
  step(IC<1>{}, IC<0xb1>{}, r & 1);       // quad_perm [1, 0, 3, 2]
  return v[0];
}

// EPI_CE_P of the wave's 128x128 block (rows are vocabulary entries, columns tokens) from transposed accumulators: a lane holds four consecutive
// tokens of a row per tile.  The probabilities go out as in store_rows; the columns' maxima and sums are formed over the lane's eight rows
// and then over the sixteen lanes that share its columns, 64 columns at a time, one per lane.  Frozen head of 151936 x 5120, 2040 tokens,
// staged through LDS 4964 us, from the registers 4867; the trainable one of 2048, 4096 tokens 6434 and 6200.  A number takes two conversions, a
// maximum, a sum and an exponential; besides, the four copies of `columns` with 48 numbers a lane each need more than the 512 registers:
// 99 are spilled (184 bytes a lane; 203 instructions, all behind the K loop), and a chunk of 32768 x 4096 writes 310 MB for 256 MB of probabilities.
RP_DEV void store_ce_p(const GemmArgs& p, f32x4 (&acc)[8][8], int m0, int n0, int wm, int wn, int lane, int part_row) {
  constexpr float LOG2E = 1.4426950408889634f, CAP = RP_CE_P_CLAMP * LOG2E;
  const int r16 = lane & 15, g = lane >> 4;
  const bool hi = r16 & 8;
  const int rows = p.M - m0 < 256 ? p.M - m0 : 256, w0 = wm * 128;
  const uint32_t ldc2 = (uint32_t)p.ldc * 2u;
  const rsrc_t rc = make_rsrc(static_cast<const char*>(p.C) + (long)m0 * p.ldc * 2, (uint32_t)(((long)(rows - 1) * p.ldc + p.N) * 2));
  const rsrc_t rl = make_rsrc(p.lse, (uint32_t)p.N * 4u), rt = make_rsrc(p.labels, (uint32_t)p.N * 4u);
  auto columns = [&](auto qtag, auto fulltag) __attribute__((always_inline)) {
    constexpr int q = decltype(qtag)::value;
    constexpr bool FULL = decltype(fulltag)::value;
    const int c0 = n0 + wn * 128 + 64 * q;
    const int line = c0 + (hi ? 32 : 0) + pair_column(g);
    const uint32_t at = (line < p.N ? (uint32_t)line * 2u : OOB) + (uint32_t)(r16 & 7) * ldc2;      // (past the end stays past the end)
    float nr[16], mx[16], sum[16];
    bool any = false;       // one of the lane's tokens has its label in the block
    auto label_row = [&](uint32_t t) { return (int)t - p.row_offset - m0 - w0; };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + 16 * j + 4 * g;
      const uint4 l = buf_load16(rl, (uint32_t)c * 4u, 0), t = buf_load16(rt, (uint32_t)c * 4u, 0);      // past the end: zeros
      const uint32_t lw[4] = {l.x, l.y, l.z, l.w}, tw[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        nr[4 * j + e] = -LOG2E * __uint_as_float(lw[e]);
        any |= c < p.N && (uint32_t)label_row(tw[e]) < 128u;
        mx[4 * j + e] = -INFINITY;
        sum[4 * j + e] = 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool in = FULL || w0 + 16 * i + r16 < rows;
      uint2 pk[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float z = acc_read(acc[i][4 * q + j], e);
          if constexpr (!FULL) z = in ? z : -INFINITY;       // (no probability, no maximum)
          mx[4 * j + e] = fmaxf(mx[4 * j + e], z);
          x[e] = __builtin_amdgcn_exp2f(fminf(fmaf(z, LOG2E, nr[4 * j + e]), CAP));
          sum[4 * j + e] += x[e];
        }
        pk[j] = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      }
      uint4 v[2];
      to_lines(hi, join_pair(pk[0], pk[1]), join_pair(pk[2], pk[3]), v[0], v[1]);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        buf_store16(rc, at + (uint32_t)(w0 + i * 16 + 8 * w) * ldc2, v[w]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_amdgcn_ballot_w64(any)) {      // rare
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = c0 + 16 * j + 4 * g;
        const uint4 t = buf_load16(rt, (uint32_t)c * 4u, 0);
        const uint32_t tw[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int lab = label_row(tw[e]);
          float z = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float x = acc_read(acc[i][4 * q + j], e);
            z = lab >> 4 == i ? x : z;
          }
          if (c < p.N && (uint32_t)lab < 128u && (lab & 15) == r16) p.zlab[c + e] = z;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    const float m = reduce_columns(mx, r16, [](float a, float b) { return fmaxf(a, b); }), s = reduce_columns(sum, r16, [](float a, float b) { return a + b; });
    const int col = c0 + 16 * (r16 >> 2) + 4 * g + (r16 & 3);
    if (col < p.N) p.part[(long)part_row * p.part_ld + col] = make_float2(m, s);
  };
  if (rows == 256) {
    columns(IC<0>{}, std::true_type{});
    columns(IC<1>{}, std::true_type{});
  } else {
    columns(IC<0>{}, std::false_type{});
    columns(IC<1>{}, std::false_type{});
  }
}

// TB: the B operand is [K, N] (reduction index strided, the NN product); its units keep that layout and its fragments
// are read with the transposing LDS load.  TA (with TB: the TN product): the same for A, which is [K, M].
// GRP: grouped mode.  A group's last tile of 256 rows is rarely full (2048 tokens on 8 of 128 experts: 128 rows per expert on
// average), and what its empty rows cost is the matrix pipe's time and power.  The two wave rows take alternate blocks of 32 rows,
// and the K loop exists for one to four blocks per wave (NI): a tile of `rows` rows runs ceil(rows / 64) / 4 of the MFMAs.  Measured
// with that and the tile order of the plain products, us: h = 4096, 128 experts of 1536, backward stage of 256 | 2048 | 8192 tokens
// 2326 -> 2250 | 3664 -> 3510 | 13270 -> 12950;  h = 2880, 32 experts of 2880, forward of 1000 | 8192 tokens 659 -> 636 |
// 2995 -> 2876.  What bounds the 128-row tiles then is the experts' weights (gate/up 3.5 GB in 706 us, matrix pipe 31 % busy).
// blk: the output tile of the product (-1: the workgroup's number); grouped: the entry gm of the table and the tile column gn.
// ONCE: B is loaded non-temporally (see gemm_once_kernel).
template <bool TA, bool TB, bool GRP, bool ONCE = false, int OUT = OUT_ROWS>
RP_DEV void dtl_block(const GemmArgs& p, int blk, int gm = 0, int gn = 0) {
  static_assert((!TA || TB) && !(GRP && TA), "not a layout of this library");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  int tile_m, tile_n, m0, Mlim = p.M;
  const bf16* Bbase = static_cast<const bf16*>(p.B);
  int NI = 4;                                  // 32-row blocks of a wave that hold rows
  if constexpr (GRP) {
    tile_m = gm;
    tile_n = gn;
    const int4 g = p.grp_tab[tile_m];
    m0 = g.y;
    Mlim = g.y + g.z;
    NI = __builtin_amdgcn_readfirstlane((g.z + 63) >> 6);
    Bbase += (long)g.x * p.grp_strideB;
  } else {
    // narrow outputs (up to 24 tile columns) sweep their columns in groups of 4 tile rows, wide ones of 8: measured
    // +2-3 % at N = 5120, -1.5-2 % at N >= 10240 for groups of 4
    tile_of_block(p.M, p.N, 256, 256, tile_m, tile_n, (p.N + 255) / 256 <= 24 ? 4 : 8, blk);
    m0 = tile_m * 256;
  }
  const int n0 = tile_n * 256;
  const int nk1 = (p.K + BK - 1) / BK;
  const int nk_all = nk1 + (p.K2 + BK - 1) / BK;
  const int per_split = (nk_all + (int)gridDim.y - 1) / (int)gridDim.y;
  const int kt0 = (int)blockIdx.y * per_split;
  const int nk = (nk_all - kt0) < per_split ? (nk_all - kt0 > 0 ? nk_all - kt0 : 0) : per_split;

  // a folded tile (SwiGLU forward): every wave's block is 64 gate columns and the 64 up columns that go with them
  const int fold = (!TB && p.epi == EPI_SWIGLU_FWD) ? p.N >> 1 : 0;   // uniform

  // Load instruction i (0..7 per operand) of this wave fills the 1 KB block 8*wave + i of a unit.
  //   reduction-contiguous operand: operand rows 8*(8*wave + i) .. + 7, lane l -> row + (l >> 3), chunk position l & 7,
  //     i.e. data chunk (l & 7) ^ ((row >> 1) & 7);
  //   TB: the unit is [64 reduction rows][256 columns] (512-byte rows of sixteen 32-byte segments, the columns of one 16x16 tile each);
  //     reduction rows 2*(8*wave + i), + 1, lane l -> row + (l >> 5), chunk position l & 31, whose segment (l & 31) >> 1
  //     holds data segment ((l & 31) >> 1) ^ seg_swizzle(row).
  uint32_t voA[8], voB[8];
  int lch[2];     // the lane's data chunk in even / odd instructions (rows 8 apart flip bit 2 of the swizzle)
  auto b_offset = [&](int i, long ldb) -> uint32_t {   // byte offset of the lane's chunk of load i of a B unit at reduction offset 0
    if constexpr (!TB) {
      const int r = 8 * (8 * wave + i) + (lane >> 3);
      const int ch = (lane & 7) ^ ((r >> 1) & 7);
      const int gl = fold ? (n0 >> 1) + (r >> 7) * 64 + (r & 63) : n0 + r;    // gate column, or output column
      const int gn = fold ? gl + ((r >> 6) & 1) * fold : gl;
      return gl < (fold ? fold : p.N) ? (uint32_t)((long)gn * ldb + ch * 8) * 2u : OOB;
    } else {
      const int kr = 2 * (8 * wave + i) + (lane >> 5);
      const int pos = lane & 31;
      const int gn = n0 + ((pos >> 1) ^ seg_swizzle(kr)) * 16 + (pos & 1) * 8;
      return gn < p.N ? (uint32_t)((long)kr * ldb + gn) * 2u : OOB;
    }
  };
  auto a_offset = [&](int i, long lda, bool first) -> uint32_t {   // the same for A (rows of a transposed A are not mapped)
    if constexpr (!TA) {
      const int r = 8 * (8 * wave + i) + (lane >> 3);
      const int ch = (lane & 7) ^ ((r >> 1) & 7);
      const int gm = m0 + r;
      if (!first) return gm < p.M ? (uint32_t)((long)gm * lda + ch * 8) * 2u : OOB;
      const long srcm = (p.row_map && gm < Mlim) ? p.row_map[gm] : gm;
      return gm < Mlim ? (uint32_t)(srcm * lda + ch * 8) * 2u : OOB;
    } else {
      const int kr = 2 * (8 * wave + i) + (lane >> 5);
      const int pos = lane & 31;
      const int gm = m0 + ((pos >> 1) ^ seg_swizzle(kr)) * 16 + (pos & 1) * 8;
      return gm < (first ? Mlim : p.M) ? (uint32_t)((long)kr * lda + gm) * 2u : OOB;
    }
  };
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 8 * (8 * wave + i) + (lane >> 3);
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    lch[i & 1] = ch;
    voA[i] = a_offset(i, p.lda, true);
    voB[i] = b_offset(i, p.ldb);
  }
  const i32x4 rsA = raw_rsrc(p.A, p.bytesA), rsB = raw_rsrc(Bbase, p.bytesB);
  i32x4 rsA2 = rsA, rsB2 = rsB;
  if (p.K2 > 0) {
    rsA2 = raw_rsrc(p.A2, p.bytesA2);
    rsB2 = raw_rsrc(p.B2, p.bytesB2);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t lds_wave = lds0 + (uint32_t)wave * 8192u;

  // Loads are issued tile by tile in order (B of a tile, then A); the state of the tile being loaded: its offsets and
  // descriptors (first or second operand pair), its reduction offset, the masks that send the chunks past the end of the
  // reduction outside the descriptor (all zero except in the last tile of an operand pair), and its two ring slots.
  uint32_t vcA[8], vcB[8];
  i32x4 rcA = rsA, rcB = rsB;
#pragma unroll
  for (int i = 0; i < 8; ++i) { vcA[i] = voA[i]; vcB[i] = voB[i]; }
  int ld_kt = kt0, ld_k0 = kt0 * BK, ld_Klim = p.K;
  bool ld_second = false, ld_live = true;
  uint32_t ld_soff = 0, ld_soffB = 0;
  uint32_t ld_kstepA = TA ? (uint32_t)p.lda * 2u : 2u;
  uint32_t ld_kstepB = TB ? (uint32_t)p.ldb * 2u : 2u;   // bytes per reduction index in the B operand
  uint32_t ld_ring = 0;          // byte offset of the ring slot of the tile's B unit; its A unit is the next slot
  uint32_t ld_ldsB = 0, ld_ldsA = 0;
  // before the loads of local tile s = 0, 1, 2, ..., in three parts (for slots of their own in the K loop); tiles past
  // the end take neither of the two rare paths, which drain the loads in flight
  auto setup_pair = [&](int s) {
    ld_live = s < nk;
    if (ld_live && !ld_second && ld_kt >= nk1) {   // uniform, at most once per kernel: on to the second operand pair
      asm volatile("" ::: "memory");    // (keeps this a branch: as selects it would cost dozens of instructions per tile)
      ld_second = true;
      ld_k0 = (ld_kt - nk1) * BK;
      ld_Klim = p.K2;
      rcA = rsA2;
      rcB = rsB2;
      if (p.K2 > 0) {   // the offsets of the second pair are worked out here rather than kept in registers through the loop
        if constexpr (TB) ld_kstepB = (uint32_t)p.ldb2 * 2u;
        if constexpr (TA) ld_kstepA = (uint32_t)p.lda2 * 2u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          vcA[i] = a_offset(i, p.lda2, false);
          vcB[i] = b_offset(i, p.ldb2);
        }
      }
      // Whatever the compiler reloads from scratch memory on this path counts in vmcnt like the loads above; left
      // pending, its own s_waitcnt before the first use of such a register would sit in the K loop and drain the
      // pipeline every tile.
      __builtin_amdgcn_s_waitcnt(0x0070);
    }
    ld_soff = s < nk ? (uint32_t)ld_k0 * ld_kstepA : OOB;   // (from s, not from the flag: the scalar offset has to stay provably wave-uniform)
    ld_soffB = s < nk ? (uint32_t)ld_k0 * ld_kstepB : OOB;
    ++ld_kt;
  };
  auto setup_mask = [&]() {
    if (ld_live && ld_k0 + BK > ld_Klim) {   // uniform: the last tile of an operand pair that is not a multiple of 64 deep
      asm volatile("" ::: "memory");
      // chunks past the end of the reduction move outside the descriptor; the offsets are not needed unmasked again
      // (the next tile belongs to the other pair, whose offsets are worked out afresh, or lies past the end)
      const uint32_t mk0 = (ld_k0 + lch[0] * 8 < ld_Klim) ? 0u : OOB, mk1 = (ld_k0 + lch[1] * 8 < ld_Klim) ? 0u : OOB;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t mkr = (ld_k0 + 2 * (8 * wave + i) + (lane >> 5) < ld_Klim) ? 0u : OOB;   // row-wise, for [K, X] units
        vcA[i] |= TA ? mkr : ((i & 1) ? mk1 : mk0);
        vcB[i] |= TB ? mkr : ((i & 1) ? mk1 : mk0);
      }
      __builtin_amdgcn_s_waitcnt(0x0070);   // as at the end of the pair switch
    }
    ld_k0 += BK;
  };
  auto setup_lds = [&]() {
    ld_ldsB = lds_wave + ld_ring;
    ld_ring = ld_ring + UNIT_BYTES == (uint32_t)DTL_SMEM ? 0u : ld_ring + UNIT_BYTES;
    ld_ldsA = lds_wave + ld_ring;
    ld_ring = ld_ring + UNIT_BYTES == (uint32_t)DTL_SMEM ? 0u : ld_ring + UNIT_BYTES;
  };
  auto tile_setup = [&](int s) { setup_pair(s); setup_mask(); setup_lds(); };
  auto issue_b = [&](auto itag) __attribute__((always_inline)) {
    constexpr int i = decltype(itag)::value;
    load_to_lds<i * 1024, ONCE>(ld_ldsB, vcB[i], rcB, ld_soffB);
  };
  auto issue_a = [&](auto itag) __attribute__((always_inline)) {
    constexpr int i = decltype(itag)::value;
    load_to_lds<i * 1024>(ld_ldsA, vcA[i], rcA, ld_soff);
  };

  // acc[i][j]: 16x16 tile (i, j) of the wave's 8 x 8
  f32x4 acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fragments: lane -> row lane % 16 of a tile, eight reduction indices from 8 (lane / 16) on of a 32-deep step, i.e. the 16-byte chunk
  // 4 ks + lane / 16 at chunk position chunk ^ ((row >> 1) & 7).  fkA[ks] / fkB[ks]: byte offset of the lane's chunk of step ks in the
  // wave's first tile of a unit; tile i (j) lies another 2 KB further each.  Grouped: blocks of 32 rows alternate between the wave rows.
  // B's fragments have a set of registers per step; those of A are read again as soon as their eight MFMAs are through, but for the last
  // two, which alternate.
  const int r16 = lane & 15, g16 = lane >> 4;
  uint32_t fkA[2], fkB[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint32_t ch = (uint32_t)((4 * ks + g16) ^ ((r16 >> 1) & 7)) * 16u;
    fkA[ks] = (uint32_t)((wm * (GRP ? 32 : 128) + r16) * 128) + ch;
    fkB[ks] = (uint32_t)((wn * 128 + r16) * 128) + ch;
  }
  uint4 af[10], bfr[2][8];
  // register of A's tile i in the steps of parity s
  auto areg = [](int s, int i) constexpr { return i < 6 ? i : i + 2 * s; };
  // A transposed operand's fragment is two transposing reads (reduction rows +0..3 and +4..7 of the lane's eight): byte offset of the
  // lane's first read of step 0 for tile x of the operand -- reduction row 8 g16 + r16 / 4, the tile's segment moved by the row's
  // swizzle (the same for both reads and both steps), columns 4 (r16 % 4) of the segment.
  [[maybe_unused]] uint32_t fkBt[8], fkAt[8];
  {
    const int kr = 8 * g16 + (r16 >> 2);
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      fkBt[x] = (uint32_t)(kr * 512 + ((wn * 8 + x) ^ seg_swizzle(kr)) * 32 + (r16 & 3) * 8);
      fkAt[x] = (uint32_t)(kr * 512 + ((wm * 8 + x) ^ seg_swizzle(kr)) * 32 + (r16 & 3) * 8);
    }
  }
  auto read_tr = [&](uint4& f, uint32_t off, int half) __attribute__((always_inline)) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(smem + off + half * 2048));
    const uint2 u = __builtin_bit_cast(uint2, v);
    if (half == 0) { f.x = u.x; f.y = u.y; }
    else { f.z = u.x; f.w = u.y; }
  };
  // read number n (0 .. RB - 1) of B's fragments of a step into register set s, read number n of A's; ringA, ringB: the units' offsets
  constexpr int RB = TB ? 16 : 8, RA = TA ? 16 : 8;
  auto read_b = [&](auto stag, auto ntag, uint32_t ringB) __attribute__((always_inline)) {
    constexpr int st = decltype(stag)::value, n = decltype(ntag)::value;
    if constexpr (TB) read_tr(bfr[st][n >> 1], ringB + fkBt[n >> 1] + st * 16384, n & 1);
    else bfr[st][n] = *reinterpret_cast<const uint4*>(smem + (ringB + fkB[st]) + n * 2048);
  };
  auto read_a = [&](auto stag, auto ntag, uint32_t ringA) __attribute__((always_inline)) {
    constexpr int st = decltype(stag)::value, n = decltype(ntag)::value;
    if constexpr (TA) read_tr(af[areg(st, n >> 1)], ringA + fkAt[n >> 1] + st * 16384, n & 1);
    else af[areg(st, n)] = *reinterpret_cast<const uint4*>(smem + (ringA + fkA[st]) + (GRP ? (n >> 1) * 8192 + (n & 1) * 2048 : n * 2048));
  };

  // prologue: tiles 0 and 1 set out (in the order of the K loop: B, then A); tile 0 has landed everywhere after the barrier
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    tile_setup(s);
    issue_b(IC<0>{}); issue_b(IC<1>{}); issue_b(IC<2>{}); issue_b(IC<3>{}); issue_b(IC<4>{}); issue_b(IC<5>{}); issue_b(IC<6>{}); issue_b(IC<7>{});
    issue_a(IC<0>{}); issue_a(IC<1>{}); issue_a(IC<2>{}); issue_a(IC<3>{}); issue_a(IC<4>{}); issue_a(IC<5>{}); issue_a(IC<6>{}); issue_a(IC<7>{});
  }
  tile_setup(2);
  __builtin_amdgcn_s_waitcnt(0x0f70 | (16 & 15) | ((16 >> 4) << 14));   // vmcnt(16)
  __syncthreads();
  for_seq([&](auto n) __attribute__((always_inline)) { read_b(IC<0>{}, n, 0u); }, std::make_integer_sequence<int, RB>{});
  for_seq([&](auto n) __attribute__((always_inline)) { read_a(IC<0>{}, n, (uint32_t)UNIT_BYTES); }, std::make_integer_sequence<int, RA>{});

  // Slot plan of tile t: 128 slots of one MFMA, step s = slots 64 s .. 64 s + 63, the eight MFMAs of A's tile i in slots 8 i .. 8 i + 7 of a
  // step.  With one wave per SIMD whatever a slot issues beside its MFMA has to fit into the 16 cycles that runs; a slot holds at most
  // one memory instruction, and the reads and loads are spread evenly.
  //   step 0, slots 2 .. 57      the fragment reads of step 1: B's, then A's tiles 6, 7 (which alternate their registers), 0, 1, .. 5
  //   slots 4 .. 60              the loads of B of tile t+2; its ring slot (A of tile t-1) is free since the barrier of tile t-1
  //   slot  BAR = 74             every read of this tile has returned.  vmcnt(8): the wave's loads of tile t+1 have landed (those of B of tile
  //                              t+2 may be in flight); barrier: tile t+1 is complete in LDS, this tile's two ring slots are free
  //   slots 76 .. 127            the reads of step 0 of tile t+1
  //   slots 77 .. 112            the loads of A of tile t+2, into the slot of B of this tile
  //   slots 120, 123             the state of the loads of tile t+3
  auto main_loop = [&](auto nitag) __attribute__((always_inline)) {
    constexpr int NB = decltype(nitag)::value;   // blocks of 32 rows
    using P = SlotPlan<RB, RA>;
    uint32_t ringB = 0, ringA = UNIT_BYTES;      // units of the tile whose fragments are read
    for (int t = 0; t < nk; ++t) {
      auto slot = [&](auto sltag) __attribute__((always_inline)) {
        constexpr int sl = decltype(sltag)::value, st = sl >> 6, i = (sl & 63) >> 3, j = sl & 7;
        if constexpr (sl == P::BAR) {
          __builtin_amdgcn_s_waitcnt(0x0f70 | 8);
          __syncthreads();
        }
        if constexpr (i < 2 * NB) {
          if constexpr (OUT == OUT_COLS) mfma16_in_place(acc[i][j], af[areg(st, i)], bfr[st][j]);
          else mfma16_in_place(acc[i][j], bfr[st][j], af[areg(st, i)]);      // the transposed tile
        }
        constexpr int rd = P::read(sl);
        if constexpr (rd >= 0) {
          constexpr int rs = sl < 64 ? 1 : 0;    // the step whose fragments these are
          if constexpr (rd < RB) read_b(IC<rs>{}, IC<rd>{}, ringB);
          else {
            constexpr int n = P::a_read(rd - RB), tile = TA ? n >> 1 : n;
            if constexpr (tile < 2 * NB) read_a(IC<rs>{}, IC<n>{}, ringA);
          }
        }
        if constexpr (sl == 66) {
          ringB = ringB + 2 * UNIT_BYTES >= (uint32_t)DTL_SMEM ? ringB + 2 * UNIT_BYTES - DTL_SMEM : ringB + 2 * UNIT_BYTES;
        }
        if constexpr (sl == 68) {
          ringA = ringA + 2 * UNIT_BYTES >= (uint32_t)DTL_SMEM ? ringA + 2 * UNIT_BYTES - DTL_SMEM : ringA + 2 * UNIT_BYTES;
        }
        constexpr int ld = P::load(sl);
        if constexpr (ld >= 0 && ld < 8) issue_b(IC<ld>{});
        if constexpr (ld >= 8) issue_a(IC<ld - 8>{});
        if constexpr (sl == 120) setup_pair(t + 3);
        if constexpr (sl == 123) { setup_mask(); setup_lds(); }
        __builtin_amdgcn_sched_barrier(0);
      };
      for_seq(slot, std::make_integer_sequence<int, 128>{});
    }
  };
  if constexpr (GRP) {
    switch (NI) {
      case 1: main_loop(IC<1>{}); break;
      case 2: main_loop(IC<2>{}); break;
      case 3: main_loop(IC<3>{}); break;
      default: main_loop(IC<4>{});
    }
  } else {
    main_loop(IC<4>{});
  }
  asm volatile("s_nop 7\n\ts_nop 7");   // the last MFMA has retired; the copies out of the accumulators are invisible to the hazard checks
  if constexpr (OUT != OUT_COLS) {
    // (nothing here reads LDS; the empty loads past the end still write it, but it is the workgroup's to its end)
    if constexpr (OUT == OUT_CE_P) store_ce_p(p, acc, m0, n0, wm, wn, lane, p.part_row0 + tile_m * 2 + wm);
    else store_rows<GRP, OUT == OUT_SWIGLU_BWD>(p, acc, m0, Mlim, n0, wm, wn, lane, fold);
  } else {
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the empty loads past the end write LDS too
    __syncthreads();                      // every wave is done with the operand stages: the epilogue reuses the LDS
    // The accumulators live in the AGPR half of the register file, which only MFMAs and copies can address.  Left to the
    // compiler all 256 are copied out at once behind the loop and half of them spilled; here each 128x64 half is copied
    // out right before its epilogue.
    f32x16 half[TM][TN];
    auto write_half = [&](auto htag) __attribute__((always_inline)) {
      constexpr int h = decltype(htag)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) half[i][j][v] = acc_read(acc[2 * i + (v >> 3)][4 * h + 2 * j + ((v >> 2) & 1)], v & 3);
      epilogue<true>(p, Mlim, half, smem, wave, lane, m0 + wm * 128, n0 + wn * 128 + 64 * h, p.part_row0 + tile_m * 2 + wm);
    };
    write_half(IC<0>{});
    write_half(IC<1>{});
  }
}

// The entry of the table and the tile column of a workgroup of a grouped product (the table's length is known on the device only:
// surplus workgroups leave).
RP_DEV bool grouped_tile(const GemmArgs& p, int& tile_m, int& tile_n) {
  const int ntiles = *p.grp_ntiles;
  if ((int)blockIdx.x >= ntiles * ((p.N + 255) / 256)) return false;
  tile_of_block(ntiles * 256, p.N, 256, 256, tile_m, tile_n, 4);
  return true;
}

template <bool TA, bool TB, bool GRP, int OUT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_dtl_kernel(const GemmArgs p) {
  int tile_m = 0, tile_n = 0;
  if constexpr (GRP) {
    if (!grouped_tile(p, tile_m, tile_n)) return;
  }
  if constexpr (OUT == OUT_COLS && TB) {      // only the atomic output comes here with these layouts
    GemmArgs q = p;
    q.epi = EPI_F32_ATOMIC;
    dtl_block<TA, TB, GRP, false, OUT>(q, -1);
  } else {
    dtl_block<TA, TB, GRP, false, OUT>(p, -1, tile_m, tile_n);
  }
}

// Grouped products whose groups have one tile each: a group's weights are then read once in the launch (every 256 columns by one
// workgroup), and loads marked non-temporal spare them the way through the caches for reuse that does not come.  What bounds these
// products is that reading alone: without any of its MFMAs gate/up of 2048 tokens on 8 of 128 experts (h = 4096, width 1536: 3.2 GB)
// took 695 us of 713, as with another half tile in flight (723) or with reductions that start at different places (708); with this
// 633, and 690 -> 675 for the gradient of the layer's input.  Stages, us (h = 4096, 128 experts | h = 2880, 32 experts of 2880):
// forward of 512, 1024, 2048, 3072 | 512, 1000, 1504 tokens 1226 -> 1151, 1373 -> 1288, 1653 -> 1565, 1954 -> 1895 | 558 -> 515,
// 614 -> 563, 700 -> 658.  With two tiles per group the second reading, which the Infinity Cache serves otherwise, comes from HBM:
// 4096 | 2048 tokens (256 rows per group) 2585 -> 2620 | 908 -> 907, gemm_pair_kernel 620 -> 751.  The caller draws the line (grp_once).
template <bool TB>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_once_kernel(const GemmArgs p) {
  int tile_m = 0, tile_n = 0;
  if (!grouped_tile(p, tile_m, tile_n)) return;
  dtl_block<false, TB, true, true>(p, -1, tile_m, tile_n);
}

// Two grouped products that read the same weights, NT and NN, over the same table: the tiles of an entry follow each other, those of
// the first product and then those of the second, on one XCD.  The second reading of a group's weights then comes out of the Infinity
// Cache (the groups in flight have 150 MB) instead of HBM: h = 4096, 128 experts of 1536, 2048 tokens
// 413 + 333 -> 638 us; backward stage of 256 | 2048 tokens 2178 -> 2110 | 3510 -> 3369.
struct PairArgs { GemmArgs nt, nn; };
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_pair_kernel(const PairArgs a) {
  GemmArgs p = a.nt, q = a.nn;       // (the plain epilogue only, known here: it needs none of the others' code or scalars)
  p.epi = q.epi = EPI_BF16;
  p.R = q.R = nullptr;
  p.alpha = q.alpha = 1.f;
  p.K2 = q.K2 = 0;
  const int ntiles = *a.nt.grp_ntiles, c1 = (a.nt.N + 255) / 256, cols = c1 + (a.nn.N + 255) / 256;
  if ((int)blockIdx.x >= ntiles * cols) return;
  const int id = xcd_remap((int)blockIdx.x, ntiles * cols);
  const int tile_m = id / cols, c = id - tile_m * cols;
  if (c < c1) dtl_block<false, false, true>(p, -1, tile_m, c);
  else dtl_block<false, true, true>(q, -1, tile_m, c - c1);
}

// Weight gradients of a layer in one launch: C_i += A_i^T B_i (fp32), all with the same reduction.  Alone each ends in a round of
// workgroups that is partly empty (h = 2048, ffn 6144: 384, 192, 128 and 64 tiles on 256 CUs), or takes smaller tiles or a split to
// fill the chip; together they are 768 tiles, three full rounds.  Measured there, four launches -> one, us: 4096 tokens 470 -> 367,
// 2048 287 -> 224, 1024 185 -> 145 (with the eight-wave kernel 386, 221 and 137: it is behind where the launch is long).
struct WgradOne { const void *A, *B; void* C; long lda, ldb, ldc; unsigned bytesA, bytesB; int M, N, first; };
struct WgradArgs { int n, K; WgradOne g[GEMM_WGRAD_MAX]; };
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_wgrad_kernel(const WgradArgs a) {
  int i = 0;
  while (i + 1 < a.n && (int)blockIdx.x >= a.g[i + 1].first) ++i;
  const WgradOne& q = a.g[__builtin_amdgcn_readfirstlane(i)];
  GemmArgs g{};
  g.A = q.A; g.B = q.B; g.C = q.C; g.lda = q.lda; g.ldb = q.ldb; g.ldc = q.ldc; g.bytesA = q.bytesA; g.bytesB = q.bytesB;
  g.M = q.M; g.N = q.N; g.K = a.K; g.alpha = 1.f; g.beta = 1; g.epi = EPI_F32;
  dtl_block<true, true, false>(g, (int)blockIdx.x - q.first);
}

}  // namespace

template <bool TA, bool TB, bool GRP = false, int OUT = OUT_ROWS, bool ONCE = false>
static hipError_t dtl_launch_one(hipStream_t st, const GemmArgs& a) {
  static bool attr_done = false;
  auto kern = gemm_dtl_kernel<TA, TB, GRP, OUT>;
  if constexpr (ONCE) kern = gemm_once_kernel<TB>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, DTL_SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  int tiles = ((a.M + 255) / 256) * ((a.N + 255) / 256);
  if (GRP) tiles = a.grp_max_tiles * ((a.N + 255) / 256);
  RP_LAUNCH(kern, dim3(tiles, a.splits > 0 ? a.splits : 1), dim3(256), DTL_SMEM, st, a);
  return hipGetLastError();
}

hipError_t gemm_dtl_launch(hipStream_t st, const GemmArgs& a, int layout) {
  if (a.grp_tab) {
    const bool once = a.grp_once;
    if (layout == GEMM_NT) return once ? dtl_launch_one<false, false, true, OUT_ROWS, true>(st, a) : dtl_launch_one<false, false, true>(st, a);
    if (layout == GEMM_NN) return once ? dtl_launch_one<false, true, true, OUT_ROWS, true>(st, a) : dtl_launch_one<false, true, true>(st, a);
    return hipErrorInvalidValue;
  }
  const bool rows = a.epi == EPI_BF16 || a.epi == EPI_F32 || a.epi == EPI_SWIGLU_FWD;
  switch (layout) {
    case GEMM_NT:
      if (a.epi == EPI_CE_P) return dtl_launch_one<false, false, false, OUT_CE_P>(st, a);
      return rows ? dtl_launch_one<false, false>(st, a) : dtl_launch_one<false, false, false, OUT_COLS>(st, a);
    case GEMM_NN:
      if (a.epi == EPI_SWIGLU_BWD) return dtl_launch_one<false, true, false, OUT_SWIGLU_BWD>(st, a);
      if (!rows && a.epi != EPI_F32_ATOMIC) return hipErrorInvalidValue;
      return rows ? dtl_launch_one<false, true>(st, a) : dtl_launch_one<false, true, false, OUT_COLS>(st, a);
    default:
      if (!rows && a.epi != EPI_F32_ATOMIC) return hipErrorInvalidValue;
      return rows ? dtl_launch_one<true, true>(st, a) : dtl_launch_one<true, true, false, OUT_COLS>(st, a);
  }
}

hipError_t gemm_wgrad_run(hipStream_t st, int n, const GemmArgs* g) {
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_wgrad_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, DTL_SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if (n < 1 || n > GEMM_WGRAD_MAX) return hipErrorInvalidValue;
  WgradArgs a{};
  a.n = n;
  a.K = g[0].K;
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& p = g[i];
    if (p.K != a.K || p.K2 || p.epi != EPI_F32 || !p.beta || p.alpha != 1.f) return hipErrorInvalidValue;
    a.g[i] = {p.A, p.B, p.C, p.lda, p.ldb, p.ldc, p.bytesA, p.bytesB, p.M, p.N, blocks};
    blocks += ((p.M + 255) / 256) * ((p.N + 255) / 256);
  }
  RP_LAUNCH(gemm_wgrad_kernel, dim3(blocks), dim3(256), DTL_SMEM, st, a);
  return hipGetLastError();
}

hipError_t gemm_pair_run(hipStream_t st, const GemmArgs& nt, const GemmArgs& nn) {
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_pair_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, DTL_SMEM);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const PairArgs a{nt, nn};
  RP_LAUNCH(gemm_pair_kernel, dim3(nt.grp_max_tiles * ((nt.N + 255) / 256 + (nn.N + 255) / 256)), dim3(256), DTL_SMEM, st, a);
  return hipGetLastError();
}
