// Causal grouped-query attention on the gfx950 matrix cores, flash style: no s x s matrix leaves the CU, except
// that a backward with room for it keeps dS in bf16 (see attn_ds_block).
//
// All kernels compute the score tile TRANSPOSED relative to the row that is being normalised: an accumulator gives every lane one column, so
// with queries (forward, dQ) as columns the softmax reductions are in-lane plus an exchange between the lanes that share a column, and the
// probabilities already sit in the register layout the next MFMA wants as its B operand; the A operand of that MFMA is read from LDS in exactly
// that order of the reduction.  An operand whose reduction index is contiguous in memory (K for Q.K^T, V for dO.V^T, Q and dO in the score
// products of the dK/dV kernel) is read with plain 16-byte LDS loads; an operand whose reduction index is the row index of the tile (V for
// P.V, K for dS.K, Q and dO for dK/dV) is read with the transposing LDS load; nothing is transposed in registers.  Global loads are 16-byte
// buffer loads whose descriptor ends with the sequence, so rows past the end read as zero without a branch.
//
// The backward kernels use v_mfma_f32_16x16x32_bf16: a lane has four rows of a 16x16 tile, four lane groups (lane / 16) share a column, and two
// 16-row tiles make one 32-deep step, which for lane group g holds the reduction indices {4g..4g+3, 16+4g..16+4g+3}.  A wave owns 32 columns
// (two column tiles), so every fragment feeds two MFMAs.  All their tiles have the row stride D + 16, which serves both kinds of reads
// without bank conflicts.  The forward kernel uses v_mfma_f32_32x32x16_bf16 (16 rows a lane, two half-waves share a column) on a K tile of row
// stride D + 8 and a V tile of D + 32.
// What was measured, 32x32x16 | 16x16x32 everywhere, two runs each on one box, us.  Backward (strides D + 8 and D + 24 | D + 16), 4096 x 16 heads of
// 128 280 | 261, 8192 x 32 1811 | 1671, 16384 x 64 14760 | 13865, 1000 x 16 72.2 | 72.0, 2 x 508 x 32 53.5 | 51.9, 3 x 1500 x 64 heads of 64 261 | 234,
// 512 x 32 of 64 34.4 | 34.2; the strides are most of it (backward 8192 x 32 with D + 24 1802 -> 1735), and what starts the dK/dV products
// (stat_start) saves an MFMA in nine of their score phase.  Forward (D + 8 and D + 32 | D + 16), where the softmax takes as many issue slots as the
// products and the narrower tile doubles their number: 128 x 16 heads of 128 7.2 | 7.6, 1000 x 16 23.9 | 25.2, 2 x 508 x 32 15.3 | 16.0, 4096 x 32
// 141 | 146, 8192 x 16 267 | 277, 16384 x 64 3890 | 3930, 31744 x 64 14430 | 14770, 512 x 32 of 64 10.2 | 11.0, 1000 x 64 of 64 17.9 | 19.1; the
// narrower one is ahead by 1 to 3 % at 4096 x 16 and 8192 x 32 of 128 and from 3 x 1500 x 64 of 64 on (77 | 75).
//
//   forward : workgroup = NW waves x 32 queries of one head, loop over 64-key tiles up to the diagonal; NW = 8 (one
//             workgroup per CU, two sets of K/V tiles, one barrier per tile) when the grid is large enough, else 4
//   dQ      : same decomposition; recomputes S^T and dP^T, accumulates dQ^T, and works out delta = rowsum(dO * O) for itself and
//             for dK/dV, which runs behind it; with kept dS it is a product of gemm_mid.hip behind dK/dV instead
//   dK, dV  : workgroup = 128 keys against one query head, or two or four of a group one after the other
//             (heads_per_workgroup); loops over 64-query tiles from the diagonal on and accumulates dK^T, dV^T in
//             registers.  d = 128: eight waves, pairs of waves share 32 keys, split the accumulators over the head
//             dimension and the score recomputation over the queries (attn_bwd_dkv_pair_kernel); d = 64: four waves x 32
//             keys (attn_bwd_dkv_fused_kernel).  A workgroup that has a whole group stores its result; else each writes an
//             fp32 partial and a small kernel adds the group's partials in head order (no atomics, fixed order).  Several
//             workgroups per kv head is what lets the triangular work balance over the CUs.
// Launch orders keep an XCD (eight of them, each with its own L2) on few heads: see xcd_head() and the dK/dV kernels.
#include "common.hpp"
#include "kernels.hpp"
#include "gemm.hpp"
#include <stdlib.h>

namespace {

typedef __amdgpu_buffer_rsrc_t rsrc_t;

struct AttnArgs {
  const bf16 *q, *k, *v, *dout;
  bf16 *o, *dq, *dk, *dv;
  float* lse;
  const float* lse_in;
  float* delta;               // read, or (dQ kernel with o_in) worked out and written first
  const bf16* o_in;           // dQ kernel: the forward's output, delta = rowsum(dO * O) comes from it; or NULL
  float *dk_part, *dv_part;   // fp32 [T, a / hpw * d] partials of the dK/dV kernel unless a workgroup takes a whole group
  long ldq, ldk, ldv, ldo, lddo, lddq, lddk, lddv;
  int batch, seq, a, kh;
  float scale_log2e, scale;
  int fold;   // see heavy_rank()
  int hpw;    // dK/dV kernel: query heads of one group that a workgroup takes one after the other (a divisor of a / kh)
  int kblock; // dK/dV kernel: key tiles per run of one head in an XCD's launch order (0: key-tile-major order over all heads)
  bf16* ds;   // dK/dV kernel with kept dS: [batch * a] heads of k_attn_ds_bytes each (see attn_ds_block)
};

// The dK/dV kernel can leave dS (bf16, as its products take it) in memory, from which dQ = dS K is one product instead of the three
// of the dQ kernel.  A head's dS is a triangle of 64-key x 128-query blocks of 16 KB: a 128-query tile t sees the keys of blocks
// 0 .. 2t + 1, which lie one after the other.  Inside a block the sixteen 1 KB pieces are what a wave stores at once (32 keys x 16
// queries: lane l holds eight queries from 8 (l / 32) on of key l % 32), piece (key / 32) * 8 + query / 16.  Block of 64-key tile kt
// and query tile t:
RP_DEV int attn_ds_block(int t, int kt) { return t * (t + 1) + kt; }

// Launch position -> rank in the order "heaviest workgroup first".  A kernel that keeps two workgroups per CU and whose
// grid fits on the chip at once (at most 2 x 256 workgroups) has all of them resident from the start, CU c holding
// positions c and 256 + c; nothing is rescheduled later, so what counts is that every CU's pair sums to the same
// work: the second half of the grid is handed out lightest first (fold; measured 5 % on the forward kernel at 4096
// tokens, while pairing neighbouring positions instead made it 20 % slower).  Larger grids are handed out as
// workgroups finish, where heaviest-first is the right order.
RP_DEV int heavy_rank(int pos, int n, int fold) { return (fold && pos >= 256) ? n - 1 - (pos - 256) : pos; }

// Consecutive workgroups go to consecutive XCDs (eight, each with an L2 of its own).  The i-th of the nhb workgroups of a
// query tile therefore takes head (i mod 8) * nhb/8 + i/8 instead of head i: an XCD then works on nhb/8 neighbouring query
// heads, i.e. on one or two K/V heads with grouped queries, and its L2 fetches their K/V tiles once for all the workgroups
// that stream them side by side -- instead of every XCD fetching every K/V head.
RP_DEV int xcd_head(int i, int nhb) { return (nhb & 7) ? i : (i & 7) * (nhb >> 3) + (i >> 3); }

RP_DEV rsrc_t seq_rsrc(const bf16* base, long ld, int seq, int D) {
  // covers rows 0..seq-1 of one head: later rows are out of range and read as zero
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(base), 0, (int)(((long)(seq - 1) * ld + D) * 2), 0x00020000);
}
RP_DEV uint4 buf_load16(rsrc_t r, uint32_t voff) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Softmax statistics of a 64-query tile for the dK/dV kernels, one per lane: wave 0 fetches lse, wave 1 delta.  The load is only
// issued here; what the score products take is worked out when the tile is stored to LDS (stat_start), a tile later.  (Worked out
// where it is loaded, it makes the two waves wait for memory in every tile and the others for them: dK/dV of 8192 tokens, 32 heads
// of 128: 1252 -> 1109 us; 4096 x 16 heads 172 -> 162; 2048 x 64 188 -> 169.)
RP_DEV rsrc_t stat_rsrc(const float* lse, const float* delta, int wave, long head, int seq) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wave == 0 ? lse : delta) + head * seq, 0, seq * 4, 0x00020000);
}
RP_DEV float stat_load(rsrc_t r, int q) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, q * 4, 0, 0)); }

// Row stride of a tile in LDS (elements): 8 banks past a multiple of 64, so that neither the 16-byte reads of 16 rows by four lane groups nor
// the transposing ones (32 lanes a phase: eight rows of 32 bytes) meet on a bank.
constexpr int tile_ld(int d) { return d + 16; }

// ---- 64 x D tile: global -> registers -> LDS -----------------------------------------------------------------
template <int D, int NT>
struct Tile64 {
  static constexpr int CH = D / 8, NREG = 64 * CH / NT;
  static_assert((64 * CH) % NT == 0, "tile does not divide over the threads");
  // rows row0..row0+63 of a [seq, D] view with row stride ld (elements)
  static RP_DEV void load(uint4 (&r)[NREG], rsrc_t rs, long ld, int row0, int tid) {
#pragma unroll
    for (int it = 0; it < NREG; ++it) {
      const int c = it * NT + tid;
      r[it] = buf_load16(rs, (uint32_t)(((long)(row0 + c / CH) * ld + (c % CH) * 8) * 2));
    }
  }
  template <int LDS_LD>
  static RP_DEV void store(const uint4 (&r)[NREG], bf16* S, int tid) {
#pragma unroll
    for (int it = 0; it < NREG; ++it) {
      const int c = it * NT + tid;
      *reinterpret_cast<uint4*>(S + (c / CH) * LDS_LD + (c % CH) * 8) = r[it];
    }
  }
};

// A-operand fragment from a [64][LD] tile whose rows are the reduction index (keys or queries) and whose columns are
// the MFMA rows: the 8 values of lane group g = lane / 16 are tile rows {4g + e, 16 + 4g + e}, e = 0..3, at column lane % 16 -- the
// order in which two 16-row tiles of scores hold them.  base = S + tr_base(lane) + first row * LD + first column.
template <int LD>
RP_DEV uint4 read_frag_tr(const bf16* base) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(base));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(base + 16 * LD));
  const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
  return make_uint4(l2.x, l2.y, h2.x, h2.y);
}
template <int LD>
RP_DEV int tr_base(int lane) {
  return (4 * (lane >> 4) + ((lane & 15) >> 2)) * LD + 4 * (lane & 3);
}

// Two 16-row score tiles, one above the other, as the B operand of the next product: 32 reduction indices in the order of read_frag_tr.
RP_DEV uint4 pack_frag(const f32x4& a, const f32x4& b) {
  return make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3]));
}

// Sum over the four lanes that hold a column.
RP_DEV float column_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
RP_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Two waves share a SIMD in the forward kernel.  Left alone they fall into step: both issue their matrix products at
// the same time (each at half rate) and then both do their exponentials, so the matrix pipeline idles while the vector
// pipeline works and the other way round.  A wave raises its issue priority for its runs of MFMAs: whichever wave gets
// there first keeps the matrix pipeline to itself, the other one falls behind by a phase, and from then on one wave's
// exponentials run under the other wave's products (forward kernel +6 % at 8192 to 31744 tokens; the dQ kernel, whose
// vector phase is short against its three products, does not change).
#define MFMA_PHASE_BEGIN() __builtin_amdgcn_s_setprio(1)
#define MFMA_PHASE_END() __builtin_amdgcn_s_setprio(0)

// What the products of the dK/dV kernels start from for a query (wave 0: -lse / scale, wave 1: -delta; rows of the score tiles are
// queries, so a lane's four rows of a tile are four consecutive numbers: one 16-byte LDS read is the accumulators' first value, and the
// tiles come out as q.k - lse/scale and dO.v - delta); padded query rows get P = exp(-3e4 scale) = 0.
RP_DEV float stat_start(float raw, int wave, bool in, float scale) {
  return wave == 0 ? (in ? -raw / scale : -3.0e4f) : (in ? -raw : 0.f);
}

// A wave's staged 32 x D block to global.
template <int D>
RP_DEV void store_staged(const bf16* stage, bf16* __restrict__ out, long ld, int row0, int nrows, int lane) {
  __syncthreads();
#pragma unroll
  for (int it = 0; it < (32 * (D / 8)) / 64; ++it) {
    const int idx = it * 64 + lane;
    const int row = idx / (D / 8), ch = idx % (D / 8);
    if (row0 + row < nrows)
      *reinterpret_cast<uint4*>(out + (long)(row0 + row) * ld + ch * 8) =
          *reinterpret_cast<const uint4*>(stage + row * (D + 8) + ch * 8);
  }
  __syncthreads();
}

// Writes a wave's 32 x D transposed accumulator (16x16 tiles; columns = the wave's 32 rows of the output) through LDS to global.
template <int D>
RP_DEV void store_acc_T(const f32x4 (&acc)[D / 16][2], float mul, bf16* stage /* [32][D+8] */, bf16* __restrict__ out,
                        long ld, int row0, int nrows, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
    for (int c = 0; c < 2; ++c)
      *reinterpret_cast<uint2*>(stage + (16 * c + lr) * (D + 8) + 16 * dt + 4 * lg) =
          make_uint2(pack_bf16x2(acc[dt][c][0] * mul, acc[dt][c][1] * mul),
                     pack_bf16x2(acc[dt][c][2] * mul, acc[dt][c][3] * mul));
  store_staged<D>(stage, out, ld, row0, nrows, lane);
}

// Same for an fp32 destination; stage is [32][D + 4] floats per wave.
template <int D>
RP_DEV void store_acc_T_f32(const f32x4 (&acc)[D / 16][2], float mul, float* stage, float* __restrict__ out, long ld,
                            int row0, int nrows, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
    for (int c = 0; c < 2; ++c)
      *reinterpret_cast<float4*>(stage + (16 * c + lr) * (D + 4) + 16 * dt + 4 * lg) =
          make_float4(acc[dt][c][0] * mul, acc[dt][c][1] * mul, acc[dt][c][2] * mul, acc[dt][c][3] * mul);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < (32 * (D / 4)) / 64; ++it) {
    const int idx = it * 64 + lane;
    const int row = idx / (D / 4), ch = idx % (D / 4);
    if (row0 + row < nrows)
      *reinterpret_cast<float4*>(out + (long)(row0 + row) * ld + ch * 4) =
          *reinterpret_cast<const float4*>(stage + row * (D + 4) + ch * 4);
  }
  __syncthreads();
}

// ================================================================================================ forward
// The fragments of the forward kernel's 32x32 tiles.  The lane half h = lane / 32 holds, of 16 rows, {4h..4h+3, 8+4h..8+4h+3}: what read_frag_tr is
// to the 16x16 tiles; the 8 values of the A operand are tile rows 16 g + those, at column lane % 32 from x_off on.
template <int LD>
RP_DEV uint4 read_frag_tr32(const bf16* base, int g, int x_off) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const bf16* q = base + 16 * g * LD + x_off;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q + 8 * LD));
  const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
  return make_uint4(l2.x, l2.y, h2.x, h2.y);
}
template <int LD>
RP_DEV int tr_base32(int lane) {
  const int lk = lane >> 5, l16 = lane & 15, g16 = lane >> 4;
  return (4 * lk + (l16 >> 2)) * LD + 16 * (g16 & 1) + 4 * (l16 & 3);
}
RP_DEV uint4 pack_frag32(const f32x16& s, int off) {
  return make_uint4(pack_bf16x2(s[off + 0], s[off + 1]), pack_bf16x2(s[off + 2], s[off + 3]),
                    pack_bf16x2(s[off + 4], s[off + 5]), pack_bf16x2(s[off + 6], s[off + 7]));
}
// max over lanes l and l ^ 32, in the vector unit: the exchange through LDS is a round trip of the wave in every key tile.  Forward of
// 8192 tokens, 64 heads of 64: 702 -> 673 us (with the mask test on one limit per lane); the eight-wave kernel, whose waves pair up
// around that wait, is 4 % slower with it (521 -> 542) and keeps the exchange
RP_DEV float half_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// store_acc_T for 32x32 tiles.
template <int D>
RP_DEV void store_acc_T32(const f32x16 (&acc)[D / 32], float mul, bf16* stage /* [32][D+8] */, bf16* __restrict__ out, long ld, int row0, int nrows, int lane) {
  const int lr = lane & 31, lk = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) {
      const int dd = 32 * dt + 8 * vg + 4 * lk;
      *reinterpret_cast<uint2*>(stage + lr * (D + 8) + dd) =
          make_uint2(pack_bf16x2(acc[dt][4 * vg] * mul, acc[dt][4 * vg + 1] * mul),
                     pack_bf16x2(acc[dt][4 * vg + 2] * mul, acc[dt][4 * vg + 3] * mul));
    }
  store_staged<D>(stage, out, ld, row0, nrows, lane);
}

template <int D, int NW>
__global__ void __launch_bounds__(NW * 64, NW <= 4 ? 2 : 1) attn_fwd_kernel(const AttnArgs p) {
  constexpr int LDK = D + 8, LDV = D + 32, KS = D / 16, DT = D / 32, NT = NW * 64, BQ = NW * 32;
  using T64 = Tile64<D, NT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];   // fwd_smem_bytes(D, NW)
  bf16* const smem = reinterpret_cast<bf16*>(dyn_smem);
  // eight-wave workgroups have the CU to themselves: two sets of K/V tiles, one barrier per key tile
  constexpr bool DB = NW >= 8;
  constexpr int SET = 64 * LDK + 64 * LDV;
  bf16* const Ks = smem;
  bf16* const Vs = smem + 64 * LDK;

  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lk = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nQ = (p.seq + BQ - 1) / BQ;
  const int nhb = p.a * p.batch;
  const int rank = heavy_rank((int)blockIdx.x, (int)gridDim.x, p.fold);
  const int qtile = nQ - 1 - rank / nhb;     // the heaviest query tiles of every head go first
  const int hb = xcd_head(rank % nhb, nhb);
  const int hq = hb % p.a, b = hb / p.a;
  const int g = hq / (p.a / p.kh);
  const int q0 = qtile * BQ, qw0 = q0 + w * 32;
  const long tok0 = (long)b * p.seq;
  const bf16* qb = p.q + tok0 * p.ldq + hq * D;
  const rsrc_t rk = seq_rsrc(p.k + tok0 * p.ldk + g * D, p.ldk, p.seq, D);
  const rsrc_t rv = seq_rsrc(p.v + tok0 * p.ldv + g * D, p.ldv, p.seq, D);

  const int qpos = qw0 + lr;     // the lane's query
  uint4 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = make_uint4(0u, 0u, 0u, 0u);
    if (qpos < p.seq) qf[ks] = *reinterpret_cast<const uint4*>(qb + (long)qpos * p.ldq + 16 * ks + 8 * lk);
  }
  const int kv_end = (q0 + BQ < p.seq) ? (q0 + BQ) : p.seq;
  const int nkv = (kv_end + 63) / 64;

  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;

  const bf16* const kfrag0 = Ks + lr * LDK + 8 * lk;
  const bf16* const vfrag0 = Vs + tr_base32<LDV>(lane);
  uint4 kreg[T64::NREG], vreg[T64::NREG];
  T64::load(kreg, rk, p.ldk, 0, tid);
  T64::load(vreg, rv, p.ldv, 0, tid);

  if constexpr (DB) {     // tile 0 into set 0, tile 1 on its way
    T64::template store<LDK>(kreg, Ks, tid);
    T64::template store<LDV>(vreg, Vs, tid);
    if (nkv > 1) {
      T64::load(kreg, rk, p.ldk, 64, tid);
      T64::load(vreg, rv, p.ldv, 64, tid);
    }
  }
  for (int j = 0; j < nkv; ++j) {
    __syncthreads();
    if constexpr (DB) {
      // everyone is done with tile j-1: its set takes tile j+1 (in registers since the last trip), tile j+2 sets out
      if (j + 1 < nkv) {
        T64::template store<LDK>(kreg, Ks + ((j + 1) & 1) * SET, tid);
        T64::template store<LDV>(vreg, Vs + ((j + 1) & 1) * SET, tid);
      }
      if (j + 2 < nkv) {
        T64::load(kreg, rk, p.ldk, (j + 2) * 64, tid);
        T64::load(vreg, rv, p.ldv, (j + 2) * 64, tid);
      }
    } else {
      T64::template store<LDK>(kreg, Ks, tid);
      T64::template store<LDV>(vreg, Vs, tid);
      __syncthreads();
      if (j + 1 < nkv) {
        T64::load(kreg, rk, p.ldk, (j + 1) * 64, tid);
        T64::load(vreg, rv, p.ldv, (j + 1) * 64, tid);
      }
    }
    const bf16* const kfrag = kfrag0 + (DB ? (j & 1) * SET : 0);
    const bf16* const vfrag = vfrag0 + (DB ? (j & 1) * SET : 0);
    const int kv0 = j * 64;
    // Waves whose queries all precede this tile's keys (the last tile of the two upper waves) run it fully masked
    // rather than skip it: they would wait at the next barrier anyway, and a skipped update would make the compiler
    // keep a second copy of the accumulator.
    {
      f32x16 sT[2];
      const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // every LDS fragment is requested AHEAD products before the one that consumes it, so that the MFMAs do not each
      // wait out an LDS round trip
      constexpr int AHEAD = 3;
      {
        constexpr int NS = 2 * KS;
        auto sfrag_at = [&](int n) { return *reinterpret_cast<const uint4*>(kfrag + 32 * (n & 1) * LDK + 16 * (n >> 1)); };
        uint4 ring[AHEAD];
#pragma unroll
        for (int n = 0; n < AHEAD; ++n) ring[n] = sfrag_at(n);
        MFMA_PHASE_BEGIN();
#pragma unroll
        for (int n = 0; n < NS; ++n) {
          const uint4 a = ring[n % AHEAD];
          if (n + AHEAD < NS) ring[n % AHEAD] = sfrag_at(n + AHEAD);
          const int ks = n >> 1, kt = n & 1;
          sT[kt] = mfma32(a, qf[ks], ks == 0 ? zero16 : sT[kt]);
          __builtin_amdgcn_sched_barrier(0);
        }
        MFMA_PHASE_END();
      }
      // the first V fragments are requested now, under the softmax arithmetic
      constexpr int NU = 4 * DT;
      auto ufrag_at = [&](int n) { return read_frag_tr32<LDV>(vfrag, n / DT, 32 * (n % DT)); };
      uint4 uring[AHEAD];
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) uring[n] = ufrag_at(n);
      __builtin_amdgcn_sched_barrier(0);
      const bool need_mask = (kv0 + 63 > qw0) || (kv0 + 64 > p.seq);   // wave-uniform
      if (need_mask) {
        const int klim = (qpos < p.seq - 1 ? qpos : p.seq - 1) - (kv0 + 4 * lk);   // keys up to klim past the lane's first
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int v = 0; v < 16; ++v) sT[kt][v] = (32 * kt + 8 * (v >> 2) + (v & 3) > klim) ? -INFINITY : sT[kt][v];
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sT[kt][v]);
      mx = (NW < 8 ? half_max(mx) : fmaxf(mx, __shfl_xor(mx, 32, 64))) * p.scale_log2e;
      // m_run is a reference exponent, not the exact running maximum: it moves only when a row's maximum outgrows
      // it by 2^8 (the probabilities stay below 256, harmless in fp32 sums and bf16 operands), so after the first
      // few key tiles almost every tile skips the rescale of the accumulator.  The skip is a wave-uniform branch,
      // and alpha passes through an empty asm statement so that the multiplies cannot be hoisted out of it.  The first key tile
      // contains key 0 <= qpos, so m_run is finite from then on.
      const bool grow = mx > m_run + 8.f;
      if (__builtin_amdgcn_ballot_w64(grow) != 0ull) {
        const float m_new = grow ? mx : m_run;
        float alpha = fast_exp2(m_run - m_new);
        asm volatile("" : "+v"(alpha));
        l_run *= alpha;
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float e = fast_exp2(__builtin_fmaf(sT[kt][v], p.scale_log2e, -m_run));
          sT[kt][v] = e;
          psum += e;
        }
      l_run += psum;
      {
        uint4 pf[4];
#pragma unroll
        for (int gk = 0; gk < 4; ++gk)
          pf[gk] = pack_frag32(sT[gk >> 1], 8 * (gk & 1));
        MFMA_PHASE_BEGIN();
#pragma unroll
        for (int n = 0; n < NU; ++n) {
          const uint4 a = uring[n % AHEAD];
          if (n + AHEAD < NU) uring[n % AHEAD] = ufrag_at(n + AHEAD);
          oacc[n % DT] = mfma32(a, pf[n / DT], oacc[n % DT]);
          __builtin_amdgcn_sched_barrier(0);
        }
        MFMA_PHASE_END();
      }
    }
  }

  __syncthreads();
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (lk == 0 && qpos < p.seq) p.lse[((long)b * p.a + hq) * p.seq + qpos] = m_run * 0.6931471805599453f + logf(l_tot);
  store_acc_T32<D>(oacc, 1.f / l_tot, smem + w * 32 * LDK, p.o + tok0 * p.ldo + hq * D, p.ldo, qw0, p.seq, lane);
}

// ================================================================================================ delta = rowsum(dO * O)
template <int D>
__global__ void __launch_bounds__(256) attn_delta_kernel(const bf16* __restrict__ o, const bf16* __restrict__ dout,
                                                         float* __restrict__ delta, long ldo, long lddo, int batch,
                                                         int seq, int a) {
  constexpr int LPH = D / 8;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  const long item = idx / LPH;          // (token, head)
  const int sub = (int)(idx % LPH);
  const long total = (long)batch * seq * a;
  float s = 0.f;
  long t = 0;
  int h = 0;
  if (item < total) {
    t = item / a;
    h = (int)(item - t * a);
    const uint4 uo = reinterpret_cast<const uint4*>(o + t * ldo + h * D)[sub];
    const uint4 ud = reinterpret_cast<const uint4*>(dout + t * lddo + h * D)[sub];
    s = bf16_lo(uo.x) * bf16_lo(ud.x) + bf16_hi(uo.x) * bf16_hi(ud.x) + bf16_lo(uo.y) * bf16_lo(ud.y) +
        bf16_hi(uo.y) * bf16_hi(ud.y) + bf16_lo(uo.z) * bf16_lo(ud.z) + bf16_hi(uo.z) * bf16_hi(ud.z) +
        bf16_lo(uo.w) * bf16_lo(ud.w) + bf16_hi(uo.w) * bf16_hi(ud.w);
  }
#pragma unroll
  for (int off = LPH / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (item < total && sub == 0) {
    const long bi = t / seq, pos = t - bi * seq;
    delta[(bi * a + h) * seq + pos] = s;
  }
}

// ================================================================================================ dQ
template <int D, int NW>
__global__ void __launch_bounds__(NW * 64, NW <= 4 ? 2 : 1) attn_bwd_dq_kernel(const AttnArgs p) {
  // K is read both ways (plain for S, transposing for dQ += dS K) and stored once
  constexpr int LDK = tile_ld(D), LDU = LDK, KS = D / 32, DT = D / 16, NT = NW * 64, BQ = NW * 32;
  using T64 = Tile64<D, NT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];   // dq_smem_bytes(D, NW)
  bf16* const smem = reinterpret_cast<bf16*>(dyn_smem);
  bf16* const Ks = smem;
  bf16* const Vs = smem + 64 * LDU;

  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nQ = (p.seq + BQ - 1) / BQ;
  const int nhb = p.a * p.batch;
  const int rank = heavy_rank((int)blockIdx.x, (int)gridDim.x, p.fold);
  const int qtile = nQ - 1 - rank / nhb;
  const int hb = xcd_head(rank % nhb, nhb);
  const int hq = hb % p.a, b = hb / p.a;
  const int g = hq / (p.a / p.kh);
  const int q0 = qtile * BQ, qw0 = q0 + w * 32;
  const long tok0 = (long)b * p.seq;
  const bf16* qb = p.q + tok0 * p.ldq + hq * D;
  const bf16* dob = p.dout + tok0 * p.lddo + hq * D;
  const rsrc_t rk = seq_rsrc(p.k + tok0 * p.ldk + g * D, p.ldk, p.seq, D);
  const rsrc_t rv = seq_rsrc(p.v + tok0 * p.ldv + g * D, p.ldv, p.seq, D);

  uint4 qf[2][KS], dof[2][KS];     // a lane's queries: column tiles c = 0, 1 (see the forward kernel)
  float lse2[2], dl[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int qpos = qw0 + 16 * c + lr;
    const bool qok = qpos < p.seq;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      dof[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      if (qok) {
        qf[c][ks] = *reinterpret_cast<const uint4*>(qb + (long)qpos * p.ldq + 32 * ks + 8 * lg);
        dof[c][ks] = *reinterpret_cast<const uint4*>(dob + (long)qpos * p.lddo + 32 * ks + 8 * lg);
      }
    }
    const long stat = ((long)b * p.a + hq) * p.seq + qpos;
    lse2[c] = qok ? p.lse_in[stat] * 1.4426950408889634f : INFINITY;   // padded rows get P = 0
    if (p.o_in) {   // uniform: this wave is the only one that holds the row's dO, so delta costs one read of O and no kernel
      float s = 0.f;
      if (qok) {
        const bf16* orow = p.o_in + (tok0 + qpos) * p.ldo + hq * D + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const uint4 u = *reinterpret_cast<const uint4*>(orow + 32 * ks), d = dof[c][ks];
          s += bf16_lo(u.x) * bf16_lo(d.x) + bf16_hi(u.x) * bf16_hi(d.x) + bf16_lo(u.y) * bf16_lo(d.y) + bf16_hi(u.y) * bf16_hi(d.y) +
               bf16_lo(u.z) * bf16_lo(d.z) + bf16_hi(u.z) * bf16_hi(d.z) + bf16_lo(u.w) * bf16_lo(d.w) + bf16_hi(u.w) * bf16_hi(d.w);
        }
      }
      dl[c] = column_sum(s);
      if (qok && lg == 0) p.delta[stat] = dl[c];
    } else {
      dl[c] = qok ? p.delta[stat] : 0.f;
    }
  }

  const int kv_end = (q0 + BQ < p.seq) ? (q0 + BQ) : p.seq;
  const int nkv = (kv_end + 63) / 64;
  f32x4 dqacc[DT][2];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dqacc[dt][0] = dqacc[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  const bf16* const kfrag0 = Ks + lr * LDU + 8 * lg;
  const bf16* const vfrag0 = Vs + lr * LDK + 8 * lg;
  const bf16* const ktfrag0 = Ks + tr_base<LDU>(lane);
  uint4 kreg[T64::NREG], vreg[T64::NREG];
  T64::load(kreg, rk, p.ldk, 0, tid);
  T64::load(vreg, rv, p.ldv, 0, tid);
  // eight-wave workgroups have the CU to themselves: two sets of tiles, one barrier per key tile (see the forward kernel)
  constexpr bool DB = NW >= 8;
  constexpr int SET = 64 * LDU + 64 * LDK;
  auto store_tiles = [&](int set) {
    T64::template store<LDU>(kreg, Ks + set * SET, tid);
    T64::template store<LDK>(vreg, Vs + set * SET, tid);
  };
  auto load_tiles = [&](int jj) {
    T64::load(kreg, rk, p.ldk, jj * 64, tid);
    T64::load(vreg, rv, p.ldv, jj * 64, tid);
  };
  if constexpr (DB) {
    store_tiles(0);
    if (nkv > 1) load_tiles(1);
  }

  for (int j = 0; j < nkv; ++j) {
    __syncthreads();
    if constexpr (DB) {
      if (j + 1 < nkv) store_tiles((j + 1) & 1);
      if (j + 2 < nkv) load_tiles(j + 2);
    } else {
      store_tiles(0);
      __syncthreads();
      if (j + 1 < nkv) load_tiles(j + 1);
    }
    const bf16* const kfrag = kfrag0 + (DB ? (j & 1) * SET : 0);
    const bf16* const vfrag = vfrag0 + (DB ? (j & 1) * SET : 0);
    const bf16* const ktfrag = ktfrag0 + (DB ? (j & 1) * SET : 0);
    const int kv0 = j * 64;
    {   // a wave whose queries all precede this tile's keys runs it fully masked (see the forward kernel)
      const bool need_mask = (kv0 + 63 > qw0) || (kv0 + 64 > p.seq);
      const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
      // the two 32-key halves of the tile one after the other: half as many score registers live at a time
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        f32x4 sT[2][2], dpT[2][2];     // [16 keys][16 queries]
        {
          constexpr int NS = 4 * KS, AHEAD = 4;     // n = (ks * 2 + kt) * 2 + which
          auto sfrag_at = [&](int n) {
            const int row = 32 * k2 + 16 * ((n >> 1) & 1), at = 32 * (n >> 2);
            return *reinterpret_cast<const uint4*>((n & 1) ? vfrag + row * LDK + at : kfrag + row * LDU + at);
          };
          uint4 ring[AHEAD];
#pragma unroll
          for (int n = 0; n < AHEAD; ++n) ring[n] = sfrag_at(n);
#pragma unroll
          for (int n = 0; n < NS; ++n) {
            const uint4 a = ring[n % AHEAD];
            if (n + AHEAD < NS) ring[n % AHEAD] = sfrag_at(n + AHEAD);
            const int ks = n >> 2, kt = (n >> 1) & 1;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (n & 1) dpT[kt][c] = mfma16(a, dof[c][ks], ks == 0 ? zero4 : dpT[kt][c]);
              else sT[kt][c] = mfma16(a, qf[c][ks], ks == 0 ? zero4 : sT[kt][c]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // one wave-uniform branch per half tile around two whole element loops (a test per element would be
        // compiled into a branch per element)
        if (need_mask) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int qpos = qw0 + 16 * c + lr;
            const int klim = (qpos < p.seq - 1 ? qpos : p.seq - 1) - (kv0 + 32 * k2 + 4 * lg);   // local key index <= klim
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                float pr = fast_exp2(__builtin_fmaf(sT[kt][c][e], p.scale_log2e, -lse2[c]));
                pr = (16 * kt + e > klim) ? 0.f : pr;
                sT[kt][c][e] = pr * (dpT[kt][c][e] - dl[c]);   // dS^T
              }
          }
        } else {
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                sT[kt][c][e] = fast_exp2(__builtin_fmaf(sT[kt][c][e], p.scale_log2e, -lse2[c])) * (dpT[kt][c][e] - dl[c]);   // dS^T
        }
        {   // the DT pairs of accumulator updates as one sequence, K^T fragments requested AHEAD pairs early
          constexpr int AHEAD = 2;
          const uint4 df[2] = {pack_frag(sT[0][0], sT[1][0]), pack_frag(sT[0][1], sT[1][1])};
          auto ufrag_at = [&](int n) { return read_frag_tr<LDU>(ktfrag + 32 * k2 * LDU + 16 * n); };
          uint4 uring[AHEAD];
#pragma unroll
          for (int n = 0; n < AHEAD; ++n) uring[n] = ufrag_at(n);
#pragma unroll
          for (int n = 0; n < DT; ++n) {
            const uint4 a = uring[n % AHEAD];
            if (n + AHEAD < DT) uring[n % AHEAD] = ufrag_at(n + AHEAD);
#pragma unroll
            for (int c = 0; c < 2; ++c) dqacc[n][c] = mfma16(a, df[c], dqacc[n][c]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  }
  __syncthreads();
  store_acc_T<D>(dqacc, p.scale, smem + w * 32 * LDK, p.dq + tok0 * p.lddq + hq * D, p.lddq, qw0, p.seq, lane);
}

// P = exp(s) and dS = P dP in place, for 32 queries (rows) x 32 keys of the dK/dV kernels; q0: the query of row 0 of this lane.
RP_DEV void softmax_grad(f32x4 (&s)[2][2], f32x4 (&dp)[2][2], bool need_mask, int q0, const int (&kpos)[2], int seq, float scale_log2e) {
  if (need_mask) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const bool kok = kpos[c] < seq;
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float pr = fast_exp2(s[qt][c][e] * scale_log2e);
          pr = (kpos[c] > q0 + 16 * qt + e || !kok) ? 0.f : pr;
          s[qt][c][e] = pr;
          dp[qt][c][e] = pr * dp[qt][c][e];
        }
    }
  } else {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pr = fast_exp2(s[qt][c][e] * scale_log2e);
          s[qt][c][e] = pr;
          dp[qt][c][e] = pr * dp[qt][c][e];
        }
  }
}

// ================================================================================================ dK, dV in one kernel
// One wave per SIMD at head dimension 128 (the K and V fragments plus both accumulators take more than 256 registers
// per lane), two at 64; four recomputed/updated products per tile.  A version split into a dV and a dK kernel at two
// waves per SIMD each (the scores recomputed in both) was as fast at best once the LDS reads here were issued ahead
// of their MFMAs (sequence 8192 to 31744: 0 to 3 % slower; 16 % slower at head dimension 64) and is gone.  Staggering
// the two 32-query halves so that one half's exponentials sit in the slots of the other half's MFMAs was 12-20 % slower
// (a wave issues in order: the dependent multiply-exp-multiply chains hold back the next MFMA).  Two sets of LDS tiles
// at d = 128 (the next query tile stored during the updates, one barrier per tile instead of two) changed nothing.
template <int D, bool MULTI>
__global__ void __launch_bounds__(256) attn_bwd_dkv_fused_kernel(const AttnArgs p) {
  const int hpw = MULTI ? p.hpw : 1;
  constexpr int LDK = tile_ld(D), KS = D / 32, DT = D / 16;
  using T64 = Tile64<D, 256>;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  bf16* const smem = reinterpret_cast<bf16*>(dyn_smem);             // 2*64*LDK elements; one layout for both kinds of reads, see the pair kernel
  bf16* const Qs = smem;
  bf16* const dOs = smem + 64 * LDK;
  float* const stat = reinterpret_cast<float*>(smem + 2 * 64 * LDK);     // [2][64], see stat_start

  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ah = p.a / hpw, nhb = ah * p.batch;     // workgroups per key tile
  // Workgroups of one query head stream the same Q and dO tiles, a few tiles apart (key tile j starts at query tile 2j
  // and all advance at the same pace).  Consecutive workgroups go to consecutive XCDs, so XCD x (launch positions x,
  // x + 8, ...) takes nhb/8 neighbouring heads and walks them in runs of `kblock` key tiles: its 32 resident workgroups
  // are two such runs, and the XCD's L2 fetches a Q/dO tile once for a whole run.  Key tile 0 sees every query, so the
  // order is still heaviest first at the grain of a run; positions past the last key tile (ragged last run) exit.
  int kvt, hb;
  if (p.kblock) {
    const int hp = nhb >> 3, per = hp * p.kblock;
    const int s = (int)blockIdx.x >> 3, r = s % per;
    hb = ((int)blockIdx.x & 7) * hp + r / p.kblock;
    kvt = (s / per) * p.kblock + r % p.kblock;
    if (kvt * 128 >= p.seq) return;          // uniform over the workgroup, before any barrier
  } else {
    kvt = (int)blockIdx.x / nhb;             // key tile 0 sees every query: heaviest first, for every head
    hb = (int)blockIdx.x % nhb;
  }
  const int hg = hb % ah, b = hb / ah;                 // heads hg * hpw ..
  const int grp = p.a / p.kh;
  const int g = hg * hpw / grp;
  const int kv0 = kvt * 128, kw0 = kv0 + 32 * w;
  const long tok0 = (long)b * p.seq;
  const bf16* kb = p.k + tok0 * p.ldk + g * D;
  const bf16* vb = p.v + tok0 * p.ldv + g * D;
  // a lane's keys are kw0 + lr and kw0 + 16 + lr (column tiles c = 0, 1)
  const int kpos[2] = {kw0 + lr, kw0 + 16 + lr};

  uint4 kf[2][KS], vf[2][KS];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      vf[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      if (kpos[c] < p.seq) {
        kf[c][ks] = *reinterpret_cast<const uint4*>(kb + (long)kpos[c] * p.ldk + 32 * ks + 8 * lg);
        vf[c][ks] = *reinterpret_cast<const uint4*>(vb + (long)kpos[c] * p.ldv + 32 * ks + 8 * lg);
      }
    }
  f32x4 dkacc[DT][2], dvacc[DT][2];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) dkacc[dt][0] = dkacc[dt][1] = dvacc[dt][0] = dvacc[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nQ = (p.seq + 63) / 64;
  const int qt0 = kv0 / 64;
  const int niter = nQ - qt0;

  const bf16* qfrag = Qs + lr * LDK + 8 * lg;
  const bf16* dofrag = dOs + lr * LDK + 8 * lg;
  const bf16* qtfrag = Qs + tr_base<LDK>(lane);
  const bf16* dotfrag = dOs + tr_base<LDK>(lane);

  uint4 qreg[T64::NREG], doreg[T64::NREG];
  float st_reg = 0.f;
  int pf_h = hg * hpw;                   // head and (with several) query tile that are fetched next
  [[maybe_unused]] int pf_it = 0;
  rsrc_t rq = seq_rsrc(p.q + tok0 * p.ldq + pf_h * D, p.ldq, p.seq, D);
  rsrc_t rdo = seq_rsrc(p.dout + tok0 * p.lddo + pf_h * D, p.lddo, p.seq, D);
  rsrc_t rst = stat_rsrc(p.lse_in, p.delta, w, (long)b * p.a + pf_h, p.seq);
  auto prefetch = [&](int nxt) {
    const int q0 = (qt0 + (MULTI ? pf_it : nxt)) * 64;
    T64::load(qreg, rq, p.ldq, q0, tid);
    T64::load(doreg, rdo, p.lddo, q0, tid);
    if (w < 2) st_reg = stat_load(rst, q0 + lane);
    if constexpr (MULTI) {
      if (++pf_it == niter) {
        pf_it = 0;
        ++pf_h;
        rq = seq_rsrc(p.q + tok0 * p.ldq + pf_h * D, p.ldq, p.seq, D);      // (past the last head: never loaded from)
        rdo = seq_rsrc(p.dout + tok0 * p.lddo + pf_h * D, p.lddo, p.seq, D);
        rst = stat_rsrc(p.lse_in, p.delta, w, (long)b * p.a + pf_h, p.seq);
      }
    }
  };
  const int total = niter * hpw;       // query tiles of all the workgroup's heads
  if (total > 0) prefetch(0);

  int it_cur = 0;                        // query tile of the current head
  for (int ia = 0; ia < total; ++ia) {
    const int it = MULTI ? it_cur : ia;
    if constexpr (MULTI) it_cur = it_cur + 1 == niter ? 0 : it_cur + 1;
    __syncthreads();
    T64::template store<LDK>(qreg, Qs, tid);
    T64::template store<LDK>(doreg, dOs, tid);
    if (w < 2) stat[64 * w + lane] = stat_start(st_reg, w, (qt0 + it) * 64 + lane < p.seq, p.scale);
    __syncthreads();
    if (ia + 1 < total) prefetch(ia + 1);
    const int q0 = (qt0 + it) * 64;
    {   // a wave whose keys all follow this tile's queries runs it fully masked (see the forward kernel)
      const bool need_mask = (q0 < kw0 + 31) || (kw0 + 32 > p.seq);   // wave-uniform
      // the two 32-query halves of the tile one after the other: half as many score registers live at a time
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        f32x4 s[2][2], dp[2][2], s0[2], dp0[2];     // [16 queries][16 keys]; what they start from
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
          s0[qt] = *reinterpret_cast<const f32x4*>(stat + 32 * t2 + 16 * qt + 4 * lg);
          dp0[qt] = *reinterpret_cast<const f32x4*>(stat + 64 + 32 * t2 + 16 * qt + 4 * lg);
        }
        // Little else covers the LDS latency, so every fragment is requested AHEAD pairs of MFMAs before the pair that consumes it.
        // Score phase: alternately S and dP.
        constexpr int AHEAD = 4;
        {
          constexpr int NS = 4 * KS;     // n = (ks * 2 + qt) * 2 + which
          auto sfrag_at = [&](int n) { return *reinterpret_cast<const uint4*>(((n & 1) ? dofrag : qfrag) + (32 * t2 + 16 * ((n >> 1) & 1)) * LDK + 32 * (n >> 2)); };
          uint4 ring[AHEAD];
#pragma unroll
          for (int n = 0; n < AHEAD; ++n) ring[n] = sfrag_at(n);
#pragma unroll
          for (int n = 0; n < NS; ++n) {
            const uint4 a = ring[n % AHEAD];
            if (n + AHEAD < NS) ring[n % AHEAD] = sfrag_at(n + AHEAD);
            const int ks = n >> 2, qt = (n >> 1) & 1;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (n & 1) dp[qt][c] = mfma16(a, vf[c][ks], ks == 0 ? dp0[qt] : dp[qt][c]);
              else s[qt][c] = mfma16(a, kf[c][ks], ks == 0 ? s0[qt] : s[qt][c]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // the first fragments of the update phase are requested now, under the exponentials
        constexpr int NU = 2 * DT;
        auto ufrag_at = [&](int n) { return read_frag_tr<LDK>(((n & 1) ? qtfrag : dotfrag) + 32 * t2 * LDK + 16 * (n >> 1)); };
        uint4 uring[AHEAD];
#pragma unroll
        for (int n = 0; n < AHEAD; ++n) uring[n] = ufrag_at(n);
        __builtin_amdgcn_sched_barrier(0);
        // rows of the score tiles are queries: q = q0 + 32*t2 + 16*qt + 4*lg + e
        // the branch is taken per tile, not per element: away from the diagonal nothing below compares positions
        softmax_grad(s, dp, need_mask, q0 + 32 * t2 + 4 * lg, kpos, p.seq, p.scale_log2e);
        // the 2*DT pairs of accumulator updates as one sequence, fragments AHEAD pairs early
        {
          const uint4 pfg[2] = {pack_frag(s[0][0], s[1][0]), pack_frag(s[0][1], s[1][1])};
          const uint4 dfg[2] = {pack_frag(dp[0][0], dp[1][0]), pack_frag(dp[0][1], dp[1][1])};
#pragma unroll
          for (int n = 0; n < NU; ++n) {
            const uint4 a = uring[n % AHEAD];
            if (n + AHEAD < NU) uring[n % AHEAD] = ufrag_at(n + AHEAD);
            const int dt = n >> 1;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (n & 1) dkacc[dt][c] = mfma16(a, dfg[c], dkacc[dt][c]);
              else dvacc[dt][c] = mfma16(a, pfg[c], dvacc[dt][c]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  }
  __syncthreads();
  if (grp == hpw) {
    store_acc_T<D>(dkacc, p.scale, smem + w * 32 * (D + 8), p.dk + tok0 * p.lddk + g * D, p.lddk, kw0, p.seq, lane);
    store_acc_T<D>(dvacc, 1.f, smem + w * 32 * (D + 8), p.dv + tok0 * p.lddv + g * D, p.lddv, kw0, p.seq, lane);
  } else {
    float* const stage = reinterpret_cast<float*>(smem) + w * 32 * (D + 4);
    const long ldp = (long)ah * D;
    store_acc_T_f32<D>(dkacc, p.scale, stage, p.dk_part + tok0 * ldp + hg * D, ldp, kw0, p.seq, lane);
    store_acc_T_f32<D>(dvacc, 1.f, stage, p.dv_part + tok0 * ldp + hg * D, ldp, kw0, p.seq, lane);
  }
}

// The same products with two waves per SIMD.  A workgroup is eight waves: the 32 keys of key group w = wave / 2 are shared
// by a pair of waves, and wave h = wave % 2 of the pair keeps the accumulators of one half of the head dimension only
// (dK^T, dV^T rows [h*D/2, (h+1)*D/2): half the registers).  The scores need the whole head dimension, so the pair splits
// them by queries instead: wave h recomputes S and dP for the 32 queries of half h of the tile, turns them into P and dS, and
// hands both (already in the operand layout of the update products, identical in the two waves since they own the same
// keys) to its partner through LDS.  Every wave then updates its half of the accumulators with its own 32 queries --
// before the workgroup barrier that publishes the exchange -- and with the partner's 32 queries after it.  Same number of
// MFMAs per workgroup as the one-wave-per-SIMD kernel, same LDS fragment traffic per CU, 8 KB of exchange per pair and tile.
// DS: dS is kept as well (see attn_ds_block): a wave stores its 32 keys x 32 queries of every tile, 16 bytes of a key's row per lane
// after one exchange between neighbouring lane groups.  The stores are older than the next tile's loads and overlap the updates, and go past
// the L2 (ordinary stores push the Q and dO tiles out of it, +1 %).  In a stage, us, dQ by recomputation -> from kept dS (with the delta
// kernel): 8192 tokens, 32 heads dK/dV 1121 -> 1209 and dQ 717 -> 553, 4096 x 16 heads 140 -> 157 and 120 -> 92; the stage 7664 -> 7600 and
// 1602 -> 1585, 2048 x 64 heads 3178 -> 3145, 2 x 508 x 32 1067 -> 1064.
template <int D, bool MULTI, bool DS>
__global__ void __launch_bounds__(512) attn_bwd_dkv_pair_kernel(const AttnArgs p) {
  const int hpw = MULTI ? p.hpw : 1;
  // One LDS layout serves both kinds of fragment reads (tile_ld), so that every Q and dO tile is stored once.  No unit is more than half
  // busy: the waves wait on their own chain.
  constexpr int LDU = tile_ld(D), KS = D / 32, DH = D / 32;     // DH: 16-row tiles of half the head dimension
  static_assert(D % 32 == 0, "the head dimension is split over two waves");
  using T64 = Tile64<D, 512>;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  bf16* const smem = reinterpret_cast<bf16*>(dyn_smem);             // two sets (tile parity) of Q | dO, then the exchange
  constexpr int TSET = 2 * 64 * LDU;
  uint4* const exch = reinterpret_cast<uint4*>(smem + 2 * TSET);    // [8 waves][4 fragments][64 lanes]
  float* const stat = reinterpret_cast<float*>(exch + 8 * 4 * 64);  // [2 sets][2][64], see stat_start

  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int w8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = w8 >> 1, h = w8 & 1;
  const int ah = p.a / hpw, nhb = ah * p.batch;
  int kvt, hb;                                 // launch order: see attn_bwd_dkv_fused_kernel
  if (p.kblock) {
    const int hp = nhb >> 3, per = hp * p.kblock;
    const int s = (int)blockIdx.x >> 3, r = s % per;
    hb = ((int)blockIdx.x & 7) * hp + r / p.kblock;
    kvt = (s / per) * p.kblock + r % p.kblock;
    if (kvt * 128 >= p.seq) return;
  } else {
    kvt = (int)blockIdx.x / nhb;
    hb = (int)blockIdx.x % nhb;
  }
  const int hg = hb % ah, b = hb / ah;
  const int grp = p.a / p.kh;
  const int g = hg * hpw / grp;
  const int kv0 = kvt * 128, kw0 = kv0 + 32 * w;
  const long tok0 = (long)b * p.seq;
  const bf16* kb = p.k + tok0 * p.ldk + g * D;
  const bf16* vb = p.v + tok0 * p.ldv + g * D;
  // a lane's keys are kw0 + lr and kw0 + 16 + lr (column tiles c = 0, 1)
  const int kpos[2] = {kw0 + lr, kw0 + 16 + lr};

  uint4 kf[2][KS], vf[2][KS];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      vf[c][ks] = make_uint4(0u, 0u, 0u, 0u);
      if (kpos[c] < p.seq) {
        kf[c][ks] = *reinterpret_cast<const uint4*>(kb + (long)kpos[c] * p.ldk + 32 * ks + 8 * lg);
        vf[c][ks] = *reinterpret_cast<const uint4*>(vb + (long)kpos[c] * p.ldv + 32 * ks + 8 * lg);
      }
    }
  f32x4 dkacc[DH][2], dvacc[DH][2];
#pragma unroll
  for (int dt = 0; dt < DH; ++dt) dkacc[dt][0] = dkacc[dt][1] = dvacc[dt][0] = dvacc[dt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nQ = (p.seq + 63) / 64;
  const int qt0 = kv0 / 64;
  const int niter = nQ - qt0;

  // this wave's 32 queries of a tile: rows 32*h .. 32*h + 31
  const bf16* qfrag = smem + (32 * h + lr) * LDU + 8 * lg;
  const bf16* dofrag = qfrag + 64 * LDU;
  // this wave's half of the head dimension: columns 16*DH*h .. of the transposed tiles
  const bf16* qtfrag = smem + tr_base<LDU>(lane) + 16 * DH * h;
  const bf16* dotfrag = qtfrag + 64 * LDU;
  uint4* const ex_mine = exch + (w8 * 4) * 64 + lane;
  const uint4* const ex_theirs = exch + ((w8 ^ 1) * 4) * 64 + lane;

  uint4 qreg[T64::NREG], doreg[T64::NREG];
  float st_reg = 0.f;
  int pf_h = hg * hpw;                   // head and (with several) query tile that are fetched next
  [[maybe_unused]] int pf_it = 0;
  rsrc_t rq = seq_rsrc(p.q + tok0 * p.ldq + pf_h * D, p.ldq, p.seq, D);
  rsrc_t rdo = seq_rsrc(p.dout + tok0 * p.lddo + pf_h * D, p.lddo, p.seq, D);
  rsrc_t rst = stat_rsrc(p.lse_in, p.delta, w8, (long)b * p.a + pf_h, p.seq);
  auto prefetch = [&](int nxt) {
    const int q0 = (qt0 + (MULTI ? pf_it : nxt)) * 64;
    T64::load(qreg, rq, p.ldq, q0, tid);
    T64::load(doreg, rdo, p.lddo, q0, tid);
    if (w8 < 2) st_reg = stat_load(rst, q0 + lane);
    if constexpr (MULTI) {
      if (++pf_it == niter) {
        pf_it = 0;
        ++pf_h;
        rq = seq_rsrc(p.q + tok0 * p.ldq + pf_h * D, p.ldq, p.seq, D);      // (past the last head: never loaded from)
        rdo = seq_rsrc(p.dout + tok0 * p.lddo + pf_h * D, p.lddo, p.seq, D);
        rst = stat_rsrc(p.lse_in, p.delta, w8, (long)b * p.a + pf_h, p.seq);
      }
    }
  };
  const int total = niter * hpw;       // query tiles of all the workgroup's heads
  if (total > 0) prefetch(0);

  constexpr int AHEAD = 2;     // two waves per SIMD cover each other's LDS latency: a short ring is enough
  // the update products of one 32-query half t2 with the fragments pf (P) and df (dS): 2 * DH pairs of MFMAs
  auto update_half = [&](int set, int t2, const uint4 (&pf)[2], const uint4 (&df)[2]) {
    constexpr int NU = 2 * DH;     // n = dt * 2 + which
    auto ufrag_at = [&](int n) { return read_frag_tr<LDU>(((n & 1) ? qtfrag : dotfrag) + set * TSET + 32 * t2 * LDU + 16 * (n >> 1)); };
    uint4 uring[AHEAD];
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) uring[n] = ufrag_at(n);
    MFMA_PHASE_BEGIN();
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      const uint4 a = uring[n % AHEAD];
      if (n + AHEAD < NU) uring[n % AHEAD] = ufrag_at(n + AHEAD);
      const int dt = n >> 1;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (n & 1) dkacc[dt][c] = mfma16(a, df[c], dkacc[dt][c]);
        else dvacc[dt][c] = mfma16(a, pf[c], dvacc[dt][c]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    MFMA_PHASE_END();
  };

  // Two barriers per tile.  After the first one every wave is done with the previous tile's score phase and has
  // published its fragments: the new tile is stored (into the other set) and, meanwhile, the
  // accumulators are updated with the partner's half of the PREVIOUS tile, whose set is still in place.
  auto partner_update = [&](int it_prev) {
    const uint4 ppf[2] = {ex_theirs[0], ex_theirs[64]};
    const uint4 pdf[2] = {ex_theirs[128], ex_theirs[192]};
    update_half(it_prev & 1, h ^ 1, ppf, pdf);
  };
  int it_cur = 0;                        // query tile of the current head
  [[maybe_unused]] const uint32_t ds_lane = (uint32_t)((w & 1) * 8192 + h * 2048 + (lg & 1) * 1024 + (lg >> 1) * 512 + lr * 16);    // where the lane stores in a block
  [[maybe_unused]] const uint32_t ds_bytes = (uint32_t)attn_ds_block((nQ + 1) / 2, 0) * 16384u;
  [[maybe_unused]] int ds_h = b * p.a + hg * hpw;
  for (int ia = 0; ia < total; ++ia) {
    const int it = MULTI ? it_cur : ia;
    if constexpr (MULTI) it_cur = it_cur + 1 == niter ? 0 : it_cur + 1;
    __syncthreads();
    bf16* const q_set = smem + (ia & 1) * TSET;
    T64::template store<LDU>(qreg, q_set, tid);
    T64::template store<LDU>(doreg, q_set + 64 * LDU, tid);
    if (w8 < 2) stat[128 * (ia & 1) + 64 * w8 + lane] = stat_start(st_reg, w8, (qt0 + it) * 64 + lane < p.seq, p.scale);
    if (ia > 0) partner_update(ia - 1);
    __syncthreads();
    if (ia + 1 < total) prefetch(ia + 1);
    const int q0 = (qt0 + it) * 64;
    const int qh0 = q0 + 32 * h;                                            // first query of this wave's half
    const bool need_mask = (qh0 < kw0 + 31) || (kw0 + 32 > p.seq);          // wave-uniform
    f32x4 s[2][2], dp[2][2], s0[2], dp0[2];      // [16 queries][16 keys]; what they start from
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      s0[qt] = *reinterpret_cast<const f32x4*>(stat + 128 * (ia & 1) + 32 * h + 16 * qt + 4 * lg);
      dp0[qt] = *reinterpret_cast<const f32x4*>(stat + 128 * (ia & 1) + 64 + 32 * h + 16 * qt + 4 * lg);
    }
    {
      constexpr int NS = 4 * KS;     // n = (ks * 2 + qt) * 2 + which
      auto sfrag_at = [&](int n) { return *reinterpret_cast<const uint4*>(((n & 1) ? dofrag : qfrag) + (ia & 1) * TSET + 16 * ((n >> 1) & 1) * LDU + 32 * (n >> 2)); };
      uint4 ring[AHEAD];
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) ring[n] = sfrag_at(n);
      MFMA_PHASE_BEGIN();
#pragma unroll
      for (int n = 0; n < NS; ++n) {
        const uint4 a = ring[n % AHEAD];
        if (n + AHEAD < NS) ring[n % AHEAD] = sfrag_at(n + AHEAD);
        const int ks = n >> 2, qt = (n >> 1) & 1;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          if (n & 1) dp[qt][c] = mfma16(a, vf[c][ks], ks == 0 ? dp0[qt] : dp[qt][c]);
          else s[qt][c] = mfma16(a, kf[c][ks], ks == 0 ? s0[qt] : s[qt][c]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      MFMA_PHASE_END();
    }
    // rows of the score tiles are queries: q = qh0 + 16*qt + 4*lg + e
    softmax_grad(s, dp, need_mask, qh0 + 4 * lg, kpos, p.seq, p.scale_log2e);
    const uint4 pfg[2] = {pack_frag(s[0][0], s[1][0]), pack_frag(s[0][1], s[1][1])};
    const uint4 dfg[2] = {pack_frag(dp[0][0], dp[1][0]), pack_frag(dp[0][1], dp[1][1])};
    // the partner read last tile's fragments before the barrier above: the slots are free
    ex_mine[0] = pfg[0]; ex_mine[64] = pfg[1]; ex_mine[128] = dfg[0]; ex_mine[192] = dfg[1];
    if constexpr (DS) {
      // fragment c holds, for key 16c + lr and lane group lg, queries {4lg..4lg+3, 16+4lg..16+4lg+3} of 32: after the exchange between
      // neighbouring groups eight queries from 16 (lg & 1) + 8 (lg >> 1) on
      const rsrc_t rds = __builtin_amdgcn_make_buffer_rsrc(p.ds + (size_t)ds_h * (ds_bytes / 2), 0, (int)ds_bytes, 0x00020000);
      const int j = qt0 + it;
      const uint32_t at = (uint32_t)attn_ds_block(j >> 1, 2 * kvt + (w >> 1)) * 16384u + (uint32_t)((j & 1) * 4096);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const auto p0 = __builtin_amdgcn_permlane16_swap(dfg[c].x, dfg[c].z, false, false);
        const auto p1 = __builtin_amdgcn_permlane16_swap(dfg[c].y, dfg[c].w, false, false);
        const u32x4 o = {p0[0], p1[0], p0[1], p1[1]};
        __builtin_amdgcn_raw_buffer_store_b128(o, rds, (int)(ds_lane + 256 * c), (int)at, 2);
      }
      if (MULTI && it + 1 == niter) ++ds_h;
    }
    update_half(ia & 1, h, pfg, dfg);
  }
  __syncthreads();
  if (total > 0) partner_update(total - 1);
  __syncthreads();
  if (grp == hpw) {
    bf16* const stage = smem + w8 * 32 * (D / 2 + 8);
    store_acc_T<D / 2>(dkacc, p.scale, stage, p.dk + tok0 * p.lddk + g * D + h * (D / 2), p.lddk, kw0, p.seq, lane);
    store_acc_T<D / 2>(dvacc, 1.f, stage, p.dv + tok0 * p.lddv + g * D + h * (D / 2), p.lddv, kw0, p.seq, lane);
  } else {
    float* const stage = reinterpret_cast<float*>(smem) + w8 * 32 * (D / 2 + 4);
    const long ldp = (long)ah * D;
    store_acc_T_f32<D / 2>(dkacc, p.scale, stage, p.dk_part + tok0 * ldp + hg * D + h * (D / 2), ldp, kw0, p.seq, lane);
    store_acc_T_f32<D / 2>(dvacc, 1.f, stage, p.dv_part + tok0 * ldp + hg * D + h * (D / 2), ldp, kw0, p.seq, lane);
  }
}

// dk[t, g, :] = sum of the fp32 partials of group g (a of them per token, one for hpw query heads), in head order; same for dv.
template <int D>
__global__ void __launch_bounds__(256) attn_dkv_reduce_kernel(const float* __restrict__ dk_part, const float* __restrict__ dv_part,
                                                              bf16* __restrict__ dk, bf16* __restrict__ dv, long lddk,
                                                              long lddv, long T, int a, int kh) {
  constexpr int CH = D / 8;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  const long per = T * kh * CH;
  if (idx >= 2 * per) return;
  const bool is_v = idx >= per;
  const long i = is_v ? idx - per : idx;
  const int ch = (int)(i % CH);
  const int g = (int)((i / CH) % kh);
  const long t = i / ((long)CH * kh);
  const int grp = a / kh;
  const float* src = (is_v ? dv_part : dk_part) + t * (long)a * D + (long)g * grp * D + ch * 8;
  float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0;
  for (int j = 0; j < grp; ++j) {
    const float4 x0 = *reinterpret_cast<const float4*>(src + (long)j * D);
    const float4 x1 = *reinterpret_cast<const float4*>(src + (long)j * D + 4);
    s0.x += x0.x; s0.y += x0.y; s0.z += x0.z; s0.w += x0.w;
    s1.x += x1.x; s1.y += x1.y; s1.z += x1.z; s1.w += x1.w;
  }
  bf16* dst = is_v ? dv + t * lddv + g * D + ch * 8 : dk + t * lddk + g * D + ch * 8;
  *reinterpret_cast<uint4*>(dst) = make_uint4(pack_bf16x2(s0.x, s0.y), pack_bf16x2(s0.z, s0.w), pack_bf16x2(s1.x, s1.y),
                                              pack_bf16x2(s1.z, s1.w));
}

// operand tiles, or the epilogue's staging of every wave's 32 x d block, whichever is larger
constexpr int max_i(int a, int b) { return a > b ? a : b; }
constexpr int fwd_smem_bytes(int d, int nw) { return max_i((nw >= 8 ? 2 : 1) * (64 * (d + 8) + 64 * (d + 32)), nw * 32 * (d + 8)) * 2; }
constexpr int dq_smem_bytes(int d, int nw) { return max_i((nw >= 8 ? 2 : 1) * (2 * 64 * tile_ld(d)), nw * 32 * (d + 8)) * 2; }
constexpr int dkv_fused_smem_bytes(int d) { return max_i(2 * 64 * tile_ld(d) * 2 + 512, 4 * 32 * (d + 4) * 4); }
constexpr int dkv_pair_smem_bytes(int d) { return 2 * (2 * 64 * tile_ld(d)) * 2 + 8 * 4 * 64 * 16 + 1024; }
void fill_common(AttnArgs& p, int batch, int seq, int a, int kh, int d) {
  p.batch = batch; p.seq = seq; p.a = a; p.kh = kh;
  p.scale = 1.0f / sqrtf((float)d);
  p.scale_log2e = p.scale * 1.4426950408889634f;
}

template <typename K>
hipError_t set_smem(K kern, int bytes, bool& done) {
  if (done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done = true;
  return e;
}

template <int D, int NW>
hipError_t launch_fwd(hipStream_t st, const AttnArgs& p) {
  constexpr int BQ = NW * 32;
  static bool done = false;
  hipError_t e = set_smem(attn_fwd_kernel<D, NW>, fwd_smem_bytes(D, NW), done);
  if (e != hipSuccess) return e;
  const int grid = ((p.seq + BQ - 1) / BQ) * p.a * p.batch;
  AttnArgs pf = p;
  pf.fold = NW <= 4 && grid > 256 && grid <= 512;
  RP_LAUNCH((attn_fwd_kernel<D, NW>), dim3(grid), dim3(NW * 64), fwd_smem_bytes(D, NW), st, pf);
  return hipGetLastError();
}

template <int D, bool MULTI>
hipError_t launch_dkv_fused_one(hipStream_t st, const AttnArgs& p, int grid) {
  static bool done = false;
  hipError_t e = set_smem(attn_bwd_dkv_fused_kernel<D, MULTI>, dkv_fused_smem_bytes(D), done);
  if (e != hipSuccess) return e;
  RP_LAUNCH((attn_bwd_dkv_fused_kernel<D, MULTI>), dim3(grid), dim3(256), dkv_fused_smem_bytes(D), st, p);
  return hipGetLastError();
}
template <int D>
hipError_t launch_dkv_fused(hipStream_t st, const AttnArgs& p, int grid) {
  return p.hpw > 1 ? launch_dkv_fused_one<D, true>(st, p, grid) : launch_dkv_fused_one<D, false>(st, p, grid);
}

template <int D, bool MULTI, bool DS>
hipError_t launch_dkv_pair_one(hipStream_t st, const AttnArgs& p, int grid) {
  static bool done = false;
  hipError_t e = set_smem(attn_bwd_dkv_pair_kernel<D, MULTI, DS>, dkv_pair_smem_bytes(D), done);
  if (e != hipSuccess) return e;
  RP_LAUNCH((attn_bwd_dkv_pair_kernel<D, MULTI, DS>), dim3(grid), dim3(512), dkv_pair_smem_bytes(D), st, p);
  return hipGetLastError();
}
template <int D>
hipError_t launch_dkv_pair(hipStream_t st, const AttnArgs& p, int grid) {
  if (p.ds) return p.hpw > 1 ? launch_dkv_pair_one<D, true, true>(st, p, grid) : launch_dkv_pair_one<D, false, true>(st, p, grid);
  return p.hpw > 1 ? launch_dkv_pair_one<D, true, false>(st, p, grid) : launch_dkv_pair_one<D, false, false>(st, p, grid);
}

template <int D, int NW>
hipError_t launch_dq(hipStream_t st, const AttnArgs& p) {
  constexpr int BQ = NW * 32;
  static bool done = false;
  hipError_t e = set_smem(attn_bwd_dq_kernel<D, NW>, dq_smem_bytes(D, NW), done);
  if (e != hipSuccess) return e;
  const int grid = ((p.seq + BQ - 1) / BQ) * p.a * p.batch;
  AttnArgs pf = p;
  pf.fold = NW <= 4 && grid > 256 && grid <= 512;
  RP_LAUNCH((attn_bwd_dq_kernel<D, NW>), dim3(grid), dim3(NW * 64), dq_smem_bytes(D, NW), st, pf);
  return hipGetLastError();
}

// Query heads of a group that a dK/dV workgroup takes one after the other, summing them in its accumulators: every doubling halves
// the fp32 partials that are written and read back (147 MB each way at 3 x 1500 tokens, 64 heads of 64) and the workgroups'
// start and end, and doubles the longest chain (key tile 0 sees every query tile).  It pays while that chain is short against
// the work per CU.  Measured, backward in us, one head | two | four, with chain / work per CU of the last two in brackets:
//   d = 128: 8192 x 32 heads 1669 | 1624 (.49) | 1620 (.98);  4096 x 64: 950 | 885 (.48) | 886 (.97);  2 x 2048 x 64:
//            580 | 513 (.47) | 489 (.94);  4096 x 32: 478 | 457 (.97) | 610
//   d = 64 (two workgroups share a CU, a chain runs at half the pace): 3 x 1500 x 64: 252 | 232 (.41) | 242 (.82);
//            8192 x 64: 1780 | 1733 (.25) | 1786 (.49);  2048 x 64: 151 | 162 (.94) | 226
// Groups of two heads in one key tile, or two, take both heads as well, beside that rule: the chain is then two to eight query tiles
// longer, 1 to 4 us, and the partials and the launch that adds them are 3 us and what their traffic takes.  Forward and backward of the
// attention entry points, us, one head | two:  d = 64, 4 heads: 1 x 64 tokens 19.2 | 17.0, 1 x 128 24.3 | 22.2, 64 x 128 25.5 | 23.2;  d = 128,
// 16 heads: 1 x 64 24.0 | 21.6, 1 x 128 31.4 | 30.8, 4 x 128 36.5 | 31.5.  Two key tiles, heads x sequences at d = 64 and d = 128: 4: 28.6 | 30.4 and
// 39.1 | 42.0, 16: 29.4 | 30.8 and 40.8 | 42.6, 32: 30.3 | 31.6 and 43.2 | 43.0, 64: 32.4 | 31.6 and 45.7 | 44.0, 256: 44.0 | 37.1 and 82.6 | 58.8;
// 48 heads x sequences, 160 and 256 tokens: 26.6 | 26.0 and 31.4 | 31.4, 36.8 | 35.2 and 46.2 | 43.3.
// (One tile, 4 heads, d = 128, 1 x 128 tokens: 30.5 | 30.5.)
// Orders by runs of key tiles (from 96 tiles on, see k_attn_bwd) keep one head: 16384 x 64 13100 | 13040 | 13270.
int heads_per_workgroup(int seq, int batch, int a, int kh, int d) {
  const long nkv = (seq + 127) / 128;
  const double per_cu = (double)a * batch * nkv * (nkv + 1) / 256.0, most = d == 128 ? 1.0 : 0.45;
  if (a == 2 * kh && (nkv == 1 || (nkv == 2 && a * batch >= (d == 128 ? 48 : 64)))) return 2;
  int hpw = 1;
  while (nkv < 96 && hpw < 4 && (a / kh) % (2 * hpw) == 0 && 2.0 * hpw * 2.0 * nkv <= most * per_cu) hpw *= 2;
  return hpw;
}

}  // namespace

// ------------------------------------------------------------------------------------------------ launchers
hipError_t k_attn_fwd(hipStream_t st, const void* q, const void* k, const void* v, void* o, float* lse, long ldq,
                      long ldk, long ldv, long ldo, int batch, int seq, int a, int kh, int d) {
  if (batch * seq == 0) return hipSuccess;
  AttnArgs p = {};
  p.q = (const bf16*)q; p.k = (const bf16*)k; p.v = (const bf16*)v; p.o = (bf16*)o; p.lse = lse;
  p.ldq = ldq; p.ldk = ldk; p.ldv = ldv; p.ldo = ldo;
  fill_common(p, batch, seq, a, kh, d);
  // workgroup = 4 waves x 32 queries; 64 queries per wave halve the LDS reads per MFMA but spill at d = 128
  // eight waves per workgroup (256 queries) store every K/V tile once for twice the products; enough workgroups needed.  Four | eight, us: 8192 x 32
  // heads 510 | 487, 4096 x 64 269 | 263, 8192 x 24 (768 workgroups) 402 | 387, 4096 x 32 (512) 137 | 132, 2048 x 64 (512) 77.3 | 76.1, but with short
  // chains 4 x 1024 x 64 (1024) 93.7 | 100.8; dQ with the rest of the backward 1658 | 1625, 878 | 877, 1303 | 1295, 461 | 444, 256 | 253, 291 | 302
  // (d = 128 only: at d = 64 the four-wave kernel fits three waves per SIMD and is 20 % faster than the eight-wave one)
  const bool big = (long)((seq + 255) / 256) * a * batch >= 1024;
  if (d == 128 && big) return launch_fwd<128, 8>(st, p);
  if (d == 128) return launch_fwd<128, 4>(st, p);
  if (d == 64) return launch_fwd<64, 4>(st, p);
  return hipErrorInvalidValue;
}

hipError_t k_attn_delta(hipStream_t st, const void* o, const void* dout, float* delta, long ldo, long lddo, int batch,
                        int seq, int a, int d) {
  const long items = (long)batch * seq * a * (d / 8);
  if (items == 0) return hipSuccess;
  const int grid = (int)((items + 255) / 256);
  if (d == 128) RP_LAUNCH(attn_delta_kernel<128>, dim3(grid), dim3(256), 0, st, (const bf16*)o, (const bf16*)dout, delta, ldo, lddo, batch, seq, a);
  else if (d == 64) RP_LAUNCH(attn_delta_kernel<64>, dim3(grid), dim3(256), 0, st, (const bf16*)o, (const bf16*)dout, delta, ldo, lddo, batch, seq, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

int k_attn_dkv_partials(int batch, int seq, int a, int kh, int d) {
  const int ah = a / heads_per_workgroup(seq, batch, a, kh, d);
  return ah == kh ? 0 : ah;
}

size_t k_attn_ds_bytes(int seq, int d) {
  const size_t n = ((size_t)seq + 127) / 128, bytes = n * (n + 1) * 16384;
  return d == 128 && bytes < ((size_t)1 << 31) ? bytes : 0;     // addressed with 31-bit offsets
}

hipError_t k_attn_bwd(hipStream_t st, int part, const void* q, const void* k, const void* v, const void* dout,
                      const float* lse, float* delta, void* dq, void* dk, void* dv, float* scratch, long ldq,
                      long ldk, long ldv, long lddo, long lddq, long lddk, long lddv, int batch, int seq, int a, int kh,
                      int d, void* ds, const void* o, long ldo) {
  if (batch * seq == 0) return hipSuccess;
  if (ds && k_attn_ds_bytes(seq, d) == 0) return hipErrorInvalidValue;
  AttnArgs p = {};
  p.ds = (bf16*)ds; p.o_in = (const bf16*)o; p.ldo = ldo;
  p.q = (const bf16*)q; p.k = (const bf16*)k; p.v = (const bf16*)v; p.dout = (const bf16*)dout;
  p.lse_in = lse; p.delta = delta; p.dq = (bf16*)dq; p.dk = (bf16*)dk; p.dv = (bf16*)dv;
  p.ldq = ldq; p.ldk = ldk; p.ldv = ldv; p.lddo = lddo; p.lddq = lddq; p.lddk = lddk; p.lddv = lddv;
  fill_common(p, batch, seq, a, kh, d);
  if (d != 128 && d != 64) return hipErrorInvalidValue;
  if (a != kh && !scratch) return hipErrorInvalidValue;
  const long T = (long)batch * seq;
  p.hpw = heads_per_workgroup(seq, batch, a, kh, d);
  const int ah = a / p.hpw;     // partials per token
  p.dk_part = scratch;
  p.dv_part = scratch ? scratch + T * a * d : nullptr;
  hipError_t e = hipSuccess;
  if (part == 2) {   // sum of the group's partials
    if (ah == kh) return hipSuccess;
    const long items = 2 * T * kh * (d / 8);
    const int grid = (int)((items + 255) / 256);
    if (d == 128) RP_LAUNCH(attn_dkv_reduce_kernel<128>, dim3(grid), dim3(256), 0, st, p.dk_part, p.dv_part, p.dk, p.dv, lddk, lddv, T, ah, kh);
    else RP_LAUNCH(attn_dkv_reduce_kernel<64>, dim3(grid), dim3(256), 0, st, p.dk_part, p.dv_part, p.dk, p.dv, lddk, lddv, T, ah, kh);
    return hipGetLastError();
  }
  if (part == 0) {
    const int nkv = (seq + 127) / 128, nhb = ah * batch;
    int nk = nkv * nhb;                               // one workgroup per 128 keys and hpw query heads
    // XCD-aware order (see the kernel) from 96 key tiles on: 5-7 % at 16-32 k tokens; below that the re-fetches it saves
    // do not matter and the plain order balances the few rounds of workgroups better (4096 tokens: 10 % slower with it)
    if (nhb % 8 == 0 && nkv >= 96) {
      p.kblock = nkv >= 192 ? 32 : 16;
      nk = ((nkv + p.kblock - 1) / p.kblock) * p.kblock * nhb;
    }
    if (d == 128) return launch_dkv_pair<128>(st, p, nk);
    return launch_dkv_fused<64>(st, p, nk);   // d = 64: its registers already allow two waves per SIMD
  } else if (ds) {
    return gemm_attn_dq(st, ds, k_attn_ds_bytes(seq, d), k, ldk, dq, lddq, batch, seq, a, kh, d, p.scale);
  } else {
    const bool big = (long)((seq + 255) / 256) * a * batch >= 1024;
    if (d == 128 && big) return launch_dq<128, 8>(st, p);
    return d == 128 ? launch_dq<128, 4>(st, p) : launch_dq<64, 4>(st, p);
  }
  return hipGetLastError();
}
