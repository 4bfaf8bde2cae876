// Cross-entropy bookkeeping around the LM-head GEMMs: the logits are reduced inside the GEMM epilogue to per-token
// (max, sum exp) partials, one per 128 vocabulary rows; these kernels merge the partials and produce the loss and the
// per-token gradient coefficient.
#include "common.hpp"
#include "kernels.hpp"
#include "gemm.hpp"

namespace {

// lse[t] = log sum_v exp(z[t, v]) from P partial (max, sum) pairs per token; part is [P][ld] so reads are coalesced
// over tokens.  A block handles 16 tokens with 64 slices of the partials each (a thread's chain of dependent
// exponentials is P/64 long), merged through LDS in two steps.
__global__ void __launch_bounds__(1024) ce_lse_kernel(const float2* __restrict__ part, int P, long ld, float* __restrict__ lse, int T) {
  constexpr int NS = 64;
  __shared__ float2 red[NS][17];
  const int tl = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int t = blockIdx.x * 16 + tl;
  float m = -INFINITY, s = 0.f;
  auto merge = [&](const float2 v) {
    if (v.x > -INFINITY) {
      const float mn = fmaxf(m, v.x);
      s = s * __expf(m - mn) + v.y * __expf(v.x - mn);
      m = mn;
    }
  };
  if (t < T)
    for (int i = sl; i < P; i += NS) merge(part[(long)i * ld + t]);
  red[sl][tl] = make_float2(m, s);
  __syncthreads();
  if (sl < 8) {   // slices sl, sl + 8, ..., in a fixed order
    for (int i = sl + 8; i < NS; i += 8) merge(red[i][tl]);
    red[sl][tl] = make_float2(m, s);
  }
  __syncthreads();
  if (sl == 0 && t < T) {
    for (int i = 1; i < 8; ++i) merge(red[i][tl]);
    lse[t] = m + logf(s);
  }
}

// One block: counts the valid tokens, loss = sum(lse - z_label) / n_valid, coef[t] = grad_scale / n_valid or 0.
// lse[t] is lse[t] + log l[t] where l is given (the reference exponents and normalisers of the one-sweep schedule).
// last: the sums that the last chunk still owes l.
__global__ void __launch_bounds__(1024) ce_finalize_kernel(const float* __restrict__ lse, float* __restrict__ l, const float* __restrict__ zlab,
                                                           const int* __restrict__ labels, float grad_scale,
                                                           float* __restrict__ coef, float* __restrict__ loss_out, int T, const CeSums last) {
  __shared__ float red[16];
  __shared__ int redi[16];
  __shared__ float bc;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int owed = last.part ? *last.flag : 0;      // uniform; waited for behind the loop, which is run again where it is set
  int cnt = 0;
  float sum = 0.f;
  auto add_up = [&]() {
    cnt = 0;
    sum = 0.f;
    for (int t = tid; t < T; t += 1024) {
      if (labels[t] != -100) { ++cnt; sum += (l ? lse[t] + logf(l[t]) : lse[t]) - zlab[t]; }
    }
  };
  add_up();
  if (owed) {      // all threads on min(T, 1024) tokens at a time, the rows split over what is left of them
    __shared__ float part[1024];
    const int width = T < 1024 ? (T + 63) / 64 * 64 : 1024, ns = 1024 / width, sl = tid / width, tl = tid - sl * width;
    for (int t0 = 0; t0 < T; t0 += width) {
      const int t = t0 + tl;
      float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;   // four chains, merged in a fixed order
      if (t < T && sl < ns) {
        int i = sl;
        for (; i + 3 * ns < last.rows; i += 4 * ns) {
          s0 += last.part[(long)i * T + t].y; s1 += last.part[(long)(i + ns) * T + t].y;
          s2 += last.part[(long)(i + 2 * ns) * T + t].y; s3 += last.part[(long)(i + 3 * ns) * T + t].y;
        }
        for (; i < last.rows; i += ns) s0 += last.part[(long)i * T + t].y;
      }
      part[tid] = (s0 + s1) + (s2 + s3);
      __syncthreads();
      if (sl == 0 && t < T) {
        float s = part[tl];
        for (int k = 1; k < ns; ++k) s += part[k * width + tl];
        l[t] += s;
      }
      __syncthreads();      // (also makes l visible to the threads that read it below)
    }
    add_up();
  }
  sum = wave_sum(sum);
  float fc = wave_sum((float)cnt);
  if (lane == 0) { red[w] = sum; redi[w] = (int)(fc + 0.5f); }
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
    int n = 0;
    for (int i = 0; i < 16; ++i) { s += red[i]; n += redi[i]; }
    loss_out[0] = n > 0 ? s / (float)n : 0.f;
    bc = n > 0 ? grad_scale / (float)n : 0.f;
  }
  __syncthreads();
  const float c = bc;
  for (int t = tid; t < T; t += 1024) coef[t] = labels[t] != -100 ? c : 0.f;
}

// ---- frozen head: one sweep over the vocabulary (no dW, so the softmax normaliser is only needed at the end) ---------
// Per vocabulary chunk the logits Z^T [vc, T] (fp32) are turned into p = exp(z - m_t) against a per-token reference
// exponent m_t, and acc_t = sum_v p_tv W_v, l_t = sum_v p_tv are carried from chunk to chunk; when a chunk's maximum
// outgrows the reference by more than 8 (in e-units), the reference moves and acc_t, l_t (or the p kept so far) are rescaled.  At the end
// lse_t = m_t + log l_t and dx_t = coef_t (acc_t / l_t - W[y_t]).
//
// After the first chunk the logits GEMM writes p itself (EPI_CE_P) against the reference as it stands, together with the
// chunk's column maxima and sums; only when some token's maximum outgrows its reference by more than RP_CE_P_LIMIT does
// the chunk take the path above (a device flag switches those kernels on; they return at once otherwise).

constexpr int CE_PROB_ROWS = 128;

// Sixteen waves share 64 tokens (lane = token) and split the rows of a [rows][T] array; red[wave][token] is theirs to merge.
constexpr int CE_SLICES = 16;

// m[t] = max over the rows of z [rows][T], l[t] = 0, alpha[t] = 1: the reference exponents a sweep starts from; and zeroes the label
// logits and the chunks' flags.
__global__ void __launch_bounds__(1024) ce_ref_init_kernel(const float* __restrict__ z, int rows, int T, float* __restrict__ m,
                                                           float* __restrict__ l, float* __restrict__ alpha, float* __restrict__ zlab,
                                                           int* __restrict__ flags, int nflags) {
  if (blockIdx.x == 0 && (int)threadIdx.x < nflags) flags[threadIdx.x] = 0;
  __shared__ float red[CE_SLICES][64];
  const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6, t = blockIdx.x * 64 + lane;
  float mx = -INFINITY;
  if (t < T)
    for (int r = sl; r < rows; r += CE_SLICES) mx = fmaxf(mx, z[(long)r * T + t]);
  red[sl][lane] = mx;
  __syncthreads();
  if (sl == 0 && t < T) {
    for (int k = 1; k < CE_SLICES; ++k) mx = fmaxf(mx, red[k][lane]);
    m[t] = mx; l[t] = 0.f; alpha[t] = 1.f; zlab[t] = 0.f;
  }
}

// What EPI_CE_P left per token: l_out[t] = l_in[t] + the chunk's sum (.y of the partial rows, sixteen interleaved chains merged
// in a fixed order), and *flag = 1 when some token's maximum (.x) lies more than RP_CE_P_LIMIT above its reference exponent:
// the chunk is then done again by the kernels behind the flag, which leave its sums to the next reader of l: here those of the chunk
// before (prev) are added to l_in first, with no launch of their own (4 us in every chunk, flag or not) and without counting blocks off
// (the fence that takes in every block of the apply kernel: 3.6 ms of 57 at 16384 tokens with eight chunks done again).  Bound by reading the partials once: 10 + 5.6 us in two kernels
// before (one thread per token in the sum), 5 us, at 2040 tokens and 32768 vocabulary rows.
__global__ void __launch_bounds__(1024) ce_chunk_stats_kernel(const float2* __restrict__ part, int nslab, int T, const float* __restrict__ m,
                                                              float* __restrict__ l_in, float* __restrict__ l_out, int* __restrict__ flag, const CeSums prev) {
  __shared__ float2 red[CE_SLICES][64];
  const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6, t = blockIdx.x * 64 + lane;
  const int owed = prev.part ? *prev.flag : 0;      // uniform; waited for behind the loop
  float lin = sl == 0 && t < T ? l_in[t] : 0.f;
  float mx = -INFINITY, sum = 0.f;
  if (t < T)
    for (int i = sl; i < nslab; i += CE_SLICES) {
      const float2 v = part[(long)i * T + t];
      mx = fmaxf(mx, v.x);
      sum += v.y;
    }
  if (owed) {
    float s = 0.f;
    if (t < T)
      for (int i = sl; i < prev.rows; i += CE_SLICES) s += prev.part[(long)i * T + t].y;
    red[sl][lane].x = s;
    __syncthreads();
    if (sl == 0 && t < T) {
      for (int k = 1; k < CE_SLICES; ++k) s += red[k][lane].x;
      lin += s;
      l_in[t] = lin;
    }
    __syncthreads();
  }
  red[sl][lane] = make_float2(mx, sum);
  __syncthreads();
  if (sl == 0 && t < T) {
    for (int k = 1; k < CE_SLICES; ++k) { mx = fmaxf(mx, red[k][lane].x); sum += red[k][lane].y; }
    l_out[t] = lin + sum;
    if (mx > m[t] + RP_CE_P_LIMIT) *flag = 1;   // every writer stores the same value
  }
}

// Behind the flag.  Moves the reference exponent of every token that this chunk outgrew and rescales what was summed before the
// chunk; alpha[t] is the factor acc_t and the stored probabilities must be multiplied with (1 for most tokens).
__global__ void __launch_bounds__(256) ce_chunk_ref_kernel(const float2* __restrict__ pmax, int nslab, int T, float* __restrict__ m,
                                                           const float* __restrict__ l_in, float* __restrict__ l_out,
                                                           float* __restrict__ alpha, const int* __restrict__ run_flag) {
  if (*run_flag == 0) return;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= T) return;
  float cm = -INFINITY;
  for (int i = 0; i < nslab; ++i) cm = fmaxf(cm, pmax[(long)i * T + t].x);
  const float mo = m[t];
  float a = 1.f;
  if (cm > mo + 8.f) {
    // by a whole number k of ln 2, to the first such value that is not below the chunk's maximum: the factor 2^-k then multiplies
    // what is stored in 16 bits without rounding it again (rounded, 2^-9 of everything before the chunk, and the same way for equal
    // probabilities: 3.1e-3 of dx where 2048 equal logits are outgrown by 9)
    const float k = ceilf((cm - mo) * 1.44269504f);
    const bool far = k > 300.f;            // nothing before the chunk is left (also where either maximum is infinite)
    a = far ? 0.f : ldexpf(1.f, -(int)k);
    m[t] = far ? cm : fmaf(k, 0.693147181f, mo);
  }
  l_out[t] = l_in[t] * a;
  alpha[t] = a;
}

// p[r][t] = exp(z[r][t] - m[t]) as bf16; the fp32 sum over the block's CE_PROB_ROWS rows goes to the .y half of the
// block's row of the partial array (whose .x half holds the column maxima the logits GEMM left there, one row of
// partials per CE_PROB_ROWS vocabulary rows): no atomics, whoever reads the normaliser next adds the rows (CeSums).
RP_DEV void chunk_prob(int bx, int by, const float* __restrict__ z, int vc, int T, const float* __restrict__ m, bf16* __restrict__ p,
                       float2* __restrict__ part) {
  const int t = (bx * 256 + threadIdx.x) * 4;      // four tokens per thread: 16-byte loads, 8-byte stores
  if (t >= T) return;
  const int r0 = by * CE_PROB_ROWS, r1 = min(r0 + CE_PROB_ROWS, vc);
  const float4 mm = *reinterpret_cast<const float4*>(m + t);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  auto one = [&](const float4& zz, int r) {
    const float p0 = __expf(zz.x - mm.x), p1 = __expf(zz.y - mm.y), p2 = __expf(zz.z - mm.z), p3 = __expf(zz.w - mm.w);
    s.x += p0; s.y += p1; s.z += p2; s.w += p3;
    *reinterpret_cast<uint2*>(p + (long)r * T + t) = make_uint2(pack_bf16x2(p0, p1), pack_bf16x2(p2, p3));
  };
  int r = r0;
  for (; r + 8 <= r1; r += 8) {          // eight rows in flight per thread
    float4 zz[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) zz[k] = *reinterpret_cast<const float4*>(z + (long)(r + k) * T + t);
#pragma unroll
    for (int k = 0; k < 8; ++k) one(zz[k], r + k);
  }
  for (; r < r1; ++r) one(*reinterpret_cast<const float4*>(z + (long)r * T + t), r);
  float2* const row = part + (long)by * T + t;
  row[0].y = s.x; row[1].y = s.y; row[2].y = s.z; row[3].y = s.w;
}

// acc[t, :] *= alpha[t] for the rows whose reference moved.  One wave per row, blocks bx of nb.
RP_DEV void rescale_rows(int bx, int nb, float* __restrict__ acc, const float* __restrict__ alpha, int T, int h) {
  const int lane = threadIdx.x & 63;
  for (int t = bx * 4 + (threadIdx.x >> 6); t < T; t += nb * 4) {
    const float a = alpha[t];
    if (a == 1.f) continue;
    float4* row = reinterpret_cast<float4*>(acc + (long)t * h);
    for (int c = lane; c < h / 4; c += 64) { float4 v = row[c]; v.x *= a; v.y *= a; v.z *= a; v.w *= a; row[c] = v; }
  }
}

// One sweep with a trainable head: the probabilities of every chunk stay in memory ([V, T] bf16, against the reference
// exponent), and the weight gradient is formed afterwards as  dW = P'^T^T xs,  P'[v, t] = p[v, t] - l_t [v = y_t],
// xs_t = (coef_t / l_t) xf_t  (= sum_t coef_t (p_tv / l_t - [v = y_t]) xf_t).
//
// p[r, t] *= alpha[t] for the rows r < rows stored so far, where a token's reference moved (alpha != 1).  Blocks bx of nb.
RP_DEV void rescale_p(int bx, int nb, bf16* __restrict__ p, long rows, int T, const float* __restrict__ alpha) {
  const int t8 = T >> 3;
  const long total = rows * t8;
  for (long idx = (long)bx * 256 + threadIdx.x; idx < total; idx += (long)nb * 256) {
    const int c = (int)(idx % t8);
    const float4 a0 = *reinterpret_cast<const float4*>(alpha + c * 8), a1 = *reinterpret_cast<const float4*>(alpha + c * 8 + 4);
    if (a0.x == 1.f && a0.y == 1.f && a0.z == 1.f && a0.w == 1.f && a1.x == 1.f && a1.y == 1.f && a1.z == 1.f && a1.w == 1.f) continue;
    uint4* const q = reinterpret_cast<uint4*>(p) + idx;
    const uint4 v = *q;
    *q = make_uint4(pack_bf16x2(bf16_lo(v.x) * a0.x, bf16_hi(v.x) * a0.y), pack_bf16x2(bf16_lo(v.y) * a0.z, bf16_hi(v.y) * a0.w),
                    pack_bf16x2(bf16_lo(v.z) * a1.x, bf16_hi(v.z) * a1.y), pack_bf16x2(bf16_lo(v.w) * a1.z, bf16_hi(v.w) * a1.w));
  }
}

// Behind the flag, in one launch: the chunk's probabilities from its fp32 logits, and the rescale of the rows of acc and of the
// probabilities stored before the chunk (p_all, `rows` of them).  Blocks [0, np) probabilities, [np, np + nr) acc, then p_all.
__global__ void __launch_bounds__(256) ce_chunk_apply_kernel(const float* __restrict__ z, int vc, int T, const float* __restrict__ m,
                                                             bf16* p, float2* __restrict__ part, const float* __restrict__ alpha,
                                                             float* __restrict__ acc, int h, bf16* p_all, long rows, int bx_prob, int np,
                                                             int nr, const int* __restrict__ run_flag) {
  if (*run_flag == 0) return;
  const int b = (int)blockIdx.x;
  if (b < np) chunk_prob(b % bx_prob, b / bx_prob, z, vc, T, m, p, part);
  else if (b < np + nr) rescale_rows(b - np, nr, acc, alpha, T, h);
  else rescale_p(b - np - nr, (int)gridDim.x - np - nr, p_all, rows, T, alpha);
}

// p[y_t, t] -= l_t for every token whose label takes part in the loss (coef != 0) and lies inside the vocabulary (one
// element per token, all in different columns: no two threads touch the same one), and
// xs[t, :] = xf[t, :] * coef[t] / l[t]  (bf16; zero rows for ignored tokens).  One wave per token.
__global__ void __launch_bounds__(256) ce_patch_scale_kernel(bf16* __restrict__ p, int T, int V, const int* __restrict__ labels,
                                                             const float* __restrict__ l, const float* __restrict__ coef,
                                                             const bf16* __restrict__ xf, bf16* __restrict__ xs, int h) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  const float lt = l[t], s = coef[t] == 0.f ? 0.f : coef[t] / lt;
  const int y = labels[t];
  if (lane == 0 && coef[t] != 0.f && y >= 0 && y < V) {
    bf16* const e = p + (long)y * T + t;
    *e = (bf16)((float)*e - lt);
  }
  const uint4* src = reinterpret_cast<const uint4*>(xf + (long)t * h);
  uint4* dst = reinterpret_cast<uint4*>(xs + (long)t * h);
  for (int c = lane; c < h / 8; c += 64) {
    const uint4 v = src[c];
    dst[c] = make_uint4(pack_bf16x2(bf16_lo(v.x) * s, bf16_hi(v.x) * s), pack_bf16x2(bf16_lo(v.y) * s, bf16_hi(v.y) * s),
                        pack_bf16x2(bf16_lo(v.z) * s, bf16_hi(v.z) * s), pack_bf16x2(bf16_lo(v.w) * s, bf16_hi(v.w) * s));
  }
}

}  // namespace

hipError_t k_ce_ref_init(hipStream_t st, const float* z, int rows, int T, float* m, float* l, float* alpha, float* zlab, int* flags, int nflags) {
  if (T == 0) return hipSuccess;
  if (nflags > 1024) return hipErrorInvalidValue;
  RP_LAUNCH(ce_ref_init_kernel, dim3((T + 63) / 64), dim3(1024), 0, st, z, rows, T, m, l, alpha, zlab, flags, nflags);
  return hipGetLastError();
}

hipError_t k_ce_chunk_stats(hipStream_t st, const float2* part, int nparts, int T, const float* m, float* l_in, float* l_out, int* flag,
                            const CeSums& prev) {
  if (T == 0) return hipSuccess;
  RP_LAUNCH(ce_chunk_stats_kernel, dim3((T + 63) / 64), dim3(1024), 0, st, part, nparts, T, m, l_in, l_out, flag, prev);
  return hipGetLastError();
}

hipError_t k_ce_chunk_redo(hipStream_t st, const float* z, int vc, int T, float2* pmax, int nparts, float* m, const float* l_in, float* l_out,
                           float* alpha, void* p, float* acc, int h, void* p_all, long rows, const int* flag, CeSums* sums) {
  *sums = CeSums{pmax, (vc + CE_PROB_ROWS - 1) / CE_PROB_ROWS, flag};
  if (T == 0 || vc == 0) return hipSuccess;
  const int nblk = (vc + CE_PROB_ROWS - 1) / CE_PROB_ROWS;
  if (T % 8 || (acc && h % 4) || nblk > nparts) return hipErrorInvalidValue;   // one partial row per CE_PROB_ROWS vocabulary rows
  const int bx = (T / 4 + 255) / 256, nr = !acc ? 0 : (T + 3) / 4 < 256 ? (T + 3) / 4 : 256, nq = p_all && rows > 0 ? 512 : 0;
  RP_LAUNCH(ce_chunk_ref_kernel, dim3((T + 255) / 256), dim3(256), 0, st, (const float2*)pmax, nparts, T, m, l_in, l_out, alpha, flag);
  RP_LAUNCH(ce_chunk_apply_kernel, dim3(bx * nblk + nr + nq), dim3(256), 0, st, z, vc, T, (const float*)m, (bf16*)p, pmax, (const float*)alpha,
            acc, h, (bf16*)p_all, rows, bx, bx * nblk, nr, flag);
  return hipGetLastError();
}

hipError_t k_ce_patch_scale(hipStream_t st, void* p, int T, int V, const int* labels, const float* l, const float* coef, const void* xf,
                            void* xs, int h) {
  if (T == 0) return hipSuccess;
  if (h % 8) return hipErrorInvalidValue;
  RP_LAUNCH(ce_patch_scale_kernel, dim3((T + 3) / 4), dim3(256), 0, st, (bf16*)p, T, V, labels, l, coef, (const bf16*)xf, (bf16*)xs, h);
  return hipGetLastError();
}

hipError_t k_ce_lse(hipStream_t st, const float2* part, int P, long part_ld, float* lse, int T) {
  if (T == 0) return hipSuccess;
  RP_LAUNCH(ce_lse_kernel, dim3((T + 15) / 16), dim3(1024), 0, st, part, P, part_ld, lse, T);
  return hipGetLastError();
}

hipError_t k_ce_finalize(hipStream_t st, const float* lse, float* l, const float* zlab, const int* labels, float grad_scale,
                         float* coef, float* loss_out, int T, const CeSums& last) {
  RP_LAUNCH(ce_finalize_kernel, dim3(1), dim3(1024), 0, st, lse, l, zlab, labels, grad_scale, coef, loss_out, T, last);
  return hipGetLastError();
}
