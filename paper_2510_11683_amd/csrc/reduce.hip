// Row and response reductions of the ELBO head:
//   log-sum-exp       combine the per-vocabulary-tile (max, sum) partials
//   per-response      l = (1/t) sum log p (Eq. per_step_loss), d, g (Eq. g),
//                     loss (Algorithm 1, L_j = -g_j/G) and the gradient scale
//   stored backward   per-row factors of the kept exponentials, their target
//                     entries (the one-hot term), H_c^T scaled by the
//                     factors, and rows outside the exponent range recomputed
//   dX                sum of the split-vocabulary partials, scattered to the
//                     masked positions
// Every reduction runs in a fixed order, so results are bit-reproducible.
#include "common.hpp"
#include "internal.hpp"

namespace bgpo {

// log-sum-exp of every row from its per-slice (max, sum) partials, and the
// target's log p.  64 rows per workgroup, one per lane, so each load of a
// slice's partials is 64 consecutive floats; the 16 waves take every 16th
// slice, 8 slices' loads in flight at a time, and are combined in LDS in a
// fixed order.
constexpr int kCombineWaves = 16;

// Whether a row's exponentials against R2 = exp_reference(z_y) may have left
// the exponent range (true for NaN).
__device__ __forceinline__ bool out_of_range(float lse2, float ztgt) {
  return !(lse2 - exp_reference(ztgt) <= kExpRange);
}

__global__ __launch_bounds__(64 * kCombineWaves) void k_combine_rows(
    const float* __restrict__ part_m, const float* __restrict__ part_s,
    const float* __restrict__ ztgt, const SampleMeta* __restrict__ meta,
    float* __restrict__ lse2, float* __restrict__ lp, uint64_t* __restrict__ row_bad, int nvt,
    int64_t ldp) {
  __shared__ float sm[kCombineWaves][64], ss[kCombineWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int row = blockIdx.x * 64 + lane;
  const int n_rows = meta->n_rows;
  if (blockIdx.x * 64 >= n_rows) return;
  float m = -INFINITY, sum = 0.f;
  if (row < n_rows) {
    for (int t0 = q; t0 < nvt; t0 += kCombineWaves * 8) {
      float mt[8], st[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int t = t0 + kCombineWaves * k;
        mt[k] = t < nvt ? part_m[(int64_t)t * ldp + row] : -INFINITY;
        st[k] = t < nvt ? part_s[(int64_t)t * ldp + row] : 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (st[k] > 0.f) {
          const float mn = fmaxf(m, mt[k]);
          sum = sum * exp2f(m - mn) + st[k] * exp2f(mt[k] - mn);
          m = mn;
        }
      }
    }
  }
  sm[q][lane] = m;
  ss[q][lane] = sum;
  __syncthreads();
  if (q == 0 && row < n_rows) {
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < kCombineWaves; ++k) M = fmaxf(M, sm[k][lane]);
    float S = 0.f;
#pragma unroll
    for (int k = 0; k < kCombineWaves; ++k)
      if (ss[k][lane] > 0.f) S += ss[k][lane] * exp2f(sm[k][lane] - M);
    const float l2 = M + log2f(S), zt = ztgt[row];
    lse2[row] = l2;
    lp[row] = zt - l2 * kLn2;
    if (row_bad) {
      const uint64_t bad = __ballot(out_of_range(l2, zt));   // (row 64 blockIdx.x is valid)
      if (lane == 0) row_bad[blockIdx.x] = bad;
    }
  }
}

hipError_t launch_combine_rows(const Workspace& ws, int V, bool mark, hipStream_t s) {
  k_combine_rows<<<(unsigned)(ws.g_used * ws.NP / 64), 64 * kCombineWaves, 0, s>>>(
      ws.part_m, ws.part_s, ws.ztgt, ws.unit(), ws.lse2, ws.lp, mark ? ws.row_bad : nullptr,
      (int)ws.nvt, ws.RP);
  return hipGetLastError();
}

// The objective's per-sample term g and its derivative dg/dl for
// d = l - l_old:
//   paper (Eq. g):  first-order Taylor bound (1 + d) A / n_t for A >= 0
//                   (Lemma 1), Jensen bound e^d A / n_t for A < 0 (Lemma 2)
//   Taylor only / Jensen only: one of the two for every sign (the ablation of
//                   Table 3)
//   exact:          exp(dbar) A / n_t with dbar the mean of d over all n_t
//                   samples, whose sum is exp(B_theta - B_old) A
//                   (Eq. elbo_ratio); dg/dl_j = exp(dbar) A / n_t
__device__ __forceinline__ void bound_term(double dj, double A, int n_t, int bound, double dbar,
                                           double* gj, double* dg) {
  if (bound == 3) {
    *gj = exp(dbar) * A / n_t;
    *dg = *gj;
  } else if (bound == 1 || (bound == 0 && A >= 0.0)) {
    *gj = (1.0 + dj) * A / n_t;
    *dg = A / n_t;
  } else {
    *gj = exp(dj) * A / n_t;
    *dg = *gj;
  }
}

// Per-response terms of the samples of a unit, one wave per (sample, response)
// segment.  Sample g of the unit is sample j0 + g; its response b has rows
// [seg_off[g (B+1) + b], seg_off[g (B+1) + b + 1]) and timestep t24[g B + b].
// The gradient scale of (g, b) goes to seq_scale[g B + b]; the loss and the
// rows' scales follow from g and seq_scale in the next kernel, when every
// segment is done.
__global__ __launch_bounds__(256) void k_seq_terms(
    const float* __restrict__ lp, const int32_t* __restrict__ seg_off,
    const uint32_t* __restrict__ t24, int B, int n_t, int j0, int n_samples,
    const float* __restrict__ adv, const double* __restrict__ ell_old, double loss_scale,
    double* __restrict__ ell, double* __restrict__ g, int32_t* __restrict__ flags,
    float* __restrict__ seq_scale, int backward, int bound, const double* __restrict__ dbar) {
  const int lane = threadIdx.x & 63, sg = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (sg >= n_samples * B) return;
  const int gs = sg / B, b = sg - gs * B, j = j0 + gs;
  const int r0 = seg_off[gs * (B + 1) + b], r1 = seg_off[gs * (B + 1) + b + 1];
  double acc = 0.0;
#pragma unroll 4
  for (int r = r0 + lane; r < r1; r += 64) acc += (double)lp[r];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane) return;
  const double t = (double)t24[sg] * (1.0 / 16777216.0);
  const double l = acc / t;                                        // Eq. per_step_loss
  const int64_t o = (int64_t)b * n_t + j;
  ell[o] = l;
  bool bad = !isfinite(l);
  if (backward) {
    const double dj = ell_old ? l - ell_old[o] : 0.0;
    double gj, dg;
    bound_term(dj, (double)adv[b], n_t, bound, dbar ? dbar[b] : 0.0, &gj, &dg);
    g[o] = gj;
    const double sc = loss_scale * dg / t;
    seq_scale[sg] = (float)sc;
    bad = bad || !isfinite(gj) || !isfinite(sc) || !isfinite((float)sc);
  }
  if (bad && flags) atomicOr(flags, kFlagNonfinite);
}

hipError_t launch_seq_terms(const Workspace& ws, int B, int n_t, int j0, const float* adv,
                            const double* ell_old, double loss_scale, double* ell, double* g,
                            int32_t* flags, bool backward, int bound, const double* dbar,
                            hipStream_t s) {
  k_seq_terms<<<(unsigned)((ws.g_used * B + 3) / 4), 256, 0, s>>>(
      ws.lp, ws.seg_off, ws.t24, B, n_t, j0, ws.g_used, adv, ell_old, loss_scale, ell, g, flags,
      ws.seq_scale, backward ? 1 : 0, bound, dbar);
  return hipGetLastError();
}

// dbar[b] = (1/n_t) sum_j (l[b][j] - l_old[b][j]), samples in order: the
// log-ratio B_theta - B_old of Eq. elbo_ratio with both ELBOs estimated on the
// same n_t masked samples.
__global__ __launch_bounds__(256) void k_mean_ratio(const double* __restrict__ ell,
                                                    const double* __restrict__ ell_old, int B,
                                                    int n_t, double* __restrict__ dbar) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  double acc = 0.0;
  for (int j = 0; j < n_t; ++j) acc += ell[(int64_t)b * n_t + j] - ell_old[(int64_t)b * n_t + j];
  dbar[b] = acc / n_t;
}

hipError_t launch_mean_ratio(const double* ell, const double* ell_old, int B, int n_t,
                             double* dbar, hipStream_t s) {
  k_mean_ratio<<<(unsigned)((B + 255) / 256), 256, 0, s>>>(ell, ell_old, B, n_t, dbar);
  return hipGetLastError();
}

// Once the unit's scales s are known: the loss, and per row what the backward
// needs.  Recompute mode: the row's scale (0 for padding), which the chunk's
// GEMM epilogue applies.  Stored mode: the forward kept
// u = 2^(z log2e - R2) (bf16) in dZ (the unit's rows from its col_off, ldz
// rows per slab), with R2 = exp_reference(z_y)
// per row; since p = u 2^(R2 - lse2),
//     dZ = s (p - onehot) = f (u - onehot 2^(lse2 - R2)),  f = s 2^(R2 - lse2)
// (differentiating Eq. per_step_loss, d l / d z = (onehot - p) / t; s carries
// -loss_scale dg/dl and the 1/t).  f (0 for padding) scales the dX rows in the
// reduction and H_c^T's columns for the dW GEMM, and the target entry becomes
// (p_y - 1) 2^(lse2 - R2), p_y from the fp32 target logit.  A row with
// lse2 - R2 > kExpRange (its target log2-probability below
// -(kExpRef + kExpRange)) was marked with the log-sum-exp: its exponentials may
// have left the range of bf16 and of the fp32 accumulators, so it is
// recomputed against R2 = lse2 (f = s), from fp32 dot products.
//
// One launch whose workgroups take one of these roles each; none reads what
// another writes (every role forms f or the marks from lse2 and the target
// logit for itself), so they run side by side.  Bound by latency and, in the
// H_c^T role, by HBM.  With the target logits in the gather's launch and one
// wave per segment in k_seq_terms, against five launches: a step of B2 L64 d128
// V1024 n_t 4 62.5 -> 55.6 us, of B3 L201 d576 V4288 n_t 6 113.5 -> 106.9 us.
struct RowTerms {
  const float *lse2, *ztgt, *seq_scale;
  const int32_t *row_tgt, *row_seq;
  const uint64_t* row_bad;
  const SampleMeta* meta;
  uint16_t *dZ, *HcT;
  const uint16_t *Hc, *WT;
  float *row_f, *row_scale;
  int64_t ldz, RP;
  int d, V;
  // the loss: g of samples j0 .. j0 + n_samples - 1
  const double* g;
  double* loss;
  double loss_scale;
  int B, n_t, j0, n_samples;
  int n_rows_wg, n_hct_wg;    // workgroups of the row and H_c^T roles

  __device__ float scale(int r) const { return seq_scale[row_seq[r]]; }
  // f of row r < n_rows
  __device__ float factor(int r) const {
    const float l2 = lse2[r], zt = ztgt[r];
    return scale(r) *
           __builtin_amdgcn_exp2f((out_of_range(l2, zt) ? l2 : exp_reference(zt)) - l2);
  }
};

// loss += the unit's terms, summed in sample-then-response order (one wave:
// 64 terms per load, added one after the other)
__device__ void add_loss(const RowTerms& p) {
  const int lane = threadIdx.x;
  const int n = p.n_samples * p.B;
  double acc = 0.0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + lane;
    double v = 0.0;
    if (i < n) v = -p.loss_scale * p.g[(int64_t)(i % p.B) * p.n_t + p.j0 + i / p.B];
    const int m = min(64, n - i0);
    for (int q = 0; q < m; ++q) acc += __shfl(v, q, 64);
  }
  if (lane == 0) p.loss[0] += acc;
}

// the row role: f and the target entry (stored), or the scale (recompute)
template <bool STORED>
__device__ void row_role(const RowTerms& p, int r) {
  if (r >= p.meta->n_rows_pad) return;
  const bool live = r < p.meta->n_rows;
  if constexpr (!STORED) {
    p.row_scale[r] = live ? p.scale(r) : 0.f;
  } else {
    p.row_f[r] = live ? p.factor(r) : 0.f;
    const float l2 = live ? p.lse2[r] : 0.f, zt = live ? p.ztgt[r] : 0.f;
    if (live && !out_of_range(l2, zt)) {   // (a marked row's target entry is recomputed too)
      const float val = (__builtin_amdgcn_exp2f(zt * kLog2e - l2) - 1.f) *
                        __builtin_amdgcn_exp2f(l2 - exp_reference(zt));
      const uint16_t b = (uint16_t)(pack_bf16x2(val, 0.f) & 0xFFFFu);
      p.dZ[slab_index(p.ldz, (int64_t)p.meta->col_off + r, p.row_tgt[r])] = b;
    }
  }
}

// the H_c^T role: H_c^T[c][col_off + r] *= f_r (bf16, nearest even) over the
// unit's columns up to col_end (its rows rounded up to 64), not its 256-row
// padding: the next unit of the dW batch starts at col_end, and with every
// sample retained its columns already hold its rows when this runs.  One
// workgroup per 64 rows and up to kHctCols hidden units; a 64 x 64 tile is
// 8 KB of the slab-major H_c^T.
constexpr int kHctCols = 512;

__device__ void hct_role(const RowTerms& p, int wg, float (&s_f)[64]) {
  const int cgroups = (p.d + kHctCols - 1) / kHctCols;
  const int r0 = wg / cgroups * 64, c0 = wg % cgroups * kHctCols;
  if (r0 >= p.meta->col_end - p.meta->col_off) return;
  const int tid = threadIdx.x, cc = tid & 7;
  if (tid < 64) s_f[tid] = r0 + tid < p.meta->n_rows ? p.factor(r0 + tid) : 0.f;
  __syncthreads();
  float fr[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) fr[e] = s_f[cc * 8 + e];
  uint16_t* base = p.HcT + slab_index(p.d, 0, (int64_t)p.meta->col_off + r0);
  const int c1 = min(p.d, c0 + kHctCols);
#pragma unroll 4
  for (int c = c0 + (tid >> 3); c < c1; c += 32) {
    uint4* q = reinterpret_cast<uint4*>(base + (int64_t)c * 64 + cc * 8);
    const uint4 v = *q;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = pack_bf16x2(__uint_as_float(w[e] << 16) * fr[2 * e],
                         __uint_as_float(w[e] & 0xFFFF0000u) * fr[2 * e + 1]);
    *q = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// the role of the marked rows, recomputed against R2 = lse2:
// u = 2^(z log2e - lse2) = p, and p_y - 1 at the target.  One thread per
// vocabulary id; the workgroup looks for a nonzero mark word, then scans the
// unit's marks 256 rows at a time and takes the marked ones in batches of 16,
// whose fp32 logits z = H_c[row] . W^T[v] it accumulates in a fixed order over
// d.  Without marked rows it only reads the mark words.
constexpr int kFixBatch = 16;

struct FixShared {
  int list[256];
  int cnt;
  float h[kFixBatch][64];
};

__device__ void fixup_role(const RowTerms& p, int wg, FixShared& sh) {
  const int tid = threadIdx.x;
  const int v = wg * 256 + tid;
  const int N = p.meta->n_rows;
  const int64_t col_off = p.meta->col_off;
  int any = 0;
  for (int i = tid; i * 64 < N; i += 256) any |= p.row_bad[i] != 0;
  if (!__syncthreads_or(any)) return;
  for (int base = 0; base < N; base += 256) {
    if (tid == 0) sh.cnt = 0;
    __syncthreads();
    const int rr = base + tid;
    if (rr < N && (p.row_bad[rr >> 6] >> (rr & 63)) & 1) sh.list[atomicAdd(&sh.cnt, 1)] = rr;
    __syncthreads();
    const int cnt = sh.cnt;
    for (int b0 = 0; b0 < cnt; b0 += kFixBatch) {
      const int nb = min(kFixBatch, cnt - b0);
      float acc[kFixBatch];
#pragma unroll
      for (int i = 0; i < kFixBatch; ++i) acc[i] = 0.f;
      for (int kc = 0; kc < p.d; kc += 64) {
        __syncthreads();
        for (int q = tid; q < kFixBatch * 64; q += 256) {
          const int i = q >> 6, k = q & 63;
          sh.h[i][k] = i < nb ? __uint_as_float(
                                    (uint32_t)p.Hc[slab_index(p.RP, sh.list[b0 + i], kc + k)] << 16)
                              : 0.f;
        }
        __syncthreads();
        if (v < p.V) {
          const uint16_t* w = p.WT + (int64_t)v * p.d + kc;
          for (int kk = 0; kk < 64; kk += 8) {
            const uint4 wv = *reinterpret_cast<const uint4*>(w + kk);
            const uint32_t ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float w0 = __uint_as_float(ww[e] << 16), w1 = __uint_as_float(ww[e] & 0xFFFF0000u);
#pragma unroll
              for (int i = 0; i < kFixBatch; ++i)
                acc[i] = fmaf(w1, sh.h[i][kk + 2 * e + 1], fmaf(w0, sh.h[i][kk + 2 * e], acc[i]));
            }
          }
        }
      }
      if (v < p.V) {
#pragma unroll
        for (int i = 0; i < kFixBatch; ++i) {
          if (i >= nb) break;
          const int r = sh.list[b0 + i];
          const float l2 = p.lse2[r];
          const float val = v == p.row_tgt[r]
                                ? __builtin_amdgcn_exp2f(fmaf(p.ztgt[r], kLog2e, -l2)) - 1.f
                                : __builtin_amdgcn_exp2f(fmaf(acc[i], kLog2e, -l2));
          const uint16_t b = (uint16_t)(pack_bf16x2(val, 0.f) & 0xFFFFu);
          p.dZ[slab_index(p.ldz, col_off + r, v)] = b;
        }
      }
    }
    __syncthreads();   // the list is rewritten for the next rows
  }
}

// workgroup 0: the loss; then the row role, the H_c^T role, the marked rows
template <bool STORED>
__global__ __launch_bounds__(256) void k_row_terms(RowTerms p) {
  __shared__ union {
    float f[64];
    FixShared fix;
  } sh;
  int wg = blockIdx.x;
  if (wg == 0) {
    if (threadIdx.x < 64) add_loss(p);
    return;
  }
  wg -= 1;
  if (wg < p.n_rows_wg) {
    row_role<STORED>(p, wg * 256 + threadIdx.x);
    return;
  }
  if constexpr (STORED) {
    wg -= p.n_rows_wg;
    if (wg < p.n_hct_wg)
      hct_role(p, wg, sh.f);
    else
      fixup_role(p, wg - p.n_hct_wg, sh.fix);
  }
}

hipError_t launch_row_terms(const Workspace& ws, int B, int n_t, int j0, double loss_scale,
                            const double* g, double* loss, int d, int V, hipStream_t s) {
  const int64_t rows = ws.g_used * ws.NP;
  RowTerms p{ws.lse2, ws.ztgt, ws.seq_scale, ws.row_tgt, ws.row_seq, ws.row_bad,
             ws.unit(), ws.dZ, ws.HcT, ws.Hc, ws.WT, ws.row_f, ws.row_scale, ws.ldz, ws.RP, d, V,
             g, loss, loss_scale, B, n_t, j0, ws.g_used, (int)(rows / 256), 0};
  if (ws.chunk) {
    k_row_terms<false><<<(unsigned)(1 + p.n_rows_wg), 256, 0, s>>>(p);
  } else {
    p.n_hct_wg = (int)(rows / 64 * ((d + kHctCols - 1) / kHctCols));
    const unsigned wgs = (unsigned)(1 + p.n_rows_wg + p.n_hct_wg + (V + 255) / 256);
    k_row_terms<true><<<wgs, 256, 0, s>>>(p);
  }
  return hipGetLastError();
}

// The rows of a unit that add into one dX row, in sample order.  Shared head
// input (SHARED): target t is position t, whose row in sample g is
// inv[g P + t] (negative: not masked there); the samples' rows are added one
// after the other, as if each sample were reduced alone.  Per-sample head
// inputs: target t is unit row t, alone, at its sample's own dX; with a stride
// below B L d the samples' dX overlap, and they run one after the other
// (`only`: the sample of this launch, else -1).
struct DxTarget {
  const int32_t* inv;       // [G, P]
  const int32_t* idx;       // [RP]  position of a unit row
  const int32_t* row_seq;   // [RP]  g*B + b of a unit row
  int n_samples, B, only;
  int64_t P, stride, d;
  // element offset of the target's dX row (and head input row)
  template <bool SHARED>
  __device__ int64_t offset(int t) const {
    return SHARED ? (int64_t)t * d : (int64_t)(row_seq[t] / B) * stride + (int64_t)idx[t] * d;
  }
  template <bool SHARED>
  __device__ bool none(int t, const SampleMeta* um) const {
    return !SHARED && (t >= um->n_rows || (only >= 0 && row_seq[t] / B != only));
  }
  template <bool SHARED>
  __device__ int row(int g, int t) const {
    return SHARED ? inv[(int64_t)g * P + t] : t;
  }
};

// sum_s part[s][r][c .. c + 3], splits in order
__device__ __forceinline__ float4 split_sum(const float* __restrict__ part, int n_split,
                                            int64_t split_stride) {
  float4 acc = *reinterpret_cast<const float4*>(part);
#pragma unroll 4
  for (int s = 1; s < n_split; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(part + s * split_stride);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  return acc;
}

// dX[t, :] += f_r sum_s part[s][r][:] over the rows r of target t (f_r the
// stored backward's row factor, 1 without one), float4 per thread.  One launch
// per unit: bound by HBM, the partials are read once and a dX row is read and
// written once per unit instead of once per sample (B8 L512 d4096, a unit of 8
// samples with 15.2k rows in 4 splits: 191 us in one launch per sample -> 132).
template <bool SHARED>
__global__ __launch_bounds__(256) void k_dx_reduce(const float* __restrict__ part, DxTarget tg,
                                                   const SampleMeta* __restrict__ um,
                                                   const float* __restrict__ rowf,
                                                   float* __restrict__ dX, int d,
                                                   int64_t split_stride) {
  const int t = blockIdx.x;
  if (tg.none<SHARED>(t, um)) return;
  const int c = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (c >= d) return;
  const int n_split = um->dx_split;
  float4* dst = reinterpret_cast<float4*>(dX + tg.offset<SHARED>(t) + c);
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  bool any = false;
  const int n = SHARED ? tg.n_samples : 1;
  for (int g = 0; g < n; ++g) {
    const int r = tg.row<SHARED>(g, t);
    if (r < 0) continue;
    float4 acc = split_sum(part + (int64_t)r * d + c, n_split, split_stride);
    if (rowf) {
      const float f = rowf[r];
      acc.x *= f; acc.y *= f; acc.z *= f; acc.w *= f;
    }
    if (!any) o = *dst;
    any = true;
    o.x += acc.x; o.y += acc.y; o.z += acc.z; o.w += acc.w;
  }
  if (any) *dst = o;
}

static DxTarget dx_target(const Workspace& ws, int B, int d, int64_t stride) {
  return DxTarget{ws.inv, ws.idx, ws.row_seq, ws.g_used, B, -1, ws.P, stride, d};
}

// launches `run` once for the unit, or once per sample where the samples' dX
// overlap; the number of launches
template <typename F>
static int for_disjoint(DxTarget tg, F run) {
  if (tg.stride == 0 || tg.stride >= tg.P * tg.d) {
    run(tg);
    return 1;
  }
  for (tg.only = 0; tg.only < tg.n_samples; ++tg.only) run(tg);
  return tg.n_samples;
}

hipError_t launch_dx_reduce(const Workspace& ws, int B, float* dX, int64_t stride, int d,
                            hipStream_t s, int* launches) {
  const float* rowf = ws.chunk ? nullptr : ws.row_f;
  const unsigned cols = (unsigned)((d / 4 + 255) / 256);
  *launches += for_disjoint(dx_target(ws, B, d, stride), [&](const DxTarget& tg) {
    if (stride == 0)
      k_dx_reduce<true><<<dim3((unsigned)ws.P, cols), 256, 0, s>>>(ws.dx_part, tg, ws.unit(), rowf,
                                                                   dX, d, ws.RP * d);
    else
      k_dx_reduce<false><<<dim3((unsigned)(ws.g_used * ws.NP), cols), 256, 0, s>>>(
          ws.dx_part, tg, ws.unit(), rowf, dX, d, ws.RP * d);
  });
  return hipGetLastError();
}

// Split reduction followed by the backward of the final RMSNorm
// h = gamma x r, r = (mean x^2 + eps)^(-1/2), one target (see DxTarget) per
// workgroup:
//   dh       = f_row sum_s part[s][row]               (d loss / d h; f_row the
//                                                     stored backward's row
//                                                     factor, 1 without one)
//   dx_k    += r gamma_k dh_k - (r^3 / d) x_k sum_i gamma_i dh_i x_i
//   c_k      = dh_k x_k r  -> part[0][row][k], summed over rows into dgamma
// Every thread revisits only the elements it wrote, so part[0] and dx need no
// cross-thread ordering; the row dot product goes through LDS.
template <typename T, bool SHARED>
__global__ __launch_bounds__(256) void k_dx_reduce_rmsnorm(
    float* __restrict__ part, DxTarget tg, const SampleMeta* __restrict__ um,
    const float* __restrict__ rowf, const T* __restrict__ x, const float* __restrict__ gamma,
    const float* __restrict__ inv_rms, float* __restrict__ dx, int d, int64_t split_stride) {
  __shared__ float red[2][4];
  const int t = blockIdx.x;
  if (tg.none<SHARED>(t, um)) return;
  const int n_split = um->dx_split;
  const int tid = threadIdx.x;
  const int64_t off = tg.offset<SHARED>(t);
  const T* xr = x + off;
  float* dxr = dx + off;
  const int n = SHARED ? tg.n_samples : 1;
  int set = 0;
  for (int g = 0; g < n; ++g) {
    const int r = tg.row<SHARED>(g, t);
    if (r < 0) continue;                    // the same for the whole workgroup
    const float f = rowf ? rowf[r] : 1.f;   // the stored backward's row factor
    float* p0 = part + (int64_t)r * d;
    float dot = 0.f;
    for (int c = tid * 4; c < d; c += 1024) {
      float4 acc = split_sum(p0 + c, n_split, split_stride);
      acc.x *= f; acc.y *= f; acc.z *= f; acc.w *= f;
      *reinterpret_cast<float4*>(p0 + c) = acc;
      const uint2 xv = load_bf16x4(xr + c);
      const float4 gm = *reinterpret_cast<const float4*>(gamma + c);
      dot = fmaf(gm.x * acc.x, __uint_as_float(xv.x << 16), dot);
      dot = fmaf(gm.y * acc.y, __uint_as_float(xv.x & 0xFFFF0000u), dot);
      dot = fmaf(gm.z * acc.z, __uint_as_float(xv.y << 16), dot);
      dot = fmaf(gm.w * acc.w, __uint_as_float(xv.y & 0xFFFF0000u), dot);
    }
#pragma unroll
    for (int off2 = 32; off2 > 0; off2 >>= 1) dot += __shfl_xor(dot, off2, 64);
    set ^= 1;   // two sets: a set is rewritten one barrier after its last read
    if ((tid & 63) == 0) red[set][tid >> 6] = dot;
    __syncthreads();
    dot = red[set][0] + red[set][1] + red[set][2] + red[set][3];
    const float ir = inv_rms[r];
    const float cx = ir * ir * ir * dot / (float)d;
    for (int c = tid * 4; c < d; c += 1024) {
      const float4 dh = *reinterpret_cast<const float4*>(p0 + c);
      const uint2 xv = load_bf16x4(xr + c);
      const float4 gm = *reinterpret_cast<const float4*>(gamma + c);
      const float x0 = __uint_as_float(xv.x << 16), x1 = __uint_as_float(xv.x & 0xFFFF0000u);
      const float x2 = __uint_as_float(xv.y << 16), x3 = __uint_as_float(xv.y & 0xFFFF0000u);
      float4 o = *reinterpret_cast<float4*>(dxr + c);
      o.x += ir * gm.x * dh.x - cx * x0;
      o.y += ir * gm.y * dh.y - cx * x1;
      o.z += ir * gm.z * dh.z - cx * x2;
      o.w += ir * gm.w * dh.w - cx * x3;
      *reinterpret_cast<float4*>(dxr + c) = o;
      *reinterpret_cast<float4*>(p0 + c) =
          make_float4(dh.x * x0 * ir, dh.y * x1 * ir, dh.z * x2 * ir, dh.w * x3 * ir);
    }
  }
}

// dgamma[k] += sum over the unit's rows of part[0][row][k], in a fixed order:
// partial sums over chunks of kGammaRows rows (four groups of rows per
// workgroup, 256 columns), then the chunks in order.  Bound by HBM in the
// first pass (2.4k rows of 4096: 82 us with one column per thread and chunks
// of 256 rows -> 13 us for the two).
__global__ __launch_bounds__(256) void k_dgamma_partial(const float* __restrict__ part,
                                                        const SampleMeta* __restrict__ um,
                                                        float* __restrict__ gpart, int d) {
  __shared__ float4 red[3][64];
  const int n_rows = um->n_rows;
  const int r0 = blockIdx.y * kGammaRows;
  if (r0 >= n_rows) return;
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int k = blockIdx.x * 256 + lane * 4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (k < d) {
    const int ra = r0 + q * (kGammaRows / 4), rb = min(n_rows, ra + kGammaRows / 4);
#pragma unroll 8
    for (int r = ra; r < rb; ++r) {
      const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)r * d + k);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
  }
  if (q) red[q - 1][lane] = acc;
  __syncthreads();
  if (q || k >= d) return;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float4 v = red[i][lane];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  *reinterpret_cast<float4*>(gpart + (int64_t)blockIdx.y * d + k) = acc;
}

__global__ __launch_bounds__(64) void k_dgamma_final(const float* __restrict__ gpart,
                                                     const SampleMeta* __restrict__ um,
                                                     float* __restrict__ dgamma, int d) {
  const int k = blockIdx.x * 64 + threadIdx.x;
  if (k >= d) return;
  const int chunks = (um->n_rows + kGammaRows - 1) / kGammaRows;
  float acc = 0.f;
#pragma unroll 16
  for (int c = 0; c < chunks; ++c) acc += gpart[(int64_t)c * d + k];
  dgamma[k] += acc;
}

template <typename T, bool SHARED>
static int dx_reduce_rmsnorm(const Workspace& ws, int B, const void* x, const float* gamma,
                             float* dx, int64_t stride, int d, hipStream_t s) {
  return for_disjoint(dx_target(ws, B, d, stride), [&](const DxTarget& tg) {
    k_dx_reduce_rmsnorm<T, SHARED><<<(unsigned)(SHARED ? ws.P : ws.g_used * ws.NP), 256, 0, s>>>(
        ws.dx_part, tg, ws.unit(), ws.chunk ? nullptr : ws.row_f, static_cast<const T*>(x), gamma,
        ws.inv_rms, dx, d, ws.RP * d);
  });
}

hipError_t launch_dx_reduce_rmsnorm(const Workspace& ws, int B, const void* x, bool f32,
                                    const float* gamma, float* dx, int64_t stride, float* dgamma,
                                    int d, hipStream_t s, int* launches) {
  const auto reduce = f32 ? (stride ? dx_reduce_rmsnorm<float, false> : dx_reduce_rmsnorm<float, true>)
                          : (stride ? dx_reduce_rmsnorm<uint16_t, false> : dx_reduce_rmsnorm<uint16_t, true>);
  *launches += 2 + reduce(ws, B, x, gamma, dx, stride, d, s);   // (dgamma takes two)
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 g1((unsigned)((d + 255) / 256),
                (unsigned)((ws.g_used * ws.NP + kGammaRows - 1) / kGammaRows));
  k_dgamma_partial<<<g1, 256, 0, s>>>(ws.dx_part, ws.unit(), ws.gpart, d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_dgamma_final<<<(unsigned)((d + 63) / 64), 64, 0, s>>>(ws.gpart, ws.unit(), dgamma, d);
  return hipGetLastError();
}

}  // namespace bgpo
