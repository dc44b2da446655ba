// Timestep draw, Bernoulli(t) masking, stable stream compaction of the masked
// positions, gather of the masked hidden rows, and the one-off W_head
// transpose.
//
// The forward masking process (Section 2.1) masks every response token
// independently with probability t; the ELBO term (Eq. per_step_loss) only
// touches masked positions, so the rows that reach the LM-head GEMMs are the
// masked ones, compacted in ascending flat order b*L + i.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace bgpo {

constexpr int kMaskThreads = 1024;
constexpr int kMaxB = 4096;
// the single-workgroup mask kernel takes problems up to this many positions;
// larger ones go through the multi-block passes below
constexpr int64_t kSingleBlockPositions = 65536;

// Philox words for position p = b*L + i are taken from counter (i>>2, seq, j, 0);
// consecutive positions of one response share a counter block, so a thread
// caches the last block it computed.
struct MaskWalker {
  uint32_t k0, k1, seq_base;
  int L, j;
  int cached_b = -1, cached_blk = -1;
  u32x4 w;
  // the counter block of response position i of response b
  __device__ void load(int b, int i) {
    const int blk = i >> 2;
    if (blk != cached_blk || b != cached_b) {
      w = philox4x32_10(u32x4{(uint32_t)blk, seq_base + (uint32_t)b, (uint32_t)j, 0u}, k0, k1);
      cached_blk = blk;
      cached_b = b;
    }
  }
  // the Philox test of response position i of response b
  __device__ bool test(const uint32_t* sT, int b, int i) {
    load(b, i);
    return (pick_word(w, i & 3) >> 8) < sT[b];
  }
};

// Vocabulary split of the dX GEMM for a unit with row_tiles row tiles:
// the split count s minimising an estimate of the GEMM's time on the
// persistent grid, in units of one tile's 64-deep slab on one workgroup:
//   ceil(tiles / grid) rounds x (slabs per split + ~10 for the tile's
//   prologue and fp32 partial store) + pl.red / 20 per (split, row tile) for
//   the reduction of the partials (0.65 slabs of a 256-wide tile).
// A fixed split leaves most of the last round idle for some row counts
// (576 tiles on 256 workgroups use 2.25 of 3 rounds).  One wave: lane l
// estimates the split l + 1, the smallest estimate (of the smallest split)
// wins.
__device__ void choose_dx_split(int row_tiles, const DxPlan& pl, int lane, int* split, int* kslab) {
  static_assert(kMaxDxSplit <= 64, "one lane per split");
  const int sp = min(lane, pl.s_max - 1) + 1;
  // 32-bit divisions (tiles <= 16384 x 256 x 16), 64-bit cost
  const uint32_t ks = ((uint32_t)pl.kslabs + sp - 1) / sp;
  const uint32_t se = ((uint32_t)pl.kslabs + ks - 1) / ks;   // splits actually used
  const uint32_t tiles = (uint32_t)row_tiles * pl.col_tiles * se;
  const uint32_t rounds = (tiles + pl.grid - 1) / pl.grid;
  const uint64_t cost = (uint64_t)rounds * (ks + 10) * 20 + (uint64_t)pl.red * se * row_tiles;
  uint64_t best = (cost << 6) | (uint32_t)(sp - 1);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor((unsigned long long)best, off, 64);
    best = o < best ? o : best;
  }
  const int win = row_tiles > 0 ? (int)(best & 63) : 0;
  *split = row_tiles > 0 ? __shfl((int)se, win, 64) : 1;
  *kslab = row_tiles > 0 ? __shfl((int)ks, win, 64) : pl.kslabs;
}

// Pointers of a unit's row state handed to the mask kernels (all NULL but idx
// for the mask-only entry point, which writes positions to idx at row 0).
struct MaskOut {
  int32_t* idx;          // [rows]  masked flat positions, indexed by unit row
  int32_t* inv;          // [G, P]  every position's unit row (negative: not masked)
  int32_t* row_tgt;      // [rows]  target token
  int32_t* row_seq;      // [rows]  g*B + b
  int32_t* seg_off;      // [G, B+1] every sample's response offsets (unit rows)
  uint32_t* t24;         // [G, B]  every sample's timesteps
  SampleMeta* meta;      // [G]     every sample's record
  int row_cap;           // rows the unit holds (padding is written up to it)
  int max_cols;          // columns of a dW batch, 0: batches of whole units
};

// The record of a sample whose `total` masked rows follow row0 rows of its unit
// (called by one whole wave).  The unit's columns follow the prev_end columns of
// the units before it in the dW batch; with max_cols > 0, where its (padded) rows
// do not fit after them any more, it starts the next batch at column 0 and asks
// for the dW GEMM over the columns so far.
__device__ void write_record(SampleMeta* m, int row0, int prev_end, int total, int max_cols,
                             const DxPlan& plan, int lane) {
  if (!m) return;
  const int rows = row0 + total;
  const int rows_pad = (rows + kRowPad - 1) / kRowPad * kRowPad;
  const bool flush = max_cols > 0 && prev_end > max_cols - rows_pad;
  const int col0 = flush ? 0 : prev_end;
  int split, kslab;
  choose_dx_split((rows + plan.tile - 1) / plan.tile, plan, lane, &split, &kslab);
  if (lane == 0) {
    m->n_rows = rows;
    m->n_rows_pad = rows_pad;
    m->col_off = col0;
    m->col_end = col0 + (rows + 63) / 64 * 64;
    m->s_rows = total;
    m->s_row_off = row0;
    m->dx_split = split;
    m->dx_kslab = kslab;
    m->flush_cols = flush ? prev_end : 0;
  }
}

// Single-workgroup form: workgroup g handles sample j0 + g of a unit, timesteps
// in LDS, 64 positions per thread at a time (all of them in one span up to
// kSingleBlockPositions; only the mask-only entry point goes beyond), every
// thread a contiguous run
// of at most 64 positions whose mask bits stay in a register between the
// count and the output, one block-wide scan.  The first row of a sample follows
// from the mask counts of the unit's earlier samples, which every workgroup
// counts again for itself (one Philox block per four positions, the runs of
// all earlier samples spread over the threads), so that the samples of a unit
// run side by side in one launch.  Against one launch per sample: a whole step
// of 4 samples of 128 positions 117 -> 99 us, of 6 samples of 603 positions
// 192 -> 171 us.
//
// Bound by the Philox arithmetic of one compute unit and by a chain of
// latencies, so whatever does not need the timesteps is in flight before the
// barrier that publishes them (the first run's response mask, targets and
// Philox block), and the unit's record is written by the last wave while the
// others write rows: one sample of 4096 positions 7.6 -> 6.5 us, a unit of 4
// samples of 128 positions 10.8 -> 8.2, of 6 of 603 15.4 -> 11.4.
static_assert(kSingleBlockPositions <= 64 * kMaskThreads, "one span per sample in a unit");

// The response-mask bytes of positions p .. min(p + 4, p1) - 1 (p a multiple of
// 4; `words`: the mask is 4-byte aligned).
__device__ __forceinline__ uint32_t resp_word(const uint8_t* resp, int p, int p1, bool words) {
  if (words && p + 4 <= p1) return *reinterpret_cast<const uint32_t*>(resp + p);
  uint32_t r4 = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) r4 |= p + e < p1 ? (uint32_t)resp[p + e] << (8 * e) : 0u;
  return r4;
}

// The mask bits of positions p0 .. p1 - 1 (at most 64): response position i
// of response b onwards.  p0 is a multiple of 4, so that the response-mask
// bytes load four at a time; r4 holds the first four.
__device__ __forceinline__ uint64_t mask_run(MaskWalker& mw, const uint8_t* resp, bool words,
                                             const uint32_t* sT, int p0, int p1, int b, int i,
                                             uint32_t r4) {
  uint64_t bits = 0;
  for (int p = p0; p < p1; p += 4) {
    if (p > p0) r4 = resp_word(resp, p, p1, words);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (p + e < p1) {
        if (((r4 >> (8 * e)) & 255u) && mw.test(sT, b, i)) bits |= 1ull << (p - p0 + e);
        if (++i == mw.L) {
          i = 0;
          ++b;
        }
      }
    }
  }
  return bits;
}

// Inclusive sum over the lanes of a wave (data-parallel moves inside and across
// the rows of 16 lanes: no LDS round trips).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2, 3
  return v;
}

struct MaskArgs {
  const uint8_t* resp;
  const int32_t* targets;
  int B, L, n_t, j0, t_mode;
  uint32_t k0, k1, seq_base;
  MaskOut out;
  int32_t* nm_out;
  int nm_stride;
  float* t_out;
  int t_stride, V;
  const SampleMeta* prev;
  DxPlan plan;
};

template <int THREADS, int MAXB>
struct MaskShared {
  uint32_t T[MAXB];            // timesteps of MAXB / B samples at a time
  int32_t seg[MAXB + 1];
  int32_t wave[THREADS / 64], earlier[THREADS / 64];
};

// Sample j0 + g of n_samples by one workgroup of THREADS threads; B <= MAXB.
template <int THREADS, int MAXB>
__device__ __forceinline__ void mask_sample(const MaskArgs& a, int g, int n_samples,
                                            MaskShared<THREADS, MAXB>& sh) {
  constexpr int kSpan = 64 * THREADS;
  uint32_t* const sT = sh.T;
  int32_t *const sSeg = sh.seg, *const sWave = sh.wave, *const sEarlier = sh.earlier;
  const uint8_t* const resp = a.resp;
  const int32_t* const targets = a.targets;
  const int B = a.B, L = a.L, n_t = a.n_t, j0 = a.j0, t_mode = a.t_mode, V = a.V;
  const uint32_t k0 = a.k0, k1 = a.k1, seq_base = a.seq_base;
  const MaskOut& out = a.out;
  int32_t* const nm_out = a.nm_out;
  float* const t_out = a.t_out;
  const int nm_stride = a.nm_stride, t_stride = a.t_stride;
  const SampleMeta* const prev = a.prev;
  const DxPlan& plan = a.plan;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int P = B * L;
  const bool words = ((uintptr_t)resp & 3) == 0;

  // this thread's run of the first span
  int n = min(kSpan, P);
  int chunk = ((n + THREADS - 1) / THREADS + 3) & ~3;
  int p0 = min(n, tid * chunk), p1 = min(n, p0 + chunk);
  int b0 = p0 / L, i0 = p0 - b0 * L;
  uint32_t r4 = resp_word(resp, p0, p1, words);
  int32_t tgt[4] = {0, 0, 0, 0};
  const bool tgt_ahead = chunk == 4 && out.row_tgt;   // (targets of longer runs are read when written)
  if (tgt_ahead)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (p0 + e < p1) tgt[e] = targets[p0 + e];
  // the unit's columns follow the previous unit's of the dW batch
  const int prev_end = prev ? prev->col_end : 0;
  MaskWalker mw{k0, k1, seq_base, L, j0 + g};

  // counts of the unit's earlier samples, then this sample's timesteps at
  // sT + t_base
  int earlier = 0, t_base = 0;
  const int per = MAXB / B;
  const int n_runs = (n + chunk - 1) / chunk;
  for (int q0 = 0; q0 <= g; q0 += per) {
    const int nq = min(per, g + 1 - q0);
    if (q0) __syncthreads();          // the previous samples' timesteps are done with
    for (int e = tid; e < nq * B; e += THREADS) {
      const int q = e / B;
      sT[e] = timestep_t24(k0, k1, seq_base + (uint32_t)(e - q * B), j0 + q0 + q, n_t, t_mode);
    }
    if (q0 == 0 && r4) mw.load(b0, i0);
    __syncthreads();
    t_base = (nq - 1) * B;
    const int n_earlier = min(nq, g - q0);
    for (int e = tid; e < n_earlier * n_runs; e += THREADS) {
      const int q = e / n_runs, c0 = (e - q * n_runs) * chunk, c1 = min(n, c0 + chunk);
      const int b = c0 / L;
      MaskWalker me{k0, k1, seq_base, L, j0 + q0 + q};
      earlier += __popcll(mask_run(me, resp, words, sT + q * B, c0, c1, b, c0 - b * L,
                                   resp_word(resp, c0, c1, words)));
    }
  }
  earlier = wave_inclusive_sum(earlier);
  if (lane == 63) sEarlier[wave] = earlier;

  int row0 = 0, total = 0;
  for (int s0 = 0; s0 < P; s0 += kSpan) {
    if (s0) {
      n = min(kSpan, P - s0);
      chunk = ((n + THREADS - 1) / THREADS + 3) & ~3;
      p0 = s0 + min(n, tid * chunk);
      p1 = min(s0 + n, p0 + chunk);
      b0 = p0 / L;
      i0 = p0 - b0 * L;
      r4 = resp_word(resp, p0, p1, words);
    }
    const uint64_t bits = mask_run(mw, resp, words, sT + t_base, p0, p1, b0, i0, r4);
    const int cnt = __popcll(bits);
    // block-wide exclusive scan of the per-thread counts
    const int incl = wave_inclusive_sum(cnt);
    if (s0) __syncthreads();          // the previous span's wave sums are done with
    if (lane == 63) sWave[wave] = incl;
    __syncthreads();
    int base = total + incl - cnt;    // masked positions of this sample before the run
#pragma unroll
    for (int q = 0; q < THREADS / 64; ++q) {
      const int v = sWave[q];
      base += q < wave ? v : 0;
      total += v;
      row0 += s0 ? 0 : sEarlier[q];
    }
    // offsets of the responses that start in this thread's run
    for (int b = b0 + (i0 > 0); b < B && b * L < p1; ++b)
      sSeg[b] = base + __popcll(bits & ((1ull << (b * L - p0)) - 1));
    if (out.inv) {
      int32_t* const inv = out.inv + (int64_t)g * P;
      int r = row0 + base;
      for (int p = p0; p < p1; ++p) inv[p] = (bits >> (p - p0)) & 1 ? r++ : -1;
    }
    int b = b0, r = row0 + base;
    for (uint64_t m = bits; m; m &= m - 1, ++r) {
      const int o = __builtin_ctzll(m), p = p0 + o;
      out.idx[r] = p;
      if (out.row_tgt) {
        // ids outside [0, V) are clamped so that no kernel reads outside W
        const int y = !tgt_ahead ? targets[p] : o == 0 ? tgt[0] : o == 1 ? tgt[1] : o == 2 ? tgt[2] : tgt[3];
        out.row_tgt[r] = y < 0 ? 0 : (y >= V ? V - 1 : y);
        while (p >= (b + 1) * L) ++b;
        out.row_seq[r] = g * B + b;
      }
    }
  }
  if (wave == THREADS / 64 - 1)
    write_record(out.meta ? out.meta + g : nullptr, row0, prev_end, total, out.max_cols, plan, lane);
  if (tid == 0) sSeg[B] = total;
  __syncthreads();

  const int rows = row0 + total;
  for (int b = tid; b < B; b += THREADS) {
    const uint32_t T = sT[t_base + b];
    if (nm_out) nm_out[(int64_t)b * nm_stride + g] = sSeg[b + 1] - sSeg[b];
    if (t_out) t_out[(int64_t)b * t_stride + g] = (float)T * (1.0f / 16777216.0f);
    if (out.seg_off) out.seg_off[g * (B + 1) + b] = row0 + sSeg[b];
    if (out.t24) out.t24[g * B + b] = T;
  }
  if (tid == 0 && out.seg_off) out.seg_off[g * (B + 1) + B] = rows;
  // the last sample pads the unit's rows up to the next row tile
  if (g == n_samples - 1 && out.row_tgt) {
    const int pad_end = min((rows + kRowPad - 1) / kRowPad * kRowPad, out.row_cap);
    for (int r = rows + tid; r < pad_end; r += THREADS) {
      out.row_tgt[r] = 0;
      out.row_seq[r] = 0;
    }
  }
}

__global__ __launch_bounds__(kMaskThreads) void k_mask_compact(MaskArgs a) {
  __shared__ MaskShared<kMaskThreads, kMaxB> sh;
  mask_sample<kMaskThreads, kMaxB>(a, blockIdx.x, gridDim.x, sh);
}

// ---------------------------------------------------------------------------
// Multi-block form for large B*L: the same masks (the same Philox words and
// integer test), in three passes that each spread over the whole GPU:
//   k_mask_bits     one 32-bit mask word per thread (32 consecutive positions),
//                   one count per block of kMbPositions positions
//   k_mask_scan     one block: exclusive scan of the block counts, the
//                   per-response offsets (block offset + popcounts of the
//                   words before the response's first position), counts,
//                   the sample's record and the padding rows
//   k_mask_scatter  every set bit in ascending position order to its row
// so the compacted order and every count equal the single-block form's.
constexpr int kMbThreads = 256;
constexpr int kMbPositions = kMbThreads * 32;   // positions per block

__global__ __launch_bounds__(256) void k_timesteps(int B, int n_t, int j, int t_mode, uint32_t k0,
                                                   uint32_t k1, uint32_t seq_base,
                                                   uint32_t* __restrict__ t24,
                                                   float* __restrict__ t_out, int t_stride) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B) return;
  const uint32_t T = timestep_t24(k0, k1, seq_base + (uint32_t)b, j, n_t, t_mode);
  t24[b] = T;
  if (t_out) t_out[(int64_t)b * t_stride] = (float)T * (1.0f / 16777216.0f);
}

// exclusive prefix of v over the block's 256 threads (and the block total)
__device__ __forceinline__ int block_exclusive_sum(int v, int* s_wave, int* total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int base = incl - v;
  for (int q = 0; q < wave; ++q) base += s_wave[q];
  *total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
  return base;
}

__global__ __launch_bounds__(kMbThreads) void k_mask_bits(
    const uint8_t* __restrict__ resp, const uint32_t* __restrict__ t24, int L, int64_t P, int j,
    uint32_t k0, uint32_t k1, uint32_t seq_base, uint32_t* __restrict__ bits,
    int32_t* __restrict__ wprefix, int32_t* __restrict__ blk_count) {
  __shared__ int s_wave[kMbThreads / 64];
  const int tid = threadIdx.x;
  const int64_t w = (int64_t)blockIdx.x * kMbThreads + tid;
  uint32_t word = 0;
  const int64_t p0 = w * 32;
  if (p0 < P) {
    // the word's 32 response-mask bytes in two 16-byte loads (resp_mask rows
    // are contiguous; a word that crosses P reads byte by byte)
    uint8_t r[32];
    if (p0 + 32 <= P && (((uintptr_t)(resp + p0)) & 15) == 0) {
      *reinterpret_cast<uint4*>(r) = *reinterpret_cast<const uint4*>(resp + p0);
      *reinterpret_cast<uint4*>(r + 16) = *reinterpret_cast<const uint4*>(resp + p0 + 16);
    } else {
#pragma unroll
      for (int e = 0; e < 32; ++e) r[e] = p0 + e < P ? resp[p0 + e] : 0;
    }
    MaskWalker mw{k0, k1, seq_base, L, j};
    int b = (int)(p0 / L), i = (int)(p0 - (int64_t)b * L);
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      if (r[e] && mw.test(t24, b, i)) word |= 1u << e;
      if (++i == L) { i = 0; ++b; }
    }
    bits[w] = word;
  }
  int total;
  const int pre = block_exclusive_sum(__popc(word), s_wave, &total);
  if (p0 < P) wprefix[w] = pre;
  if (tid == 0) blk_count[blockIdx.x] = total;
}

constexpr int kMbMaxBlocks = (1 << 20) / kMbPositions;   // B*L <= 2^20

// masked positions before position pos < P: the block's offset, the word's
// prefix within its block, the word's bits below pos
__device__ __forceinline__ int masked_before(const uint32_t* bits, const int32_t* wprefix,
                                             const int32_t* blk_off, int64_t pos) {
  const int64_t w = pos / 32;
  return blk_off[w / kMbThreads] + wprefix[w] +
         __popc(bits[w] & ((1u << (int)(pos - w * 32)) - 1u));
}

__global__ __launch_bounds__(1024) void k_mask_scan(
    const uint32_t* __restrict__ bits, const int32_t* __restrict__ wprefix,
    const int32_t* __restrict__ blk_count,
    int32_t* __restrict__ blk_off, int nblk, int B, int L, int g, MaskOut out,
    int32_t* __restrict__ nm_out, int nm_stride, const SampleMeta* prev,
    const SampleMeta* prev_unit, DxPlan plan) {
  __shared__ int s_total;
  __shared__ int32_t s_off[kMbMaxBlocks];
  const int tid = threadIdx.x;
  if (tid == 0) {
    int acc = 0;
    for (int q = 0; q < nblk; ++q) {
      s_off[q] = acc;
      blk_off[q] = acc;   // for the scatter pass
      acc += blk_count[q];
    }
    s_total = acc;
  }
  __syncthreads();
  const int total = s_total;
  const int row0 = (g > 0 && prev) ? prev->n_rows : 0;
  const int prev_end = prev_unit ? prev_unit->col_end : 0;
  for (int b = tid; b < B; b += 1024) {
    const int s0 = masked_before(bits, wprefix, s_off, (int64_t)b * L);
    const int s1 = b + 1 < B ? masked_before(bits, wprefix, s_off, (int64_t)(b + 1) * L) : total;
    if (nm_out) nm_out[(int64_t)b * nm_stride] = s1 - s0;
    if (out.seg_off) out.seg_off[b] = row0 + s0;
  }
  const int rows = row0 + total;
  const int rows_pad = (rows + kRowPad - 1) / kRowPad * kRowPad;
  if (tid == 0 && out.seg_off) out.seg_off[B] = rows;
  if (tid < 64) write_record(out.meta, row0, prev_end, total, out.max_cols, plan, tid);
  const int pad_end = min(rows_pad, out.row_cap);
  for (int r = rows + tid; r < pad_end; r += 1024) {
    if (out.row_tgt) out.row_tgt[r] = 0;
    if (out.row_seq) out.row_seq[r] = 0;
  }
}

__global__ __launch_bounds__(kMbThreads) void k_mask_scatter(
    const uint32_t* __restrict__ bits, const int32_t* __restrict__ wprefix,
    const int32_t* __restrict__ blk_off, const int32_t* __restrict__ targets, int B, int L,
    int64_t P, int g, int V, MaskOut out, const SampleMeta* prev) {
  const int64_t w = (int64_t)blockIdx.x * kMbThreads + threadIdx.x;
  if (w * 32 >= P) return;
  const uint32_t word = bits[w];
  const int row0 = (g > 0 && prev) ? prev->n_rows : 0;
  int r = row0 + blk_off[blockIdx.x] + wprefix[w];
  if (out.inv) {
    int32_t* const inv = out.inv + (int64_t)g * P + w * 32;
    int q = r;
    for (int e = 0; e < 32 && w * 32 + e < P; ++e) inv[e] = (word >> e) & 1 ? q++ : -1;
  }
  uint32_t m = word;
  while (m) {
    const int e = __builtin_ctz(m);
    m &= m - 1;
    const int64_t p = w * 32 + e;
    if (out.idx) out.idx[r] = (int32_t)p;
    if (out.row_tgt) {
      const int y = targets[p];
      out.row_tgt[r] = y < 0 ? 0 : (y >= V ? V - 1 : y);
    }
    if (out.row_seq) out.row_seq[r] = g * B + (int)(p / L);
    ++r;
  }
}

size_t mask_scratch_bytes(int B, int L) {
  const int64_t P = (int64_t)B * L;
  const int64_t words = (P + 31) / 32, nblk = (P + kMbPositions - 1) / kMbPositions;
  return (size_t)(words * 8 + nblk * 8 + (int64_t)B * 4 + 4 * 256);
}

static MaskArgs mask_args(const uint8_t* resp, const int32_t* targets, int B, int L, int n_t, int j0,
                          int t_mode, uint64_t seed, uint32_t seq_base, const Workspace* ws,
                          int32_t* idx_out, int32_t* n_masked_out, int nm_stride, float* t_out,
                          int t_stride, int V, const SampleMeta* prev_unit, const DxPlan& plan) {
  MaskOut out{idx_out, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0};
  if (ws) {
    out.idx = ws->idx;
    out.inv = ws->inv;
    out.row_tgt = ws->row_tgt;
    out.row_seq = ws->row_seq;
    out.seg_off = ws->seg_off;
    out.t24 = ws->t24;
    out.meta = ws->meta;
    out.row_cap = (int)ws->RP;
    out.max_cols = (int)ws->max_cols;
  }
  return MaskArgs{resp, targets, B, L, n_t, j0, t_mode, (uint32_t)(seed & 0xFFFFFFFFu),
                  (uint32_t)(seed >> 32), seq_base, out, n_masked_out, nm_stride, t_out, t_stride, V,
                  prev_unit, plan};
}

hipError_t launch_masks(const uint8_t* resp, const int32_t* targets, int B, int L, int n_t, int j0,
                        int n_samples, int t_mode, uint64_t seed, uint32_t seq_base,
                        const Workspace* ws, int32_t* idx_out, int32_t* n_masked_out,
                        int nm_stride, float* t_out, int t_stride, int V,
                        const SampleMeta* prev_unit, const DxPlan& plan, void* scratch,
                        bool force_multi, hipStream_t s, int* launches) {
  const MaskArgs args = mask_args(resp, targets, B, L, n_t, j0, t_mode, seed, seq_base, ws, idx_out,
                                  n_masked_out, nm_stride, t_out, t_stride, V, prev_unit, plan);
  const MaskOut& out = args.out;
  const uint32_t k0 = (uint32_t)(seed & 0xFFFFFFFFu), k1 = (uint32_t)(seed >> 32);
  const int64_t P = (int64_t)B * L;
  if ((P <= kSingleBlockPositions && !force_multi) || !scratch) {
    k_mask_compact<<<n_samples, kMaskThreads, 0, s>>>(args);
    ++*launches;
    return hipGetLastError();
  }
  // scratch: mask words, block counts and offsets, and (without a unit) the
  // sample's timesteps
  char* sc = static_cast<char*>(scratch);
  const int64_t words = (P + 31) / 32, nblk = (P + kMbPositions - 1) / kMbPositions;
  const int64_t wbytes = (words * 4 + 255) / 256 * 256;
  uint32_t* bits = reinterpret_cast<uint32_t*>(sc);
  int32_t* wprefix = reinterpret_cast<int32_t*>(sc + wbytes);
  int32_t* blk_count = reinterpret_cast<int32_t*>(sc + 2 * wbytes);
  int32_t* blk_off = blk_count + nblk;
  uint32_t* t24_0 = out.t24 ? out.t24
                            : reinterpret_cast<uint32_t*>(sc + 2 * wbytes +
                                                          (nblk * 8 + 255) / 256 * 256);
  for (int g = 0; g < n_samples; ++g) {
    const int j = j0 + g;
    uint32_t* t24 = out.t24 ? t24_0 + (int64_t)g * B : t24_0;
    MaskOut og = out;   // this sample's share of the per-sample arrays
    if (ws) {
      og.seg_off += (int64_t)g * (B + 1);
      og.meta += g;
    }
    const SampleMeta* prev = g ? ws->meta + (g - 1) : prev_unit;
    k_timesteps<<<(unsigned)((B + 255) / 256), 256, 0, s>>>(B, n_t, j, t_mode, k0, k1, seq_base,
                                                            t24, t_out ? t_out + g : nullptr,
                                                            t_stride);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_mask_bits<<<(unsigned)nblk, kMbThreads, 0, s>>>(resp, t24, L, P, j, k0, k1, seq_base, bits,
                                                      wprefix, blk_count);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_mask_scan<<<1, 1024, 0, s>>>(bits, wprefix, blk_count, blk_off, (int)nblk, B, L, g, og,
                                   n_masked_out ? n_masked_out + g : nullptr, nm_stride, prev,
                                   prev_unit, plan);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_mask_scatter<<<(unsigned)nblk, kMbThreads, 0, s>>>(bits, wprefix, blk_off, targets, B, L, P,
                                                         g, V, og, prev);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    *launches += 4;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Row r of a unit reads the head input of sample g = row_seq[r] / B at its
// position, x + g * stride + idx[r] * d.
template <typename T>
struct RowInput {
  const T* x;
  int64_t stride;
  int B, d;
  const int32_t *idx, *row_seq;
  __device__ const T* row(int r) const {
    return x + (int64_t)(row_seq[r] / B) * stride + (int64_t)idx[r] * d;
  }
};

// The final RMSNorm of 8 elements, bf16(x * ir * gamma) (fp32 arithmetic, one
// rounding).
__device__ __forceinline__ uint4 norm8(uint4 v, float ir, const float* gamma) {
  const float4 g0 = *reinterpret_cast<const float4*>(gamma);
  const float4 g1 = *reinterpret_cast<const float4*>(gamma + 4);
  const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
  uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float lo = __uint_as_float(a[e] << 16), hi = __uint_as_float(a[e] & 0xFFFF0000u);
    a[e] = pack_bf16x2(lo * ir * gg[2 * e], hi * ir * gg[2 * e + 1]);
  }
  return make_uint4(a[0], a[1], a[2], a[3]);
}

// Target logit z[row, y] = h[row] . W[:, y] by one wave: 64 lanes split the
// d-long dot product (fp32), w the target's row of W^T; h the head input
// (through the norm with NORM).
template <bool NORM, typename T>
__device__ __forceinline__ float target_logit(const T* xr, const uint16_t* w, float ir,
                                              const float* gamma, int d, int lane) {
  float acc = 0.f;
  for (int k = lane * 8; k < d; k += 64 * 8) {
    uint4 hv = load_bf16x8(xr + k);
    if constexpr (NORM) hv = norm8(hv, ir, gamma + k);
    const uint4 wv = *reinterpret_cast<const uint4*>(w + k);
    const uint32_t ha[4] = {hv.x, hv.y, hv.z, hv.w}, wa[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(__uint_as_float(ha[e] << 16), __uint_as_float(wa[e] << 16), acc);
      acc = fmaf(__uint_as_float(ha[e] & 0xFFFF0000u), __uint_as_float(wa[e] & 0xFFFF0000u), acc);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  return acc;
}

// Inverse RMS of the masked rows of the pre-norm activations x (for the final
// RMSNorm h = gamma x r, r = (mean x^2 + eps)^(-1/2)) and the rows' target
// logits: one wave per row, fp32 sum of squares.
template <typename T>
__global__ __launch_bounds__(256) void k_row_rms(RowInput<T> in, const SampleMeta* __restrict__ meta,
                                                 const float* __restrict__ gamma, float eps,
                                                 const uint16_t* __restrict__ WT,
                                                 const int32_t* __restrict__ row_tgt,
                                                 float* __restrict__ inv_rms,
                                                 float* __restrict__ ztgt) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= meta->n_rows) return;
  const T* xr = in.row(row);
  const int d = in.d;
  float acc = 0.f;
  for (int k = lane * 8; k < d; k += 64 * 8) {
    const uint4 v = load_bf16x8(xr + k);
    const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = __uint_as_float(a[e] << 16), hi = __uint_as_float(a[e] & 0xFFFF0000u);
      acc = fmaf(lo, lo, acc);
      acc = fmaf(hi, hi, acc);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  const float ir = 1.f / sqrtf(acc / (float)d + eps);
  const float z = target_logit<true>(xr, WT + (int64_t)row_tgt[row] * d, ir, gamma, d, lane);
  if (lane == 0) {
    inv_rms[row] = ir;
    ztgt[row] = z;
  }
}

template <typename T>
static RowInput<T> row_input(const void* x, int64_t stride, int B, const Workspace& ws, int d) {
  return RowInput<T>{static_cast<const T*>(x), stride, B, d, ws.idx, ws.row_seq};
}

hipError_t launch_row_rms(const void* x, bool f32, int64_t stride, int B, const Workspace& ws,
                          const float* gamma, int d, float eps, hipStream_t s) {
  const unsigned grid = (unsigned)(ws.g_used * ws.NP / 4);
  if (f32)
    k_row_rms<float><<<grid, 256, 0, s>>>(row_input<float>(x, stride, B, ws, d), ws.unit(), gamma,
                                          eps, ws.WT, ws.row_tgt, ws.inv_rms, ws.ztgt);
  else
    k_row_rms<uint16_t><<<grid, 256, 0, s>>>(row_input<uint16_t>(x, stride, B, ws, d), ws.unit(),
                                             gamma, eps, ws.WT, ws.row_tgt, ws.inv_rms, ws.ztgt);
  return hipGetLastError();
}

// Gather: Hc[r, :] = h[r, :] and HcT[:, col_off + r] for the unit's rows r < N;
// zeros for N <= r < N_pad.  Both are slab-major (Hc with RP rows per slab,
// HcT with d), so each 64x64 tile of either is 8 KB of contiguous memory; the
// tiles are staged in LDS for the transposed copy.  With `gamma`, the input
// holds the pre-norm activations and the gathered row is the final RMSNorm of
// it.  fp32 inputs are rounded to bf16 first (load_bf16x8), then treated the
// same way.  Without the norm the launch's last workgroups (from n_tile_wg)
// form the rows' target logits, one wave per row, straight from the input;
// with it k_row_rms has done so.  Bound by HBM.
template <typename T>
__global__ __launch_bounds__(256) void k_gather(RowInput<T> in, const SampleMeta* __restrict__ meta,
                                                const float* __restrict__ gamma,
                                                const float* __restrict__ inv_rms,
                                                uint16_t* __restrict__ Hc,
                                                uint16_t* __restrict__ HcT, int64_t RP,
                                                unsigned n_tile_wg,
                                                const uint16_t* __restrict__ WT,
                                                const int32_t* __restrict__ row_tgt,
                                                float* __restrict__ ztgt) {
  __shared__ uint16_t tile[64][72];
  const int tid = threadIdx.x, d = in.d;
  const int N = meta->n_rows;
  const unsigned wg = line_index();
  if (wg >= n_tile_wg) {
    const int row = (wg - n_tile_wg) * 4 + (tid >> 6), lane = tid & 63;
    if (gamma || row >= N) return;
    const float z = target_logit<false>(in.row(row), WT + (int64_t)row_tgt[row] * d, 0.f, nullptr,
                                        d, lane);
    if (lane == 0) ztgt[row] = z;
    return;
  }
  const int cts = d / 64;
  const int r0 = (int)(wg / cts) * 64, c0 = (int)(wg % cts) * 64;
  if (r0 >= meta->n_rows_pad) return;
  const int coff = meta->col_off;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int q = tid + it * 256;
    const int row = q >> 3, ch = q & 7;
    const int r = r0 + row;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < N) {
      v = load_bf16x8(in.row(r) + c0 + ch * 8);
      if (gamma) v = norm8(v, inv_rms[r], gamma + c0 + ch * 8);
    }
    *reinterpret_cast<uint4*>(Hc + slab_index(RP, r, c0 + ch * 8)) = v;
    *reinterpret_cast<uint4*>(&tile[row][ch * 8]) = v;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int q = tid + it * 256;
    const int c = q >> 3, rch = q & 7;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = (uint32_t)tile[rch * 8 + 2 * e][c] | ((uint32_t)tile[rch * 8 + 2 * e + 1][c] << 16);
    *reinterpret_cast<uint4*>(HcT + slab_index(d, c0 + c, (int64_t)coff + r0 + rch * 8)) =
        make_uint4(w[0], w[1], w[2], w[3]);
  }
}

hipError_t launch_gather(const void* hidden, bool f32, int64_t stride, int B, const float* gamma,
                         const Workspace& ws, int d, hipStream_t s) {
  const int64_t rows = ws.g_used * ws.NP;
  const unsigned tiles = (unsigned)(rows / 64 * (d / 64));   // at most 2^26
  const dim3 grid = line_grid(tiles + (gamma ? 0 : rows / 4));
  if (f32)
    k_gather<float><<<grid, 256, 0, s>>>(row_input<float>(hidden, stride, B, ws, d), ws.unit(),
                                         gamma, ws.inv_rms, ws.Hc, ws.HcT, ws.RP, tiles, ws.WT,
                                         ws.row_tgt, ws.ztgt);
  else
    k_gather<uint16_t><<<grid, 256, 0, s>>>(row_input<uint16_t>(hidden, stride, B, ws, d),
                                            ws.unit(), gamma, ws.inv_rms, ws.Hc, ws.HcT, ws.RP,
                                            tiles, ws.WT, ws.row_tgt, ws.ztgt);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// W_head [d, V] -> WT [V, d] (row-major) and, unless Wk is NULL, Wk: W in
// slab-major order with d rows per slab (the dX GEMM's operand; each 64x64
// tile is 8 KB of contiguous memory there).  64x64 tiles through LDS; fp32 W
// is rounded to bf16 as it is read.  Bound by HBM.  With NT the outputs are
// streamed past the caches and consecutive workgroups take the k tiles of one
// 64-id vocabulary slab, so that the rows of W^T are written whole at about the
// same time; else they take the vocabulary tiles of one k slab.
template <bool NT>
__device__ __forceinline__ void store16(uint16_t* p, uint4 v) {
  typedef uint32_t vec4u __attribute__((ext_vector_type(4)));
  if constexpr (NT)
    __builtin_nontemporal_store((vec4u){v.x, v.y, v.z, v.w}, reinterpret_cast<vec4u*>(p));
  else
    *reinterpret_cast<uint4*>(p) = v;
}

typedef uint16_t WTile[64][72];

template <typename T, bool NT>
__device__ __forceinline__ void transpose_w_tile(const T* __restrict__ W, uint16_t* __restrict__ WT,
                                                 uint16_t* __restrict__ Wk, int d, int V,
                                                 unsigned wg, WTile& tile) {
  const unsigned kts = d / 64, vts = V / 64;
  if (wg >= kts * vts) return;
  const int v0 = (int)(NT ? wg / kts : wg % vts) * 64;
  const int k0 = (int)(NT ? wg % kts : wg / vts) * 64;
  const int tid = threadIdx.x;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int q = tid + it * 256;
    const int kr = q >> 3, ch = q & 7;
    const uint4 v = load_bf16x8(W + (int64_t)(k0 + kr) * V + v0 + ch * 8);
    *reinterpret_cast<uint4*>(&tile[kr][ch * 8]) = v;
    if (Wk) store16<NT>(Wk + slab_index(d, k0 + kr, v0 + ch * 8), v);
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int q = tid + it * 256;
    const int v = q >> 3, kch = q & 7;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = (uint32_t)tile[kch * 8 + 2 * e][v] | ((uint32_t)tile[kch * 8 + 2 * e + 1][v] << 16);
    store16<NT>(WT + (int64_t)(v0 + v) * d + k0 + kch * 8, make_uint4(w[0], w[1], w[2], w[3]));
  }
}

template <typename T, bool NT>
__global__ __launch_bounds__(256) void k_transpose_w(const T* __restrict__ W,
                                                     uint16_t* __restrict__ WT,
                                                     uint16_t* __restrict__ Wk, int d, int V) {
  __shared__ WTile tile;
  transpose_w_tile<T, NT>(W, WT, Wk, d, V, line_index(), tile);
}

// The start of a call in one launch: the masks of its first unit (one workgroup
// per sample, the first ones) beside the copies of W, neither of which reads
// what the other writes.  Against two launches: a step of B2 L64 d128 V1024 n_t 4
// 46 -> 42 us, of B4 L128 d2048 V8192 n_t 4 176 -> 167, of B4 L256 d2048 V32000
// n_t 4 917 -> 910, one sample of B8 L512 d4096 V126464 7.66 -> 7.63 ms.
constexpr int kPrepMaxB = 512, kPrepPositions = 64 * 256;

template <typename T, bool NT>
__global__ __launch_bounds__(256, 8) void k_masks_and_w(MaskArgs a, int n_samples,
                                                        const T* __restrict__ W,
                                                        uint16_t* __restrict__ WT,
                                                        uint16_t* __restrict__ Wk, int d) {
  __shared__ union {
    MaskShared<256, kPrepMaxB> mask;
    WTile tile;
  } sh;
  const unsigned wg = line_index();
  if (wg < (unsigned)n_samples)
    mask_sample<256, kPrepMaxB>(a, wg, n_samples, sh.mask);
  else
    transpose_w_tile<T, NT>(W, WT, Wk, d, a.V, wg - n_samples, sh.tile);
}

// Bytes of an output of k_transpose_w from which it is streamed, well past what
// the 256 MB last-level cache keeps for the GEMMs: 1.04 GB (d 4096 V 126464) 612
// -> 577 us with both outputs; 0.54 GB 312 and 320, 0.13 GB 69 and 83 streamed.
constexpr int64_t kStreamBytes = int64_t(768) << 20;

hipError_t launch_transpose_w(const void* W, bool f32, uint16_t* WT, uint16_t* Wk, int d, int V,
                              hipStream_t s) {
  const dim3 grid = line_grid((int64_t)(V / 64) * (d / 64));   // at most 2^24 workgroups
  const bool nt = (int64_t)d * V * 2 >= kStreamBytes;
  if (f32)
    (nt ? k_transpose_w<float, true> : k_transpose_w<float, false>)<<<grid, 256, 0, s>>>(
        static_cast<const float*>(W), WT, Wk, d, V);
  else
    (nt ? k_transpose_w<uint16_t, true> : k_transpose_w<uint16_t, false>)<<<grid, 256, 0, s>>>(
        static_cast<const uint16_t*>(W), WT, Wk, d, V);
  return hipGetLastError();
}

// Whether the masks of n_samples samples are drawn beside the copies of W.  A
// workgroup of 256 threads takes twice as long as k_mask_compact's for a unit
// of many positions (8 samples of 4096: 47 us and 20), so they are drawn there
// if they are few or if the copies take longer (6 d V bytes at 5 TB/s against
// about 1.2 ns per position).
static bool masks_beside_w(int B, int L, int d, int V, int n_samples) {
  const int64_t P = (int64_t)B * L;
  return B <= kPrepMaxB && P <= kPrepPositions &&
         n_samples * P <= std::max<int64_t>(8192, (int64_t)d * V / 1024);
}

hipError_t launch_masks_and_w(const void* W, bool f32, const uint8_t* resp, const int32_t* targets,
                              int B, int L, int d, int n_t, int j0, int t_mode, uint64_t seed,
                              uint32_t seq_base, const Workspace& ws, int32_t* n_masked_out,
                              float* t_out, int V, const DxPlan& plan, hipStream_t s, bool* masks_done) {
  *masks_done = masks_beside_w(B, L, d, V, ws.g_used);
  if (!*masks_done) return launch_transpose_w(W, f32, ws.WT, ws.Wk, d, V, s);
  const MaskArgs a = mask_args(resp, targets, B, L, n_t, j0, t_mode, seed, seq_base, &ws, nullptr,
                               n_masked_out, n_t, t_out, n_t, V, nullptr, plan);
  const dim3 grid = line_grid(ws.g_used + (int64_t)(V / 64) * (d / 64));
  const bool nt = (int64_t)d * V * 2 >= kStreamBytes;
  if (f32)
    (nt ? k_masks_and_w<float, true> : k_masks_and_w<float, false>)<<<grid, 256, 0, s>>>(
        a, ws.g_used, static_cast<const float*>(W), ws.WT, ws.Wk, d);
  else
    (nt ? k_masks_and_w<uint16_t, true> : k_masks_and_w<uint16_t, false>)<<<grid, 256, 0, s>>>(
        a, ws.g_used, static_cast<const uint16_t*>(W), ws.WT, ws.Wk, d);
  return hipGetLastError();
}

}  // namespace bgpo
