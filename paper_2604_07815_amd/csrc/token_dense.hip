// Token-level selection over a whole context: the token-only operator of the
// paper's kernel study (Sec. 5; Double Sparsity), i.e. the token stage of
// Sec. 4.1 with every block of the unit as candidates.  For every valid token
// j of a unit:
//   l_hj = sigma * q~_h . dequant(k~_j)        (INT4 index on the channels C)
//   alpha_j = (1/G) sum_h exp(l_hj - m_h) / Z_h,  m_h, Z_h over all valid j
// then the K_t largest alpha (ties to the lower position), ascending.
//
//   pass 0: per chunk of tokens, each head's maximum logit and sum of
//           exponentials;
//   pass 1: the unit's m_h, Z_h from every chunk, then the alpha keys of the
//           chunk's tokens (recomputing the logits costs one more read of the
//           index rows, less than writing and reading them back) and the
//           unit's histogram of key buckets;
//   ds_topk_kernel: top-K_t of the unit's keys.  The histogram gives the
//           bucket that holds the K_t-th key, so one ordered pass over the
//           keys leaves the few candidates at or above it, which are selected
//           from registers.
// Three kernels compute the passes: ds_score_mfma_kernel (bf16, G <= 8),
// ds_score_wide_kernel (bf16, G = 16 or 32, d_c = 64 or 128) and
// ds_score_kernel on the vector units (fp32 queries, whose bits a bf16 operand
// would not hold, and the other index widths).
#include "attn_common.hpp"
#include "token_common.hpp"

namespace tls {

constexpr int kDsThreads = 256;
constexpr int kDsNW = kDsThreads / 64;
constexpr int kDsMaxDc = 256;
constexpr int kDsTopkThreads = 1024;
constexpr int kDsListCap = 16384;  // keys in play (or candidates) kept in LDS
constexpr int kDsMaskGroups = 4096;  // groups of 64 keys whose candidate masks are in LDS at a time
constexpr int kDsHistWords = 260;  // per unit: 256 bucket counts, the key bound, padding

// Bucket counts of a unit's keys: bucket b holds the keys with key >>
// kTopkSpreadShift == base + b, base = (bound >> kTopkSpreadShift) - 254 (an
// eighth of an octave each; bucket 0 also everything lower), as in the spread
// first pass of wg_topk_regs.  Counted in LDS per work-group (four copies),
// then added to the unit's counts in global memory, which pass 0 clears.
__device__ inline void ds_clear_hist(uint32_t* hist, int unit) {
  if (hist)
    for (int i = threadIdx.x; i < kDsHistWords; i += kDsThreads) hist[size_t(unit) * kDsHistWords + i] = 0u;
}
__device__ inline int ds_bucket(uint32_t key, uint32_t bound) {
  return min(max(int(key >> kTopkSpreadShift) - (int(bound >> kTopkSpreadShift) - 254), 0), 255);
}
__device__ inline void ds_count_key(uint32_t* s_hist, uint32_t key, uint32_t bound) {
  atomicAdd(&s_hist[(threadIdx.x % kTopkHistCopies) * kTopkHistStride + ds_bucket(key, bound)], 1u);
}
__device__ inline void ds_flush_hist(const uint32_t* s_hist, uint32_t* hist, int unit, int chunk, uint32_t bound) {
  if (!hist) return;
  __syncthreads();
  uint32_t c = 0;
#pragma unroll
  for (int cp = 0; cp < kTopkHistCopies; ++cp) c += s_hist[cp * kTopkHistStride + threadIdx.x];
  if (c) atomicAdd(&hist[size_t(unit) * kDsHistWords + threadIdx.x], c);
  if (chunk == 0 && threadIdx.x == 0) hist[size_t(unit) * kDsHistWords + 256] = bound;
}

// The unit's per-head maximum and 1/Z from its chunks' statistics
// [chunk][G][2], by all 256 threads: thread t folds chunks t / G, t / G +
// 256 / G, ... of head t % G, then lanes and waves are combined in a fixed
// order; first the maximum, then the sum against it.  s_part: [4][G][2]; the
// results are in s_mz after the caller's next barrier.
template <int G>
__device__ inline void ds_unit_norm(const float* st, int nc, float (*s_part)[G][2], float (*s_mz)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, h = tid % G;
  const float2* s2 = reinterpret_cast<const float2*>(st);
  float M = -INFINITY;
  for (int c = tid / G; c < nc; c += kDsThreads / G) M = fmaxf(M, s2[size_t(c) * G + h].x);
#pragma unroll
  for (int o = G; o < 64; o <<= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
  if (lane < G) s_part[wid][lane][0] = M;
  lds_barrier();
  M = s_part[0][h][0];
#pragma unroll
  for (int w = 1; w < kDsNW; ++w) M = fmaxf(M, s_part[w][h][0]);
  float Z = 0.f;
  if (M != -INFINITY)
    for (int c = tid / G; c < nc; c += kDsThreads / G) {
      const float2 e = s2[size_t(c) * G + h];
      if (e.x != -INFINITY) Z += e.y * __builtin_amdgcn_exp2f(e.x - M);
    }
#pragma unroll
  for (int o = G; o < 64; o <<= 1) Z += __shfl_xor(Z, o, 64);
  if (lane < G) s_part[wid][lane][1] = Z;
  lds_barrier();
  if (tid < G) {
    Z = (s_part[0][tid][1] + s_part[1][tid][1]) + (s_part[2][tid][1] + s_part[3][tid][1]);
    s_mz[tid][0] = M;
    s_mz[tid][1] = Z > 0.f ? 1.0f / Z : 0.f;
  }
}

// ---------------------------------------------------------------------------
// bf16, G <= 8: a lane owns its tokens, the code contraction runs on the matrix
// cores (lane_dots).  Bound by HBM (24 bytes per token and pass at d_c = 32) and by
// vector issue, about 90 instructions per 64 tokens: 128 units of 73k tokens, 226
// MB, take 45 us (pass 0) and 49 us (pass 1) against 78 us each on the vector
// units, which spend some 200 instructions on extracting codes and
// multiply-adds.  A work-group takes kDsSteps steps of four tokens per thread,
// the next step's rows requested before the last is used.
// ---------------------------------------------------------------------------
constexpr int kDsTpt = 4, kDsSteps = 4;
constexpr int kDsMfmaChunk = kDsThreads * kDsTpt * kDsSteps;

// NGR: 32-channel groups (1 unrolls the steps, with their loads in two register
// sets; 0 takes any d_c).
template <int G, int NGR, bool KEYS>
__global__ __launch_bounds__(kDsThreads, G <= 4 ? 4 : 2) void ds_score_mfma_kernel(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int d, int d_c,
    int T, float sigma, int nchunks, float* __restrict__ stats, uint32_t* __restrict__ keys,
    uint32_t* __restrict__ hist, uint32_t* err) {
  constexpr int TPT = kDsTpt, STEP = kDsThreads * TPT, HS = (G + 3) / 4;
  __shared__ __attribute__((aligned(16))) uint16_t s_qt[(kDsMaxDc / 32) * HS * 4 * 32];  // [group][set][head][position]
  __shared__ float s_red[kDsNW][G][2], s_mz[G][2];
  __shared__ uint32_t s_hist[KEYS ? kTopkHistWords : 1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  // pass 1 walks the chunks backwards: the rows that pass 0 read last may
  // still be in the Infinity Cache
  const int unit = KEYS ? int(gridDim.y - 1 - blockIdx.y) : int(blockIdx.y);
  const int chunk = KEYS ? int(gridDim.x - 1 - blockIdx.x) : int(blockIdx.x);
  const int s = unit / H_kv, g = unit % H_kv;
  int n = ctx_lens[s];
  if (n < 0 || n > T) {
    if (tid == 0 && chunk == 0) set_error(err, 1u);
    n = n < 0 ? 0 : T;
  }
  if (!KEYS && chunk == 0) ds_clear_hist(hist, unit);
  const int j0 = chunk * kDsMfmaChunk;
  if (j0 >= n) return;
  const int ngr = NGR > 0 ? NGR : d_c / 32, rowb = ngr * 16;
  const size_t ubase = size_t(unit) * T;
  const uint8_t* ucodes = codes + ubase * rowb;
  const uint8_t* uqp = reinterpret_cast<const uint8_t*>(qparams + ubase * ngr * 2);
  // index rows of a step's tokens, group gr (rows past the end: the last valid one)
  auto request = [&](uint4 (&cw)[TPT], float2 (&pr)[TPT], int st, int gr) {
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
      const uint32_t row = uint32_t(min(j0 + st * STEP + t * kDsThreads + tid, n - 1));
      cw[t] = ld16(ucodes + row * uint32_t(rowb) + gr * 16);
      pr[t] = *reinterpret_cast<const float2*>(uqp + row * uint32_t(ngr * 8) + gr * 8);
    }
  };
  uint4 cw[2][TPT];
  float2 pr[2][TPT];
  request(cw[0], pr[0], 0, 0);
  __builtin_amdgcn_sched_barrier(0);  // the first rows are in flight during the prologue
  if constexpr (KEYS) {
    for (int i = tid; i < kTopkHistWords; i += kDsThreads) s_hist[i] = 0u;
  }
  for (int i = tid; i < ngr * HS * 128; i += kDsThreads) {
    const int x = i & 31, h = ((i >> 7) % HS) * 4 + ((i >> 5) & 3), gr = i / (128 * HS);
    int ch = channels[g * d_c + gr * 32 + (x & ~7) + codes_chan(x & 7)];
    if (ch < 0 || ch >= d) {
      set_error(err, 32u);
      ch = 0;
    }
    s_qt[i] = h < G ? q[(size_t(s) * H_q + size_t(g) * G + h) * d + ch] : uint16_t(0);
  }
  if constexpr (KEYS)
    ds_unit_norm<G>(stats + size_t(unit) * nchunks * G * 2, (n + kDsMfmaChunk - 1) / kDsMfmaChunk, s_red, s_mz);
  lds_barrier();

  const float sigma2 = sigma * 1.4426950408889634f, invG = 1.0f / float(G);
  float m[G], z[G];  // running maximum and sum (pass 0), or the unit's maximum and 1/Z (pass 1)
  float bsum = 0.f;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = KEYS ? s_mz[h][0] : -INFINITY;
    z[h] = KEYS ? s_mz[h][1] : 0.f;
    if constexpr (KEYS) bsum = fmaf(1.0f, z[h], bsum);
  }
  const uint32_t bound = KEYS ? alpha_key(bsum * invG) : 0u;
  bf16x8_t qa[HS][4];  // A operand of each tile
  f32x4_t qsum[HS];    // the sums of q~ of the group
  auto load_q = [&](int gr) { lane_operands<HS>(s_qt + gr * HS * 128, qa, qsum); };
  // a step's base-2 logits (pass 0), or those minus the maxima (pass 1), of the thread's tokens
  auto finish = [&](float (&l)[TPT][G], int st) {
    const int j = j0 + st * STEP + tid;
    const bool full = j0 + (st + 1) * STEP <= n;  // uniform
    if constexpr (!KEYS) {
      if (!full) {
#pragma unroll
        for (int t = 0; t < TPT; ++t)
#pragma unroll
          for (int h = 0; h < G; ++h) l[t][h] = j + t * kDsThreads < n ? l[t][h] : -INFINITY;
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float mn = m[h];
#pragma unroll
        for (int t = 0; t < TPT; ++t) mn = fmaxf(mn, l[t][h]);
        const float mr = mn == -INFINITY ? 0.f : mn;  // no valid token yet: every exponential is 0
        float zz = z[h] * __builtin_amdgcn_exp2f(m[h] - mr);
#pragma unroll
        for (int t = 0; t < TPT; ++t) zz += __builtin_amdgcn_exp2f(l[t][h] - mr);
        z[h] = zz;
        m[h] = mn;
      }
    } else {
#pragma unroll
      for (int t = 0; t < TPT; ++t) {
        float a = 0.f;
#pragma unroll
        for (int h = 0; h < G; ++h) a = fmaf(__builtin_amdgcn_exp2f(l[t][h]), z[h], a);
        if (full || j + t * kDsThreads < n) {
          const uint32_t key = alpha_key(a * invG);
          keys[ubase + j + t * kDsThreads] = key;
          ds_count_key(s_hist, key, bound);
        }
      }
    }
  };
  if constexpr (NGR == 1) {
    load_q(0);
#pragma unroll
    for (int st = 0; st < kDsSteps; ++st) {
      if (j0 + st * STEP >= n) break;  // uniform
      if (st + 1 < kDsSteps && j0 + (st + 1) * STEP < n) request(cw[(st + 1) & 1], pr[(st + 1) & 1], st + 1, 0);
      __builtin_amdgcn_sched_barrier(0);
      float l[TPT][G];
#pragma unroll
      for (int t = 0; t < TPT; ++t) {
        f32x4_t acc[HS];
        lane_dots<HS>(cw[st & 1][t], qa, acc);
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const float qs = qsum[h / 4][h % 4];
          const float v = sigma2 * fmaf(pr[st & 1][t].x, acc[h / 4][h % 4], pr[st & 1][t].y * qs);
          l[t][h] = KEYS ? v - m[h] : v;
        }
      }
      finish(l, st);
    }
  } else {
    for (int st = 0; st < kDsSteps; ++st) {
      if (j0 + st * STEP >= n) break;  // uniform
      float l[TPT][G];
#pragma unroll
      for (int t = 0; t < TPT; ++t)
#pragma unroll
        for (int h = 0; h < G; ++h) l[t][h] = 0.f;
#pragma unroll 1
      for (int gr = 0; gr < ngr; ++gr) {
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
          cw[1][t] = cw[0][t];
          pr[1][t] = pr[0][t];
        }
        const int gr1 = gr + 1 == ngr ? 0 : gr + 1, st1 = gr1 == 0 ? st + 1 : st;
        if (st1 < kDsSteps && j0 + st1 * STEP < n) request(cw[0], pr[0], st1, gr1);
        __builtin_amdgcn_sched_barrier(0);
        load_q(gr);
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
          f32x4_t acc[HS];
          lane_dots<HS>(cw[1][t], qa, acc);
#pragma unroll
          for (int h = 0; h < G; ++h) {
            const float qs = qsum[h / 4][h % 4];
            l[t][h] += fmaf(pr[1][t].x, acc[h / 4][h % 4], pr[1][t].y * qs);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < TPT; ++t)
#pragma unroll
        for (int h = 0; h < G; ++h) l[t][h] = KEYS ? sigma2 * l[t][h] - m[h] : sigma2 * l[t][h];
      finish(l, st);
    }
  }
  if constexpr (KEYS) {
    ds_flush_hist(s_hist, hist, unit, chunk, bound);
  } else {
    // this chunk's maximum and sum of exponentials per head
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float M = wave_max_f32(m[h]);
      const float Z = wave_sum_f32(z[h] == 0.f ? 0.f : z[h] * __builtin_amdgcn_exp2f(m[h] - (M == -INFINITY ? 0.f : M)));
      if (lane == 0) {
        s_red[wid][h][0] = M;
        s_red[wid][h][1] = Z;
      }
    }
    __syncthreads();
    if (tid < G) {
      float M = s_red[0][tid][0], Z = 0.f;
#pragma unroll
      for (int w = 1; w < kDsNW; ++w) M = fmaxf(M, s_red[w][tid][0]);
#pragma unroll
      for (int w = 0; w < kDsNW; ++w)
        if (s_red[w][tid][0] != -INFINITY) Z += s_red[w][tid][1] * __builtin_amdgcn_exp2f(s_red[w][tid][0] - M);
      float* sp = stats + ((size_t(unit) * nchunks + chunk) * G + tid) * 2;
      sp[0] = M;
      sp[1] = Z;
    }
  }
}

// ---------------------------------------------------------------------------
// bf16, G = 16 HT (absorbed MLA), d_c = 32 NGR: the contraction on
// v_mfma_f32_16x16x32_bf16 as in token_score_mfma_kernel (A = 16 heads' q~ of
// one group, B = 16 tokens' codes).  A wave walks its tiles of 16 tokens TL
// at a time; lane (lg, t16) of a result holds token t16 for heads 4lg + r.
// ---------------------------------------------------------------------------
constexpr int kDsWideChunk = 1024;  // tokens per work-group

template <int HT, int NGR, bool KEYS>
__global__ __launch_bounds__(kDsThreads, 2) void ds_score_wide_kernel(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int d, int T,
    float sigma, int nchunks, float* __restrict__ stats, uint32_t* __restrict__ keys, uint32_t* __restrict__ hist,
    uint32_t* err) {
  constexpr int G = 16 * HT, DC = 32 * NGR, TL = NGR == 4 ? 2 : 4;
  constexpr int STEPS = kDsWideChunk / (kDsNW * TL * 16);
  __shared__ __attribute__((aligned(16))) uint16_t s_qt[G * DC];  // [head][group][lane group][8]
  __shared__ float s_red[kDsNW][G][2], s_mz[G][2];
  __shared__ uint32_t s_hist[KEYS ? kTopkHistWords : 1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int t16 = lane & 15, lg = lane >> 4;
  const int unit = KEYS ? int(gridDim.y - 1 - blockIdx.y) : int(blockIdx.y);  // as in ds_score_mfma_kernel
  const int chunk = KEYS ? int(gridDim.x - 1 - blockIdx.x) : int(blockIdx.x);
  const int s = unit / H_kv, g = unit % H_kv;
  int n = ctx_lens[s];
  if (n < 0 || n > T) {
    if (tid == 0 && chunk == 0) set_error(err, 1u);
    n = n < 0 ? 0 : T;
  }
  if (!KEYS && chunk == 0) ds_clear_hist(hist, unit);
  const int j0 = chunk * kDsWideChunk;
  if (j0 >= n) return;
  const size_t ubase = size_t(unit) * T;
  uint32_t cx[TL][NGR];
  float2 pq[TL][NGR];
  // tile tl of step st: tokens j0 + (st * 4 + wid) * 16 TL + tl * 16 + t16
  auto request = [&](int st) {
#pragma unroll
    for (int tl = 0; tl < TL; ++tl) {
      const int j = j0 + (st * kDsNW + wid) * (TL * 16) + tl * 16 + t16;
      const size_t row = ubase + size_t(min(j, n - 1));
#pragma unroll
      for (int gr = 0; gr < NGR; ++gr) {
        cx[tl][gr] = *reinterpret_cast<const uint32_t*>(codes + row * (DC / 2) + gr * 16 + lg * 4);
        pq[tl][gr] = *reinterpret_cast<const float2*>(qparams + (row * NGR + gr) * 2);
      }
    }
  };
  request(0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (KEYS) {
    for (int i = tid; i < kTopkHistWords; i += kDsThreads) s_hist[i] = 0u;
  }
  {
    // thread t holds q~ positions t % DC of heads t / DC + j (256 / DC)
    static_assert(kDsThreads % DC == 0 && G * DC % kDsThreads == 0, "q~ entries per thread");
    const int x = tid % DC;
    int ch = channels[g * DC + (x & ~7) + codes_chan(x & 7)];
    if (ch < 0 || ch >= d) {
      set_error(err, 32u);
      ch = 0;
    }
#pragma unroll
    for (int j = 0; j < G * DC / kDsThreads; ++j)
      s_qt[tid + j * kDsThreads] = q[(size_t(s) * H_q + size_t(g) * G + j * (kDsThreads / DC) + tid / DC) * d + ch];
  }
  if constexpr (KEYS)
    ds_unit_norm<G>(stats + size_t(unit) * nchunks * G * 2, (n + kDsWideChunk - 1) / kDsWideChunk, s_red, s_mz);
  lds_barrier();
  bf16x8_t qa[HT][NGR];
  f32x4_t qs[HT][NGR];  // sums of q~ of heads ht*16 + 4lg + r (B = 1)
  const bf16x8_t one = __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
#pragma unroll
  for (int ht = 0; ht < HT; ++ht)
#pragma unroll
    for (int gr = 0; gr < NGR; ++gr) {
      qa[ht][gr] = *reinterpret_cast<const bf16x8_t*>(&s_qt[(ht * 16 + t16) * DC + gr * 32 + lg * 8]);
      qs[ht][gr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ht][gr], one, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
  const float sigma2 = sigma * 1.4426950408889634f;
  const float invG = 1.0f / float(G);
  float m[HT][4], z[HT][4];  // running maximum and sum (pass 0), or the unit's maximum and 1/Z (pass 1)
  float bsum = 0.f;
#pragma unroll
  for (int ht = 0; ht < HT; ++ht)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m[ht][r] = KEYS ? s_mz[ht * 16 + lg * 4 + r][0] : -INFINITY;
      z[ht][r] = KEYS ? s_mz[ht * 16 + lg * 4 + r][1] : 0.f;
      if constexpr (KEYS) bsum = fmaf(1.0f, z[ht][r], bsum);
    }
  const uint32_t bound = KEYS ? alpha_key(xrows_sum(bsum) * invG) : 0u;  // summed in the keys' own order
#pragma unroll 1
  for (int st = 0; st < STEPS; ++st) {
    if (j0 + st * kDsNW * TL * 16 >= n) break;  // uniform
    float lgt[TL][HT][4];
#pragma unroll
    for (int tl = 0; tl < TL; ++tl) {
      const bool ok = j0 + (st * kDsNW + wid) * (TL * 16) + tl * 16 + t16 < n;
      float v[HT][4];
#pragma unroll
      for (int ht = 0; ht < HT; ++ht)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[ht][r] = 0.f;
#pragma unroll
      for (int gr = 0; gr < NGR; ++gr) {
        const bf16x8_t b = __builtin_bit_cast(bf16x8_t, codes_bf16(cx[tl][gr]));
        const float sc = pq[tl][gr].x, mn = pq[tl][gr].y;
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) {
          const f32x4_t acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ht][gr], b, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[ht][r] += fmaf(sc, acc[r], mn * qs[ht][gr][r]);
        }
      }
#pragma unroll
      for (int ht = 0; ht < HT; ++ht)
#pragma unroll
        for (int r = 0; r < 4; ++r) lgt[tl][ht][r] = ok ? sigma2 * v[ht][r] : -INFINITY;
    }
    if (st + 1 < STEPS) request(st + 1);  // clamped rows: in range also past the end
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!KEYS) {
#pragma unroll
      for (int ht = 0; ht < HT; ++ht)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float mn = m[ht][r];
#pragma unroll
          for (int tl = 0; tl < TL; ++tl) mn = fmaxf(mn, lgt[tl][ht][r]);
          if (mn != -INFINITY) {
            float zz = m[ht][r] == -INFINITY ? 0.f : z[ht][r] * __builtin_amdgcn_exp2f(m[ht][r] - mn);
#pragma unroll
            for (int tl = 0; tl < TL; ++tl) zz += __builtin_amdgcn_exp2f(lgt[tl][ht][r] - mn);
            z[ht][r] = zz;
            m[ht][r] = mn;
          }
        }
    } else {
#pragma unroll
      for (int tl = 0; tl < TL; ++tl) {
        float a = 0.f;
#pragma unroll
        for (int ht = 0; ht < HT; ++ht)
#pragma unroll
          for (int r = 0; r < 4; ++r) a = fmaf(__builtin_amdgcn_exp2f(lgt[tl][ht][r] - m[ht][r]), z[ht][r], a);
        a = xrows_sum(a);
        const int j = j0 + (st * kDsNW + wid) * (TL * 16) + tl * 16 + t16;
        if (lg == tl && j < n) {
          const uint32_t key = alpha_key(a * invG);
          keys[ubase + j] = key;
          ds_count_key(s_hist, key, bound);
        }
      }
    }
  }
  if constexpr (KEYS) {
    ds_flush_hist(s_hist, hist, unit, chunk, bound);
  } else {
    // combine the 16 token lanes of each head, then the waves
#pragma unroll
    for (int ht = 0; ht < HT; ++ht)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float mm = m[ht][r], zz = z[ht][r];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
          const float m2 = __shfl_xor(mm, o, 64), z2 = __shfl_xor(zz, o, 64);
          const float mn = fmaxf(mm, m2);
          if (mn != -INFINITY)
            zz = (mm == -INFINITY ? 0.f : zz * __builtin_amdgcn_exp2f(mm - mn)) +
                 (m2 == -INFINITY ? 0.f : z2 * __builtin_amdgcn_exp2f(m2 - mn));
          mm = mn;
        }
        if (t16 == 0) {
          s_red[wid][ht * 16 + lg * 4 + r][0] = mm;
          s_red[wid][ht * 16 + lg * 4 + r][1] = zz;
        }
      }
    __syncthreads();
    if (tid < G) {
      float mm = s_red[0][tid][0], zz = 0.f;
#pragma unroll
      for (int w = 1; w < kDsNW; ++w) mm = fmaxf(mm, s_red[w][tid][0]);
#pragma unroll
      for (int w = 0; w < kDsNW; ++w)
        if (s_red[w][tid][0] != -INFINITY) zz += s_red[w][tid][1] * __builtin_amdgcn_exp2f(s_red[w][tid][0] - mm);
      float* sp = stats + ((size_t(unit) * nchunks + chunk) * G + tid) * 2;
      sp[0] = mm;
      sp[1] = zz;
    }
  }
}

template <int G>
__host__ __device__ constexpr int ds_tpt() { return G <= 8 ? 4 : 1; }  // tokens per thread
template <int G>
__host__ __device__ constexpr int ds_chunk() { return kDsThreads * ds_tpt<G>(); }

template <class E, int G>
__global__ __launch_bounds__(kDsThreads) void ds_score_kernel(
    const typename E::T* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int d, int d_c,
    int T, float sigma, int pass, int nchunks, float* __restrict__ stats, uint32_t* __restrict__ keys,
    uint32_t* __restrict__ hist, uint32_t* err) {
  constexpr int TPT = ds_tpt<G>();
  constexpr int CH = ds_chunk<G>();
  __shared__ __attribute__((aligned(16))) float s_q[kDsMaxDc * G];  // [channel][head]
  __shared__ float s_qs[(kDsMaxDc / 32) * G];                       // [group][head]: sum of q~ over the group
  __shared__ float s_red[kDsNW][G][2];
  __shared__ float s_mz[G][2];
  __shared__ float s_tmp[kDsThreads];
  __shared__ int s_ch[kDsMaxDc];
  __shared__ uint32_t s_hist[kTopkHistWords];
  const int chunk = blockIdx.x, unit = blockIdx.y;
  const int s = unit / H_kv, g = unit % H_kv;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  int n = ctx_lens[s];
  if (n < 0 || n > T) {
    if (tid == 0 && chunk == 0) set_error(err, 1u);
    n = n < 0 ? 0 : T;
  }
  const int j0 = chunk * CH;
  if (pass == 0 && chunk == 0) ds_clear_hist(hist, unit);
  if (pass == 1 && j0 >= n) return;
  if (pass == 1)
    for (int i = tid; i < kTopkHistWords; i += kDsThreads) s_hist[i] = 0u;
  const int ngr = d_c / 32;
  // the group's channel ids once (every head uses the same), then the q~ gather
  for (int c = tid; c < d_c; c += kDsThreads) {
    int ch = channels[g * d_c + c];
    if (ch < 0 || ch >= d) {
      set_error(err, 32u);
      ch = 0;
    }
    s_ch[c] = ch;
  }
  __syncthreads();
  for (int i = tid; i < G * d_c; i += kDsThreads) {
    const int h = i / d_c, c = i % d_c;
    s_q[c * G + h] = E::to_f(q[(size_t(s) * H_q + size_t(g) * G + h) * d + s_ch[c]]);
  }
  __syncthreads();
  for (int i = tid; i < G * ngr; i += kDsThreads) {
    const int gr = i / G, h = i % G;
    float a = 0.f;
    for (int c = 0; c < 32; ++c) a += s_q[(gr * 32 + c) * G + h];
    s_qs[gr * G + h] = a;
  }
  // the unit's normalisers from every chunk (pass 1): thread t folds chunks
  // t / G, t / G + 256 / G, ... of head t % G, then the partials of each head
  // are combined in a fixed order
  if (pass == 1) {
    const int h = tid % G, ks = kDsThreads / G;
    const float* st = stats + size_t(unit) * nchunks * G * 2;
    float M = -INFINITY;
#pragma unroll 4
    for (int c = tid / G; c < nchunks; c += ks) M = fmaxf(M, st[(c * G + h) * 2]);
    s_tmp[tid] = M;
    __syncthreads();
    if (tid < G) {
      float m = -INFINITY;
      for (int k = 0; k < ks; ++k) m = fmaxf(m, s_tmp[k * G + tid]);
      s_mz[tid][0] = m;
    }
    __syncthreads();
    M = s_mz[h][0];
    float Z = 0.f;
    if (M != -INFINITY) {
#pragma unroll 4
      for (int c = tid / G; c < nchunks; c += ks) {
        const float mc = st[(c * G + h) * 2], zc = st[(c * G + h) * 2 + 1];
        if (mc != -INFINITY) Z += zc * __builtin_amdgcn_exp2f(mc - M);
      }
    }
    s_tmp[tid] = Z;
    __syncthreads();
    if (tid < G) {
      float z = 0.f;
      for (int k = 0; k < ks; ++k) z += s_tmp[k * G + tid];
      s_mz[tid][1] = z > 0.f ? 1.0f / z : 0.f;
    }
  }
  __syncthreads();

  // base-2 logits of this thread's tokens j0 + tid + t*256 (-inf when invalid)
  const float sigma2 = sigma * 1.4426950408889634f;
  const size_t ubase = size_t(unit) * T;
  const int rowb = d_c / 2;
  float lg[TPT][G];
  bool ok[TPT];
#pragma unroll
  for (int t = 0; t < TPT; ++t) {
    ok[t] = j0 + tid + t * kDsThreads < n;
#pragma unroll
    for (int h = 0; h < G; ++h) lg[t][h] = 0.f;
  }
  for (int gr = 0; gr < ngr; ++gr) {
    uint4 cw[TPT];
    float2 pr[TPT];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
      const size_t row = ubase + size_t(ok[t] ? j0 + tid + t * kDsThreads : 0);
      cw[t] = ld16_stream(codes + row * rowb + gr * 16);
      pr[t] = *reinterpret_cast<const float2*>(qparams + (row * ngr + gr) * 2);
    }
    float dot[TPT][G];
#pragma unroll
    for (int t = 0; t < TPT; ++t)
#pragma unroll
      for (int h = 0; h < G; ++h) dot[t][h] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // byte b of the dword holds channels 2b (low nibble) and 2b + 1
        const int c = gr * 32 + w * 8 + e;
        const int sh = (e >> 1) * 8 + (e & 1) * 4;
        float qv[G];
        if constexpr (G % 4 == 0) {
#pragma unroll
          for (int h = 0; h < G; h += 4) {  // 16-byte aligned: G is a multiple of 4
            const float4 v = *reinterpret_cast<const float4*>(&s_q[c * G + h]);
            qv[h] = v.x;
            qv[h + 1] = v.y;
            qv[h + 2] = v.z;
            qv[h + 3] = v.w;
          }
        } else {
#pragma unroll
          for (int h = 0; h < G; ++h) qv[h] = s_q[c * G + h];
        }
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
          const uint32_t wd = w == 0 ? cw[t].x : (w == 1 ? cw[t].y : (w == 2 ? cw[t].z : cw[t].w));
          const float code = float((wd >> sh) & 15u);
#pragma unroll
          for (int h = 0; h < G; ++h) dot[t][h] = fmaf(qv[h], code, dot[t][h]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TPT; ++t)
#pragma unroll
      for (int h = 0; h < G; ++h) lg[t][h] += fmaf(pr[t].y, s_qs[gr * G + h], pr[t].x * dot[t][h]);
  }
#pragma unroll
  for (int t = 0; t < TPT; ++t)
#pragma unroll
    for (int h = 0; h < G; ++h) lg[t][h] = ok[t] ? sigma2 * lg[t][h] : -INFINITY;

  if (pass == 0) {
    // this chunk's maximum and sum of exponentials per head
    float mx[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float m = -INFINITY;
#pragma unroll
      for (int t = 0; t < TPT; ++t) m = fmaxf(m, lg[t][h]);
      mx[h] = wave_max_f32(m);
      if (lane == 0) s_red[wid][h][0] = mx[h];
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float m = s_red[0][h][0];
#pragma unroll
      for (int w = 1; w < kDsNW; ++w) m = fmaxf(m, s_red[w][h][0]);
      mx[h] = m;
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float z = 0.f;
      if (mx[h] != -INFINITY)
#pragma unroll
        for (int t = 0; t < TPT; ++t) z += __builtin_amdgcn_exp2f(lg[t][h] - mx[h]);
      z = wave_sum_f32(z);
      if (lane == 0) s_red[wid][h][1] = z;
    }
    __syncthreads();
    if (tid < G) {
      float m = s_red[0][tid][0], z = 0.f;
      for (int w = 1; w < kDsNW; ++w) m = fmaxf(m, s_red[w][tid][0]);
      for (int w = 0; w < kDsNW; ++w) z += s_red[w][tid][1];
      float* st = stats + ((size_t(unit) * nchunks + chunk) * G + tid) * 2;
      st[0] = m;
      st[1] = z;
    }
    return;
  }
  // pass 1: alpha keys (a NaN alpha, from NaN inputs, ranks as 0)
  const float invG = 1.0f / float(G);
  float bsum = 0.f;
#pragma unroll
  for (int h = 0; h < G; ++h) bsum = fmaf(1.0f, s_mz[h][1], bsum);
  const uint32_t bound = alpha_key(bsum * invG);
#pragma unroll
  for (int t = 0; t < TPT; ++t) {
    const int j = j0 + tid + t * kDsThreads;
    if (j >= n) continue;
    float a = 0.f;
#pragma unroll
    for (int h = 0; h < G; ++h) a = fmaf(__builtin_amdgcn_exp2f(lg[t][h] - s_mz[h][0]), s_mz[h][1], a);
    const uint32_t key = alpha_key(a * invG);
    keys[ubase + j] = key;
    ds_count_key(s_hist, key, bound);
  }
  ds_flush_hist(s_hist, hist, unit, chunk, bound);
}

// One work-group per unit.  With the bucket counts of pass 1 the bucket of the
// K_t-th key is known at once; one pass over the keys (16 per thread, the next
// 16 requested before the last are compacted) lists the positions of the keys
// at or above its lower end in order, and the selection finishes on those keys
// in registers.  The pass has no barrier: a ballot per 64 keys leaves their
// candidate mask in LDS, and once per 262144 keys each thread expands the masks
// of four groups at most behind one prefix sum.  At 128 units of 73k keys: 60 us
// for a radix pass at a time, 27 with an ordered compaction (two barriers) per
// 16384 keys, 20.7 so; 32 keys per thread in flight: 21-23.
// Without counts, where every key is selected, where the bucket is the lowest
// (it also holds everything below 32 octaves) or the highest (it also holds
// everything above: a key exceeds the bound by the rounding of its logits,
// which pass 1 computes without pass 0's rounding of the product with sigma,
// i.e. by octaves where they are above 2^22), or where more candidates than
// kDsListCap remain, the keys are streamed once per radix pass.
template <int EPT>
__device__ inline void ds_select_list(const uint32_t* keys, const int32_t* list, int cnt, int K_t, int32_t* out,
                                      uint32_t* scratch, const TopkStart& start) {
  uint32_t kr[EPT];
  int32_t pos[EPT];
#pragma unroll
  for (int j = 0; j < EPT; ++j) {
    const int i = int(threadIdx.x) + j * kDsTopkThreads;
    pos[j] = list[min(i, cnt - 1)];
  }
#pragma unroll
  for (int j = 0; j < EPT; ++j) {
    const int i = int(threadIdx.x) + j * kDsTopkThreads;
    const uint32_t key = keys[pos[j]];
    kr[j] = i < cnt ? key : kInvalidKey;
  }
  wg_topk_resume<kDsTopkThreads, EPT>(kr, K_t, out, K_t, [&](int j, int) { return pos[j]; }, scratch, start);
}

__global__ __launch_bounds__(kDsTopkThreads) void ds_topk_kernel(const uint32_t* __restrict__ keys,
                                                                  const uint32_t* __restrict__ hist,
                                                                  const int32_t* __restrict__ ctx_lens, int H_kv,
                                                                  int T, int K_t, int32_t* __restrict__ token_ids,
                                                                  uint32_t* arrive) {
  constexpr int NT = kDsTopkThreads, EPT = kTopkMaxEPT, TILE = NT * EPT;
  extern __shared__ uint32_t smem[];
  uint32_t* scratch = smem;
  uint32_t* list = smem + topk_scratch_words(NT);
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (arrive && tid == 0) arrive[unit] = 0u;
  int n = ctx_lens[unit / H_kv];
  n = n < 0 ? 0 : (n > T ? T : n);
  const uint32_t* uk = keys + size_t(unit) * T;
  int32_t* out = token_ids + size_t(unit) * K_t;
  if (hist && n > K_t) {
    const uint32_t* h = hist + size_t(unit) * kDsHistWords;
    // group j of wave w in batch t: positions t TILE + (16 w + j) 64 + lane
    uint32_t kr[EPT];
    auto request = [&](int t) {
#pragma unroll
      for (int j = 0; j < EPT; ++j) kr[j] = uk[min(t * TILE + (wid * EPT + j) * 64 + lane, n - 1)];
    };
    request(0);
    // the bucket: lane L of every wave holds buckets 255 - 4L .. 252 - 4L
    const uint4 c = *reinterpret_cast<const uint4*>(h + 252 - 4 * lane);
    const uint32_t bound = h[256];
    const uint32_t c0 = c.w, c1 = c0 + c.z, c2 = c1 + c.y, c3 = c2 + c.x;
    const uint32_t incl = wave_incl_scan_u32(c3), excl = incl - c3;
    const uint32_t kt = uint32_t(K_t);
    // (the counts cover every key and n > K_t, so some lane reaches K_t)
    const int src = __ffsll((unsigned long long)__ballot(incl >= kt)) - 1;
    const int q = excl + c0 >= kt ? 0 : (excl + c1 >= kt ? 1 : (excl + c2 >= kt ? 2 : 3));
    const uint32_t before = excl + (q == 0 ? 0u : (q == 1 ? c0 : (q == 2 ? c1 : c2)));
    const uint32_t here = q == 0 ? c.w : (q == 1 ? c.z : (q == 2 ? c.y : c.x));
    const int digit = __builtin_amdgcn_readlane(255 - 4 * lane - q, src);
    const uint32_t above = uint32_t(__builtin_amdgcn_readlane(int(before), src));
    const uint32_t bucket = uint32_t(__builtin_amdgcn_readlane(int(here), src));
    const int cnt = int(above + bucket);
    if (digit > 0 && digit < 255 && cnt <= kDsListCap) {
      const uint32_t lowest = uint32_t(int(bound >> kTopkSpreadShift) - 254 + digit) << kTopkSpreadShift;
      uint32_t* wsum = scratch + align4w_c(kTopkPasses * kTopkHistWords);
      uint2* masks = reinterpret_cast<uint2*>(list + kDsListCap);
      topk_prepare<NT>(scratch);
      int base = 0;
      for (int t0 = 0; t0 * TILE < n; t0 += kDsMaskGroups / (EPT * NT / 64)) {
        const int end = min(n, t0 * TILE + kDsMaskGroups * 64);
        for (int t = t0; t * TILE < end; ++t) {
          uint32_t mlo = 0u, mhi = 0u;
          const int p0 = t * TILE + wid * EPT * 64;
#pragma unroll
          for (int j = 0; j < EPT; ++j) {
            const int left = n - (p0 + j * 64);  // keys of the group (uniform)
            const uint64_t m = __ballot(kr[j] >= lowest) & (left >= 64 ? ~0ull : (left > 0 ? (1ull << left) - 1ull : 0ull));
            mlo = lane == j ? uint32_t(m) : mlo;
            mhi = lane == j ? uint32_t(m >> 32) : mhi;
          }
          if ((t + 1) * TILE < n) request(t + 1);
          if (lane < EPT) masks[(t - t0) * (TILE / 64) + wid * EPT + lane] = make_uint2(mlo, mhi);
        }
        __syncthreads();
        const int groups = (end - t0 * TILE + 63) / 64, per = (groups + NT - 1) / NT;
        uint64_t m[kDsMaskGroups / NT];
        int c = 0;
#pragma unroll
        for (int i = 0; i < kDsMaskGroups / NT; ++i) {
          const int g = tid * per + i;
          const bool ok = i < per && g < groups;
          const uint2 w = masks[ok ? g : 0];
          m[i] = ok ? uint64_t(w.y) << 32 | w.x : 0ull;
          c += __popcll(m[i]);
        }
        const uint32_t incl_c = wave_incl_scan_u32(uint32_t(c));
        if (lane == 63) wsum[wid] = incl_c;
        __syncthreads();
        const uint32_t ws = wsum[lane & 15];
        const uint32_t wincl = wave_incl_scan_u32(lane < NT / 64 ? ws : 0u);
        int off = base + int(incl_c) - c + (wid ? __builtin_amdgcn_readlane(int(wincl), wid - 1) : 0);
        base += __builtin_amdgcn_readlane(int(wincl), NT / 64 - 1);
#pragma unroll
        for (int i = 0; i < kDsMaskGroups / NT; ++i) {
          const int p = t0 * TILE + (tid * per + i) * 64;
          for (uint64_t w = m[i]; w; w &= w - 1) list[off++] = uint32_t(p + __builtin_ctzll(w));
        }
        __syncthreads();  // the masks are rewritten by the next round; the list is complete after the last
      }
      const TopkStart start{lowest, K_t - int(above), int(bucket)};
      const int32_t* pos = reinterpret_cast<const int32_t*>(list);
      if (cnt <= 4 * NT) ds_select_list<4>(uk, pos, cnt, K_t, out, scratch, start);
      else if (cnt <= 8 * NT) ds_select_list<8>(uk, pos, cnt, K_t, out, scratch, start);
      else ds_select_list<16>(uk, pos, cnt, K_t, out, scratch, start);
      return;
    }
  }
  wg_topk_global<kDsTopkThreads>(uk, n, K_t, out, K_t, scratch, list, kDsListCap);
}

// Which kernel computes the passes.
static bool ds_use_mfma(const Problem& P) { return P.dtype == 1 && P.G <= 8; }
static bool ds_use_wide(const Problem& P) {
  return P.dtype == 1 && (P.G == 16 || P.G == 32) && (P.d_c == 64 || P.d_c == 128);
}

static int ds_chunk_tokens(const Problem& P) {
  if (ds_use_mfma(P)) return kDsMfmaChunk;
  if (ds_use_wide(P)) return kDsWideChunk;
  return P.G <= 8 ? ds_chunk<8>() : ds_chunk<16>();
}

size_t ds_stats_floats(const Problem& P) {
  const int ch = ds_chunk_tokens(P);
  return size_t(P.units) * ((P.T + ch - 1) / ch) * P.G * 2;
}

size_t ds_hist_words(const Problem& P) { return size_t(P.units) * kDsHistWords; }

bool ds_supported(const Problem& P) {
  return (P.G == 1 || P.G == 2 || P.G == 4 || P.G == 8 || P.G == 16 || P.G == 32) && P.d_c <= kDsMaxDc;
}

struct DsArgs {
  const void* q;
  const uint8_t* codes;
  const float* qparams;
  const int32_t* channels;
  const int32_t* ctx_lens;
  float* stats;
  uint32_t* keys;
  uint32_t* hist;
  uint32_t* err;
};

template <class E, int G>
static void launch_ds_vector(const Problem& P, const DsArgs& a, dim3 grid, int nchunks, hipStream_t st) {
  using S = typename E::T;
  for (int pass = 0; pass < 2; ++pass)
    ds_score_kernel<E, G><<<grid, kDsThreads, 0, st>>>((const S*)a.q, a.codes, a.qparams, a.channels, a.ctx_lens, P.H_q,
                                                       P.H_kv, P.d_qk, P.d_c, P.T, P.sigma, pass, nchunks, a.stats,
                                                       a.keys, a.hist, a.err);
}

template <int G, int NGR>
static void launch_ds_mfma_n(const Problem& P, const DsArgs& a, dim3 grid, int nchunks, hipStream_t st) {
  ds_score_mfma_kernel<G, NGR, false><<<grid, kDsThreads, 0, st>>>(
      (const uint16_t*)a.q, a.codes, a.qparams, a.channels, a.ctx_lens, P.H_q, P.H_kv, P.d_qk, P.d_c, P.T, P.sigma,
      nchunks, a.stats, a.keys, a.hist, a.err);
  ds_score_mfma_kernel<G, NGR, true><<<grid, kDsThreads, 0, st>>>(
      (const uint16_t*)a.q, a.codes, a.qparams, a.channels, a.ctx_lens, P.H_q, P.H_kv, P.d_qk, P.d_c, P.T, P.sigma,
      nchunks, a.stats, a.keys, a.hist, a.err);
}

template <int G>
static void launch_ds_mfma(const Problem& P, const DsArgs& a, dim3 grid, int nchunks, hipStream_t st) {
  if (P.d_c == 32) launch_ds_mfma_n<G, 1>(P, a, grid, nchunks, st);
  else launch_ds_mfma_n<G, 0>(P, a, grid, nchunks, st);
}

template <int HT, int NGR>
static void launch_ds_wide(const Problem& P, const DsArgs& a, dim3 grid, int nchunks, hipStream_t st) {
  ds_score_wide_kernel<HT, NGR, false><<<grid, kDsThreads, 0, st>>>(
      (const uint16_t*)a.q, a.codes, a.qparams, a.channels, a.ctx_lens, P.H_q, P.H_kv, P.d_qk, P.T, P.sigma, nchunks,
      a.stats, a.keys, a.hist, a.err);
  ds_score_wide_kernel<HT, NGR, true><<<grid, kDsThreads, 0, st>>>(
      (const uint16_t*)a.q, a.codes, a.qparams, a.channels, a.ctx_lens, P.H_q, P.H_kv, P.d_qk, P.T, P.sigma, nchunks,
      a.stats, a.keys, a.hist, a.err);
}

hipError_t launch_token_select_dense(const Problem& P, const void* q, const uint8_t* codes, const float* qparams,
                                     const int32_t* channels, const int32_t* ctx_lens, int K_t, float* stats,
                                     uint32_t* keys, uint32_t* hist, int32_t* token_ids, uint32_t* arrive,
                                     uint32_t* err, hipStream_t st) {
  if (!ds_supported(P)) return hipErrorInvalidValue;
  const DsArgs a{q, codes, qparams, channels, ctx_lens, stats, keys, hist, err};
  const int ch = ds_chunk_tokens(P), nchunks = (P.T + ch - 1) / ch;
  const dim3 grid(nchunks, P.units);
  if (ds_use_mfma(P)) {
    switch (P.G) {
      case 1: launch_ds_mfma<1>(P, a, grid, nchunks, st); break;
      case 2: launch_ds_mfma<2>(P, a, grid, nchunks, st); break;
      case 4: launch_ds_mfma<4>(P, a, grid, nchunks, st); break;
      default: launch_ds_mfma<8>(P, a, grid, nchunks, st); break;
    }
  } else if (ds_use_wide(P)) {
    if (P.G == 32 && P.d_c == 128) launch_ds_wide<2, 4>(P, a, grid, nchunks, st);
    else if (P.G == 32) launch_ds_wide<2, 2>(P, a, grid, nchunks, st);
    else if (P.d_c == 128) launch_ds_wide<1, 4>(P, a, grid, nchunks, st);
    else launch_ds_wide<1, 2>(P, a, grid, nchunks, st);
  } else if (P.dtype == 1) {
    if (P.G == 16) launch_ds_vector<BF16, 16>(P, a, grid, nchunks, st);
    else launch_ds_vector<BF16, 32>(P, a, grid, nchunks, st);
  } else {
    switch (P.G) {
      case 1: launch_ds_vector<F32, 1>(P, a, grid, nchunks, st); break;
      case 2: launch_ds_vector<F32, 2>(P, a, grid, nchunks, st); break;
      case 4: launch_ds_vector<F32, 4>(P, a, grid, nchunks, st); break;
      case 8: launch_ds_vector<F32, 8>(P, a, grid, nchunks, st); break;
      case 16: launch_ds_vector<F32, 16>(P, a, grid, nchunks, st); break;
      default: launch_ds_vector<F32, 32>(P, a, grid, nchunks, st); break;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = (size_t(topk_scratch_words(kDsTopkThreads)) + kDsListCap + 2 * kDsMaskGroups) * sizeof(uint32_t);
  e = allow_dynamic_lds(reinterpret_cast<const void*>(ds_topk_kernel), lds);
  if (e != hipSuccess) return e;
  ds_topk_kernel<<<P.units, kDsTopkThreads, lds, st>>>(keys, hist, ctx_lens, P.H_kv, P.T, K_t, token_ids, arrive);
  return hipGetLastError();
}

}  // namespace tls
