// Fine token selection inside the selected blocks (AsyncTLS Sec. 4.1).
//
// Candidate slots of a unit: slot = i*B + o for the i-th entry of its block
// list and offset o; the slot is a valid candidate when that entry is a
// block id >= 0 and token id*B + o < ctx_len.  With an ascending block list,
// slot order is token order, so lowest-slot tie-breaking is lowest-position
// tie-breaking.
//
// token_score_*_kernel: per slot and head, l = sigma * q~_h . dequant(code_j)
//   (mfma: bf16 with 16 or 32 heads; lane: bf16 up to 8 heads; row: 1, 2, 4 or
//   8 heads on the vector units, the fp32 layout; token_score_kernel: the rest).
//   With dequant = min + code*scale per 32-channel group this is
//   sigma * sum_grp (min_grp * sum_c q~_hc + scale_grp * sum_c q~_hc code_c):
//   the integer codes enter the dot product directly.  Also emits each
//   work-group's per-head (max, sum exp) of its slots.
// token_alpha_topk_kernel: per-head normalisers over all candidates, then
//   alpha_j = (1/G) sum_h exp(l_hj - m_h) / Z_h as an orderable key, and the
//   K_t largest alpha as ascending token positions (4 or 8 heads; 16 or 32 with
//   up to 1024 candidates; otherwise token_alpha_kernel(_g), token_topk_kernel).
#include <type_traits>

#include "token_common.hpp"

namespace tls {

constexpr int kMaxG = 32;
constexpr int kMaxGroups = 8;  // d_c <= 256

template <class E>
__global__ __launch_bounds__(256) void token_score_kernel(
    const typename E::T* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ block_ids, int K_b,
    const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int G, int d, int d_c, int B, int T, float sigma,
    float* __restrict__ logits, float* __restrict__ stats, uint32_t* __restrict__ kinfo, uint32_t* err) {
  __shared__ float s_qt[kMaxG * 256];
  __shared__ float s_qsum[kMaxG * kMaxGroups];
  __shared__ float s_red[4 * kMaxG];
  __shared__ int s_ch[kMaxGroups * 32];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  if (chunk == 0 && threadIdx.x == 0) kinfo[2 * size_t(unit)] = 0u;  // arrivals of the alpha stage
  const int s = unit / H_kv, g = unit % H_kv;
  int n = ctx_lens[s];
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  const int ngr = d_c / 32;
  const int S = K_b * B;
  const typename E::T* qg = q + (size_t(s) * H_q + size_t(g) * G) * d;
  // the group's channel ids once (every head uses the same), then the q~ gather
  if (threadIdx.x < d_c) {
    int ch = channels[g * d_c + threadIdx.x];
    if (ch < 0 || ch >= d) {  // caller-supplied channel id out of range
      set_error(err, 32u);
      ch = 0;
    }
    s_ch[threadIdx.x] = ch;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < G * d_c; i += 256) {
    const int h = i / d_c, c = i % d_c;
    s_qt[i] = E::to_f(qg[size_t(h) * d + s_ch[c]]);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < G * ngr; i += 256) {
    const int h = i / ngr, gr = i % ngr;
    float acc = 0.f;
    for (int c = 0; c < 32; ++c) acc += s_qt[h * d_c + gr * 32 + c];
    s_qsum[i] = acc;
  }
  __syncthreads();

  const int slot = chunk * kTokenSlotsPerWG + threadIdx.x;
  const int32_t* bl = block_ids + size_t(unit) * K_b;
  int tok = 0;
  const bool valid = slot < S && slot_token(bl, K_b, B, m, n, slot, &tok, err);
  float acc[kMaxG];
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) acc[h] = 0.f;
  if (valid) {
    const size_t row = size_t(unit) * T + tok;
    const uint8_t* crow = codes + row * (d_c / 2);
    const float* prow = qparams + row * ngr * 2;
    for (int gr = 0; gr < ngr; ++gr) {
      const uint4 cw = ld16_stream(crow + gr * 16);
      const float scale = prow[gr * 2 + 0], mn = prow[gr * 2 + 1];
      float cf[32];
      unpack_nibbles8(cw.x, cf + 0);
      unpack_nibbles8(cw.y, cf + 8);
      unpack_nibbles8(cw.z, cf + 16);
      unpack_nibbles8(cw.w, cf + 24);
#pragma unroll
      for (int h = 0; h < kMaxG; ++h) {
        if (h < G) {
          const float* qt = s_qt + h * d_c + gr * 32;
          float dot = 0.f;
#pragma unroll
          for (int c = 0; c < 32; ++c) dot = fmaf(qt[c], cf[c], dot);
          acc[h] += mn * s_qsum[h * ngr + gr] + scale * dot;
        }
      }
    }
  }
  // logits and this work-group's per-head softmax statistics
  float* lg = logits + size_t(unit) * G * S;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) {
    if (h < G) {
      const float l = valid ? sigma * acc[h] : -INFINITY;
      acc[h] = l;
      if (slot < S) lg[size_t(h) * S + slot] = l;
      const float wm = wave_max<64>(l);
      if (lane == 0) s_red[wid * kMaxG + h] = wm;
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) {
    if (h < G) {
      const float M = fmaxf(fmaxf(s_red[h], s_red[kMaxG + h]), fmaxf(s_red[2 * kMaxG + h], s_red[3 * kMaxG + h]));
      acc[h] = (valid && M != -INFINITY) ? __expf(acc[h] - M) : 0.f;
    }
  }
  __syncthreads();
  __shared__ float s_sum[4 * kMaxG];
#pragma unroll
  for (int h = 0; h < kMaxG; ++h) {
    if (h < G) {
      const float ws = wave_sum<64>(acc[h]);
      if (lane == 0) s_sum[wid * kMaxG + h] = ws;
    }
  }
  __syncthreads();
  if (threadIdx.x < G) {
    const int h = threadIdx.x;
    const float M = fmaxf(fmaxf(s_red[h], s_red[kMaxG + h]), fmaxf(s_red[2 * kMaxG + h], s_red[3 * kMaxG + h]));
    const float Z = ((s_sum[h] + s_sum[kMaxG + h]) + s_sum[2 * kMaxG + h]) + s_sum[3 * kMaxG + h];
    float* st = stats + ((size_t(unit) * gridDim.x + chunk) * G + h) * 2;
    st[0] = M;
    st[1] = Z;
  }
}

// One work-group's per-head maximum and sum of exponentials, from its waves'
// (lane 0 of each has written s_red[wave][head] = {max, sum}).
template <int NH>
__device__ inline void write_chunk_stats(const float (*s_red)[NH][2], int G, float* st) {
  __syncthreads();
  if (int(threadIdx.x) < G) {
    const int h = threadIdx.x;
    float M = -INFINITY, Z = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_red[w][h][0]);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (s_red[w][h][0] != -INFINITY) Z += s_red[w][h][1] * __expf(s_red[w][h][0] - M);
    st[2 * h] = M;
    st[2 * h + 1] = Z;
  }
}

// The same for fp32 queries (and index widths without a matrix-core kernel)
// with G = 1, 2, 4 or 8: a latency chain at the sizes it runs at, so the
// loads leave in two rounds (block-list entry, context length and channel ids;
// then q~ and the slot's rows) with one barrier, a row is dequantised in
// registers and meets the heads' q~ of a channel in one LDS read.  fp32 queries
// take sum_c q~_c (min + scale code_c) with each term centred, which rounds
// less than min and scale parts apart (alpha against 64 bits, 4 heads of 128
// channels: 1.22e-7 rms, 1.89e-7 apart).  2 units of 4 heads, 512 slots: 9.4 ->
// 4 us; bf16, 256 units of 8 heads, 96 channels, 8192 slots, the whole selection:
// 202 -> 115.
template <class E, int G>
__global__ __launch_bounds__(256) void token_score_row_kernel(
    const typename E::T* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ block_ids, int K_b,
    const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int d, int d_c, int B, int T, float sigma,
    float* __restrict__ logits, float* __restrict__ stats, uint32_t* __restrict__ kinfo, uint32_t* err) {
  __shared__ __attribute__((aligned(16))) float s_q[kMaxGroups * 32 * G];  // [channel][head]
  __shared__ float s_qs[E::kIsBf16 ? kMaxGroups : 1][G];
  __shared__ float s_red[4][G][2];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  if (chunk == 0 && threadIdx.x == 0) kinfo[2 * size_t(unit)] = 0u;  // arrivals of the alpha stage
  const int s = unit / H_kv, g = unit % H_kv;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int S = K_b * B, ngr = d_c / 32;
  const int slot = chunk * kTokenSlotsPerWG + tid;
  int n = ctx_lens[s];
  const int blk = block_ids[size_t(unit) * K_b + min(tok_block(min(slot, S - 1), B), K_b - 1)];
  int ch = tid < d_c ? channels[g * d_c + tid] : 0;  // d_c <= 256
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  if (ch < 0 || ch >= d) {
    set_error(err, 32u);
    ch = 0;
  }
  if (slot < S && blk >= m) set_error(err, 2u);
  const int tok = blk * B + tok_offset(slot, B);
  const bool valid = slot < S && blk >= 0 && blk < m && tok < n;
  typename E::T qv[G];
  const typename E::T* qg = q + (size_t(s) * H_q + size_t(g) * G) * d;
  if (tid < d_c) {
#pragma unroll
    for (int h = 0; h < G; ++h) qv[h] = qg[size_t(h) * d + ch];
  }
  const size_t row = size_t(unit) * T + (valid ? tok : 0);
  const uint8_t* crow = codes + row * (d_c / 2);
  const float2* prow = reinterpret_cast<const float2*>(qparams + row * ngr * 2);
  uint4 cw = ld16(crow);
  float2 pr = prow[0];
  __builtin_amdgcn_sched_barrier(0);
  if (tid < d_c) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      s_q[tid * G + h] = E::to_f(qv[h]);
      if constexpr (E::kIsBf16) {  // the group's 32 channels are two DPP rows
        const uint32_t r16 = row16_reduce_bits(__float_as_uint(E::to_f(qv[h])), [](uint32_t u, uint32_t v) {
          return __float_as_uint(__uint_as_float(u) + __uint_as_float(v));
        });
        const auto sw = __builtin_amdgcn_permlane16_swap(r16, r16, false, false);
        if (tid % 32 == 0) s_qs[tid / 32][h] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
      }
    }
  }
  lds_barrier();
  float acc[G];
#pragma unroll
  for (int h = 0; h < G; ++h) acc[h] = 0.f;
#pragma unroll 1
  for (int gr = 0; gr < ngr; ++gr) {
    const uint4 c = cw;
    const float2 p = pr;
    if (gr + 1 < ngr) {
      cw = ld16(crow + (gr + 1) * 16);
      pr = prow[gr + 1];
    }
    const float* qr = s_q + gr * 32 * G;
    const uint32_t wd[4] = {c.x, c.y, c.z, c.w};
    // the group's sum, rounded at its own size and not at that of all groups;
    // the products of bf16 queries and codes are exact, so those take the
    // codes and the sum of q~ apart
    float part[G];
#pragma unroll
    for (int h = 0; h < G; ++h) part[h] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      float f[8];
      unpack_nibbles8(wd[w], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = E::kIsBf16 ? f[e] : fmaf(p.x, f[e], p.y);
#pragma unroll
        for (int h = 0; h < G; ++h) part[h] = fmaf(qr[(w * 8 + e) * G + h], x, part[h]);
      }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) acc[h] += E::kIsBf16 ? fmaf(p.x, part[h], p.y * s_qs[gr][h]) : part[h];
  }
  float* lg = logits + size_t(unit) * G * S + slot;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float l = valid ? sigma * acc[h] : -INFINITY;
    if (slot < S) lg[size_t(h) * S] = l;
    const float M = wave_max_f32(l);
    const float Z = wave_sum_f32(l == -INFINITY ? 0.f : __expf(l - M));
    if (lane == 0) {
      s_red[wid][h][0] = M;
      s_red[wid][h][1] = Z;
    }
  }
  write_chunk_stats<G>(s_red, G, stats + (size_t(unit) * gridDim.x + chunk) * G * 2);
}

// bf16, G <= 4 HS, d_c = 32 NGR, where the fused kernel does not apply (more
// than four heads or one group, larger budgets): the same two rounds of
// requests, the contraction of a lane's slot on the matrix cores (lane_dots).
// 32 units of 8 heads, d_c = 64, 4096 slots: 18.3 -> 7.1 us.
template <int HS, int NGR>
__global__ __launch_bounds__(256) void token_score_lane_kernel(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ block_ids, int K_b,
    const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int G, int d, int B, int T, float sigma,
    float* __restrict__ logits, float* __restrict__ stats, uint32_t* __restrict__ kinfo, uint32_t* err) {
  constexpr int DC = 32 * NGR, NQ = NGR * HS * 128, PER = (NQ + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t s_qt[NQ];  // [group][set][head][position]
  __shared__ float s_red[4][4 * HS][2];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  if (chunk == 0 && threadIdx.x == 0) kinfo[2 * size_t(unit)] = 0u;  // arrivals of the alpha stage
  const int s = unit / H_kv, g = unit % H_kv;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int S = K_b * B;
  const int slot = chunk * kTokenSlotsPerWG + tid;
  int n = ctx_lens[s];
  const int blk = block_ids[size_t(unit) * K_b + min(tok_block(min(slot, S - 1), B), K_b - 1)];
  int ch[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = min(tid + j * 256, NQ - 1), x = i & 31;
    ch[j] = channels[g * DC + i / (128 * HS) * 32 + (x & ~7) + codes_chan(x & 7)];
  }
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  if (slot < S && blk >= m) set_error(err, 2u);
  const int tok = blk * B + tok_offset(slot, B);
  const bool valid = slot < S && blk >= 0 && blk < m && tok < n;
  uint16_t qv[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (ch[j] < 0 || ch[j] >= d) {
      set_error(err, 32u);
      ch[j] = 0;
    }
    const int i = min(tid + j * 256, NQ - 1), h = ((i >> 7) % HS) * 4 + ((i >> 5) & 3);
    const uint16_t v = q[(size_t(s) * H_q + size_t(g) * G + min(h, G - 1)) * d + ch[j]];
    qv[j] = h < G ? v : uint16_t(0);
  }
  __builtin_amdgcn_sched_barrier(0);
  const size_t row = size_t(unit) * T + (valid ? tok : 0);
  uint4 cw[NGR];
  float2 pr[NGR];
#pragma unroll
  for (int gr = 0; gr < NGR; ++gr) {
    cw[gr] = ld16(codes + row * (DC / 2) + gr * 16);
    pr[gr] = *reinterpret_cast<const float2*>(qparams + (row * NGR + gr) * 2);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (tid + j * 256 < NQ) s_qt[tid + j * 256] = qv[j];
  lds_barrier();
  float l[4 * HS];
#pragma unroll
  for (int h = 0; h < 4 * HS; ++h) l[h] = 0.f;
#pragma unroll
  for (int gr = 0; gr < NGR; ++gr) {
    bf16x8_t qa[HS][4];
    f32x4_t qsum[HS], acc[HS];
    lane_operands<HS>(s_qt + gr * HS * 128, qa, qsum);
    lane_dots<HS>(cw[gr], qa, acc);
#pragma unroll
    for (int h = 0; h < 4 * HS; ++h) {
      const float qs = qsum[h / 4][h % 4];
      l[h] += fmaf(pr[gr].x, acc[h / 4][h % 4], pr[gr].y * qs);
    }
  }
  float* lg = logits + size_t(unit) * G * S + slot;
#pragma unroll
  for (int h = 0; h < 4 * HS; ++h) {
    if (h < G) {  // uniform
      const float v = valid ? sigma * l[h] : -INFINITY;
      if (slot < S) lg[size_t(h) * S] = v;
      const float M = wave_max_f32(v);
      const float Z = wave_sum_f32(v == -INFINITY ? 0.f : __expf(v - M));
      if (lane == 0) {
        s_red[wid][h][0] = M;
        s_red[wid][h][1] = Z;
      }
    }
  }
  write_chunk_stats<4 * HS>(s_red, G, stats + (size_t(unit) * gridDim.x + chunk) * G * 2);
}

// The same logits and statistics with the code contraction on the matrix
// cores, for bf16 with G a multiple of 16 (the absorbed MLA layout: 32 heads
// over d_c = 128 channels).  A work-group (4 waves) takes 256 slots; each
// wave takes four 16-slot tiles.  Per tile and 32-channel group,
// v_mfma_f32_16x16x32_bf16 with A = q~ (16 heads x 32 channels, exact in
// bf16) and B = the tile's codes, entering as the bf16 number 128 + c (one
// byte permute per two codes; exact) gives dot'_hj = dot_hj + 128 sum_c q~_hc,
// so per group l gains sigma (scale_j dot'_hj + (min_j - 128 scale_j) qsum_h).
// Lane (g, i) of the result holds slot i of the tile for heads 4g..4g+3.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 ts_bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float ts_f32x4_t;
typedef uint32_t ts_u32x4_t __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ inline float dpp_row_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xF, 0xF, false));
}

template <int HT, int NGR>
__global__ __launch_bounds__(256) void token_score_mfma_kernel(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ codes, const float* __restrict__ qparams,
    const int32_t* __restrict__ channels, const int32_t* __restrict__ block_ids, int K_b,
    const int32_t* __restrict__ ctx_lens, int H_q, int H_kv, int d, int B, int T, float sigma,
    float* __restrict__ logits, float* __restrict__ stats, uint32_t* __restrict__ kinfo, uint32_t* err) {
  constexpr int G = 16 * HT, DC = 32 * NGR;
  constexpr uint32_t kBase = 0x43434343u;  // high byte of bf16(128 + c), c < 16
  // q~ in operand order: [head][group][lane group g][8], channel g*8 + {0,2,4,6,1,3,5,7}
  __shared__ __attribute__((aligned(16))) uint16_t s_qt[G * DC];
  __shared__ float s_qs[G * NGR];
  __shared__ float s_red[4][G][2];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  if (chunk == 0 && threadIdx.x == 0) kinfo[2 * size_t(unit)] = 0u;  // arrivals of the alpha stage
  const int s = unit / H_kv, g = unit % H_kv;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t16 = lane & 15, lg = lane >> 4;
  const int S = K_b * B;
  const uint16_t* qg = q + (size_t(s) * H_q + size_t(g) * G) * d;
  const int32_t* bl = block_ids + size_t(unit) * K_b;
  // Two rounds of requests, each with every load in flight at once (loads
  // are unconditional at clamped addresses, so that none is sunk into a
  // branch and waited for alone):
  // 1. the context length, the block-list entries of the four tiles' slots
  //    and the channel id of this thread's q~ position;
  // 2. the q~ elements, then the tiles' index rows (so that the wait for q~
  //    does not cover the rows).
  // Thread t holds q~ entries t + 256 j: with 256 a multiple of DC they all
  // lie at operand position x = t % DC, of heads j (256 / DC) + t / DC.
  static_assert(256 % DC == 0 && G * DC % 256 == 0, "q~ entries per thread");
  constexpr int PER = G * DC / 256;
  const int x = tid % DC;
  int n = ctx_lens[s];
  int blk[4];
#pragma unroll
  for (int tl = 0; tl < 4; ++tl) {
    const int slot = chunk * kTokenSlotsPerWG + w * 64 + tl * 16 + t16;
    blk[tl] = bl[min(tok_block(min(slot, S - 1), B), K_b - 1)];
  }
  int ch;
  {
    const int e = x & 7;
    ch = channels[g * DC + (x & ~7) + ((e & 3) << 1) + (e >> 2)];  // channel index of position x
  }
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  if (ch < 0 || ch >= d) {
    set_error(err, 32u);
    ch = 0;
  }
  uint16_t qv[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) qv[j] = qg[size_t(j * (256 / DC) + tid / DC) * d + ch];
  __builtin_amdgcn_sched_barrier(0);
  bool valid[4];
  uint32_t cx[4][NGR];
  float2 pqv[4][NGR];
#pragma unroll
  for (int tl = 0; tl < 4; ++tl) {
    const int slot = chunk * kTokenSlotsPerWG + w * 64 + tl * 16 + t16;
    const int b = blk[tl];
    if (slot < S && b >= m) set_error(err, 2u);
    const int tok = b * B + tok_offset(slot, B);
    valid[tl] = slot < S && b >= 0 && b < m && tok < n;
    const size_t row = size_t(unit) * T + (valid[tl] ? tok : 0);
#pragma unroll
    for (int grp = 0; grp < NGR; ++grp) {
      cx[tl][grp] = *reinterpret_cast<const uint32_t*>(codes + row * (DC / 2) + grp * 16 + lg * 4);
      pqv[tl][grp] = *reinterpret_cast<const float2*>(qparams + (row * NGR + grp) * 2);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // q~ to LDS in operand order, and each (head, 32-channel group) sum over
  // the 32 lanes that hold its positions (a 32-lane aligned half-wave): DPP
  // sums inside each 16-lane row, then the two rows' sums exchanged
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    s_qt[tid + j * 256] = qv[j];
    const uint32_t r16 = row16_reduce_bits(uint32_t(qv[j]) << 16, [](uint32_t u, uint32_t v) {
      return __float_as_uint(__uint_as_float(u) + __uint_as_float(v));
    });
    const auto sw = __builtin_amdgcn_permlane16_swap(r16, r16, false, false);
    if ((tid & 31) == 0)
      s_qs[(j * (256 / DC) + tid / DC) * NGR + x / 32] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  __syncthreads();
  // A operands: head ht*16 + t16, channels of group grp at lane group lg
  ts_bf16x8_t qa[HT][NGR];
#pragma unroll
  for (int ht = 0; ht < HT; ++ht)
#pragma unroll
    for (int grp = 0; grp < NGR; ++grp)
      qa[ht][grp] = *reinterpret_cast<const ts_bf16x8_t*>(&s_qt[(ht * 16 + t16) * DC + grp * 32 + lg * 8]);
  float qs[HT][4][NGR];  // heads ht*16 + 4lg + r
#pragma unroll
  for (int ht = 0; ht < HT; ++ht)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int grp = 0; grp < NGR; ++grp) qs[ht][r][grp] = s_qs[(ht * 16 + lg * 4 + r) * NGR + grp];

  float lgt[4][HT][4];  // [tile][ht][r]
#pragma unroll
  for (int tl = 0; tl < 4; ++tl) {
    const int slot = chunk * kTokenSlotsPerWG + w * 64 + tl * 16 + t16;
    ts_f32x4_t acc[HT][NGR];
#pragma unroll
    for (int ht = 0; ht < HT; ++ht)
#pragma unroll
      for (int grp = 0; grp < NGR; ++grp) acc[ht][grp] = ts_f32x4_t{0.f, 0.f, 0.f, 0.f};
    float sc[NGR], off[NGR];
#pragma unroll
    for (int grp = 0; grp < NGR; ++grp) {
      const uint32_t x = cx[tl][grp];
      sc[grp] = pqv[tl][grp].x;
      off[grp] = pqv[tl][grp].y - 128.0f * pqv[tl][grp].x;
      const uint32_t lo = x & 0x0f0f0f0fu, hi = (x >> 4) & 0x0f0f0f0fu;
      const ts_u32x4_t bw = {__builtin_amdgcn_perm(kBase, lo, 0x04010400u), __builtin_amdgcn_perm(kBase, lo, 0x04030402u),
                             __builtin_amdgcn_perm(kBase, hi, 0x04010400u), __builtin_amdgcn_perm(kBase, hi, 0x04030402u)};
      const ts_bf16x8_t b = __builtin_bit_cast(ts_bf16x8_t, bw);
#pragma unroll
      for (int ht = 0; ht < HT; ++ht)
        acc[ht][grp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ht][grp], b, acc[ht][grp], 0, 0, 0);
    }
    // validity of slot t16 for the result lanes (lane (lg, t16) holds slot t16)
#pragma unroll
    for (int ht = 0; ht < HT; ++ht)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = 0.f;
#pragma unroll
        for (int grp = 0; grp < NGR; ++grp) v += fmaf(sc[grp], acc[ht][grp][r], off[grp] * qs[ht][r][grp]);
        lgt[tl][ht][r] = valid[tl] ? sigma * v : -INFINITY;
      }
    if (slot < S) {
      float* lg_out = logits + size_t(unit) * G * S + slot;
#pragma unroll
      for (int ht = 0; ht < HT; ++ht)
#pragma unroll
        for (int r = 0; r < 4; ++r) lg_out[size_t(ht * 16 + lg * 4 + r) * S] = lgt[tl][ht][r];
    }
  }
  // this work-group's per-head max and sum of exponentials (a DPP row holds
  // the 16 slots of one head)
  auto row16 = [](float v, bool is_max) {
    float o = dpp_row_move<0xB1>(v);
    v = is_max ? fmaxf(v, o) : v + o;
    o = dpp_row_move<0x4E>(v);
    v = is_max ? fmaxf(v, o) : v + o;
    o = dpp_row_move<0x141>(v);
    v = is_max ? fmaxf(v, o) : v + o;
    o = dpp_row_move<0x140>(v);
    return is_max ? fmaxf(v, o) : v + o;
  };
#pragma unroll
  for (int ht = 0; ht < HT; ++ht)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float mx = fmaxf(fmaxf(lgt[0][ht][r], lgt[1][ht][r]), fmaxf(lgt[2][ht][r], lgt[3][ht][r]));
      mx = row16(mx, true);
      float sm = 0.f;
      if (mx != -INFINITY) {
#pragma unroll
        for (int tl = 0; tl < 4; ++tl) sm += lgt[tl][ht][r] == -INFINITY ? 0.f : __expf(lgt[tl][ht][r] - mx);
      }
      sm = row16(sm, false);
      if (t16 == 0) {
        s_red[w][ht * 16 + lg * 4 + r][0] = mx;
        s_red[w][ht * 16 + lg * 4 + r][1] = sm;
      }
    }
  __syncthreads();
  if (tid < G) {
    float M = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) M = fmaxf(M, s_red[v][tid][0]);
    float Z = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (s_red[v][tid][0] != -INFINITY) Z += s_red[v][tid][1] * __expf(s_red[v][tid][0] - M);
    }
    float* st = stats + ((size_t(unit) * gridDim.x + chunk) * G + tid) * 2;
    st[0] = M;
    st[1] = Z;
  }
}

// Work-group 0 of a unit's alpha kernel also writes the unit's number of
// valid candidate slots and the key of a bound on every alpha key: with each
// exponential <= 1, the alpha of a slot is at most (1/G) sum_h 1/Z_h summed
// in the key loop's order (rounding is monotone), so the top-K_t kernel needs
// no statistics pass of its own.  All 256 threads call it; b_first is the
// list entry bl[threadIdx.x] (any value where threadIdx.x >= K_b), requested
// by the caller with its other loads.
__device__ inline void write_unit_info(const int32_t* bl, int b_first, int K_b, int B, int m, int n,
                                       const float* s_iz, int G, float invG, uint32_t* kinfo, int unit,
                                       uint32_t* s_cnt) {
  uint32_t c = 0;
  for (int i = threadIdx.x; i < K_b; i += 256) {
    const int b = i == int(threadIdx.x) ? b_first : bl[i];
    if (b >= 0 && b < m) c += uint32_t(min(B, n - b * B));
  }
  c = wave_reduce_bits(c, [](uint32_t a, uint32_t b) { return a + b; });
  if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    float bsum = 0.f;
    for (int h = 0; h < G; ++h) bsum = fmaf(1.0f, s_iz[h], bsum);
    kinfo[2 * size_t(unit)] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    kinfo[2 * size_t(unit) + 1] = __float_as_uint(fmaxf(bsum * invG, 0.f)) | 0x80000000u;
  }
}

__global__ __launch_bounds__(256) void token_alpha_kernel(
    const float* __restrict__ logits, const float* __restrict__ stats, int n_tchunks,
    const int32_t* __restrict__ block_ids, int K_b, const int32_t* __restrict__ ctx_lens, int H_kv, int G,
    int B, int T, uint32_t* __restrict__ keys, uint32_t* __restrict__ kinfo) {
  __shared__ float s_m[kMaxG], s_iz[kMaxG];
  __shared__ uint32_t s_cnt[4];
  const int unit = blockIdx.y;
  const int s = unit / H_kv;
  int n = ctx_lens[s];
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  const int S = K_b * B;
  if (threadIdx.x < G) {
    const int h = threadIdx.x;
    const float* st = stats + size_t(unit) * n_tchunks * G * 2;
    float M = -INFINITY;
    for (int c = 0; c < n_tchunks; ++c) M = fmaxf(M, st[(c * G + h) * 2]);
    float Z = 0.f;
    if (M != -INFINITY)
      for (int c = 0; c < n_tchunks; ++c) {
        const float mc = st[(c * G + h) * 2], zc = st[(c * G + h) * 2 + 1];
        if (mc != -INFINITY) Z += zc * __expf(mc - M);
      }
    s_m[h] = M;
    s_iz[h] = Z > 0.f ? 1.0f / Z : 0.f;
  }
  __syncthreads();
  const float invG = 1.0f / float(G);
  const int32_t* bl = block_ids + size_t(unit) * K_b;
  if (blockIdx.x == 0)
    write_unit_info(bl, threadIdx.x < K_b ? bl[threadIdx.x] : -1, K_b, B, m, n, s_iz, G, invG, kinfo, unit, s_cnt);
  const float* lg = logits + size_t(unit) * G * S;
  for (int slot = blockIdx.x * 256 + threadIdx.x; slot < S; slot += gridDim.x * 256) {
    int tok;
    uint32_t key = kInvalidKey;
    if (slot_token(bl, K_b, B, m, n, slot, &tok, nullptr)) {
      float a = 0.f;
      for (int h = 0; h < G; ++h) a += __expf(lg[size_t(h) * S + slot] - s_m[h]) * s_iz[h];
      key = alpha_key(a * invG);
    }
    keys[size_t(unit) * S + slot] = key;
  }
}

// token_alpha_kernel with the head count fixed at compile time, for a grid
// of one slot per thread: 256/G lanes combine each head's work-group
// statistics, and every request of a work-group leaves at once before the
// first is used (its lanes' statistics, the block-list entries of its slots
// and of the unit information, the slots' G logits; unconditional loads at
// clamped addresses), so the kernel waits for one memory round trip.
template <int G>
__global__ __launch_bounds__(256) void token_alpha_kernel_g(
    const float* __restrict__ logits, const float* __restrict__ stats, int n_tchunks,
    const int32_t* __restrict__ block_ids, int K_b, const int32_t* __restrict__ ctx_lens, int H_kv, int B, int T,
    uint32_t* __restrict__ keys, uint32_t* __restrict__ kinfo) {
  constexpr int TPH = 256 / G;  // lanes per head (a power of two)
  constexpr int kC = 8;         // statistics chunks per lane requested together
  __shared__ float s_m[G], s_iz[G];
  __shared__ uint32_t s_cnt[4];
  const int unit = blockIdx.y, tid = threadIdx.x;
  const int s = unit / H_kv;
  const int S = K_b * B;
  const int h = tid / TPH, j = tid % TPH;
  const float2* st = reinterpret_cast<const float2*>(stats) + size_t(unit) * n_tchunks * G;
  const int32_t* bl = block_ids + size_t(unit) * K_b;
  const float* lg = logits + size_t(unit) * G * S;
  const int slot = blockIdx.x * 256 + tid, sl = min(slot, S - 1);
  float2 sv[kC];
#pragma unroll
  for (int c = 0; c < kC; ++c) sv[c] = st[size_t(min(j + c * TPH, n_tchunks - 1)) * G + h];
  __builtin_amdgcn_sched_barrier(0);
  const int b_slot = bl[tok_block(sl, B)];
  const int b_first = bl[min(tid, K_b - 1)];
  float v[G];
#pragma unroll
  for (int hh = 0; hh < G; ++hh) v[hh] = lg[size_t(hh) * S + sl];
  __builtin_amdgcn_sched_barrier(0);
  int n = ctx_lens[s];
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  {
    // chunks j, j + TPH, ... in ascending order, then the lanes' tree (the
    // requested entries are used through selects, not branches, so that
    // no load is sunk into a branch; adding +0 leaves Z >= +0 unchanged)
    float M = -INFINITY;
#pragma unroll
    for (int c = 0; c < kC; ++c) M = fmaxf(M, j + c * TPH < n_tchunks ? sv[c].x : -INFINITY);
    for (int c = j + kC * TPH; c < n_tchunks; c += TPH) M = fmaxf(M, st[size_t(c) * G + h].x);
#pragma unroll
    for (int o = TPH / 2; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
    float Z = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int c = 0; c < kC; ++c) {
        const bool ok = j + c * TPH < n_tchunks && sv[c].x != -INFINITY;
        Z += ok ? sv[c].y * __expf(sv[c].x - M) : 0.f;
      }
      for (int c = j + kC * TPH; c < n_tchunks; c += TPH) {
        const float2 e = st[size_t(c) * G + h];
        if (e.x != -INFINITY) Z += e.y * __expf(e.x - M);
      }
    }
#pragma unroll
    for (int o = TPH / 2; o > 0; o >>= 1) Z += __shfl_xor(Z, o, 64);
    if (j == 0) {
      s_m[h] = M;
      s_iz[h] = Z > 0.f ? 1.0f / Z : 0.f;
    }
  }
  __syncthreads();
  const float invG = 1.0f / float(G);
  if (blockIdx.x == 0) write_unit_info(bl, b_first, K_b, B, m, n, s_iz, G, invG, kinfo, unit, s_cnt);
  if (slot < S) {
    const int t = b_slot * B + tok_offset(slot, B);
    uint32_t key = kInvalidKey;
    if (b_slot >= 0 && b_slot < m && t < n) {
      float a = 0.f;
#pragma unroll
      for (int hh = 0; hh < G; ++hh) a += __expf(v[hh] - s_m[hh]) * s_iz[hh];
      key = alpha_key(a * invG);
    }
    keys[size_t(unit) * S + slot] = key;
  }
}

// Alpha and the top-K_t in one launch: a work-group of 1024 threads computes the
// keys of 1024 slots, stores them past the L2s (as SplitOut's partials) and
// counts itself in; the unit's last one reads all of them back into registers
// and selects, from bounds it knows (each exponential is <= 1, so alpha is at
// most (1/G) sum_h 1/Z_h summed in the key loop's order).  A latency chain: every
// request of a work-group leaves at once before the first is used (statistics,
// block-list entries, the slot's G logits; unconditional loads at clamped
// addresses).  With one work-group per unit it is a single pass.  Against an
// alpha and a top-K_t launch: 2 units of 512 slots 6.6 -> 4.8 us, 32 units of 8
// heads and 4096 slots 9.9 -> 9.4.  Storing, counting and reading back cost what
// a launch does, and with 16 or 32 heads more (32 heads, whole step of 8 units
// and 8192 slots 53.4 us against 52.7 in two launches, 2 units and 6400 slots
// 41.8 against 40.5), so those take it only in the single-pass form; spreading a
// slot's heads over four threads changed nothing.
template <int G, int EPT>
__global__ __launch_bounds__(1024) void token_alpha_topk_kernel(
    const float* __restrict__ logits, const float* __restrict__ stats, int n_tchunks,
    const int32_t* __restrict__ block_ids, int K_b, const int32_t* __restrict__ ctx_lens, int H_kv, int B, int T,
    int K_t, uint32_t* __restrict__ keys, uint32_t* __restrict__ kinfo, int32_t* __restrict__ token_ids,
    float* __restrict__ token_scores, uint32_t* arrive) {
  constexpr int NT = 1024, TPH = 256 / G;  // statistics: TPH lanes per head (a power of two) of the first 256 threads
  constexpr int kC = 8;                    // statistics chunks per lane requested together
  __shared__ float s_m[G], s_iz[G];
  __shared__ uint32_t s_cnt[4], s_last;
  extern __shared__ uint32_t smem[];
  uint32_t* scratch = smem;
  int32_t* s_bl = reinterpret_cast<int32_t*>(smem + topk_scratch_words(NT));
  const int unit = blockIdx.y, tid = threadIdx.x;
  if (arrive && blockIdx.x == 0 && tid == 0) arrive[unit] = 0u;
  const int s = unit / H_kv;
  const int S = K_b * B;
  const int h = (tid & 255) / TPH, j = tid % TPH;
  const float2* st = reinterpret_cast<const float2*>(stats) + size_t(unit) * n_tchunks * G;
  const int32_t* bl = block_ids + size_t(unit) * K_b;
  const float* lg = logits + size_t(unit) * G * S;
  const int slot = blockIdx.x * NT + tid, sl = min(slot, S - 1);
  float2 sv[kC];
  if (tid < 256) {
#pragma unroll
    for (int c = 0; c < kC; ++c) sv[c] = st[size_t(min(j + c * TPH, n_tchunks - 1)) * G + h];
  }
  __builtin_amdgcn_sched_barrier(0);
  const int b_slot = bl[tok_block(sl, B)];
  const int b_first = bl[min(tid, K_b - 1)];
  float v[G];
#pragma unroll
  for (int hh = 0; hh < G; ++hh) v[hh] = lg[size_t(hh) * S + sl];
  __builtin_amdgcn_sched_barrier(0);
  int n = ctx_lens[s];
  n = n < 0 ? 0 : (n > T ? T : n);
  const int m = (n + B - 1) / B;
  topk_prepare<NT>(scratch);
  for (int i = tid; i < K_b; i += NT) s_bl[i] = i == tid ? b_first : bl[i];
  if (tid < 256) {
    // chunks j, j + TPH, ... in ascending order, then the lanes' tree (the
    // requested entries are used through selects, not branches, so that
    // no load is sunk into a branch; adding +0 leaves Z >= +0 unchanged)
    float M = -INFINITY;
#pragma unroll
    for (int c = 0; c < kC; ++c) M = fmaxf(M, j + c * TPH < n_tchunks ? sv[c].x : -INFINITY);
    for (int c = j + kC * TPH; c < n_tchunks; c += TPH) M = fmaxf(M, st[size_t(c) * G + h].x);
#pragma unroll
    for (int o = TPH / 2; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
    float Z = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int c = 0; c < kC; ++c) {
        const bool ok = j + c * TPH < n_tchunks && sv[c].x != -INFINITY;
        Z += ok ? sv[c].y * __expf(sv[c].x - M) : 0.f;
      }
      for (int c = j + kC * TPH; c < n_tchunks; c += TPH) {
        const float2 e = st[size_t(c) * G + h];
        if (e.x != -INFINITY) Z += e.y * __expf(e.x - M);
      }
    }
#pragma unroll
    for (int o = TPH / 2; o > 0; o >>= 1) Z += __shfl_xor(Z, o, 64);
    if (j == 0) {
      s_m[h] = M;
      s_iz[h] = Z > 0.f ? 1.0f / Z : 0.f;
    }
    // the unit's valid candidates
    uint32_t c = 0;
    for (int i = tid; i < K_b; i += 256) {
      const int b = i == tid ? b_first : bl[i];
      if (b >= 0 && b < m) c += uint32_t(min(B, n - b * B));
    }
    c = wave_reduce_bits(c, [](uint32_t a, uint32_t b) { return a + b; });
    if ((tid & 63) == 0) s_cnt[tid >> 6] = c;
  }
  __syncthreads();
  const float invG = 1.0f / float(G);
  uint32_t key = kInvalidKey;
  {
    const int t = b_slot * B + tok_offset(slot, B);
    if (slot < S && b_slot >= 0 && b_slot < m && t < n) {
      float a = 0.f;
#pragma unroll
      for (int hh = 0; hh < G; ++hh) a += __expf(v[hh] - s_m[hh]) * s_iz[hh];
      key = alpha_key(a * invG);
    }
  }
  uint32_t kr[EPT];
  if (EPT == 1 || gridDim.x == 1) {
    kr[0] = key;
#pragma unroll
    for (int e = 1; e < EPT; ++e) kr[e] = kInvalidKey;
  } else {
    uint32_t* uk = keys + size_t(unit) * S;
    if (slot < S) __hip_atomic_store(uk + slot, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");  // this wave's keys are in memory
    __syncthreads();
    if (tid == 0) s_last = __hip_atomic_fetch_add(kinfo + 2 * size_t(unit), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_last != gridDim.x - 1) return;  // uniform
    asm volatile("" : : : "memory");
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int p = tid + e * NT;
      kr[e] = __hip_atomic_load(uk + min(p, S - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (p >= S) kr[e] = kInvalidKey;
    }
  }
  float bsum = 0.f;
#pragma unroll
  for (int hh = 0; hh < G; ++hh) bsum = fmaf(1.0f, s_iz[hh], bsum);
  const TopkKnown known{s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3], alpha_key(bsum * invG), 0x80000000u};
  wg_topk_regs<NT, EPT, true>(kr, K_t, token_ids + size_t(unit) * K_t, K_t,
                              token_scores ? token_scores + size_t(unit) * K_t : nullptr,
                              [=](int, int p) { return int32_t(s_bl[tok_block(p, B)] * B + tok_offset(p, B)); }, scratch,
                              &known);
}

// Top-K_t of the alpha keys of each unit, one work-group per unit.  Thread t
// holds the keys of slots t + 1024 j (j < EPT), requested together straight
// into registers.
template <int EPT>
__global__ __launch_bounds__(1024) void token_topk_kernel(const uint32_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ kinfo,
                                                           const int32_t* __restrict__ block_ids, int K_b,
                                                           int B, int K_t, int32_t* __restrict__ token_ids,
                                                           float* __restrict__ token_scores, uint32_t* arrive) {
  extern __shared__ uint32_t smem[];
  uint32_t* scratch = smem;
  int32_t* s_bl = reinterpret_cast<int32_t*>(smem + topk_scratch_words(1024));
  const int S = K_b * B;
  const int unit = blockIdx.x;
  if (arrive && threadIdx.x == 0) arrive[unit] = 0u;
  uint32_t kr[EPT];
#pragma unroll
  for (int j = 0; j < EPT; ++j) {
    const int p = threadIdx.x + j * 1024;
    kr[j] = p < S ? keys[size_t(unit) * S + p] : kInvalidKey;
  }
  // the valid count and the key bound from the alpha kernel; every valid key
  // is >= the key of +0
  const TopkKnown known{kinfo[2 * size_t(unit)], kinfo[2 * size_t(unit) + 1], 0x80000000u};
  for (int i = threadIdx.x; i < K_b; i += 1024) s_bl[i] = block_ids[size_t(unit) * K_b + i];
  topk_prepare<1024>(scratch);
  __syncthreads();
  wg_topk_regs<1024, EPT, true>(kr, K_t, token_ids + size_t(unit) * K_t, K_t,
                                token_scores ? token_scores + size_t(unit) * K_t : nullptr,
                                [=](int, int slot) { return int32_t(s_bl[tok_block(slot, B)] * B + tok_offset(slot, B)); }, scratch,
                                &known);
}

template <int HT, int NGR>
static void launch_score_mfma(const Problem& P, const void* q, const uint8_t* codes, const float* qparams,
                              const int32_t* channels, const int32_t* block_ids, int K_b, const int32_t* ctx_lens,
                              float* logits, float* stats, int n_tchunks, uint32_t* kinfo, uint32_t* err,
                              hipStream_t st) {
  token_score_mfma_kernel<HT, NGR><<<dim3(n_tchunks, P.units), 256, 0, st>>>(
      (const uint16_t*)q, codes, qparams, channels, block_ids, K_b, ctx_lens, P.H_q, P.H_kv, P.d_qk, P.B, P.T,
      P.sigma, logits, stats, kinfo, err);
}

hipError_t launch_token_score(const Problem& P, const void* q, const uint8_t* codes, const float* qparams,
                              const int32_t* channels, const int32_t* block_ids, int K_b,
                              const int32_t* ctx_lens, float* logits, float* stats, int n_tchunks, uint32_t* kinfo,
                              uint32_t* err, hipStream_t st) {
  if (P.dtype == 1 && (P.G == 16 || P.G == 32) && (P.d_c == 64 || P.d_c == 128)) {
    if (P.G == 32 && P.d_c == 128) launch_score_mfma<2, 4>(P, q, codes, qparams, channels, block_ids, K_b, ctx_lens, logits, stats, n_tchunks, kinfo, err, st);
    else if (P.G == 32) launch_score_mfma<2, 2>(P, q, codes, qparams, channels, block_ids, K_b, ctx_lens, logits, stats, n_tchunks, kinfo, err, st);
    else if (P.d_c == 128) launch_score_mfma<1, 4>(P, q, codes, qparams, channels, block_ids, K_b, ctx_lens, logits, stats, n_tchunks, kinfo, err, st);
    else launch_score_mfma<1, 2>(P, q, codes, qparams, channels, block_ids, K_b, ctx_lens, logits, stats, n_tchunks, kinfo, err, st);
    return hipGetLastError();
  }
  dim3 grid(n_tchunks, P.units);
  if (P.dtype == 1 && P.G <= 8 && (P.d_c == 32 || P.d_c == 64 || P.d_c == 128)) {
    auto go = [&](auto kern) {
      kern<<<grid, 256, 0, st>>>((const uint16_t*)q, codes, qparams, channels, block_ids, K_b, ctx_lens, P.H_q, P.H_kv,
                                 P.G, P.d_qk, P.B, P.T, P.sigma, logits, stats, kinfo, err);
    };
    if (P.G <= 4) {
      if (P.d_c == 32) go(token_score_lane_kernel<1, 1>);
      else if (P.d_c == 64) go(token_score_lane_kernel<1, 2>);
      else go(token_score_lane_kernel<1, 4>);
    } else {
      if (P.d_c == 32) go(token_score_lane_kernel<2, 1>);
      else if (P.d_c == 64) go(token_score_lane_kernel<2, 2>);
      else go(token_score_lane_kernel<2, 4>);
    }
    return hipGetLastError();
  }
  auto rows = [&](auto elem) {
    using E = decltype(elem);
    using T = typename E::T;
    auto go = [&](auto kern) {
      kern<<<grid, 256, 0, st>>>((const T*)q, codes, qparams, channels, block_ids, K_b, ctx_lens, P.H_q, P.H_kv, P.d_qk,
                                 P.d_c, P.B, P.T, P.sigma, logits, stats, kinfo, err);
    };
    switch (P.G) {
      case 1: go(token_score_row_kernel<E, 1>); return;
      case 2: go(token_score_row_kernel<E, 2>); return;
      case 4: go(token_score_row_kernel<E, 4>); return;
      case 8: go(token_score_row_kernel<E, 8>); return;
      default:
        token_score_kernel<E><<<grid, 256, 0, st>>>((const T*)q, codes, qparams, channels, block_ids, K_b, ctx_lens,
                                                    P.H_q, P.H_kv, P.G, P.d_qk, P.d_c, P.B, P.T, P.sigma, logits,
                                                    stats, kinfo, err);
    }
  };
  if (P.dtype == 1) rows(BF16{});
  else rows(F32{});
  return hipGetLastError();
}

hipError_t launch_token_alpha_topk(const Problem& P, const float* logits, const float* stats, int n_tchunks,
                                   const int32_t* block_ids, int K_b, const int32_t* ctx_lens, int K_t, uint32_t* keys,
                                   uint32_t* kinfo, int32_t* token_ids, float* token_scores, uint32_t* arrive,
                                   hipEvent_t topk_begin, hipStream_t st) {
  const int S = K_b * P.B;
  const size_t lds = (topk_scratch_words(1024) + size_t(align4w(K_b))) * sizeof(uint32_t);
  const int ept = (S + 1023) / 1024;
  auto one = [&](auto kern) {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    if (topk_begin) (void)hipEventRecord(topk_begin, st);
    kern<<<dim3(ept, P.units), 1024, lds, st>>>(logits, stats, n_tchunks, block_ids, K_b, ctx_lens, P.H_kv, P.B, P.T,
                                                K_t, keys, kinfo, token_ids, token_scores, arrive);
    return hipGetLastError();
  };
  auto by_slots = [&](auto g) {
    constexpr int G = decltype(g)::value;
    if (ept <= 1) return one(token_alpha_topk_kernel<G, 1>);
    if (ept <= 2) return one(token_alpha_topk_kernel<G, 2>);
    if (ept <= 4) return one(token_alpha_topk_kernel<G, 4>);
    if (ept <= 8) return one(token_alpha_topk_kernel<G, 8>);
    return one(token_alpha_topk_kernel<G, 16>);
  };
  if (P.G == 4) return by_slots(std::integral_constant<int, 4>{});
  if (P.G == 8) return by_slots(std::integral_constant<int, 8>{});
  if (P.G == 16 && ept == 1) return one(token_alpha_topk_kernel<16, 1>);
  if (P.G == 32 && ept == 1) return one(token_alpha_topk_kernel<32, 1>);
  // two launches
  const dim3 grid((S + 255) / 256, P.units);
  auto alpha = [&](auto kern) {
    kern<<<grid, 256, 0, st>>>(logits, stats, n_tchunks, block_ids, K_b, ctx_lens, P.H_kv, P.B, P.T, keys, kinfo);
  };
  if (P.G == 16) alpha(token_alpha_kernel_g<16>);
  else if (P.G == 32) alpha(token_alpha_kernel_g<32>);
  else
    token_alpha_kernel<<<grid, 256, 0, st>>>(logits, stats, n_tchunks, block_ids, K_b, ctx_lens, P.H_kv, P.G, P.B, P.T,
                                             keys, kinfo);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (topk_begin) (void)hipEventRecord(topk_begin, st);
  auto go = [&](auto kern) {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    kern<<<P.units, 1024, lds, st>>>(keys, kinfo, block_ids, K_b, P.B, K_t, token_ids, token_scores, arrive);
    return hipGetLastError();
  };
  if (ept <= 1) return go(token_topk_kernel<1>);
  if (ept <= 2) return go(token_topk_kernel<2>);
  if (ept <= 4) return go(token_topk_kernel<4>);
  if (ept <= 8) return go(token_topk_kernel<8>);
  return go(token_topk_kernel<16>);
}

}  // namespace tls
