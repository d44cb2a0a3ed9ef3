// Exact attention over the selected tokens for the absorbed MLA layout
// (AsyncTLS Sec. 4.1 final step; MLA collapsed to one shared latent head,
// Sec. 3): per unit, 16 or 32 query heads share every 576-dim row
// [latent; rope]; the value is the row's first 512 dims.
//
//   scores S = Q K^T (heads x tokens x 576) and O += P V (heads x 512 x
//   tokens) are dense contractions, so both run on the matrix cores:
//   * a work-group of TT x HT waves walks its split in chunks of 16 TT tokens,
//     double buffered.  Rows are gathered whole into LDS with
//     global_load_lds_dwordx4 (64 consecutive 16-byte pieces per instruction,
//     i.e. 8 or 9 cache lines), piece p of row r at position p with its low
//     three bits XORed by r / 2, which spreads both operand reads below
//     evenly over the LDS banks;
//   * wave (token tile tt, head tile ht) holds its 16 heads' queries as
//     operands in registers (72 VGPRs) and computes the 16 x 16 tile
//     S^T = K Q^T by 18 v_mfma_f32_16x16x32_bf16;
//   * softmax in base 2 against a running maximum that is only raised when a
//     logit exceeds it by more than 2^8: as a rule the probabilities of a
//     chunk need no exchange between the waves, and a chunk costs two
//     barriers (rows landed; probabilities written).  A wave that sees a
//     larger logit sets a flag, and the chunk then takes the exact maximum
//     over the token tiles, with two more barriers (always the first chunk,
//     rarely a later one);
//   * wave w owns output dims [512 w / NW, ...): O += P V by
//     v_mfma_f32_16x16x32_bf16 over 32 tokens, P rounded to bf16 for 32 heads
//     and entered as three bf16 parts that hold all 24 bits of its fp32 value
//     for 16 heads.  The two products agree on the
//     order of the 32 tokens (4 lg + r of two token tiles), so that a lane's
//     own scores are its A operand and two ds_read_b64_tr_b16 its B operand.
// The work-group writes normalised partials and their log-sum-exp; the merge
// kernel combines the splits.
//
// What bounds it: per chunk the LDS moves 2.3 KB per token (gather, K read by
// the HT head tiles, V), about 1 us per 64 tokens, under the 2.4 us the rows
// take at HBM rate, so long splits are HBM-bound as long as rows stay in
// flight: two work-groups of TT = 2 (80 KB of LDS) share a compute unit and
// one's gathers cover the other's barriers.  A split of one chunk is a chain
// of latencies instead: TT = 4 takes 64 tokens in one pass.  Measured (8 units
// x 65536 tokens, 604 MB, attention and merge): 112 us, 5.4 TB/s; 243 us for
// 32-token chunks with the queries in LDS (one work-group per compute unit),
// five barriers per chunk and gathers of 64 rows' single pieces, each its own
// cache line.  16 heads ran on the vector kernel before, with fp32
// probabilities: a two-level step of 1, 16 and 48 sequences (2048 of 8192
// tokens) took 85.8, 153 and 386 us with it, 42.4, 54.3 and 78.6 with this one.
// Their three parts cost up to 1 us of that (42.7, 53.7, 77.4 with one bf16
// part, whose error from 64 bits is 2.05e-3 in the 2-norm; 1.648e-3 with three,
// as on the vector kernel, which is the rounding of the output).  32 heads
// keep one part: 2.06e-3.
#include "attn_common.hpp"

namespace tls {

namespace {

constexpr int kMlaDqk = 576, kMlaDv = 512;
constexpr int kMlaPieces = kMlaDqk / 8;  // 16-byte pieces per row
constexpr int kMlaMaxTPW = 1024;         // tokens per work-group

// position of piece p of a row with swizzle z (0..7): within the row's
// aligned groups of eight pieces
__device__ inline int swz_piece(int p, int z) { return (p & ~7) | ((p ^ z) & 7); }

template <int HT, int TT>
struct AttnMlaLds {
  static constexpr int CT = 16 * TT;
  alignas(16) uint4 kv[2][CT * kMlaPieces];
  // bf16 parts of a probability: 16 heads leave the matrix cores room for all of fp32
  static constexpr int PP = HT == 1 ? 3 : 1;
  alignas(16) uint2 p[PP][TT / 2][HT][64][2];  // [part][token tile pair][ht][lane][tile of the pair]
  int src[kMlaMaxTPW];                     // row gathered for each entry
  uint64_t valid[kMlaMaxTPW / CT];         // valid entries of each chunk
  float cmax[TT][HT * 16], l[TT][HT * 16], sc[HT * 16], m[HT * 16];
  int raise[2];
};

}  // namespace

template <int HT, int TT>
__global__ __launch_bounds__(64 * HT * TT, 2) void attn_mla_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ Kp, const int32_t* __restrict__ slot_map,
    int64_t n_slots, const TokenList tl, const int32_t* __restrict__ ctx_lens, int H_q,
    int H_kv, int T, int B, int m_max, int K_t, int tpw, float sigma, float* __restrict__ po,
    float* __restrict__ plse, uint32_t* err) {
  constexpr int NW = HT * TT, CT = 16 * TT, G = 16 * HT;
  constexpr int NG = kMlaPieces * CT / 64 / NW;  // gathers per wave per chunk
  constexpr int DW = kMlaDv / NW, NNT = DW / 16;  // output dims (tiles) per wave
  constexpr int KS = TT / 2;                      // 32-token steps of the second product
  constexpr int PP = AttnMlaLds<HT, TT>::PP;
  constexpr float kLog2e = 1.4426950408889634f;
  constexpr float kRaise = 8.0f;
  static_assert(NG * NW * 64 == kMlaPieces * CT && DW % 64 == 0 && TT % 2 == 0, "tile geometry");
  __shared__ AttnMlaLds<HT, TT> lds;

  const int unit = blockIdx.y, split = blockIdx.x, nsplit = gridDim.x;
  const int s = unit / H_kv, g = unit % H_kv;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t16 = lane & 15, lg = lane >> 4;
  const int tt = w / HT, ht = w % HT;  // score tile of this wave
  int n = ctx_lens[s];
  n = n < 0 ? 0 : (n > T ? T : n);
  const int p0 = split * tpw;
  const int cnt = max(0, min(tpw, K_t - p0));
  const int nch = (cnt + CT - 1) / CT;

  // this wave's queries: head ht*16 + t16, channels kk*32 + lg*8 .. +8, requested
  // behind the list entries (whose wait would cover them) and in flight with the
  // first rows; ahead of them where no entry is loaded
  bf16x8_t qb[kMlaPieces / 4];
  auto load_q = [&] {
    const uint16_t* qh = q + (size_t(s) * H_q + size_t(g) * G + ht * 16 + t16) * kMlaDqk + lg * 8;
#pragma unroll
    for (int kk = 0; kk < kMlaPieces / 4; ++kk) qb[kk] = *reinterpret_cast<const bf16x8_t*>(qh + kk * 32);
  };
  const bool direct = tl.kind == kListAll && !slot_map;  // uniform
  if (direct) load_q();

  // resolve entries to rows of the unit's K base; a skipped entry gathers a
  // valid row of the same chunk (its probability is zero and its values are
  // finite), or row 0 when the chunk has none (the chunk is then not consumed)
  for (int i0 = w * 64; i0 < nch * CT; i0 += NW * 64) {
    const int i = i0 + lane;
    int row = -1;
    if (i < cnt) {
      bool bad = false;
      const int tok = list_token(tl, unit, p0 + i, n, &bad);
      if (bad) {
        set_error(err, 4u);
      } else if (tok >= 0) {
        if (!slot_map) {
          row = tok;
        } else {
          const int slot = slot_map[size_t(unit) * m_max + tok_block(tok, B)];
          if (slot >= 0 && slot < n_slots) row = slot * B + tok_offset(tok, B);
          else set_error(err, 8u);
        }
      }
    }
    const uint64_t vm = __builtin_amdgcn_ballot_w64(row >= 0);
    int src = row;
    if constexpr (CT == 64) {
      if (row < 0) src = vm ? __builtin_amdgcn_readlane(row, __builtin_ctzll(vm)) : 0;
      if (lane == 0) lds.valid[i0 / CT] = vm;
    } else {  // two chunks of 32 entries
      const uint32_t v0 = uint32_t(vm), v1 = uint32_t(vm >> 32);
      const int s0 = v0 ? __builtin_amdgcn_readlane(row, __builtin_ctz(v0)) : 0;
      const int s1 = v1 ? __builtin_amdgcn_readlane(row, 32 + __builtin_ctz(v1)) : 0;
      if (row < 0) src = lane < 32 ? s0 : s1;
      if (lane == 0) lds.valid[i0 / CT] = v0;
      if (lane == 32 && i0 / CT + 1 < nch) lds.valid[i0 / CT + 1] = v1;
    }
    if (i < nch * CT) lds.src[i] = src;
  }
  if (!direct) load_q();
  if (tid < 2) lds.raise[tid] = 0;
  const size_t ubase = slot_map ? size_t(unit) * size_t(n_slots) * B : size_t(unit) * T;
  const uint8_t* Kb = reinterpret_cast<const uint8_t*>(Kp + ubase * kMlaDqk);
  lds_barrier();

  // chunk c's gathers by this wave: positions (NG w + j) 64 + lane of the
  // chunk's CT x 72 pieces
  int grow[NG], gpiece[NG];
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const int x = (NG * w + j) * 64 + lane;
    grow[j] = x / kMlaPieces;
    gpiece[j] = swz_piece(x % kMlaPieces, (grow[j] >> 1) & 7) * 16;
  }
  auto issue = [&](const int c, const int b) {
    int rows[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) rows[j] = lds.src[c * CT + grow[j]];
#pragma unroll
    for (int j = 0; j < NG; ++j)
      gather16_to_lds(Kb + (size_t(uint32_t(rows[j])) * (kMlaDqk * 2) + gpiece[j]), &lds.kv[b][(NG * w + j) * 64]);
  };

  f32x4_t acc[HT][NNT];
#pragma unroll
  for (int a = 0; a < HT; ++a)
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt) acc[a][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY;  // head ht*16 + t16, base 2 (the same in every wave of the head tile)
  float l_lane = 0.f;       // this lane's share of the head's sum
  const float sl2 = sigma * kLog2e;
  if (nch > 0) issue(0, 0);
  for (int c = 0; c < nch; ++c) {
    const int b = c & 1;
    wave_fence();
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    lds_barrier();  // chunk c has landed for every wave; chunk c - 1 is consumed
    if (c + 1 < nch) issue(c + 1, b ^ 1);
    wave_fence();
    if (tid == 0) lds.raise[b ^ 1] = 0;  // chunk c - 1's flag, read before the barrier above
    const uint64_t vm = lds.valid[c];
    if (vm == 0) continue;  // uniform over the work-group: nothing to consume
    const uint32_t vmask = uint32_t(vm >> (tt * 16)) & 0xffffu;
    // S^T tile: rows = tokens tt*16 + 4lg + r, col = head ht*16 + t16
    f32x4_t st = {0.f, 0.f, 0.f, 0.f}, st1 = {0.f, 0.f, 0.f, 0.f};
    {
      const uint4* row = &lds.kv[b][(tt * 16 + t16) * kMlaPieces];
      const int z = t16 >> 1;
#pragma unroll
      for (int kk = 0; kk < kMlaPieces / 4; kk += 2) {
        const bf16x8_t k0 = __builtin_bit_cast(bf16x8_t, row[4 * kk + (lg ^ z)]);
        const bf16x8_t k1 = __builtin_bit_cast(bf16x8_t, row[4 * kk + ((4 + lg) ^ z)]);
        st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qb[kk], st, 0, 0, 0);
        st1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qb[kk + 1], st1, 0, 0, 0);
      }
    }
    float z[4], zmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[r] = ((vmask >> (lg * 4 + r)) & 1u) ? (st[r] + st1[r]) * sl2 : -INFINITY;
      zmax = fmaxf(zmax, z[r]);
    }
    // probabilities against the maximum m, to this wave's half of the operand
    // (m is -inf while every logit of the head is -inf or NaN: none counts)
    auto write_p = [&](const float m) {
      float ps = 0.f;
      short pb[PP][4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float p = z[r] == -INFINITY || m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(z[r] - m);
        ps += p;
        if constexpr (PP == 1) {
          pb[0][r] = bf16_bits_rne(p);
        } else {  // eight leading bits at a time: every difference is exact, the last part is what is left
#pragma unroll
          for (int k = 0; k < PP; ++k) {
            pb[k][r] = short(__float_as_uint(p) >> 16);
            p -= __uint_as_float(__float_as_uint(p) & 0xffff0000u);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < PP; ++k)
        lds.p[k][tt >> 1][ht][lane][tt & 1] = __builtin_bit_cast(uint2, i16x4_t{pb[k][0], pb[k][1], pb[k][2], pb[k][3]});
      return ps;
    };
    float ps = 0.f;
    const bool larger = zmax > m_run + kRaise;  // also while m_run is -inf
    if (__builtin_amdgcn_ballot_w64(larger) != 0) {
      if (lane == 0) lds.raise[b] = 1;
    } else {
      ps = write_p(m_run);
    }
    lds_barrier();  // the probabilities (or the flag) are written
    if (__builtin_amdgcn_readfirstlane(lds.raise[b]) != 0) {
      const float cm = xrows_max(zmax);
      if (lg == 0) lds.cmax[tt][ht * 16 + t16] = cm;
      lds_barrier();
      float cmax = lds.cmax[0][ht * 16 + t16];
#pragma unroll
      for (int v = 1; v < TT; ++v) cmax = fmaxf(cmax, lds.cmax[v][ht * 16 + t16]);
      const float m_new = cmax > m_run + kRaise ? cmax : m_run;
      const float sc = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      ps = write_p(m_new);
      if (tt == 0 && lg == 0) lds.sc[ht * 16 + t16] = sc;
      l_lane *= sc;
      m_run = m_new;
      lds_barrier();
#pragma unroll
      for (int a = 0; a < HT; ++a) {
        float f[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = lds.sc[a * 16 + lg * 4 + r];
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[a][nt][r] *= f[r];
      }
    }
    l_lane += ps;
    // O += P V for this wave's output dims
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8_t pa[PP][HT];
#pragma unroll
      for (int k = 0; k < PP; ++k)
#pragma unroll
        for (int a = 0; a < HT; ++a) pa[k][a] = *reinterpret_cast<const bf16x8_t*>(&lds.p[k][ks][a][lane][0]);
      // V operand: rows ks*32 + 4lg + (t16 / 4) and 16 more, dims 16nt + 4 (t16 % 4) .. +4
      const int vz = (lg * 2 + (t16 >> 3)) & 7;  // the rows' swizzle
      const uint8_t* vrow = reinterpret_cast<const uint8_t*>(&lds.kv[b][(ks * 32 + lg * 4 + (t16 >> 2)) * kMlaPieces]);
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt) {
        const int piece = DW / 8 * w + (2 * nt & ~7) + ((((2 * nt) & 7) + ((t16 & 3) >> 1)) ^ vz);
        const uint8_t* addr = vrow + piece * 16 + (t16 & 1) * 8;
        const i16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)addr);
        const i16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(addr + 16 * kMlaPieces * 16));
        const bf16x8_t vb = __builtin_bit_cast(
            bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
        for (int a = 0; a < HT; ++a)
#pragma unroll
          for (int k = PP - 1; k >= 0; --k)
            acc[a][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[k][a], vb, acc[a][nt], 0, 0, 0);
      }
    }
  }
  // normalised partial output and lse; lane (lg, t16): heads a*16 + 4lg + r, dim DW w + 16nt + t16
  l_lane = xrows_sum(l_lane);
  if (lg == 0) {
    lds.l[tt][ht * 16 + t16] = l_lane;
    if (tt == 0) lds.m[ht * 16 + t16] = m_run;
  }
  __syncthreads();
  const size_t pbase = (size_t(unit) * nsplit + split) * G;
#pragma unroll
  for (int a = 0; a < HT; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int h = a * 16 + lg * 4 + r;
      float L = 0.f;
#pragma unroll
      for (int v = 0; v < TT; ++v) L += lds.l[v][h];
      const float inv = L > 0.f ? 1.0f / L : 0.f;
#pragma unroll
      for (int nt = 0; nt < NNT; ++nt) {
        // (a sum that is NaN leaves its split out with 16 heads, as on the
        // vector kernel, and makes the output NaN with 32)
        const float o = acc[a][nt][r] * inv;
        po[(pbase + h) * kMlaDv + DW * w + 16 * nt + t16] = HT == 1 && !(L > 0.f) ? 0.f : o;
      }
    }
  if (tid < G) {
    float L = 0.f;
#pragma unroll
    for (int v = 0; v < TT; ++v) L += lds.l[v][tid];
    plse[pbase + tid] = L > 0.f ? (lds.m[tid] + __log2f(L)) * 0.6931471805599453f : -INFINITY;
  }
}

bool mla_mfma_ok(const Problem& P) {
  return P.mla && P.dtype == 1 && P.d_qk == kMlaDqk && P.d_v == kMlaDv && (P.G == 32 || P.G == 16);
}

int mla_mfma_tokens_per_split() { return kMlaMaxTPW; }

// Split count.  More splits shorten a work-group's chain of 64-token chunks
// (about 1.9 us each) but each adds a partial of G x 512 floats per unit,
// written and read back (128 KB of traffic for 32 heads: 0.026 us, the unit of
// the costs below), so the two are weighed, with at most one work-group per
// compute unit.  The merge reads four partials at a time below eight splits and
// the rest one after another (0.3 us each), and from eight on in two columns of
// loads.  Attention and merge, 32 heads, against the former one work-group per
// compute unit (b units of K tokens, us): 8 x 2048: 16 splits 18.7, 32 splits
// 22.3; 16 x 2048: 8 splits 23.4, 16 splits 23.9; 8 x 8192: 32 splits 30.3, 16
// splits 31.5, 64 splits 33.8.  With 32 heads a split may be as short as 32
// tokens, which take half of a chunk's time: few units with few tokens (32-token
// splits against 64-token ones): 1 x 300 11.6, 13.2; 8 x 300 14.2, 14.9; 4 x 500
// 13.4, 14.0; but 8 x 500 15.6, 15.0; 1 x 2048 14.9, 14.8; and where the longer
// splits are four (200 tokens) 13.7, 13.3 with 2 units.
int mla_mfma_splits(const Problem& P, int K_t) {
  constexpr int kChunk = 64;
  const long chunk_cost = 73 * 32 / P.G;  // in partials of one split and unit
  const int need = (K_t + kMlaMaxTPW - 1) / kMlaMaxTPW;
  const int ct = P.G == 32 ? kChunk / 2 : kChunk;  // the smallest split
  int max_ns = device_cus() / P.units;
  if (max_ns > (K_t + ct - 1) / ct) max_ns = (K_t + ct - 1) / ct;
  if (max_ns > kMaxSplits) max_ns = kMaxSplits;
  int best = need;
  long best_cost = -1;
  for (int ns = need; ns <= max_ns; ++ns) {
    const int tokens = (K_t + ns - 1) / ns;
    const long chain = tokens <= kChunk / 2 ? chunk_cost / 2 : (tokens + kChunk - 1) / kChunk * chunk_cost;
    const long cost = chain + long(ns) * P.units + (ns >= 8 ? ns / 4 : (ns > 4 ? (ns - 4) * 12 : 0));
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = ns;
    }
  }
  return best;
}

template <int HT, int TT>
static hipError_t launch_mla_t(const Problem& P, const void* q, const KvView& kv, const TokenList& tl,
                               const int32_t* ctx_lens, int K_t, int nsplit, float* po, float* plse, uint32_t* err,
                               hipStream_t st) {
  constexpr int CT = 16 * TT;
  const int tpw = ((K_t + nsplit - 1) / nsplit + CT - 1) / CT * CT;
  if (tpw > kMlaMaxTPW) return hipErrorInvalidValue;
  attn_mla_mfma_kernel<HT, TT><<<dim3(nsplit, P.units), 64 * HT * TT, 0, st>>>(
      (const uint16_t*)q, (const uint16_t*)kv.k, kv.slot_map, kv.n_slots, tl, ctx_lens, P.H_q, P.H_kv, P.T, P.B,
      P.m_max, K_t, tpw, P.sigma, po, plse, err);
  return hipGetLastError();
}

// 64-token chunks where every work-group has a compute unit to itself (3
// units of 65536 tokens in 64 splits: 53 us against 59), two work-groups of
// 32-token chunks per compute unit where there are more (8 such units: 113 us
// against 122), and 32-token chunks for splits that have no more tokens (see
// mla_mfma_splits).  16 heads have half the waves per token tile and
// always take 64 tokens.
hipError_t launch_attention_mla_mfma(const Problem& P, const void* q, const KvView& kv, const TokenList& tl,
                                     const int32_t* ctx_lens, int K_t, int nsplit, float* po, float* plse,
                                     uint32_t* err, hipStream_t st) {
  if (P.G == 16) return launch_mla_t<1, 4>(P, q, kv, tl, ctx_lens, K_t, nsplit, po, plse, err, st);
  if (long(P.units) * nsplit <= device_cus() && K_t > 32 * nsplit)
    return launch_mla_t<2, 4>(P, q, kv, tl, ctx_lens, K_t, nsplit, po, plse, err, st);
  return launch_mla_t<2, 2>(P, q, kv, tl, ctx_lens, K_t, nsplit, po, plse, err, st);
}

}  // namespace tls
