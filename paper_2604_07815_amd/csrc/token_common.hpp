// Helpers shared by the token-selection kernels.
#pragma once

#include "attn_common.hpp"
#include "kernels.hpp"

namespace tls {

// Eight 4-bit codes of one packed dword (byte i = code[2i] | code[2i+1] << 4)
// as floats, in channel order.
__device__ inline void unpack_nibbles8(uint32_t w, float* f) {
  const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
  f[0] = float(lo & 0xffu);         f[1] = float(hi & 0xffu);
  f[2] = float((lo >> 8) & 0xffu);  f[3] = float((hi >> 8) & 0xffu);
  f[4] = float((lo >> 16) & 0xffu); f[5] = float((hi >> 16) & 0xffu);
  f[6] = float(lo >> 24);           f[7] = float(hi >> 24);
}

// The alpha key of a candidate: alpha >= +0 has the key bits | 2^31 (as
// float_key); a NaN alpha (NaN inputs only) ranks as 0.
__device__ inline uint32_t alpha_key(float a) { return __float_as_uint(fmaxf(a, 0.f)) | 0x80000000u; }

// A packed dword of codes (channel 2i in the low nibble of byte i) as bf16
// numbers, in the channel order 0, 2, 4, 6, 1, 3, 5, 7 of a matrix operand.  As
// an fp8 number (e4m3) a byte c < 16 is c 2^-9, subnormal up to 7 and normal
// above, so the conversion with a scale of 2^9 gives c itself: seven
// instructions, and nothing has to come off the dot afterwards.
__device__ inline uint4 codes_bf16(uint32_t w) {
  const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
  return make_uint4(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, true)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, true)));
}
// channel of position j (< 8) in that order
__device__ inline int codes_chan(int j) { return 2 * (j & 3) | (j >> 2); }

// The code contraction of 64 tokens of a wave, one per lane, with up to 4 HS
// heads on one 32-channel group.  The tokens are four tiles of 16, lane (lg,
// t16) owning token t16 of tile lg.  v_mfma_f32_16x16x32_bf16 takes B = one
// tile's codes (the lanes' dwords transposed over the lane groups with four
// swaps) and A = four heads' q~ in the rows 4 tl + r of tile tl, zeros
// elsewhere, so that the four tiles' products accumulate in one result whose
// lane (lg, t16) holds its own token's dots with heads r: nothing is
// rearranged afterwards.
//
// lane_operands: the A operands and the heads' sums of q~ (the same product
// with B = 1) from the group's q~ table [set][head of 4][32], channels in the
// order of codes_chan, zeros for the heads past G.
template <int HS>
__device__ inline void lane_operands(const uint16_t* s_qt, bf16x8_t (&qa)[HS][4], f32x4_t (&qsum)[HS]) {
  const int t16 = __lane_id() & 15, lg = __lane_id() >> 4;
  const uint4 one = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) {
    const uint4 row = *reinterpret_cast<const uint4*>(s_qt + (hs * 4 + (t16 & 3)) * 32 + lg * 8);
    qsum[hs] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tl = 0; tl < 4; ++tl) {
      qa[hs][tl] = __builtin_bit_cast(bf16x8_t, t16 >> 2 == tl ? row : make_uint4(0, 0, 0, 0));
      qsum[hs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[hs][tl], __builtin_bit_cast(bf16x8_t, one), qsum[hs], 0, 0, 0);
    }
  }
}

// Products of this lane's codes with the heads' q~.
// Every lane of the wave must be active.
template <int HS>
__device__ inline void lane_dots(const uint4& c, const bf16x8_t (&qa)[HS][4], f32x4_t (&acc)[HS]) {
  // dword lg of tile tl's token t16
  const auto a02 = __builtin_amdgcn_permlane32_swap(c.x, c.z, false, false);
  const auto a13 = __builtin_amdgcn_permlane32_swap(c.y, c.w, false, false);
  const auto b01 = __builtin_amdgcn_permlane16_swap(a02[0], a13[0], false, false);
  const auto b23 = __builtin_amdgcn_permlane16_swap(a02[1], a13[1], false, false);
  const uint32_t wd[4] = {b01[0], b01[1], b23[0], b23[1]};
#pragma unroll
  for (int hs = 0; hs < HS; ++hs) acc[hs] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int tl = 0; tl < 4; ++tl) {
    const bf16x8_t b = __builtin_bit_cast(bf16x8_t, codes_bf16(wd[tl]));
#pragma unroll
    for (int hs = 0; hs < HS; ++hs) acc[hs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[hs][tl], b, acc[hs], 0, 0, 0);
  }
}

// Candidate slot -> token position.  slot = i*B + o addresses offset o of the
// i-th entry of the unit's block list; valid when that entry is a block id
// >= 0 and the token lies below ctx_len.  Ids past the last block set
// TLS_DEVERR_BLOCK_ID and are skipped.
__device__ inline bool slot_token(const int32_t* bl, int K_b, int B, int m, int n, int slot, int* tok,
                                  uint32_t* err) {
  const int i = tok_block(slot, B), o = tok_offset(slot, B);
  if (i >= K_b) return false;
  const int blk = bl[i];
  if (blk < 0) return false;
  if (blk >= m) {
    set_error(err, 2u);
    return false;
  }
  const int t = blk * B + o;
  *tok = t;
  return t < n;
}

}  // namespace tls
