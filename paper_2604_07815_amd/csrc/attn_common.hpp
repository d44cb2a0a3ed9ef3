// Helpers shared by the attention kernels.
#pragma once

#include "kernels.hpp"

namespace tls {

// Address of token `tok`'s row in the direct layout [units][T][d] or, with a
// slot map, in the block pool [units][n_slots][B][d].  *ok turns false when
// the token's block is not resident.
template <class S>
__device__ inline const S* kv_row(const S* base, const int32_t* slot_map, int64_t n_slots, size_t unit, int T,
                                  int B, int m_max, int d, int tok, bool* ok) {
  if (!slot_map) return base + (unit * size_t(T) + size_t(tok)) * d;
  const int slot = slot_map[unit * size_t(m_max) + tok_block(tok, B)];
  if (slot < 0 || slot >= n_slots) {
    *ok = false;
    return base;
  }
  return base + ((unit * size_t(n_slots) + size_t(slot)) * B + tok_offset(tok, B)) * d;
}

// Token of entry p of a unit's work list (-1: empty).  *bad turns true for
// an explicit id at or past ctx_len n (the caller flags it and skips it).
__device__ inline int list_token(const TokenList& L, size_t unit, int p, int n, bool* bad) {
  if (L.kind == kListIds) {
    const int t = L.ids[unit * size_t(L.stride) + p];
    if (t >= n) {
      *bad = true;
      return -1;
    }
    return t < 0 ? -1 : t;
  }
  if (L.kind == kListBlocks) {
    const int blk = L.ids[unit * size_t(L.stride) + tok_block(p, L.B)];
    const int t = blk * L.B + tok_offset(p, L.B);
    return blk < 0 || t >= n ? -1 : t;
  }
  return p < n ? p : -1;
}

// s_waitcnt immediates (gfx9 encoding): vmcnt in [3:0] and [15:14],
// expcnt in [6:4], lgkmcnt in [11:8].
__host__ __device__ constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int kWaitLgkm0 = 0xC07F;

// Work-group barrier for LDS traffic only: completes this wave's LDS
// accesses, then synchronises, leaving global loads (including the
// asynchronous LDS gathers of the next chunk) in flight.  The
// wavefront-scope fences keep the compiler from moving memory accesses
// across it.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef __attribute__((address_space(3))) void lds_void;

// Asynchronous 16-byte-per-lane gather into LDS: lane i reads 16 bytes at
// `src` and the wave writes them to lds + 16*i.  Issued through inline asm so
// that the compiler does not order later LDS accesses behind it; completion
// is tracked explicitly with s_waitcnt vmcnt and a work-group barrier before
// the data is read, and the target buffer is not read or rewritten while a
// gather into it is in flight.  The s_nop is the wait state that gfx9 requires
// between a scalar write of M0 and an LDS-DMA load that reads it (the compiler
// inserts none inside an asm block).
__device__ inline void gather16_to_lds(const void* src, const void* lds) {
  // the LDS destination is wave-uniform; readfirstlane puts it in an SGPR
  const uint32_t off = uint32_t(__builtin_amdgcn_readfirstlane(int(reinterpret_cast<uintptr_t>((lds_void*)lds))));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "s"(off), "v"(src) : "m0");
}

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// Compiler-level ordering point for LDS accesses around the inline-asm
// gathers (emits no instruction at wavefront scope).
__device__ inline void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Max / sum over the lanes i, i^16, i^32, i^48 (one per DPP row) through the
// gfx950 row-swap permutes; every lane gets the same bits.
__device__ inline float xrows_max(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float xrows_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4;

__device__ inline short bf16_bits_rne(float f) {
  uint32_t u = __float_as_uint(f);  // finite, non-negative here
  u += 0x7fffu + ((u >> 16) & 1u);
  return short(u >> 16);
}

__device__ inline float exp_or_zero(float x) { return x == -INFINITY ? 0.f : expf(x); }

// ---------------------------------------------------------------------------
// Split merge by a unit's last work-group, without a launch of its own.
//
// The work-groups of a unit store their partials and count themselves in; the
// last one reads them all and writes the output.  They may run on different
// XCDs, whose L2 caches are not coherent for ordinary accesses, and a device
// fence would write back and invalidate a whole L2 (measured: 4 times the
// attention's time).  So the partials themselves are relaxed agent-scope
// atomics, 4 bytes a store and 8 a load, which go past the L2s to memory: a
// wave waits for its stores (vmcnt), the work-group meets at a barrier, and
// only then the count is raised; the last arrival's loads are issued after its
// count came back.  The count is cleared by the kernel that chose the tokens,
// earlier in the same call.
// ---------------------------------------------------------------------------
struct SplitOut {
  float* po;         // [units][nsplit][G][D]
  float* plse;       // [units][nsplit][G]
  uint32_t* arrive;  // [units] arrivals, or NULL: merge_kernel combines the partials
  void* out;         // used with arrive
  float* lse;
};

__device__ inline void store_partial(const SplitOut& so, float* p, float v) {
  if (so.arrive) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
__device__ inline float2 load_partial2(const float* p) {
  const uint64_t u = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float(uint32_t(u)), __uint_as_float(uint32_t(u >> 32)));
}

// Called by all NT threads of a work-group after its partials' stores;
// `scratch`: G * kMaxSplits + 1 words of LDS that nothing else uses any more.
// Output rows of the unit start at orow.
template <class E, int NT, int D>
__device__ inline void arrive_and_merge(const SplitOut& so, int unit, int nsplit, int G, size_t orow,
                                        uint32_t* scratch) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");  // this wave's partials are in memory
  __syncthreads();
  if (tid == 0) scratch[0] = __hip_atomic_fetch_add(so.arrive + unit, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (scratch[0] != uint32_t(nsplit - 1)) return;  // uniform
  asm volatile("" : : : "memory");
  // split weights e^{lse_i - M} / sum_j e^{lse_j - M}; lane l holds splits l, l + 64
  float* s_w = reinterpret_cast<float*>(scratch) + 1;  // [G][nsplit]
  const float* ls = so.plse + size_t(unit) * nsplit * G;
  for (int h = wid; h < G; h += NW) {
    constexpr int PER = kMaxSplits / 64;
    float l[PER], lm = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = lane + 64 * j;
      l[j] = i < nsplit ? __hip_atomic_load(ls + size_t(i) * G + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -INFINITY;
      lm = fmaxf(lm, l[j]);
    }
    const float M = wave_max_f32(lm);
    float e[PER], es = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      e[j] = M == -INFINITY ? 0.f : exp_or_zero(l[j] - M);
      es += e[j];
    }
    const float W = wave_sum_f32(es);
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (lane + 64 * j < nsplit) s_w[h * nsplit + lane + 64 * j] = W > 0.f ? e[j] / W : 0.f;
    if (lane == 0 && so.lse) so.lse[orow + h] = W > 0.f ? M + logf(W) : -INFINITY;
  }
  __syncthreads();
  const float* base = so.po + size_t(unit) * nsplit * G * D;
  const size_t stride = size_t(G) * D;
  // summed in merge_kernel's order, so that both give the same bits: with
  // eight or more splits split i belongs to partial sum i % ROWS, with fewer
  // to i % 4 (the ones past the last four to 0)
  constexpr int ROWS = 256 / (D / 4), U = ROWS > 8 ? ROWS : 16;  // U partials in flight
  static_assert(U % ROWS == 0, "partial sums per batch");
  for (int x = 2 * tid; x < G * D; x += 2 * NT) {
    const float* w = s_w + x / D * nsplit;
    float o0 = 0.f, o1 = 0.f;
    if (nsplit >= 8) {
      float2 acc[ROWS];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) acc[r] = make_float2(0.f, 0.f);
      for (int i0 = 0; i0 < nsplit; i0 += U) {
        float2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load_partial2(base + size_t(min(i0 + u, nsplit - 1)) * stride + x);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = i0 + u < nsplit;
          const float wu = in ? w[i0 + u] : 0.f;
          acc[u % ROWS].x = fmaf(wu, in ? v[u].x : 0.f, acc[u % ROWS].x);
          acc[u % ROWS].y = fmaf(wu, in ? v[u].y : 0.f, acc[u % ROWS].y);
        }
      }
      o0 = acc[0].x;
      o1 = acc[0].y;
#pragma unroll
      for (int r = 1; r < ROWS; ++r) {
        o0 += acc[r].x;
        o1 += acc[r].y;
      }
    } else {
      float2 v[8], acc[4];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = load_partial2(base + size_t(min(i, nsplit - 1)) * stride + x);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = make_float2(0.f, 0.f);
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        if (i < nsplit) {
          const int r = i < (nsplit & ~3) ? i % 4 : 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            acc[k].x = k == r ? fmaf(w[i], v[i].x, acc[k].x) : acc[k].x;
            acc[k].y = k == r ? fmaf(w[i], v[i].y, acc[k].y) : acc[k].y;
          }
        }
      }
      o0 = (acc[0].x + acc[1].x) + (acc[2].x + acc[3].x);
      o1 = (acc[0].y + acc[1].y) + (acc[2].y + acc[3].y);
    }
    typename E::T* o = static_cast<typename E::T*>(so.out) + orow * D + x;
    store_out<E>(o, o0);
    store_out<E>(o + 1, o1);
  }
}

// Transposing butterfly all-reduce over the MASK*2 lanes of a lane group:
// while more than one value is left, each xor step sends half of the values
// to the partner lane and keeps the other half, so NV values are reduced with
// NV - 1 shuffles instead of NV*log2(W).  On return v[j] holds the fully
// reduced value of original index xreduce_index<NV, W>(lane, j), for
// j < max(1, NV / W).
template <int NV, int MASK>
struct XReduce {
  __device__ static inline void run(float* v, int lane) {
    if constexpr (MASK == 0) {
      return;
    } else if constexpr (NV > 1) {
      constexpr int H = NV / 2;
      const bool upper = (lane & MASK) != 0;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const float send = upper ? v[j] : v[j + H];
        const float keep = upper ? v[j + H] : v[j];
        v[j] = keep + __shfl_xor(send, MASK, 64);
      }
      XReduce<H, MASK / 2>::run(v, lane);
    } else {
      v[0] += __shfl_xor(v[0], MASK, 64);
      XReduce<1, MASK / 2>::run(v, lane);
    }
  }
};

// The same transposing reduction with the partner lane chosen by DPP mirror
// patterns inside 16-lane rows (row_mirror, row_half_mirror, quad reverse,
// quad swap): a VALU lane move instead of an LDS-routed shuffle.  Within a
// group of W lanes the mirror partner has the opposite W/2 bit and the same
// higher bits, so the kept halves and the resulting index map are those of
// XReduce.  A 32-lane first step (W = 32) uses one xor-16 shuffle.
template <int CTRL>
__device__ inline float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xF, 0xF, false));
}

template <int W>
__device__ inline float mirror_partner(float v) {
  if constexpr (W == 32) return __shfl_xor(v, 16, 64);
  else if constexpr (W == 16) return dpp_mov<0x140>(v);  // row_mirror
  else if constexpr (W == 8) return dpp_mov<0x141>(v);   // row_half_mirror
  else if constexpr (W == 4) return dpp_mov<0x1B>(v);    // quad_perm [3,2,1,0]
  else return dpp_mov<0xB1>(v);                          // quad_perm [1,0,3,2]
}

template <int NV, int W>
struct XReduceDpp {
  __device__ static inline void run(float* v, int lane) {
    if constexpr (W < 2) {
      return;
    } else if constexpr (NV > 1) {
      constexpr int H = NV / 2;
      const bool upper = (lane & (W / 2)) != 0;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const float send = upper ? v[j] : v[j + H];
        const float keep = upper ? v[j + H] : v[j];
        v[j] = keep + mirror_partner<W>(send);
      }
      XReduceDpp<H, W / 2>::run(v, lane);
    } else {
      v[0] += mirror_partner<W>(v[0]);
      XReduceDpp<1, W / 2>::run(v, lane);
    }
  }
};

template <int NV, int W>
__device__ inline int xreduce_index(int lane, int j) {
  int idx = j, cur = NV;
#pragma unroll
  for (int mask = W / 2; mask > 0; mask >>= 1) {
    if (cur > 1) {
      cur >>= 1;
      if (lane & mask) idx += cur;
    }
  }
  return idx;
}

}  // namespace tls
