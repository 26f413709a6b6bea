// Device-side building blocks for the sampling kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace a3 {

constexpr int kWave = 64;
constexpr int32_t kMapEmpty = 0x7FFFFFFF;

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t other = __shfl_xor(v, o, kWave);
    v = other > v ? other : v;
  }
  return v;
}

// LDS traffic between the lanes of one wavefront: LDS executes a wavefront's accesses in order,
// so only the compiler has to be kept from moving them.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {  // set bits of mask in lower lanes
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A data-parallel move inside a row of 16 lanes is an operand of an ordinary vector instruction,
// where __shfl goes through the LDS unit (some hundred cycles a step).  Lanes without a source read 0.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)v, kCtrl, 0xf, 0xf, true);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;            // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;  // i -> 7 - i in a half row, i -> 15 - i in a row
constexpr int kDppShr = 0x110, kDppLast = 0x15F;           // lane i from i - n; every lane from lane 15
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;    // the row's / half's last lane to the next one

__device__ __forceinline__ uint32_t row16_incl_scan(uint32_t v) {
  v += dpp_u32<kDppShr + 1>(v);
  v += dpp_u32<kDppShr + 2>(v);
  v += dpp_u32<kDppShr + 4>(v);
  v += dpp_u32<kDppShr + 8>(v);
  return v;
}
__device__ __forceinline__ uint32_t row16_last(uint32_t v) { return dpp_u32<kDppLast>(v); }

// exclusive prefix sum across the 64 lanes of a wave, all of them active
__device__ __forceinline__ uint32_t wave_excl_scan_u32(uint32_t v) {
  uint32_t incl = row16_incl_scan(v);
  incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)incl, kDppBcast15, 0xa, 0xf, false);  // rows 1, 3
  incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int32_t)incl, kDppBcast31, 0xc, 0xf, false);  // rows 2, 3
  return incl - v;
}

// a ^ b ^ c as one instruction, where the compiler makes two of it.  The scan of a row is bound by
// the vector instructions of its Philox blocks (17 multiplies, then 32 xors, now 14 of these and
// 4 xors): 252 -> 200 cycles per 64 blocks on one SIMD; a mini-batch on 100 M nodes 868 -> 812 us.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon et al., SC'11).  One block yields the draws of four
// consecutive neighbour slots: counter (slot >> 2, node lo, node hi, hop),
// key (seed lo, seed hi); slot s reads word s & 3.
struct PhiloxKey {
  uint32_t c1, c2, c3;  // node lo, node hi, hop
  uint32_t k0, k1;      // seed lo, seed hi
};

__device__ __forceinline__ void philox4x32_10(uint32_t q, const PhiloxKey& pk, uint32_t x[4]) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
  uint32_t c0 = q, c1 = pk.c1, c2 = pk.c2, c3 = pk.c3;
  uint32_t k0 = pk.k0, k1 = pk.k1;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)M0 * c0;
    const uint64_t p1 = (uint64_t)M1 * c2;
    const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
    // where a wavefront draws for one node, only c0 differs between its lanes: c1, k0 stay scalar
    // for two rounds, c3, k1 for three
    const uint32_t n0 = r < 2 ? h1 ^ (c1 ^ k0) : xor3(h1, c1, k0);
    const uint32_t n2 = r < 1 ? h0 ^ (c3 ^ k1) : r < 2 ? c3 ^ (h0 ^ k1) : r < 3 ? h0 ^ (c3 ^ k1) : xor3(h0, c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += W0;
    k1 += W1;
  }
  x[0] = c0; x[1] = c1; x[2] = c2; x[3] = c3;
}

// log2(U), U in [1, 2^32], as Q6.32: shift-and-square on a Q1.31 mantissa,
// products truncated.  Integer only, so host and device agree bit for bit.
__device__ __forceinline__ uint64_t fixlog2_q32(uint64_t U) {
  const int e = 63 - __clzll((long long)U);
  uint32_t t = (e == 32) ? 0x80000000u : (uint32_t)(U << (31 - e));
  uint32_t frac = 0;
#pragma unroll 4
  for (int i = 1; i <= 32; ++i) {
    const uint64_t p = (uint64_t)t * t;
    const bool hi = (p >> 63) != 0;
    frac |= hi ? (1u << (32 - i)) : 0u;
    t = hi ? (uint32_t)(p >> 32) : (uint32_t)(p >> 31);
  }
  return ((uint64_t)e << 32) | frac;
}

// floor(n / w) for n < 2^54 with at most 38 significant bits (n = L << 16, L < 2^38) and
// 2^16 <= w < 2^32, given inv_w = 1.0 / w rounded to double: n is exact in a double, the product
// is within 2^-14 of n / w, so its integer part is the quotient or one beside it, and one
// correction by the remainder makes it exact.  A dozen instructions where the 64-bit division
// takes some eighty.
__device__ __forceinline__ uint64_t div_by_weight(uint64_t n, uint32_t w, double inv_w) {
  uint64_t q = (uint64_t)((double)n * inv_w);
  const int64_t r = (int64_t)(n - q * (uint64_t)w);
  if (r < 0) q -= 1;
  else if (r >= (int64_t)w) q += 1;
  return q;
}

// Alg. 2, key step in the log domain: -log2(u)/w in Q32 with u = (x+1)/2^32; inv_w = 1.0 / w_q16.
__device__ __forceinline__ uint64_t sample_key(uint32_t x, uint32_t w_q16, double inv_w) {
  const uint64_t L = (32ull << 32) - fixlog2_q32((uint64_t)x + 1);
  return div_by_weight(L << 16, w_q16, inv_w);
}

// order of equal-weight slots: larger draw first, then smaller slot
__device__ __forceinline__ uint64_t draw_order_key(uint32_t x, uint32_t slot) {
  return ((uint64_t)(~x) << 32) | slot;
}

}  // namespace a3
