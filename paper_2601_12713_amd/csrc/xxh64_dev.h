// XXH64 building blocks for gfx950, from the public xxHash specification:
// five 64-bit primes, four accumulators over 32-byte stripes, the 8/4/1-byte
// remainder steps and the final avalanche. The library runs the four
// accumulators of one input on four adjacent lanes of a wavefront.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace odp {

constexpr uint64_t kP1 = 0x9E3779B185EBCA87ull;
constexpr uint64_t kP2 = 0xC2B2AE3D27D4EB4Full;
constexpr uint64_t kP3 = 0x165667B19E3779F9ull;
constexpr uint64_t kP4 = 0x85EBCA77C2B2AE63ull;
constexpr uint64_t kP5 = 0x27D4EB2F165667C5ull;

__device__ __forceinline__ uint64_t rotl64(uint64_t x, int r) { return (x << r) | (x >> (64 - r)); }

// One stripe word folded into one accumulator.
__device__ __forceinline__ uint64_t xx_round(uint64_t acc, uint64_t w) {
  acc += w * kP2;
  acc = rotl64(acc, 31);
  return acc * kP1;
}

__device__ __forceinline__ uint64_t xx_merge(uint64_t h, uint64_t v) {
  h ^= xx_round(0, v);
  return h * kP1 + kP4;
}

// Initial value of accumulator `a` (0..3) for `seed`.
__device__ __forceinline__ uint64_t xx_acc_init(uint64_t seed, int a) {
  return a == 0 ? seed + kP1 + kP2 : a == 1 ? seed + kP2 : a == 2 ? seed : seed - kP1;
}

// Folds the four accumulators into the running hash (inputs of >= 32 bytes).
__device__ __forceinline__ uint64_t xx_converge(uint64_t v1, uint64_t v2, uint64_t v3, uint64_t v4) {
  uint64_t h = rotl64(v1, 1) + rotl64(v2, 7) + rotl64(v3, 12) + rotl64(v4, 18);
  h = xx_merge(h, v1);
  h = xx_merge(h, v2);
  h = xx_merge(h, v3);
  return xx_merge(h, v4);
}

__device__ __forceinline__ uint64_t xx_step8(uint64_t h, uint64_t w) {
  h ^= xx_round(0, w);
  return rotl64(h, 27) * kP1 + kP4;
}
__device__ __forceinline__ uint64_t xx_step4(uint64_t h, uint32_t w) {
  h ^= uint64_t(w) * kP1;
  return rotl64(h, 23) * kP2 + kP3;
}
__device__ __forceinline__ uint64_t xx_step1(uint64_t h, uint8_t b) {
  h ^= uint64_t(b) * kP5;
  return rotl64(h, 11) * kP1;
}

__device__ __forceinline__ uint64_t xx_avalanche(uint64_t h) {
  h ^= h >> 33;
  h *= kP2;
  h ^= h >> 29;
  h *= kP3;
  h ^= h >> 32;
  return h;
}

// Little-endian 8 bytes at any address, from the two or three 4-byte words that
// hold them (nothing else is touched), without a branch: loads under one are
// waited for before the next is issued (20,000 buffers up to 1 MiB at byte
// addresses: 977 -> 724 us against a second 8-byte load where p needs one).
__device__ __forceinline__ uint64_t load64_any(const uint8_t* p) {
  typedef uint64_t u64_a4 __attribute__((aligned(4)));
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  const uint64_t w = *reinterpret_cast<const u64_a4*>(a & ~uintptr_t(3));
  const uint32_t last = *reinterpret_cast<const uint32_t*>((a + 7) & ~uintptr_t(3));
  const uint32_t w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32), sh = (uint32_t)(a & 3);
  return (uint64_t)__builtin_amdgcn_alignbyte(w1, w0, sh) | (uint64_t)__builtin_amdgcn_alignbyte(last, w1, sh) << 32;
}

// Little-endian first min(avail, 8) bytes at p (any address, avail > 0); the
// bytes above them are undefined. Only 8-byte granules that hold some of
// [p, p + avail) are read.
__device__ __forceinline__ uint64_t load64_part(const uint8_t* p, uint32_t avail) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  const uint64_t* q = reinterpret_cast<const uint64_t*>(a & ~uintptr_t(7));
  const uint32_t o = uint32_t(a & 7);
  uint64_t v = q[0] >> (8 * o);
  if (o + (avail < 8 ? avail : 8) > 8) v |= q[1] << (64 - 8 * o);  // o > 0 here
  return v;
}

// The remainder steps over the rem (1..31) bytes held in four words.
__device__ __forceinline__ uint64_t xx_tail_words(uint64_t h, uint64_t x0, uint64_t x1, uint64_t x2, uint64_t x3,
                                                  uint32_t rem) {
  const uint32_t n8 = rem >> 3;
  if (n8 > 0) h = xx_step8(h, x0);
  if (n8 > 1) h = xx_step8(h, x1);
  if (n8 > 2) h = xx_step8(h, x2);
  uint64_t x = n8 == 0 ? x0 : n8 == 1 ? x1 : n8 == 2 ? x2 : x3;
  if (rem & 4) {
    h = xx_step4(h, (uint32_t)x);
    x >>= 32;
  }
  for (uint32_t r = rem & 3; r > 0; --r, x >>= 8) h = xx_step1(h, (uint8_t)x);
  return h;
}

// Lane k of each group of four lanes, broadcast to the group (DPP quad_perm,
// a VALU move: no LDS round trip on the accumulator chain). Every lane of the
// group must be active.
template <int K>
__device__ __forceinline__ uint64_t xx_quad_bcast(uint64_t x) {
  constexpr int ctrl = K * 0x55;  // quad_perm:[K,K,K,K]
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, ctrl, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), ctrl, 0xF, 0xF, false);
  return ((uint64_t)hi << 32) | lo;
}

// Gathers the accumulator of lanes 4g..4g+3 into all four lanes.
__device__ __forceinline__ void xx_gather4(uint64_t acc, uint64_t& v1, uint64_t& v2, uint64_t& v3, uint64_t& v4) {
  v1 = xx_quad_bcast<0>(acc);
  v2 = xx_quad_bcast<1>(acc);
  v3 = xx_quad_bcast<2>(acc);
  v4 = xx_quad_bcast<3>(acc);
}

// XXH64 of `nw` little-endian u64 words (a tree node's children), computed by
// the four lanes 4g..4g+3 together; every one of them returns the digest.
// `w` may point to LDS or global memory.
__device__ __forceinline__ uint64_t xx_words4(const uint64_t* w, uint32_t nw, uint64_t seed) {
  const int a = threadIdx.x & 3;
  uint32_t nstripes = nw / 4;
  uint64_t acc = xx_acc_init(seed, a);
  for (uint32_t s = 0; s < nstripes; ++s) acc = xx_round(acc, w[s * 4 + a]);
  uint64_t v1, v2, v3, v4;
  xx_gather4(acc, v1, v2, v3, v4);
  uint64_t h = nstripes ? xx_converge(v1, v2, v3, v4) : seed + kP5;
  h += uint64_t(nw) * 8;
  for (uint32_t i = nstripes * 4; i < nw; ++i) h = xx_step8(h, w[i]);
  return xx_avalanche(h);
}

// XXH64 of exactly 64 words (a full tree node) by lanes 4g..4g+3; every lane
// returns the digest. One four-lane chain is bound by latency, not issue, so
// every stripe word and its product with P2 are formed before the chain
// starts, and only the add, the rotation and the multiply by P1 wait on the
// previous round. Same result as xx_words4(w, 64, seed).
__device__ __forceinline__ uint64_t xx_words4_full64(const uint64_t* w, uint64_t seed) {
  const int a = threadIdx.x & 3;
  uint64_t t[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) t[s] = w[s * 4 + a];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    t[s] *= kP2;
    asm volatile("" : "+v"(t[s]));  // keeps the product out of the accumulator's multiply-add
  }
  uint64_t acc = xx_acc_init(seed, a);
#pragma unroll
  for (int s = 0; s < 16; ++s) acc = rotl64(acc + t[s], 31) * kP1;
  uint64_t v1, v2, v3, v4;
  xx_gather4(acc, v1, v2, v3, v4);
  return xx_avalanche(xx_converge(v1, v2, v3, v4) + 64 * 8);
}

}  // namespace odp
