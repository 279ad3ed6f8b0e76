// Device helpers for the Moss sampling kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moss {

// Philox4x64 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC 2011).  Each round
// takes the 128-bit products of words 0 and 2 with two odd multipliers; the next
// state is (hi(M1 x2) ^ x1 ^ k0, lo(M1 x2), hi(M0 x0) ^ x3 ^ k1, lo(M0 x0)); the key
// advances by two Weyl increments between rounds.
constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// The 128-bit product a * b as four 32 x 32 -> 64-bit partial products, each one
// multiply-add (v_mad_u64_u32); none of the partial sums exceeds 64 bits.  Spelled out
// because the high half written as __umul64hi next to a 64-bit low product compiles to
// about a third more multiplies.
__device__ __forceinline__ void mul_wide(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t p = (uint64_t)a0 * b0;
  const uint64_t t = (uint64_t)a1 * b0 + (p >> 32);
  const uint64_t u = (uint64_t)a0 * b1 + (uint32_t)t;
  hi = (uint64_t)a1 * b1 + (t >> 32) + (u >> 32);
  lo = (u << 32) | (uint32_t)p;
}

// The two products of a Philox round, x0 * M0 and x2 * M1, each with its two middle partial
// products added by one multiply-add whose carry out (bit 96 of the product) becomes the
// upper word of the last addend: 4 multiply-adds and 3 other instructions a product
// against mul_wide's 9 in all (a 64-bit addend needs its upper word cleared or copied by
// moves).  The compiler has no form that yields the carry.  gfx950 wants two wait states
// between a vector instruction that writes a scalar register and a vector instruction
// that reads it, and the compiler does not look into the block for them: between each
// multiply-add and the select of its carry there are two instructions, and the block reads
// no scalar register from outside.
__device__ __forceinline__ void philox_products(uint64_t x0, uint64_t x2, uint64_t& hi0, uint64_t& lo0,
                                                uint64_t& hi1, uint64_t& lo1) {
  constexpr uint32_t a0 = (uint32_t)kPhiloxM0, a1 = (uint32_t)(kPhiloxM0 >> 32);
  constexpr uint32_t b0 = (uint32_t)kPhiloxM1, b1 = (uint32_t)(kPhiloxM1 >> 32);
  const uint32_t xl = (uint32_t)x0, xh = (uint32_t)(x0 >> 32), yl = (uint32_t)x2, yh = (uint32_t)(x2 >> 32);
  const uint64_t p = (uint64_t)xl * a0, q = (uint64_t)yl * b0;
  uint64_t m = (uint64_t)xl * a1 + (p >> 32), n = (uint64_t)yl * b1 + (q >> 32);
  uint32_t c, d;
  uint64_t cc, dd;  // the carries, one bit per lane
  asm("v_mad_u64_u32 %0, %4, %6, %8, %0\n\t"
      "v_mad_u64_u32 %1, %5, %7, %9, %1\n\t"
      "s_nop 0\n\t"
      "v_cndmask_b32_e64 %2, 0, 1, %4\n\t"
      "v_cndmask_b32_e64 %3, 0, 1, %5"
      : "+&v"(m), "+&v"(n), "=&v"(c), "=&v"(d), "=&s"(cc), "=&s"(dd)
      : "v"(xh), "v"(yh), "v"(a0), "v"(b0));
  hi0 = (uint64_t)xh * a1 + (((uint64_t)c << 32) | (m >> 32));
  lo0 = (m << 32) | (uint32_t)p;
  hi1 = (uint64_t)yh * b1 + (((uint64_t)d << 32) | (n >> 32));
  lo1 = (n << 32) | (uint32_t)q;
}

__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_bitop3_b32((int)(a >> 32), (int)(b >> 32), (int)(c >> 32), 0x96);
  return (uint64_t)hi << 32 | lo;
}

// Random words of block `blk` of sample `k`: counter (k, blk, 0, 0), key (seed, tag);
// blk, seed and tag are the same for every lane of the wave.
//
// Bound by VALU issue: every instruction of it takes an issue slot of about four cycles
// whatever it is (a v_mad_u64_u32 as a v_xor_b32), so what counts is their number.  The
// first round multiplies word 0 only (words 1 to 3 are blk, 0, 0) and the second's word 0
// is uniform and multiplied on the scalar unit.  The round keys are made opaque per
// block, so that the scalar unit computes them between the vector instructions (the
// compiler otherwise keeps forty of them live across a sampling loop, in VGPR lanes, one
// v_readlane_b32 each) and the three-way xors take one v_bitop3_b32 a word.  A round is
// 18 vector instructions, a block 194 instead of 257; alone on the chip 1.99e11 -> 2.48e11
// blocks/s, and a 256-request batch (two or three blocks a sample) 23.9 -> 22.1 ms.
__device__ __forceinline__ void philox_block(uint64_t k, uint64_t blk, uint64_t seed, uint64_t tag,
                                             uint64_t out[4]) {
  uint64_t k0 = seed, k1 = tag;
  asm volatile("" : "+s"(k0), "+s"(k1));
  uint64_t hi0, lo0, hi1, lo1;
  // round 0
  mul_wide(k, kPhiloxM0, hi0, lo0);
  const uint64_t s0 = blk ^ k0;  // word 0 of every lane
  uint64_t x2 = hi0 ^ k1;
  const uint64_t y3 = lo0;
  // round 1
  k0 += kPhiloxW0;
  k1 += kPhiloxW1;
  mul_wide(s0, kPhiloxM0, hi0, lo0);
  mul_wide(x2, kPhiloxM1, hi1, lo1);
  uint64_t x0 = hi1 ^ k0, x1 = lo1, x3 = lo0;
  x2 = y3 ^ (hi0 ^ k1);  // the bracket is uniform
#pragma unroll
  for (int round = 2; round < 10; ++round) {
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
    philox_products(x0, x2, hi0, lo0, hi1, lo1);
    x0 = xor3(hi1, x1, k0);
    x1 = lo1;
    x2 = xor3(hi0, x3, k1);
    x3 = lo0;
  }
  out[0] = x0;
  out[1] = x1;
  out[2] = x2;
  out[3] = x3;
}

// Two consecutive 32-bit words p[0], p[1] in one 8-byte load (dword alignment is enough
// for global loads on gfx950), so a guide window or a pair of row entries costs one
// memory request instead of two.
template <typename T>
__device__ __forceinline__ uint2 load_pair(const T* p) {
  static_assert(sizeof(T) == 4, "32-bit words");
  uint2 v;
  __builtin_memcpy(&v, p, sizeof(v));
  return v;
}

// floor(x * n / 2^64): a uniform index in [0, n) from one 64-bit word.
__device__ __forceinline__ uint64_t bounded(uint64_t x, uint64_t n) { return __umul64hi(x, n); }

// The same for n below 2^32.
__device__ __forceinline__ uint32_t bounded32(uint64_t x, uint32_t n) {
  return (uint32_t)(((x >> 32) * n + ((x & 0xFFFFFFFFu) * n >> 32)) >> 32);
}

// Smallest i in [lo, hi] with value(i) > r, given value(hi) > r (inverse CDF over an
// inclusive prefix; Section 4.1.3 "WeightRandomVertex", step 2).
template <typename F>
__device__ __forceinline__ int32_t first_above_by(F value, int32_t lo, int32_t hi, uint64_t r) {
  int32_t n = hi - lo;
  while (n > 0) {
    const int32_t half = n >> 1;
    if (value(lo + half) <= r) {
      lo += half + 1;
      n -= half + 1;
    } else {
      n = half;
    }
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ int32_t first_above(const T* __restrict__ acc, int32_t lo, int32_t hi, uint64_t r) {
  return first_above_by([acc](int32_t i) { return static_cast<uint64_t>(acc[i]); }, lo, hi, r);
}

// First entry above r of a row's (or an array's) prefix acc[0, len), known to lie in
// [lo, hi]: binary steps down to a window of 4 (32-bit prefixes) or 2 (64-bit) entries,
// which one 16-byte load settles.  Every step is a round trip that the whole wave waits
// for, its widest window setting the number.  The load may start before lo (so as to
// stay inside the row) and run past hi: the entries before lo are at most r, those from
// hi on above it, so counting the entries at most r gives the place either way.  Against
// binary steps to the end (and 64-bit products for the 32-bit draws): n = 1e5, m = 1e6,
// MOSS-4 for 1e7 samples, 460 -> 446 us an estimate; a 256-request batch 21.8 -> 21.1 ms.
__device__ __forceinline__ int32_t first_above_wide(const uint32_t* __restrict__ acc, int32_t len, int32_t lo,
                                                    int32_t hi, uint32_t r) {
  int32_t n = hi - lo;
  const int32_t wide = len >= 4 ? 4 : 0;
  while (n > wide) {
    const int32_t half = n >> 1;
    if (acc[lo + half] <= r) {
      lo += half + 1;
      n -= half + 1;
    } else {
      n = half;
    }
  }
  if (n > 0) {
    lo = min(lo, len - 4);
    uint4 q;
    __builtin_memcpy(&q, acc + lo, sizeof(q));
    lo += (q.x <= r) + (q.y <= r) + (q.z <= r) + (q.w <= r);
  }
  return lo;
}

__device__ __forceinline__ int32_t first_above_wide(const uint64_t* __restrict__ acc, int32_t len, int32_t lo,
                                                    int32_t hi, uint64_t r) {
  int32_t n = hi - lo;
  const int32_t wide = len >= 2 ? 2 : 0;
  while (n > wide) {
    const int32_t half = n >> 1;
    if (acc[lo + half] <= r) {
      lo += half + 1;
      n -= half + 1;
    } else {
      n = half;
    }
  }
  if (n > 0) {
    lo = min(lo, len - 2);
    ulonglong2 q;
    __builtin_memcpy(&q, acc + lo, sizeof(q));
    lo += (q.x <= r) + (q.y <= r);
  }
  return lo;
}

// Is key in the sorted row col[base .. base+len)?
__device__ __forceinline__ bool row_has(const int32_t* __restrict__ col, int32_t base, int32_t len, int32_t key) {
  int32_t lo = base, n = len;
  while (n > 1) {
    const int32_t half = n >> 1;
    if (col[lo + half] <= key) lo += half;
    n -= half;
  }
  return n == 1 && col[lo] == key;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// ---- edge hash set: open addressing with linear probing over 2^bits u64 slots ----
constexpr uint64_t kEmptySlot = ~0ull;
constexpr uint64_t kNoSlot = ~0ull - 1;  // no key and not empty: node ids stay below 2^31

__device__ __forceinline__ uint64_t edge_key(int32_t a, int32_t b) {
  const uint32_t lo = (uint32_t)min(a, b), hi = (uint32_t)max(a, b);
  return (uint64_t)lo << 32 | hi;
}

// Fibonacci hashing of a key: the two halves of key * 2^64 / phi (mod 2^64), in one
// multiply-add, two 32-bit multiplies and an add.  The slot of a key is the top bits of
// the upper half (at most 32 of them: a graph has fewer than 2^30 edges).
struct EdgeHash {
  uint32_t top, low;
};

__device__ __forceinline__ EdgeHash edge_hash(uint64_t key) {
  constexpr uint32_t c0 = 0x7F4A7C15u, c1 = 0x9E3779B9u;
  const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
  const uint64_t p = (uint64_t)lo * c0;
  return {(uint32_t)(p >> 32) + lo * c1 + hi * c0, (uint32_t)p};
}

__device__ __forceinline__ uint32_t edge_slot(EdgeHash h, int bits) { return h.top >> (32 - bits); }

__device__ __forceinline__ uint64_t edge_slot(uint64_t key, int bits) { return edge_slot(edge_hash(key), bits); }

// Settles a lookup of `key` whose home slot h held `first`: found, absent (an empty
// slot ends the probe sequence) or, rarely, more slots to walk.
__device__ __forceinline__ bool edge_hash_rest(const uint64_t* __restrict__ slots, int bits, uint64_t key, uint64_t h,
                                               uint64_t first) {
  if (first == key) return true;
  if (first == kEmptySlot) return false;
  const uint64_t mask = (1ull << bits) - 1;
  for (uint64_t i = 1; i <= mask; ++i) {
    h = (h + 1) & mask;
    const uint64_t x = slots[h];
    if (x == key) return true;
    if (x == kEmptySlot) return false;
  }
  return false;
}

// ---- edge filter: a blocked Bloom filter in front of the hash set ----
// Every edge sets 4 bits of one 64-bit word, two in each half.  A pair whose 4 bits are
// not all set is certainly not an edge, so most non-edges are settled by one read of a
// table small enough to stay cached; the others and every edge go on to the hash set.
// The word of a key is the top filter_bits bits of its hash (the high part of its home
// slot in the hash set, so the filter can be built from the set slot range by slot
// range); the 4 bit positions are the top four 5-bit fields of one more 32-bit product of
// both halves of the hash (its multiplier is the first of a 32-bit mixing function found by
// Chris Wellons' hash-prospector search, public domain).  Against the splitmix64 finaliser of the key and four 6-bit
// positions in the whole word a probe takes about 25 vector instructions instead of 70 and
// lets as many non-edges through (3.0% at 8.4 bits an edge, 5.4% at 6.7): a 256-request
// batch 22.2 -> 21.8 ms.
__device__ __forceinline__ uint2 filter_mask(EdgeHash h) {
  const uint32_t q = (h.top ^ (h.low >> 7)) * 0x2C1B3C6Du;
  return make_uint2(1u << (q >> 27) | 1u << ((q >> 22) & 31), 1u << ((q >> 17) & 31) | 1u << ((q >> 12) & 31));
}

__device__ __forceinline__ bool filter_has(uint2 word, uint2 mask) {
  return ((~word.x & mask.x) | (~word.y & mask.y)) == 0;
}

// Where a row's hub filter lies (in 8-byte words), and the word of a key in it.
__device__ __forceinline__ uint32_t hub_first(uint32_t start) { return (start + 63) / 64 * 8; }
__device__ __forceinline__ uint32_t hub_words(uint32_t start, uint32_t d) {
  return (start + d) / 64 * 8 - hub_first(start);
}
__device__ __forceinline__ uint32_t hub_word(uint32_t start, uint32_t d, EdgeHash h) {
  return hub_first(start) + __umulhi(h.top, hub_words(start, d));
}

// The steps of an inclusive scan over a wave's lanes, by moves between registers (1, 2, 4
// and 8 lanes on within the rows of 16, then lane 15 of rows 0 and 2 to the rows after
// them, then lane 31 to rows 2 and 3): step(from), where from(x) is another lane's x, or 0.
// All lanes active.  (Against shuffles through LDS, k_span_prefix over ACC_tau at m = 1e7:
// 96 -> 78 us.)
template <class Step>
__device__ __forceinline__ void wave_scan_steps(Step step) {
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false); });
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false); });
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false); });
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false); });
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false); });
  step([](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false); });
}

__device__ __forceinline__ uint32_t wave_scan32(uint32_t x) {  // inclusive sum over the lanes
  wave_scan_steps([&](auto from) { x += from(x); });
  return x;
}

// Inclusive scan over the 64 lanes of a wave; `wrapped` is set on any 64-bit wrap.
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t x, bool& wrapped) {
  wave_scan_steps([&](auto from) {
    const uint64_t z = x + ((uint64_t)from((uint32_t)(x >> 32)) << 32 | from((uint32_t)x));
    wrapped |= z < x;
    x = z;
  });
  return x;
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

__device__ __forceinline__ uint64_t wave_sum_wrap(uint64_t x, bool& wrapped) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t z = x + __shfl_xor(x, off, 64);
    wrapped |= z < x;
    x = z;
  }
  return x;
}

__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x |= __shfl_xor(x, off, 64);
  return x;
}

// C(d, 3) and C(d, 4) for d < 2^31, exactly: the factorial denominators are
// divided out of the consecutive factors before multiplying, so only the final
// product can exceed 64 bits, which sets `over`.
__device__ __forceinline__ uint64_t choose3(uint64_t d, bool& over) {
  if (d < 3) return 0;
  uint64_t f0 = d, f1 = d - 1, f2 = d - 2;
  if ((f0 & 1) == 0) f0 >>= 1; else f1 >>= 1;
  if (f0 % 3 == 0) f0 /= 3; else if (f1 % 3 == 0) f1 /= 3; else f2 /= 3;
  const uint64_t p = f0 * f1;
  over |= __umul64hi(p, f2) != 0;
  return p * f2;
}

__device__ __forceinline__ uint64_t choose4(uint64_t d, bool& over) {
  if (d < 4) return 0;
  uint64_t f[4] = {d, d - 1, d - 2, d - 3};
  // one of four consecutive numbers is a multiple of 4, the one two away is even
  int i4 = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (f[i] % 4 == 0) i4 = i;
  f[i4] /= 4;
  f[i4 < 2 ? i4 + 2 : i4 - 2] /= 2;
  bool done = false;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (!done && f[i] % 3 == 0) {
      f[i] /= 3;
      done = true;
    }
  const uint64_t p = f[0] * f[1], q = f[2] * f[3];
  over |= __umul64hi(p, q) != 0;
  return p * q;
}

}  // namespace moss
