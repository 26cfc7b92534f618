// Device kernels of the canonical k-mer counting path for gfx950 (CDNA4).
//
// Path (one call):
//   front          ASCII -> 2-bit bases (32 per uint64, base i at bits 2i) and one
//                  bit per byte: whether the window that starts there is valid (k
//                  bases of one read). A batch, packed once for several k, does so
//                  in steps: pack and read_ends (masks of invalid bytes and of
//                  reads' last bytes), valid_mask for each k.
//   window_hist    every valid window -> its shard's count: the first-level
//                  key-range shards are the top bits of the canonical key.
//   plan_shards    where each shard's slice lies and how it is split.
//   window_scatter every valid window -> its canonical key in its shard's slice of
//                  the owner-major record buffer (each owner's shards are
//                  contiguous: the owner's receive buffer), staged in LDS so that
//                  each shard gets one coalesced run per tile.
//   split_hist /   shards too large for one LDS table are split by the next key
//   plan_leaves /  bits (MSD radix step) into leaves. Small inputs are not: every
//   split_scatter  shard is a leaf.
//   leaf_count     a leaf at a time: open-addressing hash table in LDS (linear
//                  probing, CAS claim of an EMPTY slot, atomic add of the count),
//                  overflow detection, compaction, then a counting sort of the
//                  distinct keys and a rank within each of its groups (a bitonic
//                  sort where a group is large) -> sorted (key, count) pairs.
//                  Leaves that overflow get a second count with a table twice as
//                  large; what overflows that is refined under host control.
//   concat         leaves are disjoint key ranges, so concatenating their
//                  sorted pairs in key-range order gives the sorted output.
//   check          device self-check of the output.
//
// Nothing here is a dense contraction: the path is bound by HBM traffic and
// LDS atomics, not by MFMA.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kc_internal.h"

namespace kc {
namespace {

typedef unsigned __int128 u128;

// ---------------------------------------------------------------- key helpers

__device__ __forceinline__ uint64_t mask64(int k) { return k >= 32 ? ~0ull : ((1ull << (2 * k)) - 1); }
__device__ __forceinline__ u128 mask128(int k) {
  return k >= 64 ? ~(u128)0 : (((u128)1 << (2 * k)) - 1);
}

// Reverse the order of the 32 two-bit groups of a word.
__device__ __forceinline__ uint64_t rev2(uint64_t x) {
  x = __builtin_bitreverse64(x);
  return ((x >> 1) & 0x5555555555555555ull) | ((x & 0x5555555555555555ull) << 1);
}

template <typename K> struct Key;

template <> struct Key<uint64_t> {
  static constexpr bool kWide = false;
  static constexpr int kWords = 1;
  __device__ static uint32_t bits(uint64_t x, int shift, int nbits) {
    return (uint32_t)(x >> shift) & ((1u << nbits) - 1u);
  }
  // Canonical key of the window starting at bit offset s (0..62, even) of the
  // little-endian base stream held in words p0, p1 (p2 unused).
  __device__ static uint64_t canon(uint64_t p0, uint64_t p1, uint64_t, int s, int k) {
    uint64_t v = s ? (p0 >> s) | (p1 << (64 - s)) : p0;  // base j of the window at bits 2j
    v &= mask64(k);
    uint64_t rc = ~v & mask64(k);          // complement, base j at 4^j: reverse complement
    uint64_t fwd = rev2(v) >> (64 - 2 * k);  // first base most significant
    return fwd < rc ? fwd : rc;
  }
  __device__ static uint64_t mask(int k) { return mask64(k); }
  __device__ static uint64_t window(uint64_t p0, uint64_t p1, int s, int k) {
    return (s ? (p0 >> s) | (p1 << (64 - s)) : p0) & mask64(k);
  }
  __device__ static uint64_t fwd_of(uint64_t p0, uint64_t p1, uint64_t, int s, int k) {
    return rev2(window(p0, p1, s, k)) >> (64 - 2 * k);
  }
  __device__ static uint64_t rc_of(uint64_t p0, uint64_t p1, uint64_t, int s, int k) {
    return ~window(p0, p1, s, k) & mask64(k);
  }
  __device__ static uint64_t revcomp(uint64_t x, int k) { return rev2(~x & mask64(k)) >> (64 - 2 * k); }
  __device__ static bool in_range(uint64_t x, int k) { return (x & ~mask64(k)) == 0; }
};

// LDS atomics take unsigned long long; same key semantics as uint64_t.
template <> struct Key<unsigned long long> : Key<uint64_t> {};

template <> struct Key<u128> {
  static constexpr bool kWide = true;
  static constexpr int kWords = 2;
  __device__ static uint32_t bits(u128 x, int shift, int nbits) {
    return (uint32_t)(x >> shift) & ((1u << nbits) - 1u);
  }
  __device__ static u128 canon(uint64_t p0, uint64_t p1, uint64_t p2, int s, int k) {
    uint64_t lo = s ? (p0 >> s) | (p1 << (64 - s)) : p0;
    uint64_t hi = s ? (p1 >> s) | (p2 << (64 - s)) : p1;
    u128 v = (((u128)hi << 64) | lo) & mask128(k);
    u128 rc = ~v & mask128(k);
    u128 r = ((u128)rev2((uint64_t)v) << 64) | rev2((uint64_t)(v >> 64));
    u128 fwd = r >> (128 - 2 * k);
    return fwd < rc ? fwd : rc;
  }
  __device__ static u128 mask(int k) { return mask128(k); }
  __device__ static u128 window(uint64_t p0, uint64_t p1, uint64_t p2, int s, int k) {
    const uint64_t lo = s ? (p0 >> s) | (p1 << (64 - s)) : p0;
    const uint64_t hi = s ? (p1 >> s) | (p2 << (64 - s)) : p1;
    return (((u128)hi << 64) | lo) & mask128(k);
  }
  __device__ static u128 fwd_of(uint64_t p0, uint64_t p1, uint64_t p2, int s, int k) {
    const u128 v = window(p0, p1, p2, s, k);
    return (((u128)rev2((uint64_t)v) << 64) | rev2((uint64_t)(v >> 64))) >> (128 - 2 * k);
  }
  __device__ static u128 rc_of(uint64_t p0, uint64_t p1, uint64_t p2, int s, int k) {
    return ~window(p0, p1, p2, s, k) & mask128(k);
  }
  __device__ static u128 revcomp(u128 x, int k) {
    u128 c = ~x & mask128(k);
    u128 r = ((u128)rev2((uint64_t)c) << 64) | rev2((uint64_t)(c >> 64));
    return r >> (128 - 2 * k);
  }
  __device__ static bool in_range(u128 x, int k) { return (x & ~mask128(k)) == 0; }
};

// 256-bit keys (k in [65, 128]): two 128-bit halves with the operations the
// key-generic kernels apply to keys (shifts by 0..255, bitwise logic, order).
struct u256 {
  u128 lo, hi;
  u256() = default;
  __device__ constexpr u256(u128 l, u128 h) : lo(l), hi(h) {}
  __device__ constexpr u256(u128 x) : lo(x), hi(0) {}
  __device__ constexpr u256(uint64_t x) : lo(x), hi(0) {}
  __device__ constexpr u256(unsigned long long x) : lo(x), hi(0) {}
  __device__ constexpr u256(uint32_t x) : lo(x), hi(0) {}
  __device__ constexpr u256(int x) : lo((u128)(uint32_t)x), hi(0) {}
  __device__ explicit operator uint32_t() const { return (uint32_t)lo; }
  __device__ explicit operator uint64_t() const { return (uint64_t)lo; }
  __device__ explicit operator unsigned long long() const { return (unsigned long long)lo; }
};
__device__ __forceinline__ u256 operator<<(const u256& a, int s) {
  if (s == 0) return a;
  if (s >= 128) return u256((u128)0, a.lo << (s - 128));
  return u256(a.lo << s, (a.hi << s) | (a.lo >> (128 - s)));
}
__device__ __forceinline__ u256 operator>>(const u256& a, int s) {
  if (s == 0) return a;
  if (s >= 128) return u256(a.hi >> (s - 128), (u128)0);
  return u256((a.lo >> s) | (a.hi << (128 - s)), a.hi >> s);
}
__device__ __forceinline__ u256 operator|(const u256& a, const u256& b) {
  return u256(a.lo | b.lo, a.hi | b.hi);
}
__device__ __forceinline__ u256 operator&(const u256& a, const u256& b) {
  return u256(a.lo & b.lo, a.hi & b.hi);
}
__device__ __forceinline__ u256 operator~(const u256& a) { return u256(~a.lo, ~a.hi); }
__device__ __forceinline__ u256& operator|=(u256& a, const u256& b) { return a = a | b; }
__device__ __forceinline__ bool operator==(const u256& a, const u256& b) {
  return a.lo == b.lo && a.hi == b.hi;
}
__device__ __forceinline__ bool operator!=(const u256& a, const u256& b) { return !(a == b); }
__device__ __forceinline__ bool operator<(const u256& a, const u256& b) {
  return a.hi != b.hi ? a.hi < b.hi : a.lo < b.lo;
}
__device__ __forceinline__ bool operator>(const u256& a, const u256& b) { return b < a; }

// Reverse the order of the 128 two-bit groups.
__device__ __forceinline__ u256 rev2_256(const u256& v) {
  const u128 lo = ((u128)rev2((uint64_t)(v.hi >> 64)) << 0) | ((u128)rev2((uint64_t)v.hi) << 64);
  const u128 hi = ((u128)rev2((uint64_t)(v.lo >> 64)) << 0) | ((u128)rev2((uint64_t)v.lo) << 64);
  return u256(lo, hi);
}

__device__ __forceinline__ u128 low_bits128(int bits) {
  return bits >= 128 ? ~(u128)0 : (((u128)1 << bits) - 1);
}

// Keys of more than 64 bases: built from five packed words (up to 128 bases
// starting anywhere in the first word).
template <> struct Key<u256> {
  static constexpr int kWords = 4;
  __device__ static u256 mask(int k) {
    const int b = 2 * k;
    return b <= 128 ? u256(low_bits128(b), (u128)0) : u256(~(u128)0, low_bits128(b - 128));
  }
  __device__ static uint32_t bits(const u256& x, int shift, int nbits) {
    return (uint32_t)(x >> shift) & ((1u << nbits) - 1u);
  }
  // Bases [s/2, s/2 + k) of the little-endian base stream in p[0..4] (base j
  // of the window at bits 2j), s even, 0 <= s <= 62.
  __device__ static u256 window(const uint64_t (&p)[5], int s, int k) {
    uint64_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = s ? (p[i] >> s) | (p[i + 1] << (64 - s)) : p[i];
    return u256(((u128)w[1] << 64) | w[0], ((u128)w[3] << 64) | w[2]) & mask(k);
  }
  __device__ static u256 fwd_of_window(const u256& v, int k) { return rev2_256(v) >> (256 - 2 * k); }
  __device__ static u256 rc_of_window(const u256& v, int k) { return ~v & mask(k); }
  __device__ static u256 revcomp(const u256& x, int k) {
    return rev2_256(~x & mask(k)) >> (256 - 2 * k);
  }
  __device__ static bool in_range(const u256& x, int k) { return (x & ~mask(k)) == u256(0); }
};

// ---------------------------------------------------------------- block scans

// Exclusive scan of one value per thread (wave shuffles, then one wave over
// the wave totals); returns the prefix and sets *total. wsum holds TB/64 values.
template <int TB, typename T>
__device__ __forceinline__ T block_exscan(T v, T* wsum, T* total) {
  constexpr int NW = TB / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const T y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  if (wid == 0) {
    T w = lane < NW ? wsum[lane] : (T)0;
#pragma unroll
    for (int off = 1; off < NW; off <<= 1) {
      const T y = __shfl_up(w, off);
      if (lane >= off) w += y;
    }
    if (lane < NW) wsum[lane] = w;  // inclusive prefix of the wave totals
  }
  __syncthreads();
  const T before = wid ? wsum[wid - 1] : (T)0;
  *total = wsum[NW - 1];
  __syncthreads();
  return before + x - v;
}

// Exclusive scan of an LDS array a[0..n) into out[0..n); returns the total.
// If maxv is not null it receives the largest a[i].
template <int TB>
__device__ __forceinline__ uint32_t block_exscan_array(const uint32_t* a, uint32_t* out, int n,
                                                       uint32_t* wsum, uint32_t* maxv = nullptr) {
  const int per = (n + TB - 1) / TB;
  const int b = threadIdx.x * per;
  const int e = min(n, b + per);
  uint32_t s = 0, m = 0;
  for (int i = b; i < e; ++i) {
    s += a[i];
    m = max(m, a[i]);
  }
  if (maxv) {
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) atomicMax(maxv, m);
  }
  uint32_t total;
  uint32_t run = block_exscan<TB, uint32_t>(s, wsum, &total);
  for (int i = b; i < e; ++i) {
    out[i] = run;
    run += a[i];
  }
  __syncthreads();
  return total;
}

// In-place exclusive scan of a[0..n) (counts become offsets); returns the total.
template <int TB>
__device__ __forceinline__ uint32_t block_exscan_inplace(uint32_t* a, int n, uint32_t* wsum) {
  const int per = (n + TB - 1) / TB;
  const int b = threadIdx.x * per;
  const int e = min(n, b + per);
  uint32_t s = 0;
  for (int i = b; i < e; ++i) s += a[i];
  uint32_t total;
  uint32_t run = block_exscan<TB, uint32_t>(s, wsum, &total);
  for (int i = b; i < e; ++i) {
    const uint32_t x = a[i];
    a[i] = run;
    run += x;
  }
  __syncthreads();
  return total;
}

__global__ void k_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---------------------------------------------------------------- pack

// Top bit of each byte of v set iff that byte is not zero (no carry between bytes).
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) {
  return (((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) & 0x80808080u;
}
// Four bytes w at once (SWAR), bases j .. j+3 of a chunk: the 2-bit code of each
// byte from its bits 1 and 2, then the four 2-bit codes gathered into 8 bits of p; a byte is invalid iff its
// lowercase form differs from each of a, c, g, t (nonzero_bytes sets a byte's top
// bit iff the byte is not 0), the four top bits gathered into 4 bits of iv by one
// multiply.
__device__ __forceinline__ void pack4(uint32_t w, int j, uint64_t (&p)[2], uint64_t& iv) {
  const uint32_t c = ((w >> 1) ^ (w >> 2)) & 0x03030303u;
  const uint32_t t = c | (c >> 6);
  p[j >> 5] |= (uint64_t)((t & 0xFu) | ((t >> 12) & 0xF0u)) << (2 * (j & 31));
  const uint32_t l = w | 0x20202020u;
  const uint32_t bad = nonzero_bytes(l ^ 0x61616161u) & nonzero_bytes(l ^ 0x63636363u) &
                       nonzero_bytes(l ^ 0x67676767u) & nonzero_bytes(l ^ 0x74747474u);
  iv |= (uint64_t)(((bad & 0x80808080u) * 0x00204081u) >> 28) << j;
}

// Bases [64c, 64c + 64) of the n bytes at src, at any alignment: two packed
// words and the invalid mask. Bytes from n on are invalid, their codes 0. Off a
// 16-byte boundary the aligned words that hold a byte of src are loaded, all
// before any is used (byte loads, each waited for, took 7.4 us of a small input).
__device__ __forceinline__ void pack_chunk(const uint8_t* __restrict__ src, uint64_t n, uint64_t c,
                                           uint64_t (&p)[2], uint64_t& iv) {
  const uint64_t g0 = c * 64;
  p[0] = p[1] = 0;
  iv = 0;
  if (g0 >= n) {
    iv = ~0ull;
    return;
  }
  const uint8_t* const q = src + g0;
  if (((uintptr_t)q & 15) == 0 && g0 + 64 <= n) {
    const uint4* const v = (const uint4*)q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint4 x = v[i];
      pack4(x.x, i * 16, p, iv);
      pack4(x.y, i * 16 + 4, p, iv);
      pack4(x.z, i * 16 + 8, p, iv);
      pack4(x.w, i * 16 + 12, p, iv);
    }
    return;
  }
  const uint32_t sh = (uint32_t)((uintptr_t)q & 3);
  const uint32_t* const a = (const uint32_t*)(q - sh);
  const uint32_t left = (uint32_t)min((uint64_t)64, n - g0), end = left + sh;  // bytes from a
  uint32_t w[17];
#pragma unroll
  for (int i = 0; i < 17; ++i) w[i] = 4u * i < end ? a[i] : 0u;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    pack4((uint32_t)((((uint64_t)w[i + 1] << 32) | w[i]) >> (8 * sh)), 4 * i, p, iv);
  if (left < 64) {
    iv |= ~0ull << left;
    p[1] &= left > 32 ? (1ull << (2 * (left - 32))) - 1 : 0ull;
    p[0] &= left >= 32 ? ~0ull : (1ull << (2 * left)) - 1;
  }
}

// Thread c packs bytes [64c, 64c+64): two packed words, one invalid-mask word
// and one end-mask word (bit j set iff byte 64c+j is the last byte of a read).
__global__ void __launch_bounds__(256) k_pack(const uint8_t* __restrict__ src, uint64_t n_bytes,
                                              uint64_t* __restrict__ packed,
                                              uint64_t* __restrict__ inv,
                                              uint64_t* __restrict__ endm, uint64_t nchunks) {
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nchunks) return;
  uint64_t p[2], iv;
  pack_chunk(src, n_bytes, c, p, iv);
  packed[2 * c] = p[0];
  packed[2 * c + 1] = p[1];
  inv[c] = iv;
  endm[c] = 0;  // read ends are set by k_read_ends, launched after this kernel
}

// Read-end mask: bit of the last byte of every non-empty read (thread per read).
__global__ void __launch_bounds__(256) k_read_ends(const uint64_t* __restrict__ offsets,
                                                   uint64_t n_reads, uint64_t off0,
                                                   unsigned long long* __restrict__ endm) {
  const uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_reads) return;
  const uint64_t b = offsets[r], e = offsets[r + 1];
  if (e > b) {
    const uint64_t pos = e - 1 - off0;
    atomicOr(&endm[pos >> 6], 1ull << (pos & 63));
  }
}

// ---------------------------------------------------------------- windows

// Window validity. Bit j of valid[w] is set iff the window of k bytes
// starting at byte 64w + j is valid: no invalid byte in it and no read end
// before its last byte. The mask is built once per k by k_valid_mask, so that
// the window kernels test a start with one shift.

// Bits [64w, 64w + 128) of a bit array (the arrays are padded by two words).
__device__ __forceinline__ u128 load_bits(const uint64_t* __restrict__ m, uint64_t w) {
  return ((u128)m[w + 1] << 64) | m[w];
}

// r[i] = OR of x[i .. i+len) (len >= 1).
__device__ __forceinline__ u128 smear(u128 x, int len) {
  int l = 1;
  while (2 * l <= len) {
    x |= x >> l;
    l <<= 1;
  }
  if (l < len) x |= x >> (len - l);
  return x;
}

// The same over 256 bits, for keys of more than 64 bases (64 + k - 1 may pass
// 128 bits; the arrays are padded by five words).
__device__ __forceinline__ u256 load_bits256(const uint64_t* __restrict__ m, uint64_t w) {
  return u256(((u128)m[w + 1] << 64) | m[w], ((u128)m[w + 3] << 64) | m[w + 2]);
}

__device__ __forceinline__ u256 smear256(u256 x, int len) {
  int l = 1;
  while (2 * l <= len) {
    x |= x >> l;
    l <<= 1;
  }
  if (l < len) x |= x >> (len - l);
  return x;
}

// One thread per mask word w in [w_begin, w_end). Also clears the counters of
// the pipeline that starts with this kernel (z): a launch of its own for each
// array costs 4 to 5 us whatever its size, a third of a small count's time.
template <bool WIDE>
__global__ void __launch_bounds__(256) k_valid_mask(const uint64_t* __restrict__ inv,
                                                    const uint64_t* __restrict__ endm,
                                                    uint64_t w_begin, uint64_t w_end, int k,
                                                    uint64_t* __restrict__ valid, ZeroRanges z) {
#pragma unroll
  for (int r = 0; r < ZeroRanges::kN; ++r)
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < z.n[r];
         i += (uint64_t)gridDim.x * 256)
      z.p[r][i] = 0;
  const uint64_t w = w_begin + (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (w >= w_end) return;
  uint64_t bad;
  if constexpr (WIDE) {
    u256 b = smear256(load_bits256(inv, w), k);
    if (k > 1) b |= smear256(load_bits256(endm, w), k - 1);
    bad = (uint64_t)b;
  } else {
    u128 b = smear(load_bits(inv, w), k);
    if (k > 1) b |= smear(load_bits(endm, w), k - 1);
    bad = (uint64_t)b;
  }
  valid[w] = ~bad;
}

// Chunks after a window's first that it may reach into: it starts at bit 63 at
// the latest and is up to 128 (WIDE) or 64 bases long.
template <bool WIDE> constexpr int kFrontHalo = WIDE ? 2 : 1;

// First r in [lo, hi) with off[r + 1] > x, or hi; by a whole wave, 64 places a
// step. guess: about where it lies.
__device__ __forceinline__ uint64_t wave_first_end(const uint64_t* __restrict__ off, uint64_t lo,
                                                   uint64_t hi, uint64_t x, uint64_t guess) {
  const uint64_t lane = threadIdx.x & 63;
  if (hi - lo > 64) {  // 64 places about the guess: reads of like lengths are found between two
    uint64_t i = guess + 64 * lane;
    i = i < lo + 2048 ? lo : i - 2048;
    i = min(i, hi - 1);
    const int below = __popcll(__ballot(off[i + 1] <= x));
    const uint64_t last = __shfl(i, below ? below - 1 : 0), first = __shfl(i, below & 63);
    if (below) lo = last + 1;
    if (below < 64) hi = first;
  }
  while (lo < hi) {
    const uint64_t step = (hi - lo + 63) / 64;
    const uint64_t i = lo + lane * step;
    const uint64_t below = (uint64_t)__popcll(__ballot(i < hi && off[i + 1] <= x));
    hi = min(hi, lo + below * step);
    if (below) lo += (below - 1) * step + 1;
  }
  return lo;
}

// Input of a plain call in one pass: packed bases and the valid-start mask for
// k, and the counters of the pipeline cleared. A workgroup takes 256 chunks of
// 64 bytes, a thread each, and keeps the invalid and read-end masks in LDS; the
// last HALO chunks (those a window of k reaches into) are the next workgroup's
// first. The read ends among its bytes are a range of the offsets, found by
// one wave and set by all threads. Bound by reading the input (large) and by
// the number of launches (small): apart, the three kernels wrote and read the
// two masks (3/8 of a byte a base) and set the ends by an atomic each in
// memory: 20,000,000 reads 1.33 -> 0.85 ms (3.5 TB/s of bases), 1,000,000 reads
// 83 -> 60 us, 667 reads 11.8 -> 6.3 us and two launches less (whole call 101 ->
// 94 us).
template <bool WIDE>
__global__ void __launch_bounds__(256) k_front(const uint8_t* __restrict__ src, uint64_t n_bytes,
                                               const uint64_t* __restrict__ offsets,
                                               uint64_t n_reads, uint64_t off0, int k,
                                               uint64_t* __restrict__ packed,
                                               uint64_t* __restrict__ valid, uint64_t nchunks,
                                               ZeroRanges z) {
  constexpr int HALO = kFrontHalo<WIDE>;
  __shared__ uint64_t s_inv[256];
  __shared__ __align__(8) uint32_t s_end[512];  // two words a chunk
  __shared__ uint64_t s_r;
  const int t = threadIdx.x;
#pragma unroll
  for (int r = 0; r < ZeroRanges::kN; ++r)
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + t; i < z.n[r]; i += (uint64_t)gridDim.x * 256)
      z.p[r][i] = 0;
  const uint64_t c0 = (uint64_t)blockIdx.x * (256 - HALO), c = c0 + t;
  if (c0 >= nchunks) return;  // a workgroup that only clears
  s_end[t] = s_end[t + 256] = 0;
  uint64_t p[2], iv;
  pack_chunk(src, n_bytes, c, p, iv);
  s_inv[t] = iv;
  // ends e with x0 < e <= x1 are those of bases of these chunks
  const uint64_t x0 = off0 + min(n_bytes, c0 * 64), x1 = off0 + min(n_bytes, (c0 + 256) * 64);
  auto first_end = [&](uint64_t lo, uint64_t x) {
    if (t < 64) {
      const uint64_t r = wave_first_end(
          offsets, lo, n_reads, x, (uint64_t)((double)(x - off0) / (double)n_bytes * (double)n_reads));
      if (t == 0) s_r = r;
    }
    __syncthreads();
    return s_r;
  };
  constexpr int U = 4;
  for (uint64_t r = first_end(0, x0); r < n_reads;) {
    uint64_t e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t i = r + u * 256 + t;
      e[u] = i < n_reads ? offsets[i + 1] : ~0ull;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e[u] <= x1) {  // (an empty read's end is that of an earlier one too, or <= x0)
        const uint32_t b = (uint32_t)(e[u] - 1 - off0 - c0 * 64);
        atomicOr(&s_end[b >> 5], 1u << (b & 31));
      }
    // done if the last one looked at is past these chunks; many empty reads
    // with one end are passed over
    const uint64_t last = r + U * 256;
    if (last > n_reads) break;
    const uint64_t el = offsets[last];
    if (el > x1) break;
    const bool same = offsets[r + 1] == el;
    r = last;
    if (same) {
      __syncthreads();  // s_r was read by all
      r = first_end(r, el);
    }
  }
  __syncthreads();
  if (t >= 256 - HALO || c >= nchunks) return;
  *(ulonglong2*)(packed + 2 * c) = ulonglong2{p[0], p[1]};
  const uint64_t* const s_e = (const uint64_t*)s_end;
  uint64_t bad;
  if constexpr (WIDE) {
    u256 b = smear256(u256(((u128)s_inv[t + 1] << 64) | s_inv[t], (u128)s_inv[t + 2]), k);
    if (k > 1) b |= smear256(u256(((u128)s_e[t + 1] << 64) | s_e[t], (u128)s_e[t + 2]), k - 1);
    bad = (uint64_t)b;
  } else {
    u128 b = smear(((u128)s_inv[t + 1] << 64) | s_inv[t], k);
    if (k > 1) b |= smear(((u128)s_e[t + 1] << 64) | s_e[t], k - 1);
    bad = (uint64_t)b;
  }
  valid[c] = ~bad;
}

// Valid starts among the S window starts g .. g+S-1 (g a multiple of S, S
// dividing 64): bit i for start g+i.
template <int S>
__device__ __forceinline__ uint32_t valid_starts(const uint64_t* __restrict__ valid, uint64_t g) {
  return (uint32_t)(valid[g >> 6] >> (g & 63)) & (S >= 32 ? 0xFFFFFFFFu : ((1u << S) - 1u));
}

template <typename K, int S>
__device__ __forceinline__ void load_window_words(const uint64_t* __restrict__ packed, uint64_t g,
                                                  uint64_t& p0, uint64_t& p1, uint64_t& p2) {
  const uint64_t w = g >> 5;
  p0 = packed[w];
  p1 = packed[w + 1];
  p2 = Key<K>::kWide ? packed[w + 2] : 0;
}

// Canonical keys of the S windows starting at bytes g .. g+S-1 (g a multiple
// of S, S dividing 32). The first is built directly from the packed words,
// the others by rolling one base in: fwd = ((fwd << 2) | x) & mask and
// rc = (rc >> 2) | ((3 - x) << 2(k-1)), x being the base at g+i+k-1.
// Keys of invalid starts are computed too (the caller masks them).
template <typename K, int S>
__device__ __forceinline__ void canon_run(uint64_t p0, uint64_t p1, uint64_t p2, uint64_t g, int k,
                                          K (&out)[S]) {
  const int s0 = (int)(g & 31);
  out[0] = Key<K>::canon(p0, p1, p2, 2 * s0, k);
  K fwd = Key<K>::fwd_of(p0, p1, p2, 2 * s0, k);
  K rc = Key<K>::rc_of(p0, p1, p2, 2 * s0, k);
  const K mask = Key<K>::mask(k);
  const int top = 2 * (k - 1);
#pragma unroll
  for (int i = 1; i < S; ++i) {
    const int p = s0 + i + k - 1;  // position of the incoming base within words p0..p2
    const uint64_t w = p < 32 ? p0 : (p < 64 ? p1 : p2);
    const uint32_t x = (uint32_t)(w >> (2 * (p & 31))) & 3u;
    fwd = ((fwd << 2) | (K)x) & mask;
    rc = (rc >> 2) | ((K)(3u - x) << top);
    out[i] = fwd < rc ? fwd : rc;
  }
}

// canon_run for keys of more than 64 bases, from five packed words (the
// incoming base of window i sits at most 158 bases past the first word).
template <int S>
__device__ __forceinline__ void canon_run256(const uint64_t (&p)[5], uint64_t g, int k,
                                             u256 (&out)[S]) {
  const int s0 = (int)(g & 31);
  const u256 v = Key<u256>::window(p, 2 * s0, k);
  u256 fwd = Key<u256>::fwd_of_window(v, k);
  u256 rc = Key<u256>::rc_of_window(v, k);
  out[0] = fwd < rc ? fwd : rc;
  const u256 mask = Key<u256>::mask(k);
  const int top = 2 * (k - 1);
#pragma unroll
  for (int i = 1; i < S; ++i) {
    const int q = s0 + i + k - 1;  // position of the incoming base within p[0..4]
    const int wi = q >> 5;
    const uint64_t w = wi == 0 ? p[0] : wi == 1 ? p[1] : wi == 2 ? p[2] : wi == 3 ? p[3] : p[4];
    const uint32_t x = (uint32_t)(w >> (2 * (q & 31))) & 3u;
    fwd = ((fwd << 2) | u256(x)) & mask;
    rc = (rc >> 2) | (u256(3u - x) << top);
    out[i] = fwd < rc ? fwd : rc;
  }
}

template <typename K>
__device__ __forceinline__ uint32_t shard_of(const K& key, int keybits, int shard_bits) {
  return (uint32_t)(key >> (keybits - shard_bits));
}

// Sets of a batch that the bytes [g0, g1) lie in: lo to hi; any: one of them is
// in the class being counted. The same for a whole workgroup, so that its
// threads search between lo and hi only (mostly one set), and tiles of other
// classes' sets are passed over.
struct SetRange {
  uint32_t lo, hi;
  bool any;
};
__device__ __forceinline__ SetRange sets_of(const BatchSets& bs, uint64_t g0, uint64_t g1) {
  uint32_t lo = 0, hi = bs.n_sets - 1;  // last set whose first byte is <= g0
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (bs.set_byte_off[mid] <= g0) lo = mid; else hi = mid - 1;
  }
  SetRange r{lo, lo, bs.set_local[lo] != kNoSet};
  while (r.hi + 1 < bs.n_sets && bs.set_byte_off[r.hi + 1] < g1) {
    ++r.hi;
    r.any |= bs.set_local[r.hi] != kNoSet;
  }
  return r;
}

// Set of byte g among those of r.
__device__ __forceinline__ uint32_t set_of(const BatchSets& bs, const SetRange& r, uint64_t g) {
  uint32_t lo = r.lo, hi = r.hi;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (bs.set_byte_off[mid] <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Keys of a thread's S window starts. Plain counting: the canonical k-mer. In
// a batch of read sets, the key of a window is (set id within its k-class <<
// 2k) | canonical k-mer, so that sorting keys sorts by set, then k-mer; windows
// of sets outside the class are dropped from vm. Returns the updated vm.
// Cut keys (CUT, one word, see BatchSets): the key's low 64 bits, and in
// shard[] its top set_bits + kb bits.
template <typename K, typename Kc, int S, bool BATCH, bool CUT>
__device__ __forceinline__ uint32_t window_keys(const uint64_t* __restrict__ packed, uint64_t g,
                                                int k, uint32_t vm, const BatchSets& bs,
                                                const SetRange& range, K (&key)[S], int kb,
                                                uint32_t (&shard)[CUT ? S : 1]) {
  Kc c[S];
  if constexpr (Key<Kc>::kWords == 4) {
    const uint64_t w = g >> 5;
    uint64_t p[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) p[i] = packed[w + i];
    canon_run256<S>(p, g, k, c);
  } else {
    uint64_t p0, p1, p2;
    load_window_words<Kc, S>(packed, g, p0, p1, p2);
    canon_run<Kc, S>(p0, p1, p2, g, k, c);
  }
  if constexpr (!BATCH) {
#pragma unroll
    for (int i = 0; i < S; ++i) key[i] = (K)c[i];
    return vm;
  } else {
  uint32_t set = set_of(bs, range, g);
#pragma unroll
  for (int i = 0; i < S; ++i) {
    if (!(vm & (1u << i))) continue;
    while (set + 1 < bs.n_sets && g + i >= bs.set_byte_off[set + 1]) ++set;
    const uint32_t loc = bs.set_local[set];
    if (loc == kNoSet) vm &= ~(1u << i);
    // (a class of one k = 32 set has no set-id bits: no shift by the key width)
    else key[i] = (2 * k < (int)(8 * sizeof(K)) ? ((K)loc << (2 * k)) : (K)0) | (K)c[i];
    if constexpr (CUT) shard[i] = (loc << kb) | (uint32_t)((c[i] >> 1) >> (2 * k - 1 - kb));
  }
  return vm;
  }
}

// 24 bits of the packed stream (p1:p0) from bit q (q < 128 - 24).
__device__ __forceinline__ uint32_t bits24(uint64_t p0, uint64_t p1, int q) {
  const uint64_t lo = q >= 64 ? p1 >> (q - 64) : (p0 >> q) | (q ? p1 << (64 - q) : 0ull);
  return (uint32_t)lo & 0xFFFFFFu;
}

// Shard histogram over the owner scatter's tiles: tile j holds the window
// starts [w_begin + j*R*TB*S, w_begin + (j+1)*R*TB*S) ∩ [.., w_end), taken S per
// thread in R units of TB*S. The counts of the tiles of class c = j mod kXcds
// go to hist[(1 + c)*nb, ..) (gridDim.x is a multiple of R*kXcds, so all of a
// workgroup's units are of class blockIdx.x / R mod kXcds); k_plan_shards adds
// up the totals, hist[0, nb). In smaller inputs every unit has a workgroup of
// its own and a thread one step, not R dependent ones. The number of valid
// windows is the sum of the totals: counted here, by one atomic per wave on one
// word, it took most of the kernel (8,192 of them at 12 ns each; 1,000,000
// reads: 139 -> 61 us, 3.7 MB: 27.6 -> 7.5 us).
template <typename K, typename Kc, int S, int TB, bool BATCH>
__global__ void __launch_bounds__(TB) k_window_hist(const uint64_t* __restrict__ packed,
                                                    const uint64_t* __restrict__ valid,
                                                    uint64_t w_begin, uint64_t w_end,
                                                    int R, int k, int keybits,
                                                    int shard_bits, BatchSets bs,
                                                    unsigned long long* __restrict__ hist) {
  __shared__ uint32_t sh[1 << kMaxShardBits];
  const int nb = 1 << shard_bits;
  for (int i = threadIdx.x; i < nb; i += TB) sh[i] = 0;
  __syncthreads();
  // Only the shard is needed: set id bits (batch), then kb bits of the canonical
  // k-mer, whose top bits are the smaller of the top bits of fwd and of rc (if
  // those are equal, so are both keys' top bits). The top 10 bits of fwd are
  // its first 5 bases, those of rc the complements of its last 5 bases, last
  // first: whole keys are not built, whatever their width (four words: 0.50 ->
  // 0.08 ms on 1,000,000 reads).
  const int kb = BATCH ? shard_bits - (keybits - 2 * k) : shard_bits;
  const bool ends = S <= 8 && k >= 5 && kb >= 0 && kb <= 10;
  for (uint64_t unit = w_begin + (uint64_t)blockIdx.x * TB * S; unit < w_end;
       unit += (uint64_t)gridDim.x * TB * S) {
    SetRange range{0, 0, true};
    if constexpr (BATCH) {
      // (to the unit's end: a thread's S starts may pass w_end, which is rounded to
      // the scatter's starts per thread, and those there belong to the next set)
      range = sets_of(bs, unit, unit + (uint64_t)TB * S);
      if (!range.any) continue;
    }
    const uint64_t g = unit + (uint64_t)threadIdx.x * S;
    if (g >= w_end) continue;
    uint32_t vm = valid_starts<S>(valid, g);
    if (!vm) continue;
    if (ends) {
      const uint64_t w0 = g >> 5, wt = (g + k - 5) >> 5;
      const uint64_t p0 = packed[w0], p1 = packed[w0 + 1];
      const uint32_t head = bits24(p0, p1, 2 * (int)(g & 31));  // bases g .. g+11
      const uint32_t tail = Key<Kc>::kWords == 1                // bases g+k-5 .. g+k+6
                                ? bits24(p0, p1, 2 * ((int)(g & 31) + k - 5))
                                : bits24(packed[wt], packed[wt + 1], 2 * (int)((g + k - 5) & 31));
      // the 12 head bases in reverse order (each base's 2-bit code kept):
      // reverse all bits, then swap the two bits of every base
      const uint32_t hb = __builtin_bitreverse32(head) >> 8;
      const uint32_t hr = ((hb >> 1) & 0x555555u) | ((hb & 0x555555u) << 1);
      uint32_t set = BATCH ? set_of(bs, range, g) : 0u;
#pragma unroll
      for (int i = 0; i < S; ++i) {
        if (!(vm & (1u << i))) continue;
        uint32_t at = 0;
        if constexpr (BATCH) {
          while (set < range.hi && g + i >= bs.set_byte_off[set + 1]) ++set;
          const uint32_t loc = bs.set_local[set];
          if (loc == kNoSet) continue;
          at = loc << kb;
        }
        // bases g+i .. g+i+4, the first most significant
        const uint32_t f = (hr >> (2 * (7 - i))) & 0x3FFu;
        const uint32_t r = ((tail >> (2 * i)) & 0x3FFu) ^ 0x3FFu;
        atomicAdd(&sh[at + (min(f, r) >> (10 - kb))], 1u);
      }
      continue;
    }
    K keys[S];
    uint32_t none[1];
    vm = window_keys<K, Kc, S, BATCH, false>(packed, g, k, vm, bs, range, keys, 0, none);
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (vm & (1u << i)) atomicAdd(&sh[shard_of(keys[i], keybits, shard_bits)], 1u);
  }
  __syncthreads();
  unsigned long long* const hc = hist + (uint64_t)(1 + blockIdx.x / R % kXcds) * nb;
  for (int i = threadIdx.x; i < nb; i += TB)
    if (sh[i]) atomicAdd(&hc[i], (unsigned long long)sh[i]);
}

// Owner-major scatter of window records into shard slices (cursor[x*nb + i]
// starts where tile class x's part of shard i's slice begins). One tile =
// TB*S window starts: the tile's records are ranked per shard in LDS, each
// shard's run reserves its place in its class's part with one global atomic,
// and the runs leave LDS as coalesced writes.
// CUT (see BatchSets): the shard is not in the record; it is staged beside it.
template <typename K, typename Kc, int S, int TB, bool BATCH, bool CUT = false>
__device__ __forceinline__ void window_scatter_body(const uint64_t* __restrict__ packed,
                                                    const uint64_t* __restrict__ valid,
                                                    uint64_t t_begin, uint64_t t_end, int k,
                                                    int keybits, int shard_bits, BatchSets bs,
                                                    unsigned long long* __restrict__ cursor,
                                                    K* __restrict__ out) {
  constexpr int NBMAX = 1 << kMaxShardBits;
  __shared__ K stage[TB * S];
  __shared__ uint32_t loff[NBMAX];  // per shard: records in the tile, then their run offsets
  __shared__ unsigned long long gbase[NBMAX];
  __shared__ uint32_t wsum[TB / 64];
  __shared__ uint16_t stage_shard[CUT ? TB * S : 1];
  const int nb = 1 << shard_bits;
  const int kb = CUT ? shard_bits - (keybits - 2 * k) : 0;
  const uint64_t n_tiles = (t_end - t_begin + TB - 1) / TB;
  for (uint64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    // tiles of class tile mod kXcds take their runs from their own part of
    // each shard slice (cursor[class * nb + shard], sized by k_window_hist):
    // the concurrent tiles of one XCD (workgroups are dealt to the XCDs in
    // turn) then write adjacent runs, whose shared 64-byte segments meet in
    // that XCD's L2 instead of going to memory in halves
    unsigned long long* const cls_cursor = cursor + (tile % kXcds) * (uint64_t)nb;
    SetRange range{0, 0, true};
    if constexpr (BATCH) {
      range = sets_of(bs, (t_begin + tile * TB) * S, min(t_end, t_begin + (tile + 1) * TB) * S);
      if (!range.any) continue;
    }
    for (int i = threadIdx.x; i < nb; i += TB) loff[i] = 0;
    __syncthreads();
    const uint64_t t = t_begin + tile * TB + threadIdx.x;
    const uint64_t g = t * S;
    uint32_t vm = t < t_end ? valid_starts<S>(valid, g) : 0u;
    K key[S];
    uint32_t rank[S];  // (the shard is recomputed from the key: fewer live registers)
    uint32_t cut_shard[CUT ? S : 1];
    auto shard = [&](int i) {
      if constexpr (CUT) return cut_shard[i];
      else return shard_of(key[i], keybits, shard_bits);
    };
    if (vm) {
      vm = window_keys<K, Kc, S, BATCH, CUT>(packed, g, k, vm, bs, range, key, kb, cut_shard);
#pragma unroll
      for (int i = 0; i < S; ++i)
        if (vm & (1u << i)) rank[i] = atomicAdd(&loff[shard(i)], 1u);
    }
    __syncthreads();
    const uint32_t total = block_exscan_inplace<TB>(loff, nb, wsum);
    for (int i = threadIdx.x; i < nb; i += TB) {
      const uint32_t cnt = (i + 1 < nb ? loff[i + 1] : total) - loff[i];
      if (cnt) gbase[i] = atomicAdd(&cls_cursor[i], (unsigned long long)cnt);
    }
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (vm & (1u << i)) {
        const uint32_t p = loff[shard(i)] + rank[i];
        stage[p] = key[i];
        if constexpr (CUT) stage_shard[p] = (uint16_t)shard(i);
      }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < total; j += TB) {
      const K kk = stage[j];  // its shard again from the key: cheaper than staging it
      uint32_t b;
      if constexpr (CUT) b = stage_shard[j];
      else b = shard_of(kk, keybits, shard_bits);
      out[gbase[b] + (j - loff[b])] = kk;
    }
    __syncthreads();
  }
}

template <typename K, typename Kc, int S, int TB, bool BATCH>
__global__ void __launch_bounds__(TB) k_window_scatter(const uint64_t* __restrict__ packed,
                                                       const uint64_t* __restrict__ valid,
                                                       uint64_t t_begin, uint64_t t_end, int k,
                                                       int keybits, int shard_bits, BatchSets bs,
                                                       unsigned long long* __restrict__ cursor,
                                                       K* __restrict__ out) {
  window_scatter_body<K, Kc, S, TB, BATCH>(packed, valid, t_begin, t_end, k, keybits,
                                           shard_bits, bs, cursor, out);
}

// Cut keys of a batch.
template <int S, int TB>
__global__ void __launch_bounds__(TB)
k_window_scatter_cut(const uint64_t* __restrict__ packed, const uint64_t* __restrict__ valid,
                     uint64_t t_begin, uint64_t t_end, int k, int keybits, int shard_bits,
                     BatchSets bs, unsigned long long* __restrict__ cursor,
                     uint64_t* __restrict__ out) {
  window_scatter_body<uint64_t, uint64_t, S, TB, true, true>(packed, valid, t_begin, t_end, k,
                                                             keybits, shard_bits, bs, cursor, out);
}

// Plain 64-bit keys: registers capped so that two 1024-thread workgroups
// share a CU (their LDS fits twice), which hides the per-tile barriers and
// atomics. (The batch form keeps more values live and stays uncapped.)
// The same with 16 window starts per thread: a tile of 16,384 records (128 KiB
// of LDS staging, one workgroup per CU) gives each of many shards a run twice
// as long per tile.
template <typename K, typename Kc, int S, int TB, bool BATCH>
__global__ void __launch_bounds__(TB)
k_window_scatter64w(const uint64_t* __restrict__ packed, const uint64_t* __restrict__ valid, uint64_t t_begin, uint64_t t_end, int k,
                    int keybits, int shard_bits, BatchSets bs,
                    unsigned long long* __restrict__ cursor, K* __restrict__ out) {
  window_scatter_body<K, Kc, S, TB, BATCH>(packed, valid, t_begin, t_end, k, keybits,
                                           shard_bits, bs, cursor, out);
}

template <typename K, typename Kc, int S, int TB, bool BATCH>
__global__ void __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_window_scatter64(const uint64_t* __restrict__ packed, const uint64_t* __restrict__ valid, uint64_t t_begin, uint64_t t_end, int k,
                   int keybits, int shard_bits, BatchSets bs,
                   unsigned long long* __restrict__ cursor, K* __restrict__ out) {
  window_scatter_body<K, Kc, S, TB, BATCH>(packed, valid, t_begin, t_end, k, keybits,
                                           shard_bits, bs, cursor, out);
}

// ---------------------------------------------------------------- planning (one block)

constexpr int kPlanTB = 1024;
// Up to this many split items are listed by the one planning workgroup itself
// (a few rounds of its waves); more by a launch of their own.
constexpr uint64_t kFewItems = 4096;

__device__ __forceinline__ int ceil_log2_dev(uint64_t x) {
  return x <= 1 ? 0 : 64 - __builtin_clzll(x - 1);
}

// Shard plan: owner-major record ranges, split decision per shard, split
// work items, leaf slot offsets (leaf slots follow key order).
__global__ void __launch_bounds__(kPlanTB) k_plan_shards(
    unsigned long long* __restrict__ hist, const int* __restrict__ order, int shard_bits,
    int keybits, uint64_t leaf_target, uint64_t leaf_attempt, int tile,
    unsigned long long* __restrict__ sbegin, unsigned long long* __restrict__ cursor,
    SplitBin* __restrict__ bins, unsigned long long* __restrict__ item_off,
    unsigned long long* __restrict__ subhist, DevState* __restrict__ st,
    SplitItem* __restrict__ items, Leaf* __restrict__ leaves) {
  __shared__ unsigned long long wsum[kPlanTB / 64];
  __shared__ unsigned long long s_hist[kPlanTB], s_off[kPlanTB + 1], s_begin[kPlanTB];
  const int nb = 1 << shard_bits;  // <= kPlanTB
  const int t = threadIdx.x;
  unsigned long long total;
  // shard sizes: the sum over the tile classes
  unsigned long long h = 0;
  if (t < nb) {
#pragma unroll
    for (int x = 0; x < kXcds; ++x) h += hist[(uint64_t)(1 + x) * nb + t];
    hist[t] = h;
    s_hist[t] = h;
  }
  __syncthreads();
  // owner-major exclusive scan: the t-th shard in owner order
  const int co = t < nb ? order[t] : 0;
  const unsigned long long ho = t < nb ? s_hist[co] : 0ull;
  const unsigned long long b0 = block_exscan<kPlanTB, unsigned long long>(ho, wsum, &total);
  if (t == 0) st->W = total;  // every valid window has one shard
  if (t < nb) {
    sbegin[co] = b0;
    s_begin[co] = b0;
    // each class's part of the slice: after the earlier classes' records
    unsigned long long c = b0;
    for (int x = 0; x < kXcds; ++x) {
      cursor[(uint64_t)x * nb + co] = c;
      c += hist[(uint64_t)(1 + x) * nb + co];
    }
  }
  // split decision for shard t (key order)
  int nbits = 0;
  const int remaining = keybits - shard_bits;
  if (h > leaf_attempt && remaining > 0) {
    nbits = ceil_log2_dev((h + leaf_target - 1) / leaf_target);
    nbits = max(1, min(nbits, min(kSplitMaxBits, remaining)));
  }
  const unsigned long long L = h == 0 ? 0ull : (nbits ? (1ull << nbits) : 1ull);
  const unsigned long long loff = block_exscan<kPlanTB, unsigned long long>(L, wsum, &total);
  const unsigned long long n_leaves = total;
  const unsigned long long ni = nbits ? (h + tile - 1) / tile : 0ull;
  const unsigned long long ioff = block_exscan<kPlanTB, unsigned long long>(ni, wsum, &total);
  const unsigned long long n_items = total;
  if (t < nb) {
    bins[t] = SplitBin{loff, (uint32_t)(keybits - shard_bits - nbits), (uint32_t)nbits};
    item_off[t] = ioff;
    if (leaves) {  // no shard is split (leaf_attempt): a leaf each
      if (h) leaves[loff] = Leaf{s_begin[t], s_begin[t] + h, 0u, (uint32_t)shard_bits, 0u, (uint32_t)t};
    } else if (!nbits && h) {
      subhist[loff] = h;  // split shards' counters were cleared before
    }
  }
  if (t == 0) {
    item_off[nb] = n_items;
    st->n_items = n_items;
    st->n_leaves = n_leaves;
  }
  if (!items || leaves) return;  // many items: k_plan_items lists them
  if (t < nb) s_off[t] = ioff;
  if (t == 0) s_off[nb] = n_items;
  __syncthreads();
  // a shard's items by one wave
  for (int c = t >> 6; c < nb; c += kPlanTB / 64) {
    const unsigned long long i0 = s_off[c], i1 = s_off[c + 1], b = s_begin[c], e = b + s_hist[c];
    for (unsigned long long i = i0 + (t & 63); i < i1; i += 64) {
      const unsigned long long a = b + (i - i0) * (unsigned long long)tile;
      items[i] = SplitItem{a, min(e, a + (unsigned long long)tile), (uint32_t)c, 0};
    }
  }
}

// Split work items: item i belongs to the shard c with item_off[c] <= i < item_off[c+1].
__global__ void k_plan_items(const unsigned long long* __restrict__ hist,
                             const unsigned long long* __restrict__ sbegin,
                             const unsigned long long* __restrict__ item_off, int shard_bits,
                             int tile, const DevState* __restrict__ st,
                             SplitItem* __restrict__ items) {
  const int nb = 1 << shard_bits;
  const unsigned long long n = st->n_items;
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x) {
    int lo = 0, hi = nb - 1;  // last c with item_off[c] <= i
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (item_off[mid] <= i) lo = mid; else hi = mid - 1;
    }
    const unsigned long long a = sbegin[lo] + (i - item_off[lo]) * (unsigned long long)tile;
    items[i] = SplitItem{a, min(sbegin[lo] + hist[lo], a + (unsigned long long)tile), (uint32_t)lo, 0};
  }
}

// Classification of the leaves, a lane each (id i of len records; has: the
// lane has a leaf). Leaves above the small-leaf size go to a list of their own
// (order irrelevant); with huge != nullptr, leaves of more than huge_min
// records go straight to that list instead (st->n_ovf), for the second count's
// larger table: such leaves are the dense clusters that overflow the first
// table (on 40,000,000 reads at k = 31 the overflowed leaves average 147,000
// records, the others 4,600), and the first count would read part of them
// before giving up. d_zero != nullptr (no one-wave kernel follows): the counts
// of empty leaves are set to 0 there.
// (direct: the block-wide kernel takes all others straight from the leaf table,
// see leaf_lists.)
// Called by all threads of a workgroup of up to 1,024; sh holds 2 * 17 words.
// One atomic per list and workgroup: one per wave, on one word, took 130 us for
// the 2^20 leaves of 20,000,000 reads at 12 ns each (the whole kernel now 21 us).
__device__ __forceinline__ void classify_leaves(bool has, uint32_t i, uint64_t len,
                                                DevState* __restrict__ st, const LeafLists& q,
                                                uint32_t* sh, unsigned long long* base) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  const bool to_huge = has && q.huge && len > q.huge_min;
  const bool big = has && !to_huge && !q.direct && len > q.small_max;
  if (q.d_zero && has && len == 0) q.d_zero[i] = 0;
  const unsigned long long m = __ballot(big), mh = __ballot(to_huge);
  if (lane == 0) {
    sh[w] = (uint32_t)__popcll(m);
    sh[17 + w] = (uint32_t)__popcll(mh);
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    uint32_t* const c = sh + 17 * threadIdx.x;
    uint32_t run = 0;
    for (int v = 0; v < nw; ++v) {
      const uint32_t x = c[v];
      c[v] = run;
      run += x;
    }
    base[threadIdx.x] =
        run ? atomicAdd(threadIdx.x == 0 ? &st->n_large : &st->n_ovf, (unsigned long long)run) : 0;
  }
  __syncthreads();
  const unsigned long long below = (1ull << lane) - 1;
  if (big) q.large[base[0] + sh[w] + __popcll(m & below)] = i;
  if (to_huge) q.huge[base[1] + sh[17 + w] + __popcll(mh & below)] = i;
  __syncthreads();
}

__global__ void k_classify_leaves(const Leaf* __restrict__ leaves, DevState* __restrict__ st,
                                  LeafLists q) {
  __shared__ uint32_t sh[34];
  __shared__ unsigned long long base[2];
  const unsigned long long n = st->n_leaves;
  const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
  for (unsigned long long i0 = (unsigned long long)blockIdx.x * blockDim.x; i0 < n; i0 += stride) {
    const unsigned long long i = i0 + threadIdx.x;
    const Leaf lf = i < n ? leaves[i] : Leaf{0, 0, 0, 0, 0, 0};
    classify_leaves(i < n, (uint32_t)i, lf.end - lf.begin, st, q, sh, base);
  }
}

// Leaf table (key order) and sub-bin cursors: block c handles shard c. With
// q.on the leaves are classified here as well (not where pre-aggregation
// still shortens them).
__global__ void __launch_bounds__(kPlanTB) k_plan_leaves(
    const unsigned long long* __restrict__ hist, const unsigned long long* __restrict__ sbegin,
    const SplitBin* __restrict__ bins, int shard_bits,
    const unsigned long long* __restrict__ subhist, Leaf* __restrict__ leaves,
    unsigned long long* __restrict__ cursor, int merge_cshift, int ncls, uint64_t cls_stride,
    DevState* __restrict__ st, LeafLists q) {
  __shared__ unsigned long long wsum[kPlanTB / 64], base[2];
  __shared__ uint32_t sh[34];
  const int c = blockIdx.x;
  const unsigned long long h = hist[c];
  if (!h) return;
  const SplitBin b = bins[c];
  if (b.nbits == 0) {
    if (threadIdx.x == 0)
      leaves[b.hist_off] =
          Leaf{sbegin[c], sbegin[c] + h, 0u, (uint32_t)shard_bits, 0u, (uint32_t)c};
    if (q.on) classify_leaves(threadIdx.x == 0, (uint32_t)b.hist_off, h, st, q, sh, base);
    return;
  }
  const uint32_t nsub = 1u << b.nbits;  // <= kPlanTB
  const uint32_t j = threadIdx.x;
  unsigned long long n = 0;
  if (j < nsub)
    for (int x = 0; x < ncls; ++x) n += subhist[x * cls_stride + b.hist_off + j];
  unsigned long long total;
  const unsigned long long off = block_exscan<kPlanTB, unsigned long long>(n, wsum, &total);
  if (j < nsub) {
    const unsigned long long run = sbegin[c] + off;
    leaves[b.hist_off + j] = Leaf{run, run + n, 1u, (uint32_t)(shard_bits + b.nbits),
                                  (uint32_t)merge_cshift, (uint32_t)c};
    // each item class's part of the sub-bin: after the earlier classes' records
    unsigned long long at = run;
    for (int x = 0; x < ncls; ++x) {
      cursor[x * cls_stride + b.hist_off + j] = at;
      at += subhist[x * cls_stride + b.hist_off + j];
    }
  }
  if (q.on) classify_leaves(j < nsub, (uint32_t)(b.hist_off + j), n, st, q, sh, base);
}

// ---------------------------------------------------------------- refinement support

// Indices (any order) and entries of the leaves whose tables overflowed.
__global__ void k_list_overflowed(const uint32_t* __restrict__ d, uint64_t n,
                                  const Leaf* __restrict__ leaves, uint32_t* __restrict__ list,
                                  Leaf* __restrict__ out, unsigned long long* __restrict__ count) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x; i0 < n; i0 += stride) {
    const uint64_t i = i0 + threadIdx.x;
    const bool ovf = i < n && d[i] == kLeafOverflow;
    const unsigned long long m = __ballot(ovf);
    if (!m) continue;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)m) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd(count, (unsigned long long)__popcll(m));
    base = __shfl(base, leader);
    if (ovf) {
      const unsigned long long at = base + __popcll(m & ((1ull << lane) - 1));
      list[at] = (uint32_t)i;
      out[at] = leaves[i];
    }
  }
}

// Entries each old leaf occupies in the refined list: 1, or (for an
// overflowed leaf) the number of its parts, set by k_splice_root_counts.
__global__ void k_splice_counts(const uint32_t* __restrict__ d, uint64_t n,
                                uint32_t* __restrict__ cnt) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cnt[i] = d[i] == kLeafOverflow ? 0u : 1u;
}

__global__ void k_splice_root_counts(const uint32_t* __restrict__ root_leaf,
                                     const uint32_t* __restrict__ nparts, uint32_t R,
                                     uint32_t* __restrict__ cnt) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < R) cnt[root_leaf[r]] = nparts[r];
}

// Kept leaves move to pos[i]; the parts of root r fill pos[root_leaf[r]] onwards.
__global__ void k_splice_keep(const Leaf* __restrict__ leaves, const uint32_t* __restrict__ d,
                              const unsigned long long* __restrict__ pos, uint64_t n,
                              Leaf* __restrict__ out, uint32_t* __restrict__ out_d) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && d[i] != kLeafOverflow) {
    out[pos[i]] = leaves[i];
    out_d[pos[i]] = d[i];
  }
}

__global__ void k_splice_parts(const uint32_t* __restrict__ root_leaf,
                               const uint32_t* __restrict__ part_begin,
                               const uint32_t* __restrict__ nparts, uint32_t R,
                               const Leaf* __restrict__ parts, const uint32_t* __restrict__ part_d,
                               const unsigned long long* __restrict__ pos, Leaf* __restrict__ out,
                               uint32_t* __restrict__ out_d) {
  for (uint32_t r = blockIdx.x; r < R; r += gridDim.x) {
    const unsigned long long at = pos[root_leaf[r]];
    const uint32_t b = part_begin[r];
    for (uint32_t p = threadIdx.x; p < nparts[r]; p += blockDim.x) {
      out[at + p] = parts[b + p];
      out_d[at + p] = part_d[b + p];
    }
  }
}

// Output offsets: exclusive scan of the leaf counts in leaf (= key) order, in
// three steps (tile sums, scan of tile sums, tile scans). Overflowed leaves
// count zero and raise st->overflow.
constexpr int kScanTB = 256, kScanPer = 16, kScanTile = kScanTB * kScanPer;

__global__ void __launch_bounds__(kScanTB) k_scan_reduce(const uint32_t* __restrict__ d,
                                                         DevState* __restrict__ st,
                                                         unsigned long long* __restrict__ bsum) {
  __shared__ unsigned long long wsum[kScanTB / 64];
  const unsigned long long n = st->n_leaves;
  const unsigned long long base = (unsigned long long)blockIdx.x * kScanTile;
  unsigned long long s = 0;
  uint32_t ovf = 0;
  for (int j = 0; j < kScanPer; ++j) {
    const unsigned long long i = base + (unsigned long long)j * kScanTB + threadIdx.x;
    if (i < n) {
      const uint32_t x = d[i];
      if (x == kLeafOverflow) ovf = 1;
      else s += x;
    }
  }
  if (ovf) atomicOr(&st->overflow, 1u);
  unsigned long long total;
  (void)block_exscan<kScanTB, unsigned long long>(s, wsum, &total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kPlanTB) k_scan_top(unsigned long long* __restrict__ bsum,
                                                      uint32_t nblocks, DevState* __restrict__ st) {
  __shared__ unsigned long long wsum[kPlanTB / 64];
  const uint32_t per = (nblocks + kPlanTB - 1) / kPlanTB;
  const uint32_t b = threadIdx.x * per, e = min(nblocks, b + per);
  unsigned long long s = 0;
  for (uint32_t i = b; i < e; ++i) s += bsum[i];
  unsigned long long total;
  unsigned long long run = block_exscan<kPlanTB, unsigned long long>(s, wsum, &total);
  for (uint32_t i = b; i < e; ++i) {
    const unsigned long long x = bsum[i];
    bsum[i] = run;
    run += x;
  }
  if (threadIdx.x == 0) st->D = total;
}

// The call's state into host memory, once it is final: the host then only
// waits for the stream, with no copy queued behind the last kernel.
__device__ __forceinline__ void publish_state(DevState* st, DevState* pub) {
  static_assert(sizeof(DevState) % 8 == 0, "copied by words");
  // (loads past this CU's caches: some words may just have been written)
  if (pub && threadIdx.x < sizeof(DevState) / 8)
    ((unsigned long long*)pub)[threadIdx.x] =
        __hip_atomic_load((unsigned long long*)st + threadIdx.x, __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(kScanTB) k_scan_down(const uint32_t* __restrict__ d,
                                                       DevState* st,
                                                       const unsigned long long* __restrict__ bsum,
                                                       unsigned long long* __restrict__ out_off,
                                                       DevState* pub) {
  __shared__ unsigned long long wsum[kScanTB / 64];
  if (blockIdx.x == 0) publish_state(st, pub);
  const unsigned long long n = st->n_leaves;
  // thread t owns kScanPer consecutive leaves of the tile
  const unsigned long long base = (unsigned long long)blockIdx.x * kScanTile +
                                  (unsigned long long)threadIdx.x * kScanPer;
  uint32_t v[kScanPer];
  unsigned long long s = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const unsigned long long i = base + j;
    v[j] = i < n ? d[i] : 0u;
    if (v[j] == kLeafOverflow) v[j] = 0;
    s += v[j];
  }
  unsigned long long total;
  unsigned long long run = bsum[blockIdx.x] + block_exscan<kScanTB, unsigned long long>(s, wsum, &total);
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const unsigned long long i = base + j;
    if (i < n) out_off[i] = run;
    run += v[j];
  }
}

// The same by one workgroup, for up to kScanOneMax leaves: one launch instead
// of three.
constexpr uint32_t kScanOnePer = 16;
constexpr uint64_t kScanOneMax = (uint64_t)kPlanTB * kScanOnePer;
__global__ void __launch_bounds__(kPlanTB) k_scan_one(const uint32_t* __restrict__ d, DevState* st,
                                                      unsigned long long* __restrict__ out_off,
                                                      DevState* pub) {
  __shared__ unsigned long long wsum[kPlanTB / 64];
  const uint32_t n = (uint32_t)min(st->n_leaves, (unsigned long long)kScanOneMax);
  const uint32_t per = (n + kPlanTB - 1) / kPlanTB, base = threadIdx.x * per;
  uint32_t v[kScanOnePer];
  unsigned long long s = 0;
  bool ovf = false;
#pragma unroll
  for (uint32_t j = 0; j < kScanOnePer; ++j) {
    v[j] = j < per && base + j < n ? d[base + j] : 0u;
    if (v[j] == kLeafOverflow) {
      ovf = true;
      v[j] = 0;
    }
    s += v[j];
  }
  if (ovf) atomicOr(&st->overflow, 1u);
  unsigned long long total;
  unsigned long long run = block_exscan<kPlanTB, unsigned long long>(s, wsum, &total);
#pragma unroll
  for (uint32_t j = 0; j < kScanOnePer; ++j) {
    if (j < per && base + j < n) out_off[base + j] = run;
    run += v[j];
  }
  if (threadIdx.x == 0) st->D = total;
  __threadfence();
  __syncthreads();
  publish_state(st, pub);
}

// ---------------------------------------------------------------- split (MSD step)

template <typename K, int TB>
__global__ void __launch_bounds__(TB) k_split_hist(const K* __restrict__ src,
                                                   const SplitItem* __restrict__ items,
                                                   const DevState* __restrict__ st,
                                                   const SplitBin* __restrict__ bins,
                                                   unsigned long long* __restrict__ subhist,
                                                   int ncls, uint64_t cls_stride) {
  __shared__ uint32_t h[1 << kSplitMaxBits];
  const unsigned long long n_items = st->n_items;
  for (unsigned long long w = blockIdx.x; w < n_items; w += gridDim.x) {
    const SplitItem it = items[w];
    // counts of item class w mod ncls (the split scatter's cursor classes)
    unsigned long long* const sh = subhist + (w % ncls) * cls_stride;
    const SplitBin bn = bins[it.bin];
    const int nsub = 1 << bn.nbits;
    for (int i = threadIdx.x; i < nsub; i += TB) h[i] = 0;
    __syncthreads();
    // loads of a batch are issued together, then counted
    constexpr int RB = 8;
    for (uint64_t r0 = it.begin; r0 < it.end; r0 += (uint64_t)TB * RB) {
      K kb[RB];
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const uint64_t r = r0 + (uint64_t)j * TB + threadIdx.x;
        if (r < it.end) kb[j] = src[r];
      }
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const uint64_t r = r0 + (uint64_t)j * TB + threadIdx.x;
        if (r < it.end) atomicAdd(&h[Key<K>::bits(kb[j], bn.shift, bn.nbits)], 1u);
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nsub; i += TB)
      if (h[i]) atomicAdd(&sh[bn.hist_off + i], (unsigned long long)h[i]);
    __syncthreads();
  }
}

template <typename K, int TB, int R>
__global__ void __launch_bounds__(TB) k_split_scatter(const K* __restrict__ src,
                                                      K* __restrict__ dst,
                                                      const SplitItem* __restrict__ items,
                                                      const DevState* __restrict__ st,
                                                      const SplitBin* __restrict__ bins,
                                                      unsigned long long* __restrict__ cursor,
                                                      int ncls, uint64_t cls_stride) {
  constexpr int NS = 1 << kSplitMaxBits;
  __shared__ K stage[TB * R];
  __shared__ uint32_t hist[NS];  // per sub-bin: records in the tile, then their run offsets
  uint32_t* const loff = hist;
  __shared__ unsigned long long gbase[NS];
  __shared__ uint32_t wsum[TB / 64];
  const unsigned long long n_items = st->n_items;
  // the records of the workgroup's next item are loaded while the current
  // one's runs leave LDS (its keys' registers are free once it is staged)
  K key[R];
  SplitItem it = blockIdx.x < n_items ? items[blockIdx.x] : SplitItem{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const uint64_t r = it.begin + threadIdx.x + (uint64_t)j * TB;
    if (r < it.end) key[j] = src[r];
  }
  for (unsigned long long w = blockIdx.x; w < n_items; w += gridDim.x) {
    const SplitBin bn = bins[it.bin];
    const int nsub = 1 << bn.nbits;
    // items of class w mod ncls take their runs from their own part of each
    // sub-bin (as in the owner scatter: with ncls = kXcds and the workgroups
    // of one class on one XCD, the partial segments of adjacent runs meet in
    // that XCD's L2)
    unsigned long long* const cls_cursor = cursor + (w % ncls) * cls_stride;
    for (int i = threadIdx.x; i < nsub; i += TB) hist[i] = 0;
    __syncthreads();
    uint32_t sub[R], rank[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t r = it.begin + threadIdx.x + (uint64_t)j * TB;
      if (r < it.end) {
        sub[j] = Key<K>::bits(key[j], bn.shift, bn.nbits);
        rank[j] = atomicAdd(&hist[sub[j]], 1u);
      }
    }
    __syncthreads();
    const uint32_t total = block_exscan_inplace<TB>(hist, nsub, wsum);
    for (int i = threadIdx.x; i < nsub; i += TB) {
      const uint32_t cnt = (i + 1 < nsub ? loff[i + 1] : total) - loff[i];
      if (cnt) gbase[i] = atomicAdd(&cls_cursor[bn.hist_off + i], (unsigned long long)cnt);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t r = it.begin + threadIdx.x + (uint64_t)j * TB;
      if (r < it.end) {
        const uint32_t p = loff[sub[j]] + rank[j];
        stage[p] = key[j];
      }
    }
    __syncthreads();
    const unsigned long long wn = w + gridDim.x;
    const SplitItem nx = wn < n_items ? items[wn] : SplitItem{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t r = nx.begin + threadIdx.x + (uint64_t)j * TB;
      if (r < nx.end) key[j] = src[r];
    }
    for (uint32_t j = threadIdx.x; j < total; j += TB) {
      const K kk = stage[j];
      const uint32_t b = Key<K>::bits(kk, bn.shift, bn.nbits);
      dst[gbase[b] + (j - loff[b])] = kk;
    }
    it = nx;
    __syncthreads();
  }
}

// Split scatter with pre-aggregation of equal keys (the heavy-hitter
// aggregation of Section IV-D, on one tile of one shard's records: keys that
// occur many times in the input are concentrated in one shard and one
// sub-bin, where their copies meet in the tile). After the tile is staged by
// sub-bin in LDS, each thread takes R consecutive staged records; a run of
// equal keys among them (always inside one sub-bin) leaves as one record with
// its length minus one in bits [cshift, 64), where the key's top bits (the
// shard, common to the leaf) were. The first record of each thread's segment
// starts a run, so a run never exceeds R. The tile's cursors advance by the
// records written.
template <int TB, int R>
__global__ void __launch_bounds__(TB) k_split_scatter_merge(const uint64_t* __restrict__ src,
                                                            uint64_t* __restrict__ dst,
                                                            const SplitItem* __restrict__ items,
                                                            const DevState* __restrict__ st,
                                                            const SplitBin* __restrict__ bins,
                                                            unsigned long long* __restrict__ cursor,
                                                            int cshift) {
  constexpr int NS = 1 << kSplitMaxBits;
  __shared__ uint64_t stage[TB * R];
  __shared__ uint32_t loff[NS];        // per sub-bin: records of the tile, then their offsets
  __shared__ uint32_t mstart[NS + 1];  // per sub-bin: offset of its first merged record
  __shared__ uint32_t tbase[TB];       // per thread: merged records before its segment
  __shared__ unsigned long long gbase[NS];
  __shared__ uint32_t wsum[TB / 64];
  const uint64_t low = (1ull << cshift) - 1;
  const unsigned long long n_items = st->n_items;
  for (unsigned long long w = blockIdx.x; w < n_items; w += gridDim.x) {
    const SplitItem it = items[w];
    const SplitBin bn = bins[it.bin];
    const int nsub = 1 << bn.nbits;
    for (int i = threadIdx.x; i < nsub; i += TB) loff[i] = 0;
    __syncthreads();
    uint64_t key[R];
    uint32_t sub[R], rank[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t r = it.begin + threadIdx.x + (uint64_t)j * TB;
      if (r < it.end) {
        key[j] = src[r];
        sub[j] = Key<uint64_t>::bits(key[j], bn.shift, bn.nbits);
        rank[j] = atomicAdd(&loff[sub[j]], 1u);
      }
    }
    __syncthreads();
    const uint32_t total = block_exscan_inplace<TB>(loff, nsub, wsum);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t r = it.begin + threadIdx.x + (uint64_t)j * TB;
      if (r < it.end) stage[loff[sub[j]] + rank[j]] = key[j];
    }
    __syncthreads();
    // runs of equal keys in this thread's segment [R*t, R*t + R) of the stage
    const uint32_t s0 = (uint32_t)threadIdx.x * R;
    uint64_t seg[R];
    uint32_t heads = 0;  // bit j: a run starts at s0 + j
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint32_t i = s0 + j;
      seg[j] = i < total ? stage[i] : 0;
      if (i < total && (j == 0 || seg[j] != seg[j - 1])) heads |= 1u << j;
    }
    uint32_t nh_all;
    const uint32_t base = block_exscan<TB, uint32_t>(__builtin_popcount(heads), wsum, &nh_all);
    tbase[threadIdx.x] = base;
    __syncthreads();
    // merged records before each sub-bin: heads before its first staged record
    for (int b = threadIdx.x; b <= nsub; b += TB) {
      const uint32_t i = b < nsub ? loff[b] : total;
      if (i >= total) {
        mstart[b] = nh_all;
        continue;
      }
      const uint32_t t = i / R, j0 = t * R;
      uint32_t h = tbase[t];
      for (uint32_t q = j0; q < i; ++q) h += (q == j0 || stage[q] != stage[q - 1]) ? 1u : 0u;
      mstart[b] = h;
    }
    __syncthreads();  // every staged record has been read: the stage is rewritten below
    {
      uint32_t at = base;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        if (!(heads & (1u << j))) continue;
        const uint32_t rest = heads >> (j + 1);
        const uint32_t next = rest ? (uint32_t)(j + 1 + __builtin_ctz(rest)) : (uint32_t)R;
        const uint32_t end = min(next, total - s0);
        const uint64_t len = end - (uint32_t)j;
        stage[at++] = ((len - 1) << cshift) | (seg[j] & low);
      }
    }
    for (int b = threadIdx.x; b < nsub; b += TB) {
      const uint32_t cnt = mstart[b + 1] - mstart[b];
      if (cnt) gbase[b] = atomicAdd(&cursor[bn.hist_off + b], (unsigned long long)cnt);
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < nh_all; j += TB) {
      const uint64_t kk = stage[j];
      const uint32_t b = Key<uint64_t>::bits(kk, bn.shift, bn.nbits);
      dst[gbase[b] + (j - mstart[b])] = kk;
    }
    __syncthreads();
  }
}

// Records of pre-aggregated leaves end where the split scatter's cursor
// stopped (fewer records than windows).
__global__ void k_leaf_ends(Leaf* __restrict__ leaves, const unsigned long long* __restrict__ cursor,
                            const DevState* __restrict__ st) {
  const unsigned long long n = st->n_leaves;
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x)
    if (leaves[i].cshift) leaves[i].end = cursor[i];
}

// ---------------------------------------------------------------- leaf count

// Bitonic sort of (keys, counts) in LDS, n a power of two (fallback sort).
template <typename K, typename C, int TB>
__device__ __forceinline__ void bitonic_sort(K* keys, C* cnt, uint32_t n) {
  for (uint32_t size = 2; size <= n; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < n / 2; i += TB) {
        const uint32_t lo = (i / stride) * stride * 2 + (i % stride);
        const uint32_t hi = lo + stride;
        const bool asc = (lo & size) == 0;
        const K a = keys[lo], b = keys[hi];
        if ((a > b) == asc) {
          keys[lo] = b;
          keys[hi] = a;
          const C t = cnt[lo];
          cnt[lo] = cnt[hi];
          cnt[hi] = t;
        }
      }
      __syncthreads();
    }
  }
}

// Table slot of a 64-bit key: multiply-shift (Knuth) of a 32-bit fold of the
// key; collisions are resolved by linear probing, so only speed depends on it.
// (Multipliers: two 32-bit primes of Collet's xxHash, one of Wellons' hash search.)
__device__ __forceinline__ uint32_t slot_hash(uint64_t key, int bits) {
  const uint32_t f = (uint32_t)key * 0x9E3779B1u + (uint32_t)(key >> 32) * 0x85EBCA77u;
  return (f ^ (f >> 15)) * 0x2C1B3C6Du >> (32 - bits);
}

// Probes after which a lane gives its leaf up as overflowed, where the leaf has
// records enough for that (chains of a table below its limit are far shorter), and
// it looks every 64 probes whether another lane has. A batch may hold as many new
// keys as the table has slots, and each of its lanes probed a full table round, or
// 512 slots whatever the others had found: 100 overflowing leaves among 30,000
// (10 kbp reads, k = 55) took the launch from 0.9 to 1.7 ms, so 1.1; those of
// 1,000,000 reads at k = 100 3.9 -> 2.7 ms; one-word keys, 20 MB of A and T at k =
// 31 4.4 -> 3.0 ms, 4 MB of random reads at k = 32 537 -> 389 us.
constexpr uint32_t kMaxProbes = 512;  // a multiple of 64, as table sizes are

// Workgroup-scope flag in LDS (a volatile LDS variable would be accessed with
// flat instructions that also wait for all outstanding global memory operations).
__device__ __forceinline__ uint32_t ovf_get(uint32_t* f) {
  return __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void ovf_set(uint32_t* f) {
  __hip_atomic_store(f, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint32_t next_pow2(uint32_t x) {
  return x <= 2 ? 2u : 1u << (32 - __builtin_clz(x - 1));
}

// Table slots for a leaf of n records: enough that n distinct keys stay below
// 7/8 load, at least TB, at most CMAX.
template <int TB, int CMAX>
__device__ __forceinline__ uint32_t leaf_slots(uint64_t n, uint32_t cmax_rt) {
  const uint64_t want = n + n / 7 + 1;
  uint32_t c = want >= cmax_rt ? cmax_rt : next_pow2((uint32_t)want);
  return c < (uint32_t)TB ? (uint32_t)TB : c;
}

// Epilogue shared by all key widths: the table has been filled with Cn slots;
// table.load(s, ref, count) reads slot s (count 0: empty), table.bits(ref, shift,
// nbits) gives key bits of what the slot refers to and table.key(ref) its key;
// tk and tc, where the table may have been, then hold the distinct keys. These are
// grouped by a counting sort on the key bits
// just below the leaf's common prefix; each key then finds its place inside
// its group by counting the smaller keys of the group, and the pair is written
// to dst/tmp_cnt at [begin, begin + d) in key order. Keys of one group share a
// long prefix when sequencing errors sit near the k-mer's end (the erroneous
// copies of one k-mer), so groups are not always tiny; a group larger than
// kRankMax switches the leaf to a bitonic sort. Cn >> GSHIFT groups: aux holds
// 2 * Cn >> GSHIFT counters. Returns d.
// (wider keys: groups of up to 1,024 are still ranked sooner than a bitonic sort
// moves its 20 to 36 bytes a key: four words, the large leaves of 1,000,000 reads
// at k = 100, 12% repeats, 3.36 -> 2.84 ms; two words, 20 MB of reads of a genome
// of 40% repeats at k = 63 760 -> 691 us, 60 MB of it 1.80 -> 1.86 ms, and no
// difference on inputs of fewer repeats)
template <typename K> constexpr uint32_t kRankMax = sizeof(K) > 8 ? 1024 : 256;

template <typename K, int TB, int PER, int GSHIFT, typename Table>
__device__ __forceinline__ uint32_t leaf_sort_write(K* tk, uint32_t* tc, uint32_t* aux,
                                                    uint32_t* wsum, uint32_t* s_max, uint32_t Cn,
                                                    int keybits, int prefix_bits,
                                                    K* __restrict__ dst,
                                                    uint32_t* __restrict__ tmp_cnt,
                                                    uint64_t begin, const Table& table) {
  typename Table::Ref rk[PER];
  uint32_t rc[PER];
  uint32_t rank[PER], bk[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {  // slot j*TB + tid: consecutive lanes, consecutive slots
    const uint32_t s = (uint32_t)j * TB + threadIdx.x;
    rc[j] = 0;
    if (s < Cn) table.load(s, rk[j], rc[j]);
  }
  int nbk_bits = 31 - __builtin_clz(Cn) - GSHIFT;
  if (nbk_bits > keybits - prefix_bits) nbk_bits = keybits - prefix_bits;
  const uint32_t nbk = 1u << nbk_bits;
  const int shift = keybits - prefix_bits - nbk_bits;
  for (uint32_t i = threadIdx.x; i < nbk; i += TB) aux[i] = 0;
  if (threadIdx.x == 0) *s_max = 0;
  __syncthreads();  // table copied to registers; group counters cleared
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if ((uint32_t)j * TB >= Cn) break;  // uniform: Cn is a multiple of TB
    // every slot adds 0 or 1 (empty slots add 0 to a spread-out counter), so
    // no branch per slot
    const bool o = rc[j] != 0;
    const uint32_t s = (uint32_t)j * TB + threadIdx.x;
    bk[j] = o ? (nbk_bits ? table.bits(rk[j], shift, nbk_bits) : 0u) : (s & (nbk - 1));
    rank[j] = atomicAdd(&aux[bk[j]], o ? 1u : 0u);
  }
  __syncthreads();
  const uint32_t d = block_exscan_array<TB>(aux, aux + nbk, (int)nbk, wsum, s_max);
  const uint32_t maxb = *s_max;
  const uint32_t* boff = aux + nbk;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (rc[j]) {
      const uint32_t p = boff[bk[j]] + rank[j];
      tk[p] = table.key(rk[j]);
      tc[p] = rc[j];
    }
  }
  __syncthreads();
  if (maxb <= kRankMax<K>) {
    for (uint32_t i = threadIdx.x; i < d; i += TB) {
      const K x = tk[i];
      const uint32_t b = nbk_bits ? Key<K>::bits(x, shift, nbk_bits) : 0u;
      const uint32_t a = boff[b], m = aux[b];
      uint32_t r = 0;
      uint32_t t = a;
      if constexpr (sizeof(K) <= 16)
      for (; t + 4 <= a + m; t += 4)
        r += (uint32_t)(tk[t] < x) + (uint32_t)(tk[t + 1] < x) + (uint32_t)(tk[t + 2] < x) +
             (uint32_t)(tk[t + 3] < x);
      for (; t < a + m; ++t) r += tk[t] < x;
      dst[begin + a + r] = x;
      tmp_cnt[begin + a + r] = tc[i];
    }
    return d;
  }
  const uint32_t n2 = next_pow2(d);
  for (uint32_t i = d + threadIdx.x; i < n2; i += TB) {
    tk[i] = ~(K)0;
    tc[i] = 0;
  }
  __syncthreads();
  bitonic_sort<K, uint32_t, TB>(tk, tc, n2);
  for (uint32_t i = threadIdx.x; i < d; i += TB) {
    dst[begin + i] = tk[i];
    tmp_cnt[begin + i] = tc[i];
  }
  return d;
}

// One-word leaf tables: the epilogue's counting sort uses Cn/8 groups (8 KiB
// of group counters for 4,096 slots instead of 32 KiB with Cn/2), so that
// three 512-thread workgroups, 24 waves, share a CU (53 KB of LDS each, and
// registers capped for 6 waves per SIMD: 79 VGPRs, no spills): 27.1 -> 25.7
// ms for the large leaves of 40,000,000 reads at k = 31, 23.8 -> 21.9 ms at
// k = 21, against two workgroups per CU.
constexpr int kLeafGroupShift = 3;
constexpr int kLeafOccTB = 512;
constexpr int kLeafOccWaves = 6;

// Up to this many leaves, all go to the block-wide kernel: a wave alone needs
// 15 us or more for a leaf (a chain of LDS latencies) while most of the chip
// is idle, and the block-wide kernel that follows as long again; five rounds
// of 768 resident workgroups count as many leaves in less (100 kB of reads:
// 119 us by one-wave workgroups, 13 us so).
constexpr uint64_t kFewLeaves = 4096;

// Tables whose slots hold the keys themselves, for the epilogue.
template <typename K> struct TableK {
  typedef K Ref;
  const K* tk;
  const uint32_t* tc;
  __device__ __forceinline__ void load(uint32_t s, Ref& r, uint32_t& c) const {
    r = tk[s];
    c = tc[s];
  }
  __device__ __forceinline__ uint32_t bits(const Ref& r, int shift, int nbits) const {
    return Key<K>::bits(r, shift, nbits);
  }
  __device__ __forceinline__ K key(const Ref& r) const { return r; }
};

// 64-bit keys: EMPTY (all ones) is never a canonical key for k <= 32, so a
// slot is claimed by a 64-bit CAS of the key word itself; the count is then
// added with an atomic add. REFINED only names the launches that count the
// parts of overflowed leaves apart.
// MERGED: some leaves may hold pre-aggregated records (Leaf::cshift); the
// plain instantiation has no decoding in its insert loop.
// list != nullptr: the leaves listed there, *n_list of them (large ones, or
// those whose table overflowed in an earlier launch), with the records and
// distinct keys of the leaves counted added to acc[0] and acc[1]; else every
// leaf of at most small_max records. ovf_list != nullptr: the leaves whose
// table overflows are also appended there (count in st->n_ovf) for a second
// launch with a larger table.
template <int TB, int CMAX, int R, bool REFINED, bool MERGED>
__global__ void __launch_bounds__(TB)
__attribute__((amdgpu_waves_per_eu(TB == kLeafOccTB ? kLeafOccWaves : 1)))
k_leaf_count64(int keybits, uint64_t* bufA, uint64_t* bufB,
                                                     uint32_t* __restrict__ tmp_cnt,
                                                     const Leaf* __restrict__ leaves,
                                                     DevState* __restrict__ st,
                                                     uint32_t* __restrict__ d_out,
                                                     int slots_log2,
                                                     const uint32_t* __restrict__ list,
                                                     const unsigned long long* __restrict__ n_list,
                                                     uint32_t* __restrict__ ovf_list,
                                                     unsigned long long* __restrict__ acc,
                                                     uint64_t small_max) {
  __shared__ unsigned long long tk[CMAX];
  __shared__ uint32_t tc[CMAX];
  __shared__ uint32_t aux[(2 * CMAX) >> kLeafGroupShift];
  __shared__ uint32_t wsum[TB / 64];
  __shared__ uint32_t s_nd, s_max, s_cov;
  __shared__ unsigned long long s_sum, s_windows;
  __shared__ uint32_t s_ovf;  // accessed only through ovf_get / ovf_set
  const unsigned long long EMPTY = ~0ull;
  const uint32_t cmax_rt = 1u << slots_log2;
  const unsigned long long count = list ? *n_list : st->n_leaves;
  unsigned long long my_records = 0, my_distinct = 0;  // thread 0: this workgroup's totals
  for (unsigned long long it = blockIdx.x; it < count; it += gridDim.x) {
    const unsigned long long l = list ? (unsigned long long)list[it] : it;
    const Leaf lf = leaves[l];
    const uint64_t n = lf.end - lf.begin;
    if (n == 0) {
      if (threadIdx.x == 0) d_out[l] = 0;
      continue;
    }
    if (!list && n > small_max) continue;
    const uint64_t* src = lf.buf ? bufB : bufA;
    uint64_t* dst = lf.buf ? bufA : bufB;
    // A table for all records being distinct (a first try with half of that,
    // counted again if it filled up, saves clearing and compacting slots but
    // lengthens the probe chains: large leaves of 1,000,000 reads at k = 31 0.74
    // against 0.68 ms, sized by the share of distinct records 1.01 ms). With few
    // leaves the chip is not full and a leaf's chain of latencies counts, not
    // its work: room to spare then.
    const bool few = TB != 64 && count <= kFewLeaves;
    const uint32_t Cn = leaf_slots<TB, CMAX>(few ? n + n / 2 : n, cmax_rt);
    // pre-aggregated records: (count - 1) in bits [cshift, 64), the shard above
    const uint32_t cshift = MERGED ? lf.cshift : 0u;
    const uint64_t low = cshift ? (1ull << cshift) - 1 : ~0ull;
    const uint64_t top = cshift ? (uint64_t)lf.shard << cshift : 0ull;
    unsigned long long my_windows = 0;  // this thread's share of the leaf's windows
    const uint32_t cmask = Cn - 1;
    const int slot_bits = 31 - __builtin_clz(Cn);
    for (uint32_t i = threadIdx.x; i < Cn; i += TB) {
      tk[i] = EMPTY;
      tc[i] = 0;
    }
    if (threadIdx.x == 0) {
      s_nd = 0;
      s_cov = 0;
      s_windows = 0;
      __hip_atomic_store(&s_ovf, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    const uint32_t limit = Cn - (Cn >> 3);
    const bool track = n >= limit;  // fewer records than the limit cannot overflow
    // new keys are counted per wave and batch, not one by one (a shared counter
    // takes its lanes one after the other), so a batch may fill the table past
    // its limit: a probe chain that only such a table has ends the attempt
    const uint32_t max_probes = track ? min(Cn, kMaxProbes) : Cn;
    // records are loaded R per thread before inserting, so that the loads of a
    // batch are in flight together instead of one round trip per insert. The
    // probe loop has a single exit flag (always-CAS: a CAS on a slot holding
    // another key just returns that key), which keeps divergent control flow,
    // and its scalar bookkeeping, small.
    for (uint64_t base = lf.begin; base < lf.end; base += (uint64_t)TB * R) {
      if (ovf_get(&s_ovf)) break;
      unsigned long long kb[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        kb[j] = r < lf.end ? src[r] : EMPTY;
      }
      // one probe loop over the thread's R records: a lane moves on to its
      // next record as soon as the current one is placed, so a wave runs
      // about as many iterations as its slowest lane's probes in total, not
      // the sum over the R records of the slowest lane's probes (records past
      // the leaf's end, EMPTY, come last)
      unsigned long long key = EMPTY;
      uint32_t cnt = 1, pos = 0, left = 64, rounds = 0, claims = 0;  // of 64 probes each
      int j = 0;
      auto take = [&](unsigned long long x) {
        key = x;
        cnt = 1;
        if constexpr (MERGED) {
          if (cshift) {  // uniform per leaf
            cnt = (uint32_t)(x >> cshift) + 1u;
            key = top | (x & low);
            my_windows += cnt;
          }
        }
        pos = slot_hash(key, slot_bits);
        left = 64;
        rounds = 0;
      };
      bool todo = kb[0] != EMPTY;
      if (todo) take(kb[0]);
      while (todo) {
        const unsigned long long prev = atomicCAS(&tk[pos], EMPTY, key);
        const bool hit = (prev == EMPTY) | (prev == key);
        if (hit) {
          atomicAdd(&tc[pos], cnt);
          claims += prev == EMPTY ? 1u : 0u;
          ++j;
          unsigned long long nx = EMPTY;
#pragma unroll
          for (int q = 1; q < R; ++q)
            if (j == q) nx = kb[q];
          todo = nx != EMPTY;
          if (todo) take(nx);
        } else {
          pos = (pos + 1) & cmask;
          if (--left == 0) {
            // table full: the leaf overflows (or does already)
            left = 64;
            todo = ++rounds < max_probes / 64 && !ovf_get(&s_ovf);
            if (!todo) ovf_set(&s_ovf);
          }
        }
      }
      if (track) {
        // (summed by ballots of its bits: shuffles, six LDS operations in a chain,
        // made inputs of few distinct keys 4% slower, 10 MB of A 14.0 -> 14.6
        // ms; so 13.7, and 20,000,000 reads at k = 31 41.1 -> 40.7)
        uint32_t fresh = 0;
#pragma unroll
        for (int b = 0; (1 << b) <= R; ++b)
          fresh += (uint32_t)__popcll(__ballot(claims >> b & 1)) << b;
        if ((threadIdx.x & 63) == 0 && fresh && atomicAdd(&s_nd, fresh) + fresh >= limit)
          ovf_set(&s_ovf);
      }
    }
    __syncthreads();
    if (ovf_get(&s_ovf)) {
      if (threadIdx.x == 0) {
        d_out[l] = kLeafOverflow;
        // (st->overflow is raised from the leaf counts by the output-offset scan)
        if (ovf_list) ovf_list[atomicAdd(&st->n_ovf, 1ull)] = (uint32_t)l;
      }
      __syncthreads();
      continue;
    }
    // windows of the leaf: its records, or the sum of pre-aggregated counts
    unsigned long long windows = n;
    if (MERGED && cshift) {
      if (my_windows) atomicAdd(&s_windows, my_windows);
      __syncthreads();
      windows = s_windows;
    }
    if (windows > 0xFFFFFFFFull) {
      // a leaf of 2^32 windows or more may hold a count that wrapped past 32
      // bits; the counts then sum to less than the windows
      if (threadIdx.x == 0) s_sum = 0;
      __syncthreads();
      unsigned long long part = 0;
      for (uint32_t i = threadIdx.x; i < Cn; i += TB) part += tc[i];
      atomicAdd(&s_sum, part);
      __syncthreads();
      if (threadIdx.x == 0 && s_sum != windows) s_cov = 1;
    }
    const uint32_t d = leaf_sort_write<unsigned long long, TB, CMAX / TB, kLeafGroupShift>(
        tk, tc, aux, wsum, &s_max, Cn, keybits, (int)lf.bits, (unsigned long long*)dst, tmp_cnt,
        lf.begin, TableK<unsigned long long>{tk, tc});
    if (threadIdx.x == 0) {
      d_out[l] = d;
      if (s_cov) atomicOr(&st->count_overflow, 1u);
      my_records += n;
      my_distinct += d;
    }
    __syncthreads();
  }
  // one update of the shared totals per workgroup (not per leaf: same-address
  // atomics from every workgroup would serialise)
  if (TB != 64 && threadIdx.x == 0 && my_records) {
    atomicAdd(&acc[0], my_records);
    atomicAdd(&acc[1], my_distinct);
  }
}

// Hashes of the wider keys.
template <typename K> struct Hash2 {
  uint32_t pos, tag;  // independent hashes of a key
  __device__ __forceinline__ explicit Hash2(const K& key) {
    // multilinear in the key's 32-bit words (Dietzfelbinger): two sums of
    // words times odd constants, each finished by a multiply-shift. The constants
    // are the first words of pi's binary fraction, made odd.
    constexpr uint32_t c[16] = {0x243F6A89u, 0x85A308D3u, 0x13198A2Fu, 0x03707345u,
                                0xA4093823u, 0x299F31D1u, 0x082EFA99u, 0xEC4E6C89u,
                                0x452821E7u, 0x38D01377u, 0xBE5466CFu, 0x34E90C6Du,
                                0xC0AC29B7u, 0xC97C50DDu, 0x3F84D5B5u, 0xB5470917u};
    uint32_t w[2 * Key<K>::kWords];
    __builtin_memcpy(w, &key, sizeof(K));
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int i = 0; i < 2 * Key<K>::kWords; ++i) {
      a += w[i] * c[i];
      b += (w[i] ^ (w[i] >> 16)) * c[8 + i];
    }
    pos = (a ^ (a >> 15)) * 0x9216D5D9u;
    tag = (b ^ (b >> 15)) * 0x8979FB1Bu;
  }
};

// 128-bit keys of k <= 63: there is no 128-bit CAS, but the high word of a key
// is then never all ones, so a slot is claimed by a CAS of its high word (all
// ones = empty); the claimer writes the low word and publishes it with the
// count (release). A lane that finds its high word in a slot whose count is
// still 0 waits for that publication (made in the claimer's same pass), then
// compares the low word. list, n_list, ovf_list and acc as for one-word keys.
// (By a 32-bit tag and the keys compared after a barrier: 1.11 against 0.95 ms
// for the large leaves of 60 MB of 10 kbp reads at k = 55.)
template <int TB, int CMAX, int R, bool REFINED>
__global__ void __launch_bounds__(TB)
__attribute__((amdgpu_waves_per_eu(TB == kLeafOccTB ? kLeafOccWaves : 1)))
k_leaf_count128(int keybits, u128* bufA, u128* bufB, uint32_t* __restrict__ tmp_cnt,
                const Leaf* __restrict__ leaves, DevState* __restrict__ st,
                uint32_t* __restrict__ d_out, int slots_log2, const uint32_t* __restrict__ list,
                const unsigned long long* __restrict__ n_list, uint32_t* __restrict__ ovf_list,
                unsigned long long* __restrict__ acc, uint64_t small_max) {
  __shared__ u128 tk[CMAX];
  __shared__ uint32_t tc[CMAX];
  __shared__ uint32_t aux[CMAX];
  __shared__ uint32_t wsum[TB / 64];
  __shared__ uint32_t s_nd, s_max, s_cov;
  __shared__ unsigned long long s_sum;
  __shared__ uint32_t s_ovf;  // accessed only through ovf_get / ovf_set
  const uint32_t cmax_rt = 1u << slots_log2;
  const unsigned long long count = list ? *n_list : st->n_leaves;
  unsigned long long my_records = 0, my_distinct = 0;  // thread 0: this workgroup's totals
  for (unsigned long long it = blockIdx.x; it < count; it += gridDim.x) {
    const unsigned long long l = list ? (unsigned long long)list[it] : it;
    const Leaf lf = leaves[l];
    const uint64_t n = lf.end - lf.begin;
    if (n == 0) {
      if (threadIdx.x == 0) d_out[l] = 0;
      continue;
    }
    if (!list && n > small_max) continue;
    const u128* src = lf.buf ? bufB : bufA;
    u128* dst = lf.buf ? bufA : bufB;
    const bool few = TB != 64 && count <= kFewLeaves;
    const uint32_t Cn = leaf_slots<TB, CMAX>(few ? n + n / 2 : n, cmax_rt);
    const uint32_t cmask = Cn - 1;
    const int slot_bits = 31 - __builtin_clz(Cn);
    for (uint32_t i = threadIdx.x; i < Cn; i += TB) {
      tc[i] = 0;
      reinterpret_cast<unsigned long long*>(&tk[i])[1] = ~0ull;
    }
    if (threadIdx.x == 0) {
      s_nd = 0;
      __hip_atomic_store(&s_ovf, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      s_cov = 0;
    }
    __syncthreads();
    const uint32_t limit = Cn - (Cn >> 3);
    const bool track = n >= limit;  // fewer records than the limit cannot overflow
    const uint32_t max_probes = track ? min(Cn, kMaxProbes) : Cn;
    for (uint64_t base = lf.begin; base < lf.end; base += (uint64_t)TB * R) {
      if (ovf_get(&s_ovf)) break;
      u128 kb[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        kb[j] = r < lf.end ? src[r] : ~(u128)0;  // never a key: its high word is all ones
      }
      // one probe loop over the thread's R records, as for one-word keys
      u128 key = 0;
      uint32_t pos = 0, left = 64, rounds = 0, spins = 0;  // of 64 probes each
      int j = 0;
      const auto take = [&](const u128& x) {
        key = x;
        pos = Hash2<u128>(x).pos >> (32 - slot_bits);
        left = 64;
        rounds = 0;
      };
      bool todo = (unsigned long long)(kb[0] >> 64) != ~0ull;
      if (todo) take(kb[0]);
      while (todo) {
        unsigned long long* const w = reinterpret_cast<unsigned long long*>(&tk[pos]);
        const unsigned long long khi = (unsigned long long)(key >> 64);
        const unsigned long long klo = (unsigned long long)key;
        const unsigned long long prev = atomicCAS(&w[1], ~0ull, khi);
        bool hit = false, wait = false;
        if (prev == ~0ull) {
          w[0] = klo;
          __hip_atomic_store(&tc[pos], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (track && atomicAdd(&s_nd, 1u) + 1 >= limit) ovf_set(&s_ovf);
          hit = true;
        } else if (prev == khi) {
          const uint32_t c =
              __hip_atomic_load(&tc[pos], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (c == 0) {
            // the bound only guards against a hang; giving up marks the leaf
            // overflowed, so it is counted again
            wait = ++spins <= (1u << 22);
            if (!wait) {
              left = 1;
              rounds = max_probes / 64;
            }
          } else if (w[0] == klo) {
            __hip_atomic_fetch_add(&tc[pos], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            hit = true;
          }
        }
        if (hit) {
          ++j;
          u128 nx = ~(u128)0;
#pragma unroll
          for (int q = 1; q < R; ++q)
            if (j == q) nx = kb[q];
          todo = (unsigned long long)(nx >> 64) != ~0ull;
          if (todo) take(nx);
        } else if (!wait) {
          pos = (pos + 1) & cmask;
          if (--left == 0) {
            left = 64;
            todo = ++rounds < max_probes / 64 && !ovf_get(&s_ovf);
            if (!todo) ovf_set(&s_ovf);
          }
        }
      }
    }
    __syncthreads();
    if (ovf_get(&s_ovf)) {
      if (threadIdx.x == 0) {
        d_out[l] = kLeafOverflow;
        // (st->overflow is raised from the leaf counts by the output-offset scan)
        if (ovf_list) ovf_list[atomicAdd(&st->n_ovf, 1ull)] = (uint32_t)l;
      }
      __syncthreads();
      continue;
    }
    if (n > 0xFFFFFFFFull) {
      // 32-bit counts may have wrapped: they then sum to less than the records
      if (threadIdx.x == 0) s_sum = 0;
      __syncthreads();
      unsigned long long part = 0;
      for (uint32_t i = threadIdx.x; i < Cn; i += TB) part += tc[i];
      atomicAdd(&s_sum, part);
      __syncthreads();
      if (threadIdx.x == 0 && s_sum != n) s_cov = 1;
    }
    const uint32_t d = leaf_sort_write<u128, TB, CMAX / TB, 1>(
        tk, tc, aux, wsum, &s_max, Cn, keybits, (int)lf.bits, dst, tmp_cnt, lf.begin,
        TableK<u128>{tk, tc});
    if (threadIdx.x == 0) {
      d_out[l] = d;
      if (s_cov) atomicOr(&st->count_overflow, 1u);
      my_records += n;
      my_distinct += d;
    }
    __syncthreads();
  }
  if (TB != 64 && threadIdx.x == 0 && my_records) {
    atomicAdd(&acc[0], my_records);
    atomicAdd(&acc[1], my_distinct);
  }
}

// Keys of k >= 64: a slot holds where its key is, not the key: a 24-bit tag of the key's hash above the 40-bit number of the record
// that claimed it (all ones: empty), claimed by one 64-bit CAS. A record that
// meets its own tag compares its key with the claimer's, read from the leaf's
// records (which nothing writes here, so there is nothing to wait for), and
// counts in that slot if they are equal (else, one time in 2^24, it probes on).
// The R records of a thread are placed first, by tags alone, then all their
// claimers' keys are loaded together and compared. A slot takes 12 bytes of LDS
// instead of 20 to 40 (key and count), and the keys of the distinct records are
// brought to LDS only for the sort, where the slots were: two (four-word keys)
// and three workgroups share a CU. 1,000,000 reads of 150 bases at k = 100:
// large leaves 6.96 -> 2.8 ms (keys in the slots, claimed through a lock in the
// count word, one workgroup per CU; a bound is the latency of a leaf's chain of
// steps: about 1,100 records, 0.9 of them distinct).
// As for one-word keys, a leaf whose table overflows is listed for a
// second launch with one twice as large (ovf_list, n_list, acc as there).
// REFINED only names the launches that count refined parts apart.
constexpr int kWideGroupShift = 2;  // Cn/4 groups in the epilogue's counting sort

// Their tables for the epilogue: the slot's record holds the key, read once for
// its group bits and once for the key (a thread holding four keys of four
// words in between would spill).
constexpr int kIdxBits = 40;
constexpr unsigned long long kIdx = (1ull << kIdxBits) - 1;
template <typename K> struct TableW {
  typedef unsigned long long Ref;
  const unsigned long long* slot;
  const uint32_t* tc;
  const K* src;
  __device__ __forceinline__ void load(uint32_t s, Ref& r, uint32_t& c) const {
    r = slot[s] & kIdx;
    c = tc[s];
  }
  __device__ __forceinline__ uint32_t bits(Ref r, int shift, int nbits) const {
    const uint64_t* w = reinterpret_cast<const uint64_t*>(src + r) + (shift >> 6);
    const int off = shift & 63;
    uint64_t v = w[0] >> off;
    if (off + nbits > 64) v |= w[1] << (64 - off);
    return (uint32_t)v & ((1u << nbits) - 1u);
  }
  __device__ __forceinline__ K key(Ref r) const { return src[r]; }
};

template <typename K, int TB, int CMAX, int R>
__device__ __forceinline__ void leaf_countw_body(
    int keybits, K* bufA, K* bufB, uint32_t* __restrict__ tmp_cnt, const Leaf* __restrict__ leaves,
    DevState* __restrict__ st, uint32_t* __restrict__ d_out, int slots_log2,
    const uint32_t* __restrict__ list, const unsigned long long* __restrict__ n_list,
    uint32_t* __restrict__ ovf_list, unsigned long long* __restrict__ acc, uint64_t small_max) {
  __shared__ __align__(16) unsigned char raw[CMAX * sizeof(K)];  // slots, then sorted keys
  __shared__ uint32_t tc[CMAX];
  __shared__ uint32_t aux[(2 * CMAX) >> kWideGroupShift];
  __shared__ uint32_t wsum[TB / 64];
  __shared__ uint32_t s_nd, s_max, s_cov;
  __shared__ unsigned long long s_sum;
  __shared__ uint32_t s_ovf;  // accessed only through ovf_get / ovf_set
  unsigned long long* const slot = reinterpret_cast<unsigned long long*>(raw);
  const unsigned long long EMPTY = ~0ull;
  const uint32_t cmax_rt = 1u << slots_log2;
  const unsigned long long count = list ? *n_list : st->n_leaves;
  unsigned long long my_records = 0, my_distinct = 0;  // thread 0: this workgroup's totals
  for (unsigned long long it = blockIdx.x; it < count; it += gridDim.x) {
    const unsigned long long l = list ? (unsigned long long)list[it] : it;
    const Leaf lf = leaves[l];
    const uint64_t n = lf.end - lf.begin;
    if (n == 0) {
      if (threadIdx.x == 0) d_out[l] = 0;
      continue;
    }
    if (!list && n > small_max) continue;
    const K* __restrict__ src = (lf.buf ? bufB : bufA) + lf.begin;
    K* const dst = lf.buf ? bufA : bufB;
    const bool few = TB != 64 && count <= kFewLeaves;
    const uint32_t Cn = leaf_slots<TB, CMAX>(few ? n + n / 2 : n, cmax_rt);
    const uint32_t cmask = Cn - 1;
    const int slot_bits = 31 - __builtin_clz(Cn);
    for (uint32_t i = threadIdx.x; i < Cn; i += TB) {
      slot[i] = EMPTY;
      tc[i] = 0;
    }
    if (threadIdx.x == 0) {
      s_nd = 0;
      __hip_atomic_store(&s_ovf, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      s_cov = 0;
    }
    __syncthreads();
    const uint32_t limit = Cn - (Cn >> 3);
    const bool track = n >= limit;  // fewer records than the limit cannot overflow
    const uint32_t max_probes = track ? min(Cn, kMaxProbes) : Cn;
    // What a slot held before it was claimed for x. The second count looks first
    // (a slot claimed once never changes) in leaves of many records to a slot, so
    // of few keys: lanes that CAS one word take turns, but read it at once (10 MB
    // of A at k = 100 6.09 -> 5.09 ms; everywhere, 20 MB of A and T 3.47 -> 3.58).
    const bool look = TB > kLeafOccTB && n > 8ull * Cn;
    const auto claim = [&](unsigned long long* w, unsigned long long x) {
      unsigned long long v = EMPTY;
      if (look) v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      return v != EMPTY ? v : (unsigned long long)atomicCAS(w, EMPTY, x);
    };
    for (uint64_t base = 0; base < n; base += (uint64_t)TB * R) {
      if (ovf_get(&s_ovf)) break;
      K kb[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        if (r < n) kb[j] = src[r];
      }
      // a slot each, by tags: EMPTY = claimed, else what the slot held
      uint32_t pos[R], tag[R], probes[R];
      unsigned long long held[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        const Hash2<K> h(kb[j]);
        pos[j] = h.pos >> (32 - slot_bits);
        tag[j] = h.tag >> 8;
        probes[j] = 0;
        held[j] = EMPTY;
        bool todo = r < n;
        while (todo) {
          const unsigned long long prev =
              claim(&slot[pos[j]], (unsigned long long)tag[j] << kIdxBits | r);
          held[j] = prev;
          todo = prev != EMPTY && (uint32_t)(prev >> kIdxBits) != tag[j];
          if (todo) {
            pos[j] = (pos[j] + 1) & cmask;
            if ((++probes[j] & 63) == 0 && (probes[j] >= max_probes || ovf_get(&s_ovf))) {
              ovf_set(&s_ovf);  // table full: the leaf overflows
              probes[j] = Cn;
              todo = false;
            }
          }
        }
      }
      K kc[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        if (r < n && held[j] != EMPTY) kc[j] = src[held[j] & kIdx];
      }
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint64_t r = base + (uint64_t)j * TB + threadIdx.x;
        if (r >= n || probes[j] >= Cn) continue;
        bool fresh = held[j] == EMPTY;
        if (!fresh && kc[j] != kb[j]) {
          // another key with this tag: probe on, comparing at once
          bool todo = true;
          while (todo) {
            pos[j] = (pos[j] + 1) & cmask;
            if ((++probes[j] & 63) == 0 && (probes[j] >= max_probes || ovf_get(&s_ovf))) {
              probes[j] = Cn;
              break;
            }
            const unsigned long long prev =
                claim(&slot[pos[j]], (unsigned long long)tag[j] << kIdxBits | r);
            fresh = prev == EMPTY;
            todo = !fresh &&
                   !((uint32_t)(prev >> kIdxBits) == tag[j] && src[prev & kIdx] == kb[j]);
          }
          if (probes[j] >= Cn) {
            ovf_set(&s_ovf);
            continue;
          }
        }
        atomicAdd(&tc[pos[j]], 1u);
        if (track && fresh && atomicAdd(&s_nd, 1u) + 1 >= limit) ovf_set(&s_ovf);
      }
    }
    __syncthreads();
    if (ovf_get(&s_ovf)) {
      if (threadIdx.x == 0) {
        d_out[l] = kLeafOverflow;
        // (st->overflow is raised from the leaf counts by the output-offset scan)
        if (ovf_list) ovf_list[atomicAdd(&st->n_ovf, 1ull)] = (uint32_t)l;
      }
      __syncthreads();
      continue;
    }
    if (n > 0xFFFFFFFFull) {
      // 32-bit counts may have wrapped: they then sum to less than the records
      if (threadIdx.x == 0) s_sum = 0;
      __syncthreads();
      unsigned long long part = 0;
      for (uint32_t i = threadIdx.x; i < Cn; i += TB) part += tc[i];
      atomicAdd(&s_sum, part);
      __syncthreads();
      if (threadIdx.x == 0 && s_sum != n) s_cov = 1;
    }
    const uint32_t d = leaf_sort_write<K, TB, CMAX / TB, kWideGroupShift>(
        reinterpret_cast<K*>(raw), tc, aux, wsum, &s_max, Cn, keybits, (int)lf.bits, dst, tmp_cnt,
        lf.begin, TableW<K>{slot, tc, src});
    if (threadIdx.x == 0) {
      d_out[l] = d;
      if (s_cov) atomicOr(&st->count_overflow, 1u);
      my_records += n;
      my_distinct += d;
    }
    __syncthreads();
  }
  if (TB != 64 && threadIdx.x == 0 && my_records) {
    atomicAdd(&acc[0], my_records);
    atomicAdd(&acc[1], my_distinct);
  }
}

template <int TB, int CMAX, int R, bool REFINED>
__global__ void __launch_bounds__(TB)
__attribute__((amdgpu_waves_per_eu(TB == kLeafOccTB ? 4 : 1)))
k_leaf_countw128(int keybits, u128* bufA, u128* bufB, uint32_t* __restrict__ tmp_cnt,
                 const Leaf* __restrict__ leaves, DevState* __restrict__ st,
                 uint32_t* __restrict__ d_out, int slots_log2, const uint32_t* __restrict__ list,
                 const unsigned long long* __restrict__ n_list, uint32_t* __restrict__ ovf_list,
                 unsigned long long* __restrict__ acc, uint64_t small_max) {
  leaf_countw_body<u128, TB, CMAX, R>(keybits, bufA, bufB, tmp_cnt, leaves, st, d_out, slots_log2,
                                      list, n_list, ovf_list, acc, small_max);
}

template <int TB, int CMAX, int R, bool REFINED>
__global__ void __launch_bounds__(TB)
__attribute__((amdgpu_waves_per_eu(TB == kLeafOccTB ? 4 : 1)))
k_leaf_countw256(int keybits, u256* bufA, u256* bufB, uint32_t* __restrict__ tmp_cnt,
                 const Leaf* __restrict__ leaves, DevState* __restrict__ st,
                 uint32_t* __restrict__ d_out, int slots_log2, const uint32_t* __restrict__ list,
                 const unsigned long long* __restrict__ n_list, uint32_t* __restrict__ ovf_list,
                 unsigned long long* __restrict__ acc, uint64_t small_max) {
  leaf_countw_body<u256, TB, CMAX, R>(keybits, bufA, bufB, tmp_cnt, leaves, st, d_out, slots_log2,
                                      list, n_list, ovf_list, acc, small_max);
}

// ---------------------------------------------------------------- sort-based leaf count

// The paper's own way to count an owner's k-mers (counting by sorting, as in
// Algorithm 1 and by every owner in Algorithm 3), applied to a leaf: its
// records are sorted in LDS and each run of equal keys becomes one pair. A
// leaf of more records than fit is marked overflowed and cut further by key
// (refinement); a leaf whose key range is a single key is counted without
// sorting.
template <typename K, int TB>
__device__ __forceinline__ void bitonic_keys(K* keys, uint32_t n) {
  for (uint32_t size = 2; size <= n; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < n / 2; i += TB) {
        const uint32_t lo = (i / stride) * stride * 2 + (i % stride);
        const uint32_t hi = lo + stride;
        const bool asc = (lo & size) == 0;
        const K a = keys[lo], b = keys[hi];
        if ((a > b) == asc) {
          keys[lo] = b;
          keys[hi] = a;
        }
      }
      __syncthreads();
    }
  }
}

template <typename K, int TB, int SMAX>
__global__ void __launch_bounds__(TB) k_leaf_sort(int keybits, K* bufA, K* bufB,
                                                  uint32_t* __restrict__ tmp_cnt,
                                                  const Leaf* __restrict__ leaves,
                                                  DevState* __restrict__ st,
                                                  uint32_t* __restrict__ d_out,
                                                  const uint32_t* __restrict__ list) {
  __shared__ K sk[SMAX];
  __shared__ uint32_t sp[SMAX + 1];  // positions of the run starts, then n
  __shared__ uint32_t wsum[TB / 64];
  const unsigned long long count = st->n_large;
  unsigned long long my_records = 0, my_distinct = 0;
  for (unsigned long long it = blockIdx.x; it < count; it += gridDim.x) {
    const uint32_t l = list[it];
    const Leaf lf = leaves[l];
    const uint64_t n = lf.end - lf.begin;
    const K* src = lf.buf ? bufB : bufA;
    K* dst = lf.buf ? bufA : bufB;
    if ((int)lf.bits >= keybits) {  // the leaf's range is one key
      if (threadIdx.x == 0) {
        dst[lf.begin] = src[lf.begin];
        tmp_cnt[lf.begin] = (uint32_t)n;
        if (n > 0xFFFFFFFFull) atomicOr(&st->count_overflow, 1u);
        d_out[l] = 1;
        my_records += n;
        my_distinct += 1;
      }
      continue;
    }
    if (n > SMAX) {
      if (threadIdx.x == 0) {
        d_out[l] = kLeafOverflow;
        atomicOr(&st->overflow, 1u);
      }
      continue;
    }
    const uint32_t m = (uint32_t)n;
    const uint32_t n2 = next_pow2(m);
    for (uint32_t i = threadIdx.x; i < n2; i += TB) sk[i] = i < m ? src[lf.begin + i] : ~(K)0;
    __syncthreads();
    bitonic_keys<K, TB>(sk, n2);
    // run starts: thread t looks at positions [t*per, t*per + per)
    const uint32_t per = (m + TB - 1) / TB;
    const uint32_t b = threadIdx.x * per, e = min(m, b + per);
    uint32_t c = 0;
    for (uint32_t i = b; i < e; ++i) c += (i == 0 || sk[i] != sk[i - 1]) ? 1u : 0u;
    uint32_t d = 0;
    uint32_t at = block_exscan<TB, uint32_t>(c, wsum, &d);
    for (uint32_t i = b; i < e; ++i)
      if (i == 0 || sk[i] != sk[i - 1]) sp[at++] = i;
    if (threadIdx.x == 0) sp[d] = m;
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < d; q += TB) {
      const uint32_t i = sp[q];
      dst[lf.begin + q] = sk[i];
      tmp_cnt[lf.begin + q] = sp[q + 1] - i;
    }
    if (threadIdx.x == 0) {
      d_out[l] = d;
      my_records += n;
      my_distinct += d;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && my_records) {
    atomicAdd(&st->large_records, my_records);
    atomicAdd(&st->large_distinct, my_distinct);
  }
}

// Lanes of this wave whose digit d (nb bits) equals this lane's, among the
// lanes with v set (ballots over the digit's bits).
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool v, int nb) {
  uint64_t m = __ballot(v);
  for (int bit = 0; bit < nb; ++bit) {
    const bool on = (d >> bit) & 1u;
    const uint64_t set = __ballot(v && on);
    m &= on ? set : ~set;
  }
  return m;
}

// Stable LSD radix sort in LDS of n one-word keys (and their counts) by bits
// [0, nbits), 8-bit digits. Per pass, wave w walks its contiguous chunk of
// the elements 64 at a time: lanes holding the same digit find each other by
// ballots, so each digit's count per wave and each element's rank among the
// wave's equal digits come without atomics; a block scan of the counts in
// digit-major order gives every (digit, wave) its first position, and a
// second walk places the elements there in order (stable). Ping-pong between
// (ka, ca) and (kb, cb); returns true if the result ended in (kb, cb).
template <int TB>
__device__ bool lds_radix_sort64(uint64_t* ka, uint32_t* ca, uint64_t* kb, uint32_t* cb,
                                 uint32_t n, int nbits, uint32_t* whist, uint32_t* wsum) {
  constexpr int NW = TB / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t chunk = (n + NW - 1) / NW;
  const uint32_t c0 = min(n, (uint32_t)w * chunk), c1 = min(n, c0 + chunk);
  const uint64_t below = (1ull << lane) - 1;
  bool flipped = false;
  for (int shift = 0; shift < nbits; shift += 8) {
    const int nb = min(8, nbits - shift);
    for (int i = threadIdx.x; i < 256 * NW; i += TB) whist[i] = 0;
    __syncthreads();
    for (uint32_t r0 = c0; r0 < c1; r0 += 64) {
      const uint32_t i = r0 + lane;
      const bool v = i < c1;
      const uint32_t d = v ? (uint32_t)(ka[i] >> shift) & ((1u << nb) - 1u) : 0u;
      const uint64_t peers = digit_peers(d, v, nb);
      if (v && lane == __ffsll((long long)peers) - 1) whist[d * NW + w] += __popcll(peers);
    }
    __syncthreads();
    (void)block_exscan_inplace<TB>(whist, 256 * NW, wsum);
    for (uint32_t r0 = c0; r0 < c1; r0 += 64) {
      const uint32_t i = r0 + lane;
      const bool v = i < c1;
      const uint64_t key = v ? ka[i] : 0ull;
      const uint32_t d = (uint32_t)(key >> shift) & ((1u << nb) - 1u);
      const uint64_t peers = digit_peers(d, v, nb);
      if (v) {
        const uint32_t pos = whist[d * NW + w] + (uint32_t)__popcll(peers & below);
        kb[pos] = key;
        cb[pos] = ca[i];
      }
      // every lane has read its digit's base before the leader advances it
      if (v && lane == __ffsll((long long)peers) - 1) whist[d * NW + w] += __popcll(peers);
    }
    __syncthreads();
    uint64_t* tk = ka;
    ka = kb;
    kb = tk;
    uint32_t* tc = ca;
    ca = cb;
    cb = tc;
    flipped = !flipped;
  }
  return flipped;
}

// The paper's counting step on one-word keys, with a radix sort: a leaf's
// records (up to SMAX; pre-aggregated ones carry their counts) are loaded into
// LDS, radix-sorted by the key bits below the leaf's common prefix, and each
// run of equal keys becomes one pair whose count is the sum of its records'
// counts (the Sort and Accumulate of Algorithm 1, run by each owner in
// Algorithm 3, on records shaped like the HEAVY (k-mer, count) and NORMAL
// (k-mer) messages of Section IV-D). A larger leaf is marked overflowed and cut
// further by key; a leaf whose range is one key is summed without sorting.
template <int TB, int SMAX>
__global__ void __launch_bounds__(TB) k_leaf_radix64(int keybits, uint64_t* bufA, uint64_t* bufB,
                                                     uint32_t* __restrict__ tmp_cnt,
                                                     const Leaf* __restrict__ leaves,
                                                     DevState* __restrict__ st,
                                                     uint32_t* __restrict__ d_out,
                                                     const uint32_t* __restrict__ list) {
  __shared__ uint64_t ka[SMAX], kb[SMAX];
  __shared__ uint32_t ca[SMAX], cb[SMAX];
  __shared__ uint32_t sp[SMAX + 1];  // run starts; then their count prefix sums
  __shared__ uint32_t whist[256 * (TB / 64)];
  __shared__ uint32_t wsum[TB / 64];
  __shared__ unsigned long long s_sum;
  const unsigned long long count = st->n_large;
  unsigned long long my_records = 0, my_distinct = 0;
  for (unsigned long long it = blockIdx.x; it < count; it += gridDim.x) {
    const uint32_t l = list[it];
    const Leaf lf = leaves[l];
    const uint64_t n = lf.end - lf.begin;
    const uint64_t* src = lf.buf ? bufB : bufA;
    uint64_t* dst = lf.buf ? bufA : bufB;
    const uint32_t cshift = lf.cshift;
    const uint64_t low = cshift ? (1ull << cshift) - 1 : ~0ull;
    const uint64_t top = cshift ? (uint64_t)lf.shard << cshift : 0ull;
    if ((int)lf.bits >= keybits) {  // the leaf's range is one key: sum its records' counts
      if (threadIdx.x == 0) s_sum = 0;
      __syncthreads();
      unsigned long long part = 0;
      for (uint64_t r = lf.begin + threadIdx.x; r < lf.end; r += TB)
        part += cshift ? (src[r] >> cshift) + 1 : 1;
      if (part) atomicAdd(&s_sum, part);
      __syncthreads();
      if (threadIdx.x == 0) {
        const uint64_t w0 = src[lf.begin];
        dst[lf.begin] = cshift ? top | (w0 & low) : w0;
        tmp_cnt[lf.begin] = (uint32_t)s_sum;
        if (s_sum > 0xFFFFFFFFull) atomicOr(&st->count_overflow, 1u);
        d_out[l] = 1;
        my_records += n;
        my_distinct += 1;
      }
      __syncthreads();
      continue;
    }
    if (n > SMAX) {
      if (threadIdx.x == 0) {
        d_out[l] = kLeafOverflow;
        atomicOr(&st->overflow, 1u);
      }
      continue;
    }
    const uint32_t m = (uint32_t)n;
    for (uint32_t i = threadIdx.x; i < m; i += TB) {
      const uint64_t x = src[lf.begin + i];
      ka[i] = cshift ? top | (x & low) : x;
      ca[i] = cshift ? (uint32_t)(x >> cshift) + 1u : 1u;
    }
    __syncthreads();
    const bool in_b = lds_radix_sort64<TB>(ka, ca, kb, cb, m, keybits - (int)lf.bits, whist, wsum);
    const uint64_t* sk = in_b ? kb : ka;
    uint32_t* sc = in_b ? cb : ca;
    // run starts: thread t looks at positions [t*per, t*per + per)
    const uint32_t per = (m + TB - 1) / TB;
    const uint32_t b = threadIdx.x * per, e = min(m, b + per);
    uint32_t c = 0;
    for (uint32_t i = b; i < e; ++i) c += (i == 0 || sk[i] != sk[i - 1]) ? 1u : 0u;
    uint32_t d = 0;
    uint32_t at = block_exscan<TB, uint32_t>(c, wsum, &d);
    for (uint32_t i = b; i < e; ++i)
      if (i == 0 || sk[i] != sk[i - 1]) sp[at++] = i;
    if (threadIdx.x == 0) sp[d] = m;
    __syncthreads();
    // counts of the runs: exclusive prefix sums of the sorted records' counts
    const uint32_t all = block_exscan_inplace<TB>(sc, m, wsum);
    for (uint32_t q = threadIdx.x; q < d; q += TB) {
      const uint32_t i = sp[q], j = sp[q + 1];
      dst[lf.begin + q] = sk[i];
      tmp_cnt[lf.begin + q] = (j < m ? sc[j] : all) - sc[i];
    }
    if (threadIdx.x == 0) {
      d_out[l] = d;
      my_records += n;
      my_distinct += d;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && my_records) {
    atomicAdd(&st->large_records, my_records);
    atomicAdd(&st->large_distinct, my_distinct);
  }
}

// ---------------------------------------------------------------- concat + check

// Output offsets within the concat: the leaf counts of up to kFewLeaves leaves
// are summed by every workgroup for itself (4 loads a thread in flight, from
// L2) instead of by a launch before it, which took 7 us and the gap of a launch
// (5 us) for as many leaves: this launch 4.5 instead of 6.0 us for 667 reads,
// 7.7 instead of 13.2 for 40,001 trimmed ones. Returns the output place of leaf l0, the workgroup's
// first; ovf: a leaf overflowed. The first workgroup leaves the totals in st
// and copies the state to pub.
__device__ __forceinline__ unsigned long long leaf_prefix(const uint32_t* __restrict__ d,
                                                          uint32_t n, uint32_t l0, DevState* st,
                                                          DevState* pub, bool& ovf) {
  __shared__ unsigned long long s_below[4], s_all[4];
  __shared__ uint32_t s_ovf;
  if (threadIdx.x == 0) s_ovf = 0;
  __syncthreads();
  unsigned long long below = 0, all = 0;
  bool o = false;
  constexpr uint32_t U = 4;
  for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 256 * U) {
    uint32_t v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) v[u] = i0 + u * 256 < n ? d[i0 + u * 256] : 0u;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      o |= v[u] == kLeafOverflow;
      if (v[u] == kLeafOverflow) v[u] = 0;
      all += v[u];
      if (i0 + u * 256 < l0) below += v[u];
    }
  }
  for (int m = 32; m > 0; m >>= 1) {
    below += __shfl_xor(below, m);
    all += __shfl_xor(all, m);
  }
  if ((threadIdx.x & 63) == 0) {
    s_below[threadIdx.x >> 6] = below;
    s_all[threadIdx.x >> 6] = all;
  }
  if (o) atomicOr(&s_ovf, 1u);
  __syncthreads();
  ovf = s_ovf != 0;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      if (ovf) atomicOr(&st->overflow, 1u);
      __hip_atomic_store(&st->D, s_all[0] + s_all[1] + s_all[2] + s_all[3], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __threadfence();
    }
    __syncthreads();
    publish_state(st, pub);
  }
  return s_below[0] + s_below[1] + s_below[2] + s_below[3];
}

// OFFS: the output offsets are in out_off; else each workgroup takes four leaves
// and finds them itself (leaf_prefix).
template <typename K, bool OFFS>
__global__ void __launch_bounds__(256) k_concat(const K* __restrict__ bufA,
                                                const K* __restrict__ bufB,
                                                const uint32_t* __restrict__ tmp_cnt,
                                                const Leaf* __restrict__ leaves,
                                                const uint32_t* __restrict__ d,
                                                const unsigned long long* __restrict__ out_off,
                                                DevState* st, uint64_t cap,
                                                uint64_t* __restrict__ out_keys,
                                                uint32_t* __restrict__ out_counts,
                                                DevState* pub) {
  // a leaf overflowed: the host refines it and concatenates afterwards, so
  // this launch (enqueued before the host could know) has nothing to do
  const unsigned long long n_leaves = st->n_leaves;
  unsigned long long first = 0;
  if constexpr (OFFS) {
    if (st->overflow) return;
  } else {
    if (blockIdx.x && blockIdx.x * 4ull >= n_leaves) return;
    bool ovf;
    first = leaf_prefix(d, (uint32_t)n_leaves, blockIdx.x * 4, st, pub, ovf);
    if (ovf) return;
    for (uint32_t l = blockIdx.x * 4; l < blockIdx.x * 4 + (threadIdx.x >> 6) && l < n_leaves; ++l)
      first += d[l];
  }
  // one wave per leaf, many leaves in flight per CU
  const unsigned lane = threadIdx.x & 63;
  const unsigned long long nw = (unsigned long long)gridDim.x * 4;
  for (unsigned long long l = (unsigned long long)blockIdx.x * 4 + (threadIdx.x >> 6); l < n_leaves;
       l += nw) {
    const uint32_t n = d[l];
    if (n == 0 || n == kLeafOverflow) continue;
    const Leaf lf = leaves[l];
    const K* src = lf.buf ? bufA : bufB;  // sorted pairs sit in the other buffer
    const unsigned long long base = OFFS ? out_off[l] : first;
    const uint64_t lim = base >= cap ? 0 : min((uint64_t)n, cap - base);
    // U words per lane and step, all loaded before any is stored (more bytes
    // in flight per wave). Keys are copied word by word, whatever their width
    // (their words lie in memory as the output has them): a lane that stores a
    // four-word key's words touches 32 bytes in four stores of a quarter each
    // (1,000,000 reads at k = 100 0.73 -> 0.66 ms, at k = 31 0.202 -> 0.183).
    constexpr uint32_t U = 4;
    const uint64_t* const ks = (const uint64_t*)(src + lf.begin);
    uint64_t* const kd = out_keys + base * Key<K>::kWords;
    const uint64_t words = lim * Key<K>::kWords;
    const uint32_t* const cs = tmp_cnt + lf.begin;
    uint32_t* const cd = out_counts + base;
    for (uint64_t i0 = lane; i0 < words; i0 += 64 * U) {
      uint64_t x[U];
      uint32_t c[U];
      const bool both = Key<K>::kWords == 1;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint64_t i = i0 + u * 64;
        if (i < words) {
          x[u] = ks[i];
          if (both) c[u] = cs[i];
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint64_t i = i0 + u * 64;
        if (i < words) {
          kd[i] = x[u];
          if (both) cd[i] = c[u];
        }
      }
    }
    if constexpr (Key<K>::kWords > 1)
      for (uint64_t i0 = lane; i0 < lim; i0 += 64 * U) {
        uint32_t c[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
          if (i0 + u * 64 < lim) c[u] = cs[i0 + u * 64];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
          if (i0 + u * 64 < lim) cd[i0 + u * 64] = c[u];
      }
  }
}

// Batch form of concat: writes the k-mer (low 2k bits) and the set id within
// the class (the bits above) of every pair, in key order. cut_kb >= 0: of cut keys
// (see BatchSets), whose set id is the leaf's shard without its low cut_kb bits.
template <typename K>
__global__ void __launch_bounds__(256) k_concat_batch(
    const K* __restrict__ bufA, const K* __restrict__ bufB, const uint32_t* __restrict__ tmp_cnt,
    const Leaf* __restrict__ leaves, const uint32_t* __restrict__ d,
    const unsigned long long* __restrict__ out_off, const DevState* __restrict__ st, uint64_t cap,
    int k, int cut_kb, uint64_t* __restrict__ out_keys, uint32_t* __restrict__ out_counts,
    uint32_t* __restrict__ out_set) {
  if (st->overflow) return;  // the class is recounted set by set
  const unsigned long long n_leaves = st->n_leaves;
  const unsigned lane = threadIdx.x & 63;
  const unsigned long long nw = (unsigned long long)gridDim.x * 4;
  const bool has_set_bits = 2 * k < (int)(8 * sizeof(K));
  const K kmask = has_set_bits ? ((K)1 << (2 * k)) - 1 : ~(K)0;
  for (unsigned long long l = (unsigned long long)blockIdx.x * 4 + (threadIdx.x >> 6); l < n_leaves;
       l += nw) {
    const uint32_t n = d[l];
    if (n == 0 || n == kLeafOverflow) continue;
    const Leaf lf = leaves[l];
    const K* src = lf.buf ? bufA : bufB;
    const unsigned long long base = out_off[l];
    constexpr uint32_t U = 4;  // as in k_concat
    const uint64_t lim = base >= cap ? 0 : min((uint64_t)n, cap - base);
    for (uint32_t i0 = 0; i0 < lim; i0 += 64 * U) {
      K key[U];
      uint32_t cnt[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = i0 + u * 64 + lane;
        if (i < lim) {
          key[u] = src[lf.begin + i];
          cnt[u] = tmp_cnt[lf.begin + i];
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = i0 + u * 64 + lane;
        if (i >= lim) break;
        const uint64_t o = base + i;
        out_keys[o] = (uint64_t)(key[u] & kmask);
        out_set[o] = cut_kb >= 0 ? lf.shard >> cut_kb
                     : has_set_bits ? (uint32_t)(key[u] >> (2 * k))
                                    : 0u;
        out_counts[o] = cnt[u];
      }
    }
  }
}

// start[s] = index of the first pair of set s (within a class output sorted
// by set); sets without pairs get the index of the next pair. start has
// n_local + 1 entries; start[n_local] = number of pairs. A class whose leaf
// overflowed has no output (its concat returned at once, so the set ids hold
// whatever the buffer held before): all its bounds are 0, and the host counts
// the wave's sets one by one.
__global__ void k_set_bounds(const uint32_t* __restrict__ set, const DevState* __restrict__ st,
                             uint32_t n_local, unsigned long long* __restrict__ start) {
  const unsigned long long n = st->D;
  if (n == 0 || st->overflow) {
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t <= n_local; t += gridDim.x * blockDim.x)
      start[t] = 0;
    return;
  }
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x) {
    const uint32_t s = set[i];
    const uint32_t from = i == 0 ? 0u : set[i - 1] + 1;
    for (uint32_t t = from; t <= s; ++t) start[t] = i;
    if (i == n - 1)
      for (uint32_t t = s + 1; t <= n_local; ++t) start[t] = n;
  }
}

// Global output offsets of the sets (one block): set g is set_local[g] of
// class set_class[g], whose bounds start at start_base[class] in starts[].
__global__ void __launch_bounds__(kPlanTB) k_batch_offsets(
    const uint32_t* __restrict__ set_class, const uint32_t* __restrict__ set_local,
    const unsigned long long* __restrict__ starts, const unsigned long long* __restrict__ start_base,
    uint32_t n_sets, unsigned long long* __restrict__ set_off) {
  __shared__ unsigned long long wsum[kPlanTB / 64];
  const uint32_t per = (n_sets + kPlanTB - 1) / kPlanTB;
  const uint32_t b = threadIdx.x * per, e = min(n_sets, b + per);
  unsigned long long s = 0;
  for (uint32_t g = b; g < e; ++g) {
    const unsigned long long* st = starts + start_base[set_class[g]];
    s += st[set_local[g] + 1] - st[set_local[g]];
  }
  unsigned long long total;
  unsigned long long run = block_exscan<kPlanTB, unsigned long long>(s, wsum, &total);
  for (uint32_t g = b; g < e; ++g) {
    set_off[g] = run;
    const unsigned long long* st = starts + start_base[set_class[g]];
    run += st[set_local[g] + 1] - st[set_local[g]];
  }
  if (threadIdx.x == 0) set_off[n_sets] = total;
}

// Copy each set's pairs from its class output to its place in the batch
// output. Waves take chunks of consecutive output positions (coalesced
// reads and writes); the set of a chunk's first position is found by binary
// search in set_off, later positions move to the next set when they pass its
// start.
__global__ void __launch_bounds__(256) k_batch_gather(
    const uint32_t* __restrict__ set_class, const uint32_t* __restrict__ set_local,
    const unsigned long long* __restrict__ starts, const unsigned long long* __restrict__ start_base,
    const unsigned long long* __restrict__ class_base, const uint64_t* __restrict__ cls_keys,
    const uint32_t* __restrict__ cls_counts, const unsigned long long* __restrict__ set_off,
    uint32_t n_sets, uint64_t cap, uint64_t* __restrict__ out_keys,
    uint32_t* __restrict__ out_counts) {
  constexpr int kChunk = 64 * 16;
  const unsigned lane = threadIdx.x & 63;
  const unsigned long long D = min((unsigned long long)cap, set_off[n_sets]);
  const unsigned long long nchunks = (D + kChunk - 1) / kChunk;
  for (unsigned long long ch = (unsigned long long)blockIdx.x * 4 + (threadIdx.x >> 6);
       ch < nchunks; ch += (unsigned long long)gridDim.x * 4) {
    const unsigned long long o0 = ch * kChunk;
    uint32_t lo = 0, hi = n_sets - 1;  // last set starting at or before o0
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (set_off[mid] <= o0) lo = mid; else hi = mid - 1;
    }
    uint32_t g = lo;
    unsigned long long src0 = class_base[set_class[g]] +
                              starts[start_base[set_class[g]] + set_local[g]] - set_off[g];
    for (int j = 0; j < 16; ++j) {
      const unsigned long long o = o0 + (unsigned long long)j * 64 + lane;
      if (o >= D) break;
      bool moved = false;
      while (g + 1 < n_sets && o >= set_off[g + 1]) {
        ++g;
        moved = true;
      }
      if (moved)
        src0 = class_base[set_class[g]] + starts[start_base[set_class[g]] + set_local[g]] -
               set_off[g];
      out_keys[o] = cls_keys[src0 + o];
      out_counts[o] = cls_counts[src0 + o];
    }
  }
}

template <typename K>
__device__ __forceinline__ K load_out_key(const uint64_t* keys, uint64_t i) {
  if constexpr (Key<K>::kWords == 4)
    return K(((u128)keys[4 * i + 1] << 64) | keys[4 * i], ((u128)keys[4 * i + 3] << 64) | keys[4 * i + 2]);
  else if constexpr (Key<K>::kWords == 2)
    return (K)(((u128)keys[2 * i + 1] << 64) | keys[2 * i]);
  else
    return (K)keys[i];
}

template <typename K>
__global__ void __launch_bounds__(256) k_check(const uint64_t* __restrict__ keys,
                                               const uint32_t* __restrict__ counts, uint64_t n,
                                               int k, CheckResult* res) {
  unsigned long long sum = 0;
  uint32_t ns = 0, nc = 0, nr = 0, nz = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * 256) {
    const K x = load_out_key<K>(keys, i);
    if (i + 1 < n && !(x < load_out_key<K>(keys, i + 1))) ++ns;
    if (!Key<K>::in_range(x, k)) ++nr;
    else if (Key<K>::revcomp(x, k) < x) ++nc;
    if (counts[i] == 0) ++nz;
    sum += counts[i];
  }
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off);
    ns += __shfl_xor(ns, off);
    nc += __shfl_xor(nc, off);
    nr += __shfl_xor(nr, off);
    nz += __shfl_xor(nz, off);
  }
  if ((threadIdx.x & 63) == 0) {
    if (sum) atomicAdd(&res->sum_counts, sum);
    if (ns) atomicAdd(&res->not_sorted, ns);
    if (nc) atomicAdd(&res->not_canonical, nc);
    if (nr) atomicAdd(&res->out_of_range, nr);
    if (nz) atomicAdd(&res->zero_count, nz);
  }
}

constexpr int kHistTB = 256;
constexpr unsigned kHistGrid = 2048;  // a multiple of kXcds times the units of a tile (1 to 8)
constexpr int kScatterTB64 = 1024;
constexpr int kScatterTB128 = 1024;
constexpr int kSplitTB64 = 1024;
constexpr int kSplitTB128 = 512;
// Wider keys: LDS staging of 64 KiB per tile, two tiles per CU; four window
// starts per thread, so that these make 16 and 32 waves (eight starts, half as
// many waves: 1,000,000 reads at k = 100 1.16 ms, so 1.06)
constexpr int kScatterTB256 = 512;
constexpr int kScatterS256 = 4, kScatterS128 = 4;
// cut keys: tiles of 4,096 records and their shards, 52 KB, three workgroups a CU
// (four starts per thread and 1,024 threads: 512 us against 285 in the batch of 48
// sets)
constexpr int kScatterSCut = 8, kScatterTBCut = 512;
// One-word keys of a batch: the same tiles (a batch's kernel keeps too many values
// live for two workgroups of 1,024 threads a CU: 244 against 193 us in that batch).
// Both hold for large sets: 1,024 threads took 12 sets of 3 to 10 Mbp from 21.4 to
// 22.6 ms (k = 21), with cut keys from 17.6 to 18.7 (k = 32).
constexpr int kScatterTBBatch64 = 512;
inline int scatter_threads(int words, bool batch, bool cut, int starts) {
  return cut          ? kScatterTBCut
         : words == 4 ? kScatterTB256
         : words == 2 ? kScatterTB128
         : batch && starts == kWinStarts ? kScatterTBBatch64
                                         : kScatterTB64;
}
inline int scatter_starts(int words, int starts_per_thread) {
  return words == 4 ? kScatterS256 : words == 2 ? kScatterS128 : starts_per_thread == 16 ? 16 : kWinStarts;
}
constexpr int kSplitTB256 = 256;
constexpr int kSplitR = 8;
constexpr int kLeafTB = 512;
constexpr int kLeafCmax64 = 4096;
// second-chance count of overflowed one-word leaves: 8,192 slots (128 KiB of
// LDS with the epilogue's counters: one 1,024-thread workgroup per CU)
constexpr int kRescueTB = 1024;
constexpr int kRescueCmax64 = 8192;
// the same for wider keys: 4,096 slots (152 KiB for four-word keys)
constexpr int kRescueCmaxW = 4096;
inline int second_slots_log2(int words) { return words == 1 ? 13 : 12; }
constexpr unsigned kRescueGrid = 256;
constexpr int kLeafCmax128 = 2048;
constexpr int kLeafCmax256 = 2048;
// Workgroups of the block-wide leaf kernels and the split scatter, each taking
// every kManyGrid-th leaf or item. Many more than fit the chip (768 and 256):
// the hardware hands them out as workgroups finish, which evens out leaves of
// unequal cost, and there is no last round that fills a third of the chip (1,024
// workgroups of which 768 are resident: large leaves of 20,000,000 reads 14.3
// ms, so 10.7; 768: 12.1; 4,096: 11.2; 65,536: 10.8. Split scatter of
// 1,000,000 reads, 7,300 items on 2,048 workgroups: 0.51 ms, so 0.41).
constexpr unsigned kManyGrid = 16384;
constexpr int kSmallCmax64 = 1024;  // one-wave leaf kernel: slots of its private table
constexpr int kSmallCmax128 = 512;
constexpr unsigned kSmallGrid = 256 * 20;
constexpr int kSortMax64 = 5120;   // records per leaf of the sort-based count (radix: 148 KiB LDS)
constexpr int kSortMax128 = 4096;
constexpr int kSortMax256 = 2048;

inline unsigned grid_for(uint64_t n, unsigned tb, unsigned cap) {
  uint64_t g = (n + tb - 1) / tb;
  if (g > cap) g = cap;
  return g ? (unsigned)g : 1u;
}

inline unsigned persistent(uint64_t max_n, unsigned cap) {
  return (unsigned)(max_n == 0 ? 1 : (max_n < cap ? max_n : cap));
}

}  // namespace

int max_leaf_slots_log2(int words) { return words > 1 ? 11 : 12; }
int max_shard_bits() { return kMaxShardBits; }
int split_tile(int words, int records_per_thread) {
  const int r = words == 1 && records_per_thread == 16 ? 16 : kSplitR;
  return (words == 4 ? kSplitTB256 : words == 2 ? kSplitTB128 : kSplitTB64) * r;
}

hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v,
                           hipStream_t s) {
  if (!n) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_pack(const uint8_t* src, uint64_t n_bytes, const uint64_t* offsets,
                       uint64_t n_reads, uint64_t off0, uint64_t* packed, uint64_t* inv,
                       uint64_t* endm, uint64_t nchunks, hipStream_t s) {
  const unsigned grid = (unsigned)((nchunks + 255) / 256);
  hipLaunchKernelGGL(k_pack, dim3(grid), dim3(256), 0, s, src, n_bytes, packed, inv, endm, nchunks);
  if (n_reads)
    hipLaunchKernelGGL(k_read_ends, dim3((unsigned)((n_reads + 255) / 256)), dim3(256), 0, s,
                       offsets, n_reads, off0, (unsigned long long*)endm);
  return hipGetLastError();
}

hipError_t launch_front(int words, const uint8_t* src, uint64_t n_bytes, const uint64_t* offsets,
                        uint64_t n_reads, uint64_t off0, int k, uint64_t* packed, uint64_t* valid,
                        uint64_t nchunks, const ZeroRanges& z, hipStream_t s) {
  uint64_t zeros = 0;
  for (uint64_t n : z.n) zeros += n;
  const uint64_t per = 256 - (words == 4 ? kFrontHalo<true> : kFrontHalo<false>);
  const unsigned grid = (unsigned)std::max<uint64_t>(
      (nchunks + per - 1) / per, std::min<uint64_t>((zeros + 1023) / 1024, 1024));
  if (words == 4)
    hipLaunchKernelGGL(k_front<true>, dim3(grid), dim3(256), 0, s, src, n_bytes, offsets, n_reads,
                       off0, k, packed, valid, nchunks, z);
  else
    hipLaunchKernelGGL(k_front<false>, dim3(grid), dim3(256), 0, s, src, n_bytes, offsets,
                       n_reads, off0, k, packed, valid, nchunks, z);
  return hipGetLastError();
}

#define KC_WINDOW_LAUNCH(KERNEL, K, KC, TB, BATCH, GRID)                                    \
  hipLaunchKernelGGL((KERNEL<K, KC, kWinStarts, TB, BATCH>), dim3(GRID), dim3(TB), 0, s, packed, \
                     valid, t_begin, t_end, k, keybits, shard_bits, bs, ARG0, ARG1)
#define KC_WINDOW_LAUNCH_S(KERNEL, K, KC, S, TB, BATCH, GRID)                                  \
  hipLaunchKernelGGL((KERNEL<K, KC, S, TB, BATCH>), dim3(GRID), dim3(TB), 0, s, packed, valid,     \
                     t_begin, t_end, k, keybits, shard_bits, bs, ARG0, ARG1)

hipError_t launch_valid_mask(int words, const uint64_t* inv, const uint64_t* endm,
                             uint64_t byte_begin, uint64_t byte_end, int k, uint64_t* valid,
                             const ZeroRanges& z, hipStream_t s) {
  // the words the window kernels read: starts [byte_begin, byte_end) rounded
  // out to whole threads, which stay inside whole words
  const uint64_t w_begin = byte_begin >> 6;
  const uint64_t w_end = std::max(w_begin, (byte_end + 63) >> 6);
  uint64_t zeros = 0;
  for (uint64_t n : z.n) zeros += n;
  if (w_end == w_begin && !zeros) return hipSuccess;
  const unsigned grid = (unsigned)std::max<uint64_t>(
      (w_end - w_begin + 255) / 256, std::min<uint64_t>((zeros + 1023) / 1024, 1024));
  if (words == 4)
    hipLaunchKernelGGL(k_valid_mask<true>, dim3(grid), dim3(256), 0, s, inv, endm, w_begin, w_end,
                       k, valid, z);
  else
    hipLaunchKernelGGL(k_valid_mask<false>, dim3(grid), dim3(256), 0, s, inv, endm, w_begin,
                       w_end, k, valid, z);
  return hipGetLastError();
}

#define KC_HIST_LAUNCH(K, KC, BATCH)                                                            \
  hipLaunchKernelGGL((k_window_hist<K, KC, kWinStarts, kHistTB, BATCH>), dim3(grid),            \
                     dim3(kHistTB), 0, s, packed, valid, w_begin, w_end, R, k, keybits,         \
                     shard_bits, bs, hist)

hipError_t launch_window_hist(int words, const uint64_t* packed, const uint64_t* valid,
                              uint64_t byte_begin, uint64_t byte_end, int k,
                              int keybits, int shard_bits, const BatchSets* batch,
                              unsigned long long* hist, int starts_per_thread, hipStream_t s) {
  // the owner scatter's tiles (see launch_window_scatter)
  const bool cut = batch && batch->cut;
  const int S = cut ? kScatterSCut : scatter_starts(words, starts_per_thread);
  const int TBs = scatter_threads(words, batch != nullptr, cut, S);
  const uint64_t w_begin = byte_begin / S * S;
  const uint64_t w_end = (byte_end + S - 1) / S * S;
  const uint64_t unit = (uint64_t)kHistTB * kWinStarts;
  const int R = (int)((uint64_t)TBs * S / unit);  // units per tile
  const uint64_t n_units = (w_end - w_begin + unit - 1) / unit;
  // a multiple of R * kXcds workgroups (every workgroup's units share a class)
  const uint64_t step = (uint64_t)R * kXcds;
  const unsigned grid = (unsigned)std::min<uint64_t>((n_units + step - 1) / step * step, kHistGrid);
  if (grid == 0) return hipSuccess;
  const BatchSets bs = batch ? *batch : BatchSets{nullptr, nullptr, 0, false};
  const bool wide = words == 2;
  if (batch) {
    if (words == 4) return hipErrorInvalidValue;
    if (wide) KC_HIST_LAUNCH(u128, uint64_t, true);
    else KC_HIST_LAUNCH(uint64_t, uint64_t, true);
  } else {
    if (words == 4) KC_HIST_LAUNCH(u256, u256, false);
    else if (wide) KC_HIST_LAUNCH(u128, u128, false);
    else KC_HIST_LAUNCH(uint64_t, uint64_t, false);
  }
  return hipGetLastError();
}
#undef KC_HIST_LAUNCH

hipError_t launch_window_scatter(int words, const uint64_t* packed, const uint64_t* valid,
                                 uint64_t byte_begin, uint64_t byte_end,
                                 int k, int keybits, int shard_bits, const BatchSets* batch,
                                 unsigned long long* cursor, void* out, int starts_per_thread,
                                 hipStream_t s) {
  const BatchSets bs0 = batch ? *batch : BatchSets{nullptr, nullptr, 0, false};
  if (batch && batch->cut) {
    if (words != 1) return hipErrorInvalidValue;
    const uint64_t t0 = byte_begin / kScatterSCut;
    const uint64_t t1 = (byte_end + kScatterSCut - 1) / kScatterSCut;
    hipLaunchKernelGGL((k_window_scatter_cut<kScatterSCut, kScatterTBCut>),
                       dim3(grid_for(t1 - t0, kScatterTBCut, 1u << 20)), dim3(kScatterTBCut), 0, s,
                       packed, valid, t0, t1, k, keybits, shard_bits, bs0, cursor, (uint64_t*)out);
    return hipGetLastError();
  }
  if (words == 1 && starts_per_thread == 16) {
    // byte_begin is a multiple of 32 (batch classes) or 0
    constexpr int S = 16;
    const uint64_t t_begin = byte_begin / S;
    const uint64_t t_end = (byte_end + S - 1) / S;
    const BatchSets bs = bs0;
    const unsigned grid = grid_for(t_end - t_begin, kScatterTB64, 1u << 20);
#define ARG0 cursor
#define ARG1 (uint64_t*)out
    if (batch) KC_WINDOW_LAUNCH_S(k_window_scatter64w, uint64_t, uint64_t, S, kScatterTB64, true, grid);
    else KC_WINDOW_LAUNCH_S(k_window_scatter64w, uint64_t, uint64_t, S, kScatterTB64, false, grid);
#undef ARG1
#undef ARG0
    return hipGetLastError();
  }
  const int S = scatter_starts(words, starts_per_thread);
  const uint64_t t_begin = byte_begin / S;
  const uint64_t t_end = (byte_end + S - 1) / S;
  const BatchSets bs = batch ? *batch : BatchSets{nullptr, nullptr, 0, false};
#define ARG0 cursor
  if (words == 4) {
    if (batch) return hipErrorInvalidValue;
    const unsigned grid = grid_for(t_end - t_begin, kScatterTB256, 1u << 20);
#define ARG1 (u256*)out
    KC_WINDOW_LAUNCH_S(k_window_scatter, u256, u256, kScatterS256, kScatterTB256, false, grid);
#undef ARG1
  } else if (words == 2) {
    const unsigned grid = grid_for(t_end - t_begin, kScatterTB128, 1u << 20);
#define ARG1 (u128*)out
    if (batch)
      KC_WINDOW_LAUNCH_S(k_window_scatter, u128, uint64_t, kScatterS128, kScatterTB128, true, grid);
    else
      KC_WINDOW_LAUNCH_S(k_window_scatter, u128, u128, kScatterS128, kScatterTB128, false, grid);
#undef ARG1
  } else {
    const unsigned grid = grid_for(t_end - t_begin, kScatterTB64, 1u << 20);
#define ARG1 (uint64_t*)out
    if (batch)
      KC_WINDOW_LAUNCH(k_window_scatter, uint64_t, uint64_t, kScatterTBBatch64, true,
                       grid_for(t_end - t_begin, kScatterTBBatch64, 1u << 20));
    else KC_WINDOW_LAUNCH(k_window_scatter64, uint64_t, uint64_t, kScatterTB64, false, grid);
#undef ARG1
  }
#undef ARG0
  return hipGetLastError();
}
#undef KC_WINDOW_LAUNCH
#undef KC_WINDOW_LAUNCH_S

hipError_t launch_plan_shards(unsigned long long* hist, const int* order, int shard_bits,
                              int keybits, uint64_t leaf_target, uint64_t leaf_attempt,
                              int tile, unsigned long long* sbegin, unsigned long long* cursor,
                              SplitBin* bins, SplitItem* items, unsigned long long* item_off,
                              unsigned long long* subhist, uint64_t max_items, DevState* st,
                              Leaf* leaves, hipStream_t s) {
  if (leaves) leaf_attempt = ~0ull;
  const bool few = leaves || max_items <= kFewItems;
  hipLaunchKernelGGL(k_plan_shards, dim3(1), dim3(kPlanTB), 0, s, hist, order, shard_bits,
                     keybits, leaf_target, leaf_attempt, tile, sbegin, cursor, bins, item_off,
                     subhist, st, few ? items : (SplitItem*)nullptr, leaves);
  if (!few)
    hipLaunchKernelGGL(k_plan_items, dim3(grid_for(max_items, 256, 2048)), dim3(256), 0, s, hist,
                     sbegin, item_off, shard_bits, tile, st, items);
  return hipGetLastError();
}

// Inputs of one-word keys with up to kTinyLeaves leaves, and of wider keys where
// nothing is split: the second count's table for all of them from the start. There is a CU for each, or nearly, so a workgroup that fills one
// takes no longer (13.0 against 12.7 us for 667 reads), and the second launch,
// mostly with nothing to do, goes (4 to 5 us), as does the first try of a leaf that
// needs the larger table (100 kB of 80% AT at k = 55 181 -> 127 us, k = 100 129 -> 96).
constexpr uint64_t kTinyLeaves = 3 * kRescueGrid;
static bool tiny_leaves(int words, uint64_t max_leaves, int slots_log2, int mode, bool refine,
                        bool merged, bool unsplit = false) {
  return (words == 1 || unsplit) && mode != 1 && !refine && !merged && max_leaves <= kTinyLeaves &&
         slots_log2 == max_leaf_slots_log2(words);
}

// (The line: an eighth of the larger table, 1,024 bytes a shard for one-word keys
// and 512 for wider ones, so that the fullest shard of an AT-rich genome, 5 to 10%
// of the windows, overflows only where nearly all of them are distinct, which
// costs the leaf kernel twice. 100 kB of random reads with and without a split: at
// k = 31 88 against 69 us, k = 55 89 against 71, k = 100 91 against 73; of 80% AT 110
// against 79, 137 against 125 and 128 against 90; of A and T alone, which overflow,
// 150 against 260, 515 against 588 and 232 against 353. One-word keys of more than
// 256 shards, P > 256, are always split: the bound of their leaves that the host has
// is past kTinyLeaves.)
bool counts_unsplit(int words, uint64_t rec_bound, int shard_bits, uint64_t max_leaves,
                    int slots_log2) {
  if (words == 1)
    return tiny_leaves(words, max_leaves, slots_log2, 0, false, false) &&
           rec_bound <= (uint64_t)kRescueCmax64 / 8 << shard_bits;
  return max_leaves <= kFewLeaves && slots_log2 == max_leaf_slots_log2(words) &&
         rec_bound <= (uint64_t)kRescueCmaxW / 8 << shard_bits;
}

// Which leaves go where (see classify_leaves).
static LeafLists leaf_lists(int words, uint64_t max_leaves, uint32_t* d_out, uint32_t* large_list,
                            uint32_t* ovf_list, int slots_log2, int mode, bool tiny) {
  const bool one_wave = mode != 1 && words != 4 && max_leaves > kFewLeaves;
  // few leaves: the block-wide kernel goes through the leaf table itself, empty
  // leaves too, with no list between (one word that 256 planning workgroups
  // count up, and a load more per leaf)
  const bool direct = mode != 1 && max_leaves <= kFewLeaves;
  // leaves of more than 8 first tables of records go straight to the second
  // count (where it runs: launch_leaf_second)
  const bool second = mode != 1 && !tiny && slots_log2 < second_slots_log2(words) && ovf_list;
  return LeafLists{one_wave ? small_leaf_max(words) : 0, 8ull << slots_log2, large_list,
                   second ? ovf_list : nullptr, one_wave || direct ? nullptr : d_out,
                   true, one_wave, direct};
}

hipError_t launch_plan_leaves(int words, const unsigned long long* hist,
                              const unsigned long long* sbegin, const SplitBin* bins,
                              int shard_bits, const unsigned long long* subhist, Leaf* leaves,
                              unsigned long long* cursor, int merge_cshift, int ncls,
                              uint64_t cls_stride, DevState* st, uint64_t max_leaves,
                              uint32_t* d_out, uint32_t* large_list, uint32_t* ovf_list,
                              int slots_log2, int mode, hipStream_t s) {
  LeafLists q{};
  if (!merge_cshift)
    q = leaf_lists(words, max_leaves, d_out, large_list, ovf_list, slots_log2, mode,
                   tiny_leaves(words, max_leaves, slots_log2, mode, false, false));
  hipLaunchKernelGGL(k_plan_leaves, dim3(1u << shard_bits), dim3(kPlanTB), 0, s, hist, sbegin,
                     bins, shard_bits, subhist, leaves, cursor, merge_cshift, ncls, cls_stride, st,
                     q);
  return hipGetLastError();
}

hipError_t launch_leaf_ends(Leaf* leaves, const unsigned long long* cursor, const DevState* st,
                            uint64_t max_leaves, hipStream_t s) {
  hipLaunchKernelGGL(k_leaf_ends, dim3(grid_for(max_leaves, 256, 2048)), dim3(256), 0, s, leaves,
                     cursor, st);
  return hipGetLastError();
}

hipError_t launch_split_hist(int words, const void* src, const SplitItem* items,
                             const DevState* st, uint64_t max_items, const SplitBin* bins,
                             unsigned long long* subhist, int ncls, uint64_t cls_stride,
                             hipStream_t s) {
  const unsigned grid = persistent(max_items, 4096);
  if (words == 4)
    hipLaunchKernelGGL((k_split_hist<u256, 256>), dim3(grid), dim3(256), 0, s, (const u256*)src,
                       items, st, bins, subhist, ncls, cls_stride);
  else if (words == 2)
    hipLaunchKernelGGL((k_split_hist<u128, 256>), dim3(grid), dim3(256), 0, s, (const u128*)src,
                       items, st, bins, subhist, ncls, cls_stride);
  else
    hipLaunchKernelGGL((k_split_hist<uint64_t, 256>), dim3(grid), dim3(256), 0, s,
                       (const uint64_t*)src, items, st, bins, subhist, ncls, cls_stride);
  return hipGetLastError();
}

hipError_t launch_split_scatter(int words, const void* src, void* dst, const SplitItem* items,
                                const DevState* st, uint64_t max_items, const SplitBin* bins,
                                unsigned long long* cursor, int records_per_thread,
                                int merge_cshift, int ncls, uint64_t cls_stride, hipStream_t s) {
  const unsigned grid = persistent(max_items, kManyGrid);
  if (merge_cshift) {
    // one cursor per leaf: its final value is the leaf's end
    if (words != 1 || records_per_thread != 16 || ncls != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_split_scatter_merge<kSplitTB64, 16>), dim3(grid), dim3(kSplitTB64), 0,
                       s, (const uint64_t*)src, (uint64_t*)dst, items, st, bins, cursor,
                       merge_cshift);
    return hipGetLastError();
  }
  if (words == 1 && records_per_thread == 16) {
    // 16,384-record tiles: 128 KiB of LDS staging, one workgroup per CU
    hipLaunchKernelGGL((k_split_scatter<uint64_t, kSplitTB64, 16>), dim3(grid), dim3(kSplitTB64),
                       0, s, (const uint64_t*)src, (uint64_t*)dst, items, st, bins, cursor,
                       ncls, cls_stride);
    return hipGetLastError();
  }
  if (words == 4)
    hipLaunchKernelGGL((k_split_scatter<u256, kSplitTB256, kSplitR>), dim3(grid),
                       dim3(kSplitTB256), 0, s, (const u256*)src, (u256*)dst, items, st, bins,
                       cursor, ncls, cls_stride);
  else if (words == 2)
    hipLaunchKernelGGL((k_split_scatter<u128, kSplitTB128, kSplitR>), dim3(grid),
                       dim3(kSplitTB128), 0, s, (const u128*)src, (u128*)dst, items, st, bins,
                       cursor, ncls, cls_stride);
  else
    hipLaunchKernelGGL((k_split_scatter<uint64_t, kSplitTB64, kSplitR>), dim3(grid),
                       dim3(kSplitTB64), 0, s, (const uint64_t*)src, (uint64_t*)dst, items, st,
                       bins, cursor, ncls, cls_stride);
  return hipGetLastError();
}

uint64_t small_leaf_max(int words) {
  // n + n/7 + 1 <= slots of the one-wave kernel (none for four-word keys)
  return words == 4 ? 0 : words == 2 ? 447 : 895;
}

hipError_t launch_leaf_small(int words, int keybits, void* bufA, void* bufB, uint32_t* tmp_cnt,
                             const Leaf* leaves, DevState* st, uint64_t max_leaves,
                             uint32_t* d_out, uint32_t* large_list, uint32_t* ovf_list,
                             int slots_log2, hipStream_t s, int mode, bool refine, bool merged,
                             bool classified) {
  const bool wide = words == 2;
  const LeafLists q =
      leaf_lists(words, max_leaves, d_out, large_list, ovf_list, slots_log2, mode,
                 tiny_leaves(words, max_leaves, slots_log2, mode, refine, merged));
  const uint64_t small_max = q.small_max;
  if (!classified) {
    // n_large and n_ovf
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, s, &st->n_large, (uint64_t)2, 0ull);
    hipLaunchKernelGGL(k_classify_leaves, dim3(grid_for(max_leaves, 256, 2048)), dim3(256), 0, s,
                       leaves, st, q);
  }
  if (!q.one_wave) return hipGetLastError();  // the block-wide kernel takes every leaf
  const unsigned gsmall = persistent(max_leaves, kSmallGrid);
#define KC_SMALLW(KRN, FF)                                                                        \
  hipLaunchKernelGGL((KRN<64, kSmallCmax128, 8, FF>), dim3(gsmall), dim3(64), 0, s, keybits,       \
                     (u128*)bufA, (u128*)bufB, tmp_cnt, leaves, st, d_out,                        \
                     __builtin_ctz(kSmallCmax128), (const uint32_t*)nullptr,                      \
                     (const unsigned long long*)nullptr, (uint32_t*)nullptr, &st->large_records,  \
                     small_max)
#define KC_SMALL64(FF, MG)                                                                       \
  hipLaunchKernelGGL((k_leaf_count64<64, kSmallCmax64, 8, FF, MG>), dim3(gsmall), dim3(64), 0, s, \
                     keybits, (uint64_t*)bufA, (uint64_t*)bufB, tmp_cnt, leaves, st, d_out,      \
                     __builtin_ctz(kSmallCmax64), (const uint32_t*)nullptr,                      \
                     (const unsigned long long*)nullptr, (uint32_t*)nullptr, &st->large_records, \
                     small_max)
  if (wide) {
    if (keybits <= 126) {
      if (refine) KC_SMALLW(k_leaf_count128, true); else KC_SMALLW(k_leaf_count128, false);
    } else {
      if (refine) KC_SMALLW(k_leaf_countw128, true); else KC_SMALLW(k_leaf_countw128, false);
    }
  } else {
    if (merged) {
      if (refine) KC_SMALL64(true, true); else KC_SMALL64(false, true);
    } else {
      if (refine) KC_SMALL64(true, false); else KC_SMALL64(false, false);
    }
  }
#undef KC_SMALLW
#undef KC_SMALL64
  return hipGetLastError();
}

hipError_t launch_leaf_large(int words, int keybits, void* bufA, void* bufB, uint32_t* tmp_cnt,
                             const Leaf* leaves, DevState* st, uint64_t max_leaves,
                             uint32_t* d_out, int slots_log2, const uint32_t* large_list,
                             uint32_t* ovf_list, hipStream_t s, int mode, bool refine,
                             bool merged, bool unsplit) {
  const bool wide = words == 2;
  // (max_leaves is a bound, two to four times the leaves: fewer workgroups for
  // inputs of few, or most start only to end, in the way of other streams' work)
  const unsigned glarge = persistent(
      max_leaves, (unsigned)std::min<uint64_t>(std::max<uint64_t>(max_leaves / 4, 1024), kManyGrid));
  if (mode == 1) {
    if (words == 4)
      hipLaunchKernelGGL((k_leaf_sort<u256, kLeafTB, kSortMax256>), dim3(glarge), dim3(kLeafTB),
                         0, s, keybits, (u256*)bufA, (u256*)bufB, tmp_cnt, leaves, st, d_out,
                         large_list);
    else if (wide)
      hipLaunchKernelGGL((k_leaf_sort<u128, kLeafTB, kSortMax128>), dim3(glarge), dim3(kLeafTB),
                         0, s, keybits, (u128*)bufA, (u128*)bufB, tmp_cnt, leaves, st, d_out,
                         large_list);
    else
      hipLaunchKernelGGL((k_leaf_radix64<kLeafTB, kSortMax64>), dim3(glarge), dim3(kLeafTB), 0, s,
                         keybits, (uint64_t*)bufA, (uint64_t*)bufB, tmp_cnt, leaves, st, d_out,
                         large_list);
    return hipGetLastError();
  }
  // the leaves whose table overflows are listed for launch_leaf_second
  uint32_t* const second = slots_log2 < second_slots_log2(words) ? ovf_list : nullptr;
  // few leaves: from the leaf table, but for those planned for the second count
  const bool direct = max_leaves <= kFewLeaves;
  // (unsplit: none is planned for it)
  const uint64_t small_max = second && !unsplit ? 8ull << slots_log2 : ~0ull;  // (without a list)
  const uint32_t* const list = direct ? nullptr : large_list;
  if (tiny_leaves(words, max_leaves, slots_log2, mode, refine, merged, unsplit)) {
#define KC_TINY(KRN, KT, ...)                                                                     \
  hipLaunchKernelGGL((KRN<kRescueTB, __VA_ARGS__>), dim3(glarge), dim3(kRescueTB), 0, s, keybits,  \
                     (KT*)bufA, (KT*)bufB, tmp_cnt, leaves, st, d_out, slots_log2 + 1,            \
                     (const uint32_t*)nullptr, (const unsigned long long*)nullptr,                \
                     (uint32_t*)nullptr, &st->large_records, ~0ull)
    if (words == 4) KC_TINY(k_leaf_countw256, u256, kRescueCmaxW, 1, true);
    else if (wide && keybits <= 126) KC_TINY(k_leaf_count128, u128, kRescueCmaxW, 2, true);
    else if (wide) KC_TINY(k_leaf_countw128, u128, kRescueCmaxW, 2, true);
    else KC_TINY(k_leaf_count64, uint64_t, kRescueCmax64, 4, true, false);
#undef KC_TINY
    return hipGetLastError();
  }
#define KC_LARGEW(KRN, KT, CM, R, FF)                                                             \
  hipLaunchKernelGGL((KRN<kLeafTB, CM, R, FF>), dim3(glarge), dim3(kLeafTB), 0, s, keybits,        \
                     (KT*)bufA, (KT*)bufB, tmp_cnt, leaves, st, d_out, slots_log2, list,          \
                     &st->n_large, second, &st->large_records, small_max)
#define KC_LARGE64(FF, MG)                                                                      \
  hipLaunchKernelGGL((k_leaf_count64<kLeafTB, kLeafCmax64, 4, FF, MG>), dim3(glarge),            \
                     dim3(kLeafTB), 0, s, keybits, (uint64_t*)bufA, (uint64_t*)bufB, tmp_cnt,    \
                     leaves, st, d_out, slots_log2, list, &st->n_large, second,                  \
                     &st->large_records, small_max)
  if (words == 4) {
    if (refine) KC_LARGEW(k_leaf_countw256, u256, kLeafCmax256, 2, true);
    else KC_LARGEW(k_leaf_countw256, u256, kLeafCmax256, 2, false);
  } else if (wide && keybits <= 126) {
    if (refine) KC_LARGEW(k_leaf_count128, u128, kLeafCmax128, 4, true);
    else KC_LARGEW(k_leaf_count128, u128, kLeafCmax128, 4, false);
  } else if (wide) {
    if (refine) KC_LARGEW(k_leaf_countw128, u128, kLeafCmax128, 4, true);
    else KC_LARGEW(k_leaf_countw128, u128, kLeafCmax128, 4, false);
  } else {
    if (merged) {
      if (refine) KC_LARGE64(true, true); else KC_LARGE64(false, true);
    } else {
      if (refine) KC_LARGE64(true, false); else KC_LARGE64(false, false);
    }
  }
#undef KC_LARGEW
#undef KC_LARGE64
  return hipGetLastError();
}

hipError_t launch_leaf_second(int words, int keybits, void* bufA, void* bufB, uint32_t* tmp_cnt,
                              const Leaf* leaves, DevState* st, uint64_t max_leaves,
                              uint32_t* d_out, int slots_log2, const uint32_t* ovf_list,
                              hipStream_t s, int mode, bool refine, bool merged, bool unsplit) {
  if (mode == 1 || slots_log2 >= second_slots_log2(words) || !ovf_list ||
      tiny_leaves(words, max_leaves, slots_log2, mode, refine, merged, unsplit))
    return hipSuccess;
  // the leaves whose table overflowed are counted again at once by a
  // workgroup per CU with a table twice as large (a leaf overflows because of
  // its distinct keys: clusters of keys that share a long prefix, the
  // erroneous and diverged copies of frequent k-mers, which a split on the
  // next key bits barely thins out)
#define KC_SECONDW(KRN, KT, R)                                                                    \
  hipLaunchKernelGGL((KRN<kRescueTB, kRescueCmaxW, R, true>), dim3(kRescueGrid), dim3(kRescueTB),  \
                     0, s, keybits, (KT*)bufA, (KT*)bufB, tmp_cnt, leaves, st, d_out,             \
                     slots_log2 + 1, ovf_list, &st->n_ovf, (uint32_t*)nullptr,                    \
                     &st->second_records, (uint64_t)0)
  if (words != 1) {
    if (words == 4) KC_SECONDW(k_leaf_countw256, u256, 1);
    else if (keybits <= 126) KC_SECONDW(k_leaf_count128, u128, 2);
    else KC_SECONDW(k_leaf_countw128, u128, 2);
    return hipGetLastError();
  }
#undef KC_SECONDW
  if (merged)
    hipLaunchKernelGGL((k_leaf_count64<kRescueTB, kRescueCmax64, 4, true, true>),
                       dim3(kRescueGrid), dim3(kRescueTB), 0, s, keybits, (uint64_t*)bufA,
                       (uint64_t*)bufB, tmp_cnt, leaves, st, d_out, slots_log2 + 1, ovf_list,
                       &st->n_ovf, (uint32_t*)nullptr, &st->second_records, (uint64_t)0);
  else
    hipLaunchKernelGGL((k_leaf_count64<kRescueTB, kRescueCmax64, 4, true, false>),
                       dim3(kRescueGrid), dim3(kRescueTB), 0, s, keybits, (uint64_t*)bufA,
                       (uint64_t*)bufB, tmp_cnt, leaves, st, d_out, slots_log2 + 1, ovf_list,
                       &st->n_ovf, (uint32_t*)nullptr, &st->second_records, (uint64_t)0);
  return hipGetLastError();
}

hipError_t launch_list_overflowed(const uint32_t* d, uint64_t n, const Leaf* leaves,
                                  uint32_t* list, Leaf* out, unsigned long long* count,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, s, count, (uint64_t)1, 0ull);
  if (n)
    hipLaunchKernelGGL(k_list_overflowed, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, d, n,
                       leaves, list, out, count);
  return hipGetLastError();
}

hipError_t launch_splice(const Leaf* leaves, const uint32_t* d, uint64_t n,
                         const uint32_t* root_leaf, const uint32_t* part_begin,
                         const uint32_t* nparts, uint32_t R, const Leaf* parts,
                         const uint32_t* part_d, uint32_t* cnt, DevState* st,
                         unsigned long long* bsum, unsigned long long* pos, Leaf* out,
                         uint32_t* out_d, hipStream_t s) {
  const unsigned g = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(k_splice_counts, dim3(g), dim3(256), 0, s, d, n, cnt);
  if (R)
    hipLaunchKernelGGL(k_splice_root_counts, dim3((R + 255) / 256), dim3(256), 0, s, root_leaf,
                       nparts, R, cnt);
  // st->n_leaves == n here: the scan gives every old leaf its first new slot
  hipError_t e = launch_plan_out(cnt, st, bsum, n, pos, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_splice_keep, dim3(g), dim3(256), 0, s, leaves, d, pos, n, out, out_d);
  if (R)
    hipLaunchKernelGGL(k_splice_parts, dim3(R < 4096u ? R : 4096u), dim3(64), 0, s, root_leaf,
                       part_begin, nparts, R, parts, part_d, pos, out, out_d);
  return hipGetLastError();
}

uint64_t scan_blocks(uint64_t max_leaves) { return (max_leaves + kScanTile - 1) / kScanTile; }

hipError_t launch_plan_out(const uint32_t* d, DevState* st, unsigned long long* bsum,
                           uint64_t max_leaves, unsigned long long* out_off, hipStream_t s,
                           DevState* pub) {
  if (max_leaves <= kScanOneMax) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kPlanTB), 0, s, d, st, out_off, pub);
    return hipGetLastError();
  }
  const uint64_t nb = scan_blocks(max_leaves);
  if (nb > 65536u * kPlanTB) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanTB), 0, s, d, st, bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kPlanTB), 0, s, bsum, (uint32_t)nb, st);
  hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanTB), 0, s, d, st, bsum, out_off,
                     pub);
  return hipGetLastError();
}

bool concat_plans_out(uint64_t max_leaves) { return max_leaves <= kFewLeaves; }

hipError_t launch_concat(int words, const void* bufA, const void* bufB, const uint32_t* tmp_cnt,
                         const Leaf* leaves, const uint32_t* d, const unsigned long long* out_off,
                         DevState* st, uint64_t max_leaves, uint64_t cap, uint64_t* out_keys,
                         uint32_t* out_counts, hipStream_t s, DevState* pub) {
  const unsigned grid = persistent((max_leaves + 3) / 4, 16384);
#define KC_CONCAT(K, OFFS)                                                                       \
  hipLaunchKernelGGL((k_concat<K, OFFS>), dim3(grid), dim3(256), 0, s, (const K*)bufA,           \
                     (const K*)bufB, tmp_cnt, leaves, d, out_off, st, cap, out_keys, out_counts, pub)
  if (out_off) {
    if (words == 4) KC_CONCAT(u256, true);
    else if (words == 2) KC_CONCAT(u128, true);
    else KC_CONCAT(uint64_t, true);
  } else {
    // a workgroup for every four leaves
    if (!concat_plans_out(max_leaves)) return hipErrorInvalidValue;
    if (words == 4) KC_CONCAT(u256, false);
    else if (words == 2) KC_CONCAT(u128, false);
    else KC_CONCAT(uint64_t, false);
  }
#undef KC_CONCAT
  return hipGetLastError();
}

hipError_t launch_check(int words, const uint64_t* keys, const uint32_t* counts, uint64_t n,
                        int k, CheckResult* res, hipStream_t s) {
  if (!n) return hipSuccess;
  const unsigned grid = grid_for(n, 256, 4096);
  if (words == 4)
    hipLaunchKernelGGL(k_check<u256>, dim3(grid), dim3(256), 0, s, keys, counts, n, k, res);
  else if (words == 2)
    hipLaunchKernelGGL(k_check<u128>, dim3(grid), dim3(256), 0, s, keys, counts, n, k, res);
  else
    hipLaunchKernelGGL(k_check<uint64_t>, dim3(grid), dim3(256), 0, s, keys, counts, n, k, res);
  return hipGetLastError();
}

}  // namespace kc

namespace kc {

hipError_t launch_concat_batch(int words, const void* bufA, const void* bufB,
                               const uint32_t* tmp_cnt, const Leaf* leaves, const uint32_t* d,
                               const unsigned long long* out_off, const DevState* st,
                               uint64_t max_leaves, uint64_t cap, int k, int cut_kb,
                               uint64_t* out_keys, uint32_t* out_counts, uint32_t* out_set,
                               hipStream_t s) {
  const unsigned grid = persistent((max_leaves + 3) / 4, 16384);
  if (words == 4) return hipErrorInvalidValue;
  if (words == 2)
    hipLaunchKernelGGL(k_concat_batch<u128>, dim3(grid), dim3(256), 0, s, (const u128*)bufA,
                       (const u128*)bufB, tmp_cnt, leaves, d, out_off, st, cap, k, -1, out_keys,
                       out_counts, out_set);
  else
    hipLaunchKernelGGL(k_concat_batch<uint64_t>, dim3(grid), dim3(256), 0, s,
                       (const uint64_t*)bufA, (const uint64_t*)bufB, tmp_cnt, leaves, d, out_off,
                       st, cap, k, cut_kb, out_keys, out_counts, out_set);
  return hipGetLastError();
}

hipError_t launch_set_bounds(const uint32_t* set, const DevState* st, uint64_t max_pairs,
                             uint32_t n_local, unsigned long long* start, hipStream_t s) {
  hipLaunchKernelGGL(k_set_bounds, dim3(grid_for(max_pairs + n_local + 1, 256, 4096)), dim3(256),
                     0, s, set, st, n_local, start);
  return hipGetLastError();
}

hipError_t launch_batch_offsets(const uint32_t* set_class, const uint32_t* set_local,
                                const unsigned long long* starts,
                                const unsigned long long* start_base, uint32_t n_sets,
                                unsigned long long* set_off, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_offsets, dim3(1), dim3(kPlanTB), 0, s, set_class, set_local, starts,
                     start_base, n_sets, set_off);
  return hipGetLastError();
}

hipError_t launch_batch_gather(const uint32_t* set_class, const uint32_t* set_local,
                               const unsigned long long* starts,
                               const unsigned long long* start_base,
                               const unsigned long long* class_base, const uint64_t* cls_keys,
                               const uint32_t* cls_counts, const unsigned long long* set_off,
                               uint32_t n_sets, uint64_t cap, uint64_t* out_keys,
                               uint32_t* out_counts, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_gather, dim3(2048), dim3(256), 0, s, set_class,
                     set_local, starts, start_base, class_base, cls_keys, cls_counts, set_off,
                     n_sets, cap, out_keys, out_counts);
  return hipGetLastError();
}

}  // namespace kc
