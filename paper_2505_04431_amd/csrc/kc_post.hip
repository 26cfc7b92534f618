// Uses of a count result (entry points kc_spectrum and kc_filter_min_count of
// include/kc.h): the k-mer spectrum (how many distinct keys have each count)
// and the removal of keys below a minimum count, the two most common things
// done with a k-mer histogram (the paper's Section II surveys counters that
// avoid counting singletons for the same reason).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <string>

#include "../../include/kc.h"
#include "kc_host.h"

namespace {

constexpr int kTB = 256;
constexpr int kPer = 16;  // items per thread in the compaction
constexpr int kTile = kTB * kPer;
constexpr uint32_t kLdsBins = 4096;
constexpr unsigned kSpectrumGrid = 1024;
constexpr size_t kPinBytes = 1 << 20;

// Counts [i, i + 4) of an array of n, past its end 0; one 16-byte load where
// the array is aligned and all four are in range.
__device__ __forceinline__ uint4 counts4(const uint32_t* __restrict__ counts, uint64_t i,
                                         uint64_t n, bool aligned) {
  if (aligned && i + 4 <= n) return *reinterpret_cast<const uint4*>(counts + i);
  uint4 v = make_uint4(0, 0, 0, 0);
  if (i < n) v.x = counts[i];
  if (i + 1 < n) v.y = counts[i + 1];
  if (i + 2 < n) v.z = counts[i + 2];
  if (i + 3 < n) v.w = counts[i + 3];
  return v;
}

// Spectrum: bins 1..max_count-1 hold exact counts, bin max_count everything
// at or above it. Small bin indices are counted in LDS first. Bin 1 (a k-mer
// of a read error mostly occurs once: four of five pairs) is counted in a
// register, or every lane of a wave would add to one LDS word; and the grid is
// small, as each workgroup adds its bins to the same words of hist, 12 ns an
// atomic (4,096 workgroups of one count a load: 36M counts 113 us, so 47 us).
__global__ void __launch_bounds__(kTB) k_spectrum(const uint32_t* __restrict__ counts, uint64_t n,
                                                  uint32_t max_count, bool aligned,
                                                  unsigned long long* __restrict__ hist) {
  __shared__ uint32_t h[kLdsBins];
  const uint32_t nl = max_count + 1 < kLdsBins ? max_count + 1 : kLdsBins;
  for (uint32_t i = threadIdx.x; i < nl; i += kTB) h[i] = 0;
  __syncthreads();
  uint32_t ones = 0;  // below 2^32: a thread takes n / (threads of the grid) counts
  const auto add = [&](uint32_t c) {
    const uint32_t b = c < max_count ? c : max_count;
    if (b == 1) ++ones;
    else if (b < nl) atomicAdd(&h[b], 1u);
    else atomicAdd(&hist[b], 1ull);
  };
  constexpr int U = 4;
  const uint64_t stride = (uint64_t)gridDim.x * kTB * 4;
  for (uint64_t i0 = ((uint64_t)blockIdx.x * kTB + threadIdx.x) * 4; i0 < n; i0 += U * stride) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = counts4(counts, i0 + u * stride, n, aligned);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t i = i0 + u * stride;
      if (i < n) add(v[u].x);
      if (i + 1 < n) add(v[u].y);
      if (i + 2 < n) add(v[u].z);
      if (i + 3 < n) add(v[u].w);
    }
  }
  for (int off = 32; off > 0; off >>= 1) ones += __shfl_xor(ones, off);
  if ((threadIdx.x & 63) == 0 && ones) atomicAdd(&h[1], ones);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < nl; i += kTB)
    if (h[i]) atomicAdd(&hist[i], (unsigned long long)h[i]);
}

__global__ void k_zero(unsigned long long* p, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Compaction, step 1: kept pairs per tile.
__global__ void __launch_bounds__(kTB) k_keep_count(const uint32_t* __restrict__ counts,
                                                    uint64_t n, uint32_t min_count, bool aligned,
                                                    unsigned long long* __restrict__ tsum) {
  __shared__ uint32_t wsum[kTB / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  uint4 v[kPer / 4];
#pragma unroll
  for (int j = 0; j < kPer / 4; ++j)
    v[j] = counts4(counts, base + ((uint64_t)j * kTB + threadIdx.x) * 4, n, aligned);
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < kPer / 4; ++j) {
    const uint64_t i = base + ((uint64_t)j * kTB + threadIdx.x) * 4;
    c += (i < n && v[j].x >= min_count) + (i + 1 < n && v[j].y >= min_count) +
         (i + 2 < n && v[j].z >= min_count) + (i + 3 < n && v[j].w >= min_count);
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t all = 0;
    for (int w = 0; w < kTB / 64; ++w) all += wsum[w];
    tsum[blockIdx.x] = all;
  }
}

// Step 2 (one block): exclusive scan of the tile sums; *total (host
// memory) = their sum. Rows
// of kScanTB * 8 sums, eight consecutive ones a thread, loaded while the row
// before is still being scanned (a chain of latencies, not of bytes: 9,500 sums
// 23.3 us with one thread adding up 1,024 partial sums, 21,800 sums 18.9 us so).
constexpr int kScanTB = 1024, kScanPer = 8;
__global__ void __launch_bounds__(kScanTB) k_scan_tiles(unsigned long long* __restrict__ tsum,
                                                        uint64_t nt, uint64_t* total) {
  __shared__ unsigned long long wtot[2][kScanTB / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long carry = 0;
  unsigned long long v[kScanPer];
  const auto load = [&](uint64_t row) {
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const uint64_t i = row + (uint64_t)threadIdx.x * kScanPer + q;
      v[q] = i < nt ? tsum[i] : 0ull;
    }
  };
  load(0);
  int buf = 0;
  for (uint64_t row = 0; row < nt; row += (uint64_t)kScanTB * kScanPer, buf ^= 1) {
    unsigned long long now[kScanPer], s = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      now[q] = s;
      s += v[q];
    }
    load(row + (uint64_t)kScanTB * kScanPer);
    unsigned long long x = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned long long y = __shfl_up(x, (unsigned)off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wtot[buf][w] = x;
    __syncthreads();
    unsigned long long before = carry, all = 0;
#pragma unroll
    for (int t = 0; t < kScanTB / 64; ++t) {
      if (t < w) before += wtot[buf][t];
      all += wtot[buf][t];
    }
    carry += all;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const uint64_t i = row + (uint64_t)threadIdx.x * kScanPer + q;
      if (i < nt) tsum[i] = before + (x - s) + now[q];
    }
  }
  if (threadIdx.x == 0) *total = carry;
}

// Step 3: each tile writes its kept pairs in order from its offset. A wave
// takes kTile / 4 consecutive pairs, four a lane and row, and ranks them by
// ballots (the kept pairs of earlier lanes, then the lane's own earlier ones):
// one exchange between the waves per tile instead of two barriers per row
// (36M pairs of one word, 18% kept: 145 -> 110 us, bound by the keys of kept
// pairs, which touch four of five 64-byte segments). Wider keys are copied word
// by word from the wave's list of kept places, consecutive lanes consecutive
// words (a lane that copies its four pairs' keys itself stores 8 bytes 64 or
// 128 apart: 20M pairs all kept, two words 372 -> 188 us, four words 674 -> 310).
template <int W>
__global__ void __launch_bounds__(kTB) k_keep_write(const uint64_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ counts,
                                                    uint64_t n, uint32_t min_count, bool aligned,
                                                    const unsigned long long* __restrict__ tsum,
                                                    uint64_t* __restrict__ out_keys,
                                                    uint32_t* __restrict__ out_counts) {
  constexpr int ROWS = kPer / 4;
  __shared__ uint32_t wsum[kTB / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t base = (uint64_t)blockIdx.x * kTile + (uint64_t)w * (kTile / (kTB / 64));
  uint32_t c[ROWS][4];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const uint4 v = counts4(counts, base + (uint64_t)j * 256 + lane * 4, n, aligned);
    c[j][0] = v.x;
    c[j][1] = v.y;
    c[j][2] = v.z;
    c[j][3] = v.w;
  }
  const unsigned long long below = (1ull << lane) - 1;
  uint32_t rank[ROWS], keep[ROWS], sum = 0;  // rank of the lane's first kept pair in the wave
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    keep[j] = 0;
    rank[j] = sum;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t i = base + (uint64_t)j * 256 + lane * 4 + q;
      const bool k = i < n && c[j][q] >= min_count;
      const unsigned long long m = __ballot(k);
      rank[j] += __popcll(m & below);
      sum += __popcll(m);
      keep[j] |= (k ? 1u : 0u) << q;
    }
  }
  // places of the wave's kept pairs, in their order
  constexpr int PER_WAVE = kTile / (kTB / 64);
  __shared__ uint16_t s_pos[W > 1 ? kTile : 1];
  if constexpr (W > 1) {
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      uint32_t r = w * PER_WAVE + rank[j];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (keep[j] >> q & 1) s_pos[r++] = (uint16_t)(j * 256 + lane * 4 + q);
    }
  }
  if (lane == 0) wsum[w] = sum;
  __syncthreads();
  unsigned long long at = tsum[blockIdx.x];
  for (int v = 0; v < w; ++v) at += wsum[v];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    unsigned long long o = at + rank[j];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!(keep[j] >> q & 1)) continue;
      out_counts[o] = c[j][q];
      if constexpr (W == 1) out_keys[o] = keys[base + (uint64_t)j * 256 + lane * 4 + q];
      ++o;
    }
  }
  if constexpr (W > 1) {
    constexpr uint32_t U = 4;
    const uint64_t* const src = keys + W * base;
    uint64_t* const dst = out_keys + W * at;
    for (uint32_t t0 = lane; t0 < W * sum; t0 += 64 * U) {
      uint64_t x[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t t = t0 + u * 64;
        if (t < W * sum) x[u] = src[W * s_pos[w * PER_WAVE + t / W] + t % W];
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
        if (t0 + u * 64 < W * sum) dst[t0 + u * 64] = x[u];
    }
  }
}

struct Fail {
  int code;
};

void chk(hipError_t e, const char* what) {
  if (e != hipSuccess) {
    (void)hipGetLastError();
    kc::set_last_error(std::string(what) + ": " + hipGetErrorString(e));
    throw Fail{e == hipErrorOutOfMemory ? KC_E_NOMEM : KC_E_DEVICE};
  }
}

int bad(const char* msg) {
  kc::set_last_error(msg);
  return KC_E_INVAL;
}

// Temporary device memory of the merge and the filter: the calling thread's
// buffer, kept between calls (kc_release_scratch frees it).
void* post_scratch(size_t bytes, hipStream_t st) {
  std::string err;
  int code = KC_E_NOMEM;
  void* p = kc::thread_scratch(bytes, st, &err, &code);
  if (!p) {
    kc::set_last_error(err);
    throw Fail{code};
  }
  return p;
}

// Host words that kernels write their results to (with their device address):
// the calling thread's pinned staging memory.
uint64_t* post_words(size_t n, uint64_t** dev) {
  std::string err;
  int code = KC_E_NOMEM;
  void* d = nullptr;
  uint64_t* p = (uint64_t*)kc::thread_pinned(n * 8, &d, &err, &code);
  if (!p) {
    kc::set_last_error(err);
    throw Fail{code};
  }
  *dev = (uint64_t*)d;
  return p;
}

unsigned grid_of(uint64_t n, uint64_t per, unsigned cap) {
  const uint64_t g = (n + per - 1) / per;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace


extern "C" {

int kc_spectrum(const uint32_t* counts, uint64_t n, uint32_t max_count, uint64_t* host_hist,
                void* stream) {
  kc::set_last_error("");
  if (!host_hist) return bad("host_hist is NULL");
  if (n && !counts) return bad("counts is NULL");
  if (max_count < 1 || max_count > (1u << 24)) return bad("max_count must be in [1, 2^24]");
  const hipStream_t st = (hipStream_t)stream;
  try {
    const size_t bytes = (size_t)(max_count + 1) * 8;
    unsigned long long* hist = (unsigned long long*)post_scratch(bytes, st);
    hipLaunchKernelGGL(k_zero, dim3(grid_of(max_count + 1, 256, 1u << 20)), dim3(256), 0, st,
                       hist, (uint64_t)max_count + 1);
    if (n)
      hipLaunchKernelGGL(k_spectrum, dim3(grid_of(n, (uint64_t)kTB * 16, kSpectrumGrid)),
                         dim3(kTB), 0, st, counts, n, max_count, ((uintptr_t)counts & 15) == 0,
                         hist);
    chk(hipGetLastError(), "spectrum launch");
    // through pinned memory where it is small: a copy to pageable memory is
    // staged piece by piece
    uint64_t* dev = nullptr;
    uint64_t* const pin = bytes <= kPinBytes ? post_words(max_count + 1, &dev) : nullptr;
    chk(hipMemcpyAsync(pin ? pin : host_hist, hist, bytes, hipMemcpyDeviceToHost, st),
        "hipMemcpyAsync");
    chk(hipStreamSynchronize(st), "hipStreamSynchronize");
    if (pin) std::memcpy(host_hist, pin, bytes);
  } catch (const Fail& f) {
    return f.code;
  }
  return KC_OK;
}

int kc_filter_min_count(const uint64_t* keys, const uint32_t* counts, uint64_t n, int k,
                        uint32_t min_count, uint64_t* out_keys, uint32_t* out_counts,
                        uint64_t* n_out, void* stream) {
  kc::set_last_error("");
  if (!n_out) return bad("n_out is NULL");
  *n_out = 0;
  if (k < 1 || k > 128) return bad("k must be in [1, 128]");
  if (n && (!keys || !counts || !out_keys || !out_counts)) return bad("NULL array");
  if (n == 0) return KC_OK;
  const int words = k <= 32 ? 1 : (k <= 64 ? 2 : 4);
  const hipStream_t st = (hipStream_t)stream;
  const uint64_t nt = (n + kTile - 1) / kTile;
  void* d = nullptr;
  try {
    d = post_scratch((size_t)nt * 8, st);
    unsigned long long* tsum = (unsigned long long*)d;
    uint64_t* total_dev = nullptr;
    const uint64_t* const total = post_words(1, &total_dev);
    const bool aligned = ((uintptr_t)counts & 15) == 0;
    hipLaunchKernelGGL(k_keep_count, dim3((unsigned)nt), dim3(kTB), 0, st, counts, n, min_count,
                       aligned, tsum);
    hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(kScanTB), 0, st, tsum, nt, total_dev);
    if (words == 4)
      hipLaunchKernelGGL(k_keep_write<4>, dim3((unsigned)nt), dim3(kTB), 0, st, keys, counts, n,
                         min_count, aligned, tsum, out_keys, out_counts);
    else if (words == 2)
      hipLaunchKernelGGL(k_keep_write<2>, dim3((unsigned)nt), dim3(kTB), 0, st, keys, counts, n,
                         min_count, aligned, tsum, out_keys, out_counts);
    else
      hipLaunchKernelGGL(k_keep_write<1>, dim3((unsigned)nt), dim3(kTB), 0, st, keys, counts, n,
                         min_count, aligned, tsum, out_keys, out_counts);
    chk(hipGetLastError(), "filter launch");
    chk(hipStreamSynchronize(st), "hipStreamSynchronize");
    *n_out = *total;
  } catch (const Fail& f) {
    return f.code;
  }
  return KC_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- merging two results

namespace {

// Key i of a result (W = 1, 2 or 4 words, least significant first) as one
// comparable value.
struct Key4 {
  unsigned __int128 lo, hi;
};
__device__ __forceinline__ bool operator<(const Key4& a, const Key4& b) {
  return a.hi != b.hi ? a.hi < b.hi : a.lo < b.lo;
}
__device__ __forceinline__ bool operator==(const Key4& a, const Key4& b) {
  return a.hi == b.hi && a.lo == b.lo;
}

template <int W> struct KeyOf { typedef unsigned __int128 type; };
template <> struct KeyOf<4> { typedef Key4 type; };

template <int W>
__device__ __forceinline__ typename KeyOf<W>::type key_at(const uint64_t* keys, uint64_t i) {
  if constexpr (W == 4) {
    const uint64_t* p = keys + 4 * i;
    return Key4{((unsigned __int128)p[1] << 64) | p[0], ((unsigned __int128)p[3] << 64) | p[2]};
  } else if constexpr (W == 2) {
    return ((unsigned __int128)keys[2 * i + 1] << 64) | keys[2 * i];
  } else {
    return keys[i];
  }
}

template <int W>
__device__ __forceinline__ void key_put(uint64_t* keys, uint64_t i,
                                        const typename KeyOf<W>::type& v) {
  if constexpr (W == 4) {
    keys[4 * i] = (uint64_t)v.lo;
    keys[4 * i + 1] = (uint64_t)(v.lo >> 64);
    keys[4 * i + 2] = (uint64_t)v.hi;
    keys[4 * i + 3] = (uint64_t)(v.hi >> 64);
  } else if constexpr (W == 2) {
    keys[2 * i] = (uint64_t)v;
    keys[2 * i + 1] = (uint64_t)(v >> 64);
  } else {
    keys[i] = (uint64_t)v;
  }
}

// Merged positions per thread and per block (words of a key W): a block's keys
// and counts are staged in LDS, 21 KiB for one-word keys, so seven 256-thread
// blocks share a CU; wider keys take fewer positions for the same LDS. The
// number is odd so that the threads' positions spread over all LDS banks (8 a
// thread, keys 64 bytes apart: the second pass below 327 instead of 154 us).
template <int W> constexpr int kMergeItems = W == 1 ? 7 : W == 2 ? 5 : 3;
template <int W> constexpr int kMergeTileOf = kTB * kMergeItems<W>;

// Number of a's among the first d merged positions (a first on ties), by
// binary search over i in [lo, hi]: the largest i with a[i-1] <= b[d-i].
template <int W, typename I>
__device__ __forceinline__ I merge_split(const uint64_t* ak, const uint64_t* bk, I nb, I d, I lo,
                                         I hi) {
  while (lo < hi) {
    const I i = (lo + hi + 1) >> 1;  // candidate: take i items of a
    if (d - i >= nb || !(key_at<W>(bk, d - i) < key_at<W>(ak, i - 1))) lo = i;
    else hi = i - 1;
  }
  return lo;
}

// Split of every block boundary: part[2q], part[2q + 1] are the a's and b's
// before diagonal q * tile, q = 0..nblocks. A key that both inputs hold is
// never cut: if a's copy is the last one before the diagonal, b's is taken
// with it (a block has up to tile + 1 positions), so every output pair is
// made by one block. The search is a chain of dependent loads (25 halvings of
// 20M pairs: 32 us; by 4 or 16 lanes a search no less, 35 and 56 us: more
// pages are touched), so it starts where the split lies if both inputs are
// spread alike over the keys, as two results of one genome are, and widens
// from there (18.7 us).
template <int W>
__global__ void __launch_bounds__(kTB) k_merge_part(const uint64_t* __restrict__ ak, uint64_t na,
                                                    const uint64_t* __restrict__ bk, uint64_t nb,
                                                    uint64_t nblocks,
                                                    unsigned long long* __restrict__ part) {
  const uint64_t q = (uint64_t)blockIdx.x * kTB + threadIdx.x;
  if (q > nblocks) return;
  const uint64_t total = na + nb, at = q * kMergeTileOf<W>;
  const uint64_t d = at < total ? at : total;
  uint64_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
  // held(i): i a's lie before the diagonal (true up to the split, and at lo)
  const auto held = [&](uint64_t i) {
    return i == 0 || d - i >= nb || !(key_at<W>(bk, d - i) < key_at<W>(ak, i - 1));
  };
  uint64_t g = (uint64_t)((double)d * (double)na / (double)total);
  g = g < lo ? lo : g > hi ? hi : g;
  uint64_t w = kMergeTileOf<W>;
  if (held(g)) {
    lo = g;
    for (; hi - lo > w; w *= 8) {
      if (!held(lo + w)) {
        hi = lo + w - 1;
        break;
      }
      lo += w;
    }
  } else {
    hi = g - 1;  // g > lo: held(lo)
    for (; hi - lo > w; w *= 8) {
      if (held(hi - w)) {
        lo = hi - w;
        break;
      }
      hi -= w + 1;
    }
  }
  const uint64_t i = merge_split<W, uint64_t>(ak, bk, nb, d, lo, hi);
  uint64_t j = d - i;
  if (i > 0 && j < nb && key_at<W>(ak, i - 1) == key_at<W>(bk, j)) ++j;
  part[2 * q] = i;
  part[2 * q + 1] = j;
}

// One block's part of the ordered union: its a's and b's are staged in LDS
// (coalesced loads); each thread finds its diagonal there by binary search,
// with a pair of equal keys kept whole as in k_merge_part, and walks its
// kMergeItems positions once, an equal pair giving one output with the counts
// added. WRITE = false: only the number of outputs (tsum[block]); WRITE: the
// outputs, gathered in LDS by a block scan and written as one coalesced run
// from tsum[block] (the exclusive scan of the first pass's numbers).
// Reading the keys twice costs less than a merged copy of both inputs written
// and read again: bound by HBM (W = 1: 8 bytes of each input pair in the first
// pass, 12 read and 12 written in the second). 20M + 19M pairs of one-word keys,
// 34M results: 84 and 154 us, 3.7 and 5.7 TB/s; the whole call 0.31 ms (a
// merged copy by threads that read and wrote eight positions each on their
// own, then two passes over it: 1.49 of 1.91 ms in the merge itself).
template <int W, bool WRITE>
__global__ void __launch_bounds__(kTB) k_merge(const uint64_t* __restrict__ ak,
                                               const uint32_t* __restrict__ ac,
                                               const uint64_t* __restrict__ bk,
                                               const uint32_t* __restrict__ bc,
                                               const unsigned long long* __restrict__ part,
                                               unsigned long long* __restrict__ tsum,
                                               uint64_t* __restrict__ out_keys,
                                               uint32_t* __restrict__ out_counts,
                                               uint64_t* overflow) {
  constexpr int ITEMS = kMergeItems<W>, TILE = kMergeTileOf<W>;
  typedef typename KeyOf<W>::type Key;
  __shared__ uint64_t sk[W * (TILE + 1)];      // a's keys, then b's; then the outputs'
  __shared__ uint32_t sc[WRITE ? TILE + 1 : 1];  // their counts
  __shared__ uint32_t split[kTB + 1];          // per thread: a's and b's before it (16 bits each)
  __shared__ uint32_t wsum[kTB / 64];
  const uint64_t a0 = part[2 * blockIdx.x], b0 = part[2 * blockIdx.x + 1];
  const uint32_t la = (uint32_t)(part[2 * blockIdx.x + 2] - a0);
  const uint32_t lb = (uint32_t)(part[2 * blockIdx.x + 3] - b0);
  const uint32_t n = la + lb;
  // the block's key words, a's then b's, all loads in flight together (the
  // last word of a tile of TILE + 1 positions by itself)
  uint64_t v[ITEMS * W];
  uint32_t vc[WRITE ? ITEMS : 1];
  const uint64_t* const ka0 = ak + W * a0;
  const uint64_t* const kb0 = bk + W * b0 - W * (uint64_t)la;
#pragma unroll
  for (int s = 0; s < ITEMS * W; ++s) {
    const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
    if (t < W * n) v[s] = t < W * la ? ka0[t] : kb0[t];
  }
  if (WRITE) {
#pragma unroll
    for (int s = 0; s < ITEMS; ++s) {
      const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
      if (t < n) vc[s] = t < la ? ac[a0 + t] : bc[b0 + (t - la)];
    }
  }
#pragma unroll
  for (int s = 0; s < ITEMS * W; ++s) {
    const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
    if (t < W * n) sk[t] = v[s];
  }
  if (n > TILE && threadIdx.x < W) {
    const uint32_t t = W * TILE + threadIdx.x;
    sk[t] = t < W * la ? ka0[t] : kb0[t];
  }
  if (WRITE) {
#pragma unroll
    for (int s = 0; s < ITEMS; ++s) {
      const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
      if (t < n) sc[t] = vc[s];
    }
    if (n > TILE && threadIdx.x == 0) sc[TILE] = TILE < la ? ac[a0 + TILE] : bc[b0 + (TILE - la)];
  }
  __syncthreads();
  const uint64_t* const sb = sk + W * la;
  const uint32_t d = min(n, (uint32_t)threadIdx.x * ITEMS);
  uint32_t i = merge_split<W, uint32_t>(sk, sb, lb, d, d > lb ? d - lb : 0u, min(d, la));
  uint32_t j = d - i;
  if (i > 0 && j < lb && key_at<W>(sk, i - 1) == key_at<W>(sb, j)) ++j;
  split[threadIdx.x] = i << 16 | j;
  if (threadIdx.x == 0) split[kTB] = la << 16 | lb;
  __syncthreads();
  // a tile of TILE + 1 positions leaves its last one to the last thread
  const uint32_t next = split[threadIdx.x + 1], i1 = next >> 16, j1 = next & 0xFFFFu;
  Key key[WRITE ? ITEMS + 1 : 1];
  uint32_t cnt[WRITE ? ITEMS + 1 : 1];
  uint32_t u = 0;
  bool over = false;
  Key ka{}, kb{};
  if (i < i1) ka = key_at<W>(sk, i);
  if (j < j1) kb = key_at<W>(sb, j);
#pragma unroll
  for (int s = 0; s < ITEMS + 1; ++s) {
    const bool ha = i < i1, hb = j < j1;
    if (!(ha || hb)) break;
    const bool take_a = ha && (!hb || !(kb < ka)), take_b = hb && (!ha || !(ka < kb));
    if (WRITE) {
      key[s] = take_a ? ka : kb;
      const unsigned long long c =
          (unsigned long long)(take_a ? sc[i] : 0u) + (take_b ? sc[la + j] : 0u);
      over |= c > 0xFFFFFFFFull;
      cnt[s] = (uint32_t)c;
    }
    ++u;
    if (take_a && ++i < i1) ka = key_at<W>(sk, i);
    if (take_b && ++j < j1) kb = key_at<W>(sb, j);
  }
  // exclusive prefix of u over the block
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = u;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, (unsigned)off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();  // also: every thread has taken its keys and counts from LDS
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int v = 0; v < kTB / 64; ++v) {
    if (v < w) before += wsum[v];
    all += wsum[v];
  }
  if (!WRITE) {
    if (threadIdx.x == 0) tsum[blockIdx.x] = all;
    return;
  }
  const uint32_t at = before + x - u;
#pragma unroll
  for (int s = 0; s < ITEMS + 1; ++s) {
    if (s >= (int)u) break;
    key_put<W>(sk, at + s, key[s]);
    sc[at + s] = cnt[s];
  }
  if (over) *overflow = 1;
  __syncthreads();
  const unsigned long long o = tsum[blockIdx.x];
#pragma unroll
  for (int s = 0; s <= ITEMS * W; ++s) {
    const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
    if (t < W * all) out_keys[W * o + t] = sk[t];
  }
#pragma unroll
  for (int s = 0; s <= ITEMS; ++s) {
    const uint32_t t = (uint32_t)s * kTB + threadIdx.x;
    if (t < all) out_counts[o + t] = sc[t];
  }
}

template <int W>
void launch_merge(const uint64_t* ak, const uint32_t* ac, uint64_t na, const uint64_t* bk,
                  const uint32_t* bc, uint64_t nb, uint64_t nblk, unsigned long long* part,
                  unsigned long long* tsum, uint64_t* out_keys, uint32_t* out_counts,
                  uint64_t* result, hipStream_t st) {
  hipLaunchKernelGGL(k_merge_part<W>, dim3(grid_of(nblk + 1, kTB, ~0u)), dim3(kTB), 0,
                     st, ak, na, bk, nb, nblk, part);
  hipLaunchKernelGGL((k_merge<W, false>), dim3((unsigned)nblk), dim3(kTB), 0, st, ak, ac, bk, bc,
                     part, tsum, out_keys, out_counts, result + 1);
  hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(kScanTB), 0, st, tsum, nblk, result);
  hipLaunchKernelGGL((k_merge<W, true>), dim3((unsigned)nblk), dim3(kTB), 0, st, ak, ac, bk, bc,
                     part, tsum, out_keys, out_counts, result + 1);
}

}  // namespace

extern "C" int kc_merge_counts(const uint64_t* a_keys, const uint32_t* a_counts, uint64_t na,
                               const uint64_t* b_keys, const uint32_t* b_counts, uint64_t nb,
                               int k, uint64_t* out_keys, uint32_t* out_counts, uint64_t* n_out,
                               void* stream) {
  kc::set_last_error("");
  if (!n_out) return bad("n_out is NULL");
  *n_out = 0;
  if (k < 1 || k > 128) return bad("k must be in [1, 128]");
  if ((na && (!a_keys || !a_counts)) || (nb && (!b_keys || !b_counts)))
    return bad("NULL input array");
  const uint64_t n = na + nb;
  if (n && (!out_keys || !out_counts)) return bad("NULL output array");
  if (n == 0) return KC_OK;
  const int words = k <= 32 ? 1 : (k <= 64 ? 2 : 4);
  const hipStream_t st = (hipStream_t)stream;
  const uint64_t tile = words == 4 ? kMergeTileOf<4> : words == 2 ? kMergeTileOf<2> : kMergeTileOf<1>;
  const uint64_t nblk = (n + tile - 1) / tile;
  if (nblk > 0x7fffffffull) return bad("too many pairs");
  void* d = nullptr;
  try {
    // tile sums, splits
    d = post_scratch((nblk + 2 * (nblk + 1)) * 8, st);
    unsigned long long* tsum = (unsigned long long*)d;
    unsigned long long* part = tsum + nblk;
    // the number of results and whether a count passed 2^32-1, in host memory
    uint64_t* res_dev = nullptr;
    volatile uint64_t* const res = post_words(2, &res_dev);
    res[1] = 0;
    if (words == 4)
      launch_merge<4>(a_keys, a_counts, na, b_keys, b_counts, nb, nblk, part, tsum, out_keys,
                      out_counts, res_dev, st);
    else if (words == 2)
      launch_merge<2>(a_keys, a_counts, na, b_keys, b_counts, nb, nblk, part, tsum, out_keys,
                      out_counts, res_dev, st);
    else
      launch_merge<1>(a_keys, a_counts, na, b_keys, b_counts, nb, nblk, part, tsum, out_keys,
                      out_counts, res_dev, st);
    chk(hipGetLastError(), "merge launch");
    chk(hipStreamSynchronize(st), "hipStreamSynchronize");
    if (res[1]) {
      kc::set_last_error("a merged count exceeds 2^32-1");
      return KC_E_OVERFLOW;
    }
    *n_out = res[0];
  } catch (const Fail& f) {
    return f.code;
  }
  return KC_OK;
}
