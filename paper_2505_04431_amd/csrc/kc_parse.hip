// Parsing of FASTQ and FASTA text held in device memory into the reads +
// offsets form the counter takes (entry point kc_parse_fastx of include/kc.h).
// The paper leaves input parsing out of its measurements (Section VI); this
// lets a file's bytes be copied to the device as they are and counted there.
//
// Two passes over the text (tiles of 16 KiB, 16 bytes per thread and round,
// loads of whole aligned 16-byte chunks):
//   1. per tile: newlines, FASTA header starts, start of the last line, and how
//      many bytes it keeps (sequence-line bytes other than CR/LF) for every
//      state in which a line may enter it: which of a record's four lines is
//      open (FASTQ), or whether a header is (FASTA). Scans over the tiles then
//      give each tile its state, kept bytes and output offset;
//   2. kept bytes written in order, straight from the registers (a chunk's kept
//      bytes are one run in all but a few chunks), one offset per record, and
//      the FASTQ layout check.
// Nothing between the passes needs the host: the range without line ends at
// either end, the format and the outputs' room are looked at on the device,
// and one synchronization reads the results. 320 MB of FASTQ: 515 -> 314 us
// (a pass of its own for the kept bytes read the text a third time, 139 us,
// and three synchronizations took 90 us).
// Every position a kernel reads is inside [lo, hi) of the trimmed text.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/kc.h"
#include "kc_host.h"

namespace {

typedef unsigned long long ull;

constexpr int kTB = 256;
constexpr int kRounds = 4;
constexpr int kChunk = 16;
constexpr uint64_t kTile = (uint64_t)kTB * kRounds * kChunk;  // 16 KiB

struct Plus {
  __device__ ull operator()(ull a, ull b) const { return a + b; }
};
struct Max {
  __device__ ull operator()(ull a, ull b) const { return a > b ? a : b; }
};
// four 16-bit fields, each its own maximum
struct Max4 {
  __device__ ull operator()(ull a, ull b) const {
    ull r = 0;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const ull x = (a >> (16 * f)) & 0xFFFFu, y = (b >> (16 * f)) & 0xFFFFu;
      r |= (x > y ? x : y) << (16 * f);
    }
    return r;
  }
};

__device__ __forceinline__ uint32_t field(ull v, int f) { return (uint32_t)(v >> (16 * f)) & 0xFFFFu; }

// Exclusive scan over the block (NT threads) in thread order; *total
// receives the reduction of all threads. sh holds NT / 64 values; reusable on
// return.
template <class Op, int NT = kTB>
__device__ ull block_exscan(ull v, Op op, ull* sh, ull* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  ull x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const ull y = __shfl_up(x, (unsigned)d, 64);
    if (lane >= d) x = op(y, x);
  }
  ull ex = __shfl_up(x, 1u, 64);
  if (lane == 0) ex = 0;
  if (lane == 63) sh[w] = x;
  __syncthreads();
  ull before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    if (i < w) before = op(before, sh[i]);
    all = op(all, sh[i]);
  }
  __syncthreads();
  *total = all;
  return op(before, ex);
}

__device__ __forceinline__ uint32_t byte_of(const uint4& v, int j) {
  const uint32_t w = j < 4 ? v.x : j < 8 ? v.y : j < 12 ? v.z : v.w;
  return (w >> (8 * (j & 3))) & 0xFFu;
}

struct Ld {
  uint4 v;
  uint32_t m;
};

// Bytes [pos, pos + 16) of B; bit j of m is set when pos + j lies in
// [lo, hi) (other bytes read as 0). Only whole in-range chunks use the
// 16-byte load.
__device__ __forceinline__ Ld load16(const uint8_t* __restrict__ B, uint64_t pos, uint64_t lo,
                                     uint64_t hi) {
  if (pos >= lo && pos + kChunk <= hi) return Ld{*reinterpret_cast<const uint4*>(B + pos), 0xFFFFu};
  // partial chunk (first or last of the text): byte loads
  ull w0 = 0, w1 = 0;
  uint32_t m = 0;
  for (int j = 0; j < kChunk; ++j) {
    const uint64_t p = pos + j;
    if (p >= lo && p < hi) {
      const ull b = B[p];
      if (j < 8) w0 |= b << (8 * j);
      else w1 |= b << (8 * (j - 8));
      m |= 1u << j;
    }
  }
  return Ld{make_uint4((uint32_t)w0, (uint32_t)(w0 >> 32), (uint32_t)w1, (uint32_t)(w1 >> 32)), m};
}

// x's bytes as 0xFF where not zero, 0x7F where zero: (x & 0x7F..) + 0x7F.. sets
// a byte's top bit when its low seven bits are not all zero, without carries
// between bytes; OR-ing x adds its own top bit.
__device__ __forceinline__ uint32_t mark_zero(uint32_t x) {
  return ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu;
}

// Bit j set where byte j equals ch. The marks' top bits are gathered by dot
// products with the bit weights: bytes of 127 + 128 * (not equal) times 1, 2,
// .. 128 sum to 127 * 255 + 128 * (mask of the bytes not equal). (Both passes
// are bound by this arithmetic: five instructions a word, thirteen with a
// multiply that gathers four bits.)
__device__ __forceinline__ uint32_t eq_mask(const uint4& v, uint32_t ch) {
  const uint32_t c4 = ch * 0x01010101u, lo = 0x08040201u, hi = 0x80402010u, base = 0u - 127u * 255u;
  const uint32_t a = __builtin_amdgcn_udot4(
      mark_zero(v.x ^ c4), lo, __builtin_amdgcn_udot4(mark_zero(v.y ^ c4), hi, base, false), false);
  const uint32_t b = __builtin_amdgcn_udot4(
      mark_zero(v.z ^ c4), lo, __builtin_amdgcn_udot4(mark_zero(v.w ^ c4), hi, base, false), false);
  return (a >> 7 | b << 1) ^ 0xFFFFu;
}

// The tile's four chunks of this thread (round r: tile bytes
// [(r * kTB + t) * 16, +16)), their validity masks and newline masks.
struct Chunks {
  uint4 v[kRounds];
  uint32_t m[kRounds], nl[kRounds];
};

__device__ __forceinline__ Chunks load_tile(const uint8_t* __restrict__ B, uint64_t tile0,
                                            uint64_t lo, uint64_t hi) {
  Chunks c;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t pos = tile0 + ((uint64_t)r * kTB + threadIdx.x) * kChunk;
    const Ld x = pos < hi ? load16(B, pos, lo, hi) : Ld{make_uint4(0, 0, 0, 0), 0u};
    c.v[r] = x.v;
    c.m[r] = x.m;
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) c.nl[r] = eq_mask(c.v[r], '\n') & c.m[r];
  return c;
}

// Local line-start value of a chunk: tile offset of the byte after its last
// newline (1..16384), 0 when it has none.
__device__ __forceinline__ uint32_t last_start(uint32_t nlm, int r) {
  return nlm ? (uint32_t)((r * kTB + threadIdx.x) * kChunk) + (32u - __clz(nlm)) : 0u;
}

// What the passes find out, on the device and for the host.
struct Info {
  uint64_t lo, hi;      // the text without line ends at its ends, positions in B
  uint32_t fasta, first;  // format taken; the first byte
  uint32_t missing;     // 1, 2: nothing but line ends in the first, last kPeekMost bytes
  uint32_t tail;        // line ends after the last byte, if not missing
  ull newlines, headers, keep, err;  // err: first malformed FASTQ line, ~0 if none
};

// How far from its ends the device looks for a text's first and last byte, and
// the bytes it looks at in a step: a round of memory latency each, 1.0 ms for 1
// MiB of line ends. The host then goes on from there, a copy and a wait for
// each kPeek bytes, 5.2 ms a MiB. (With 4 KiB looked at here, 5,000 line ends
// before a text of 143 us cost 256 us: the passes were launched for nothing, then
// the host looked further, then they were launched again. Now they cost nothing.)
constexpr uint64_t kPeek = 4096, kPeekMost = 1 << 20;

// One block: [lo, hi), the first byte and the format, if the first and last
// kPeekMost bytes each hold a byte that is not CR/LF (else the host looks further).
__global__ void __launch_bounds__(kTB) k_fx_ends(const uint8_t* __restrict__ text, uint64_t n,
                                                 uint64_t a0, int format, Info* info) {
  __shared__ uint32_t s_head, s_tail;  // bytes before the first, after the last; ~0: none yet
  if (threadIdx.x == 0) s_head = s_tail = ~0u;
  __syncthreads();
  const uint32_t most = (uint32_t)(n < kPeekMost ? n : kPeekMost);
  bool need_head = true, need_tail = true;
  for (uint32_t c = 0; c < most && (need_head || need_tail); c += (uint32_t)kPeek) {
    uint32_t head = ~0u, tail = ~0u;
#pragma unroll
    for (uint32_t j = 0; j < kPeek / kTB; ++j) {
      const uint32_t i = c + j * kTB + threadIdx.x;
      const uint8_t x = i < most ? text[i] : '\n', y = i < most ? text[n - 1 - i] : '\n';
      if (x != '\n' && x != '\r' && head == ~0u) head = i;
      if (y != '\n' && y != '\r' && tail == ~0u) tail = i;
    }
    if (need_head && head != ~0u) atomicMin(&s_head, head);
    if (need_tail && tail != ~0u) atomicMin(&s_tail, tail);
    __syncthreads();
    need_head = s_head == ~0u;
    need_tail = s_tail == ~0u;
    __syncthreads();  // all have read them before the next step writes
  }
  if (threadIdx.x != 0) return;
  Info r = {};
  r.missing = n > most ? (need_head ? 1u : 0u) | (need_tail ? 2u : 0u) : 0u;
  const uint64_t s0 = need_head ? n : s_head;
  r.lo = a0 + s0;
  r.tail = s_tail;
  r.hi = need_tail ? r.lo : a0 + n - s_tail;
  if (r.missing) r.hi = r.lo;  // the passes that follow see no text
  r.first = s0 < n ? text[s0] : 0;
  r.fasta = format == KC_FASTA || (format == KC_FASTX_AUTO && r.first == '>');
  r.err = ~0ull;
  *info = r;
}

// A tile's kept bytes by the state at its start, 16 bits each. FASTQ: field q
// = bytes of the tile's lines q, q + 4, ... (line 0 is the one open at its
// start), so the lines with index 1 mod 4 are field (1 - first line) mod 4.
// FASTA: field 0 = bytes before the first newline (kept unless a header is
// open), field 1 = kept bytes after it.
__global__ void __launch_bounds__(kTB) k_fx_lines(const uint8_t* __restrict__ B,
                                                  const Info* __restrict__ info,
                                                  ull* __restrict__ t_nl, ull* __restrict__ t_hd,
                                                  ull* __restrict__ t_ls,
                                                  ull* __restrict__ t_cls) {
  __shared__ ull sh[kTB / 64];
  const uint64_t lo = info->lo, hi = info->hi;
  const uint32_t fasta = info->fasta;
  const uint64_t tile0 = (uint64_t)blockIdx.x * kTile;
  const Chunks c = load_tile(B, tile0, lo, hi);
  ull nl4 = 0;
  uint32_t hd = 0, ls = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    nl4 |= (ull)__popc(c.nl[r]) << (16 * r);
    const uint32_t s = last_start(c.nl[r], r);
    ls = s > ls ? s : ls;
  }
  ull tot_nl4;
  const ull ex_nl4 = block_exscan(nl4, Plus(), sh, &tot_nl4);
  ull ex_ls4 = 0, tot_ls4 = 0;
  if (fasta) {
    ull ls4 = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) ls4 |= (ull)last_start(c.nl[r], r) << (16 * r);
    ex_ls4 = block_exscan(ls4, Max4(), sh, &tot_ls4);
  }
  ull cls = 0;
  uint32_t nl_before = 0, ls_before = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    uint32_t line = nl_before + field(ex_nl4, r);  // of the chunk's first byte, in the tile
    nl_before += field(tot_nl4, r);
    // where that line starts, in the tile (0: before it)
    const uint32_t ls0 = ls_before > field(ex_ls4, r) ? ls_before : field(ex_ls4, r);
    ls_before = ls_before > field(tot_ls4, r) ? ls_before : field(tot_ls4, r);
    if (!c.m[r]) continue;
    const uint32_t body = c.m[r] & ~c.nl[r] & ~eq_mask(c.v[r], '\r');
    uint32_t hdm = 0;
    bool header = false;
    if (fasta) {
      // header starts: '>' at a line start (after a newline, or at lo)
      const uint64_t pos = tile0 + ((uint64_t)r * kTB + threadIdx.x) * kChunk;
      uint32_t starts = (c.nl[r] << 1) & 0xFFFFu;
      if (pos > lo) starts |= B[pos - 1] == '\n' ? 1u : 0u;
      else starts |= 1u << (uint32_t)(lo - pos);
      hdm = starts & eq_mask(c.v[r], '>') & c.m[r];
      hd += __popc(hdm);
      header = line && B[tile0 + ls0] == '>';
    }
    uint32_t from = 0;
    for (uint32_t rest = c.nl[r];;) {
      const uint32_t to = rest ? (uint32_t)__ffs(rest) : kChunk;  // one past the newline
      const uint32_t bytes = __popc(body & ((1u << to) - 1) & ~((1u << from) - 1));
      if (fasta) {
        if (line == 0) cls += bytes;
        else if (!header) cls += (ull)bytes << 16;
      } else {
        cls += (ull)bytes << (16 * (line & 3));
      }
      if (!rest) break;
      ++line;
      from = to;
      header = to < kChunk && (hdm >> to & 1);
      rest &= rest - 1;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    cls += __shfl_xor(cls, off);
    hd += __shfl_xor(hd, off);
    const uint32_t o = __shfl_xor(ls, off);
    ls = o > ls ? o : ls;
  }
  __shared__ ull s_cls[kTB / 64];
  __shared__ uint32_t s_hd[kTB / 64], s_ls[kTB / 64];
  if ((threadIdx.x & 63) == 0) {
    s_cls[threadIdx.x >> 6] = cls;
    s_hd[threadIdx.x >> 6] = hd;
    s_ls[threadIdx.x >> 6] = ls;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kTB / 64; ++w) {
      cls += s_cls[w];
      hd += s_hd[w];
      ls = s_ls[w] > ls ? s_ls[w] : ls;
    }
    ull nl = 0;
    for (int r = 0; r < kRounds; ++r) nl += field(tot_nl4, r);
    t_nl[blockIdx.x] = nl;
    t_hd[blockIdx.x] = hd;
    t_ls[blockIdx.x] = ls ? tile0 + ls : 0;
    t_cls[blockIdx.x] = cls;
  }
}

// Tile scans in two levels. Level 1 (many blocks): each group of 1024
// consecutive tiles is scanned in place (exclusive, from 0) and its total
// written to g[group]. Level 2 (one block): the group totals are scanned
// (exclusive; a maximum from lo); g[n_groups] = the reduction of everything. A tile's
// exclusive prefix is then op(g[tile >> 10], t[tile]). Up to three arrays
// per launch; is_max selects the running maximum instead of the sum.
constexpr int kScanGroup = 1024;

struct ScanArrays {
  ull* t[3];
  ull* g[3];
  int is_max[3];
  int n;
};

__global__ void __launch_bounds__(kScanGroup) k_fx_scan_groups(ScanArrays s, uint64_t nt) {
  __shared__ ull sh[kScanGroup / 64];
  const uint64_t i = (uint64_t)blockIdx.x * kScanGroup + threadIdx.x;
  for (int a = 0; a < s.n; ++a) {
    const ull v = i < nt ? s.t[a][i] : 0;
    ull total;
    const ull ex = s.is_max[a] ? block_exscan<Max, kScanGroup>(v, Max(), sh, &total)
                               : block_exscan<Plus, kScanGroup>(v, Plus(), sh, &total);
    if (i < nt) s.t[a][i] = ex;
    if (threadIdx.x == 0) s.g[a][blockIdx.x] = total;
  }
}

__global__ void __launch_bounds__(kScanGroup) k_fx_scan_top(ScanArrays s, uint64_t ng,
                                                            const Info* __restrict__ info) {
  __shared__ ull sh[kScanGroup / 64];
  for (int a = 0; a < s.n; ++a) {
    ull carry = s.is_max[a] ? info->lo : 0;  // the first line starts at lo
    for (uint64_t base = 0; base < ng; base += kScanGroup) {
      const uint64_t j = base + threadIdx.x;
      const ull v = j < ng ? s.g[a][j] : 0;
      ull total;
      ull ex;
      if (s.is_max[a]) {
        ex = block_exscan<Max, kScanGroup>(v, Max(), sh, &total);
        ex = ex > carry ? ex : carry;
        carry = total > carry ? total : carry;
      } else {
        ex = carry + block_exscan<Plus, kScanGroup>(v, Plus(), sh, &total);
        carry += total;
      }
      if (j < ng) s.g[a][j] = ex;
    }
    if (threadIdx.x == 0) s.g[a][ng] = carry;
  }
}

// Kept bytes of each tile from its classes and the state at its start, scanned
// within groups of kScanGroup tiles like the arrays above.
__global__ void __launch_bounds__(kScanGroup) k_fx_keep_groups(
    const uint8_t* __restrict__ B, const Info* __restrict__ info, const ull* __restrict__ t_nl,
    const ull* __restrict__ t_ls, const ull* __restrict__ g_nl, const ull* __restrict__ g_ls,
    const ull* __restrict__ t_cls, ull* __restrict__ t_keep, ull* __restrict__ g_keep,
    uint64_t nt) {
  __shared__ ull sh[kScanGroup / 64];
  const uint64_t i = (uint64_t)blockIdx.x * kScanGroup + threadIdx.x;
  ull v = 0;
  if (i < nt && info->lo < info->hi) {
    const ull cls = t_cls[i];
    if (info->fasta) {
      const ull ls = g_ls[blockIdx.x] > t_ls[i] ? g_ls[blockIdx.x] : t_ls[i];
      v = field(cls, 1) + (B[ls] == '>' ? 0 : field(cls, 0));
    } else {
      const uint32_t line = (uint32_t)(g_nl[blockIdx.x] + t_nl[i]);
      v = field(cls, (1u - line) & 3u);
    }
  }
  ull total;
  const ull ex = block_exscan<Plus, kScanGroup>(v, Plus(), sh, &total);
  if (i < nt) t_keep[i] = ex;
  if (threadIdx.x == 0) g_keep[blockIdx.x] = total;
}

// The L low bytes of v to p, any alignment.
__device__ __forceinline__ void store_bytes(uint8_t* p, unsigned __int128 v, uint32_t L) {
  if (L == kChunk) {
    __builtin_memcpy(p, &v, 16);
    return;
  }
  ull w = (ull)v;
  if (L & 8) {
    __builtin_memcpy(p, &w, 8);
    w = (ull)(v >> 64);
    p += 8;
  }
  uint32_t x = (uint32_t)w;
  if (L & 4) {
    __builtin_memcpy(p, &x, 4);
    x = (uint32_t)(w >> 32);
    p += 4;
  }
  if (L & 2) {
    p[0] = (uint8_t)x;
    p[1] = (uint8_t)(x >> 8);
    x >>= 16;
    p += 2;
  }
  if (L & 1) *p = (uint8_t)x;
}

// Pass 2: kept bytes and record offsets written, FASTQ layout checked. The
// per-round prefixes of the tile's chunks come from one block scan each, the
// four rounds packed in 16-bit fields (a round holds at most 4096 bytes).
// Nothing is written unless the outputs have room for all of it and the text
// can be of the format by its first byte and its number of lines;
// out_offsets[records] is written by the last block.
__global__ void __launch_bounds__(kTB) k_fx_write(const uint8_t* __restrict__ B, Info* info,
                                                  const ull* __restrict__ t_nl,
                                                  const ull* __restrict__ t_hd,
                                                  const ull* __restrict__ t_ls,
                                                  const ull* __restrict__ g_nl,
                                                  const ull* __restrict__ g_hd,
                                                  const ull* __restrict__ g_ls,
                                                  const ull* __restrict__ t_keep,
                                                  const ull* __restrict__ g_keep,
                                                  uint8_t* __restrict__ out_reads,
                                                  uint64_t reads_capacity,
                                                  uint64_t* __restrict__ out_offsets,
                                                  uint64_t max_records, uint64_t ng) {
  __shared__ ull sh[kTB / 64];
  const uint64_t lo = info->lo, hi = info->hi;
  if (lo >= hi) return;
  const uint32_t fasta = info->fasta;
  const ull lines = g_nl[ng] + 1, keep_all = g_keep[ng];
  const ull records = fasta ? g_hd[ng] : lines / 4;
  const bool fits = (fasta ? info->first == '>' : lines % 4 == 0) && records <= max_records;
  // (a FASTQ text that starts otherwise is refused; its layout check names line 0)
  const bool store = fits && (fasta || info->first == '@') && keep_all <= reads_capacity &&
                     (out_reads || !keep_all);
  if (!fits) return;
  if (store && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out_offsets[records] = keep_all;
  const uint64_t tile0 = (uint64_t)blockIdx.x * kTile;
  const Chunks c = load_tile(B, tile0, lo, hi);
  const uint64_t grp = blockIdx.x / kScanGroup;
  const ull c_nl = g_nl[grp] + t_nl[blockIdx.x];
  ull nl4 = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) nl4 |= (ull)__popc(c.nl[r]) << (16 * r);
  ull tot_nl4;
  const ull ex_nl4 = block_exscan(nl4, Plus(), sh, &tot_nl4);
  // FASTA: where the line open at each chunk's first byte starts
  ull ex_ls4 = 0, tot_ls4 = 0, c_ls = 0;
  if (fasta) {
    c_ls = g_ls[grp] > t_ls[blockIdx.x] ? g_ls[grp] : t_ls[blockIdx.x];
    ull ls4 = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) ls4 |= (ull)last_start(c.nl[r], r) << (16 * r);
    ex_ls4 = block_exscan(ls4, Max4(), sh, &tot_ls4);
  }

  // per chunk: line index at its first byte, line-start (FASTA: header-start)
  // and kept masks
  uint32_t keep[kRounds], starts[kRounds];
  uint32_t line0[kRounds];  // relative to c_nl
  uint32_t nl_before = 0, ls_before = 0;  // earlier rounds of this tile
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t pos = tile0 + ((uint64_t)r * kTB + threadIdx.x) * kChunk;
    line0[r] = nl_before + field(ex_nl4, r);
    const uint32_t lsl = ls_before > field(ex_ls4, r) ? ls_before : field(ex_ls4, r);
    nl_before += field(tot_nl4, r);
    ls_before = ls_before > field(tot_ls4, r) ? ls_before : field(tot_ls4, r);
    const uint32_t m = c.m[r], nlm = c.nl[r];
    keep[r] = starts[r] = 0;
    // the byte before the chunk: from the neighbour lane (its last byte is not
    // a newline where it lies before lo), or from memory
    uint32_t before = __shfl_up(nlm >> (kChunk - 1), 1u, 64);
    if (!m) continue;
    if ((threadIdx.x & 63) == 0) before = pos > lo && B[pos - 1] == '\n' ? 1u : 0u;
    uint32_t st = (nlm << 1) & 0xFFFFu;
    if (pos > lo) st |= before;
    else st |= 1u << (uint32_t)(lo - pos);
    st &= m;
    uint32_t k = 0;
    if (fasta) {
      // segments between line starts; a segment is kept unless its line is
      // a header
      const ull ls0 = lsl ? tile0 + lsl : c_ls;
      const uint32_t hdm = st & eq_mask(c.v[r], '>');
      bool hh = ls0 < pos && B[ls0] == '>';
      uint32_t from = 0;
      for (uint32_t rest = st;;) {
        const uint32_t to = rest ? (uint32_t)__ffs(rest) - 1 : kChunk;  // next line start
        if (!hh) k |= ((1u << to) - 1) & ~((1u << from) - 1);
        if (!rest) break;
        hh = hdm >> to & 1;
        from = to;
        rest &= rest - 1;
      }
      starts[r] = hdm;
    } else {
      // segments ending at newlines; lines 4i + 1 are kept
      uint32_t l = (uint32_t)c_nl + line0[r], from = 0;
      for (uint32_t rest = nlm;;) {
        const uint32_t to = rest ? (uint32_t)__ffs(rest) : kChunk;  // one past the newline
        if ((l & 3) == 1) k |= ((1u << to) - 1) & ~((1u << from) - 1);
        if (!rest) break;
        ++l;
        from = to;
        rest &= rest - 1;
      }
      // layout check at line starts: '@' on header lines, '+' on separators
      for (uint32_t s = st; s;) {
        const int j = __ffs(s) - 1;
        s &= s - 1;
        const ull lj = c_nl + line0[r] + __popc(nlm & ((1u << j) - 1));
        const uint32_t b = byte_of(c.v[r], j);
        if (((lj & 3) == 0 && b != '@') || ((lj & 3) == 2 && b != '+')) atomicMin(&info->err, lj);
      }
      starts[r] = st;
    }
    if (k) k &= m & ~nlm & ~eq_mask(c.v[r], '\r');
    keep[r] = k;
  }
  if (!store) return;

  ull kp4 = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) kp4 |= (ull)__popc(keep[r]) << (16 * r);
  ull tot_kp4;
  const ull ex_kp4 = block_exscan(kp4, Plus(), sh, &tot_kp4);
  const ull out0 = g_keep[grp] + t_keep[blockIdx.x];
  ull hd_ex4 = 0, tot_hd4 = 0;
  if (fasta) {
    ull hd4 = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) hd4 |= (ull)__popc(starts[r]) << (16 * r);
    hd_ex4 = block_exscan(hd4, Plus(), sh, &tot_hd4);
  }
  uint32_t kp_before = 0, hd_before = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const ull at = out0 + kp_before + field(ex_kp4, r);  // output position of the chunk
    kp_before += field(tot_kp4, r);
    const uint32_t km = keep[r];
    // record offsets: FASTA header starts; FASTQ starts of sequence lines
    if (fasta) {
      ull h = g_hd[grp] + t_hd[blockIdx.x] + hd_before + field(hd_ex4, r);
      for (uint32_t s = starts[r]; s;) {
        const int j = __ffs(s) - 1;
        s &= s - 1;
        out_offsets[h++] = at + __popc(km & ((1u << j) - 1));
      }
      hd_before += field(tot_hd4, r);
    } else {
      for (uint32_t s = starts[r]; s;) {
        const int j = __ffs(s) - 1;
        s &= s - 1;
        const ull lj = c_nl + line0[r] + __popc(c.nl[r] & ((1u << j) - 1));
        if ((lj & 3) == 1) out_offsets[lj >> 2] = at + __popc(km & ((1u << j) - 1));
      }
    }
    // the kept bytes, a run at a time
    uint8_t* o = out_reads + at;
    const unsigned __int128 v =
        ((unsigned __int128)((ull)c.v[r].w << 32 | c.v[r].z) << 64) | ((ull)c.v[r].y << 32 | c.v[r].x);
    for (uint32_t rest = km; rest;) {
      const int from = __ffs(rest) - 1;
      const uint32_t L = __ffs(~(rest >> from)) - 1;  // (bits 16.. of rest are 0)
      store_bytes(o, v >> (8 * from), L);
      o += L;
      rest &= ~(((1u << L) - 1) << from);
    }
  }
}

// The results, to the host.
__global__ void k_fx_publish(const Info* __restrict__ info, const ull* __restrict__ g_nl,
                             const ull* __restrict__ g_hd, const ull* __restrict__ g_keep,
                             uint64_t ng, Info* pub) {
  if (threadIdx.x != 0) return;
  Info r = *info;
  r.newlines = g_nl[ng];
  r.headers = g_hd[ng];
  r.keep = g_keep[ng];
  *pub = r;
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

int bad(const std::string& msg) {
  kc::set_last_error(msg);
  return KC_E_INVAL;
}

bool is_eol(uint8_t b) { return b == '\n' || b == '\r'; }

// First position in [lo, hi) whose byte is not CR/LF, scanning forward
// (dir > 0), or last such position + 1 scanning backward; hi / lo if none.
uint64_t trim(const uint8_t* text, uint64_t lo, uint64_t hi, int dir, hipStream_t st) {
  uint8_t buf[kPeek];
  if (dir > 0) {
    for (uint64_t p = lo; p < hi;) {
      const uint64_t n = hi - p < kPeek ? hi - p : kPeek;
      chk(hipMemcpyAsync(buf, text + p, n, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
      chk(hipStreamSynchronize(st), "hipStreamSynchronize");
      for (uint64_t i = 0; i < n; ++i)
        if (!is_eol(buf[i])) return p + i;
      p += n;
    }
    return hi;
  }
  for (uint64_t e = hi; e > lo;) {
    const uint64_t n = e - lo < kPeek ? e - lo : kPeek;
    chk(hipMemcpyAsync(buf, text + e - n, n, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
    chk(hipStreamSynchronize(st), "hipStreamSynchronize");
    for (uint64_t i = n; i > 0; --i)
      if (!is_eol(buf[i - 1])) return e - n + i;
    e -= n;
  }
  return lo;
}

// Device temporaries and host-visible words of the calling thread, kept
// between calls.
void* scratch(size_t bytes, hipStream_t st) {
  std::string err;
  int code = KC_E_NOMEM;
  void* p = kc::thread_scratch(bytes, st, &err, &code);
  if (!p) {
    kc::set_last_error(err);
    throw Fail{code};
  }
  return p;
}

}  // namespace

extern "C" int kc_parse_fastx(const uint8_t* text, uint64_t n_bytes, int format,
                              uint8_t* out_reads, uint64_t reads_capacity, uint64_t* out_offsets,
                              uint64_t max_records, uint64_t* n_records, uint64_t* n_bases,
                              int* format_out, void* stream) {
  kc::set_last_error("");
  if (!n_records || !n_bases) return bad("n_records or n_bases is NULL");
  *n_records = 0;
  *n_bases = 0;
  if (format_out) *format_out = format;
  if (format < KC_FASTX_AUTO || format > KC_FASTA) return bad("unknown format");
  if (n_bytes && !text) return bad("text is NULL");
  if (!out_offsets) return bad("out_offsets is NULL");
  const hipStream_t st = (hipStream_t)stream;
  try {
    if (!n_bytes) {
      const uint64_t zero = 0;
      chk(hipMemcpyAsync(out_offsets, &zero, 8, hipMemcpyHostToDevice, st), "hipMemcpyAsync");
      chk(hipStreamSynchronize(st), "hipStreamSynchronize");
      return KC_OK;
    }
    // positions relative to the 16-byte aligned base B; the text is [a, a + n)
    const uint64_t a = (uint64_t)(uintptr_t)text & 15u;
    const uint8_t* B = text - a;
    const uint64_t nt = (a + n_bytes + kTile - 1) / kTile;
    if (nt > 0x7fffffffull) return bad("text too large");
    const uint64_t ng = (nt + kScanGroup - 1) / kScanGroup;
    ull* t_nl = (ull*)scratch((5 * nt + 4 * (ng + 1)) * sizeof(ull) + sizeof(Info), st);
    ull* t_hd = t_nl + nt;
    ull* t_ls = t_hd + nt;
    ull* t_cls = t_ls + nt;
    ull* t_keep = t_cls + nt;
    ull* g_nl = t_keep + nt;
    ull* g_hd = g_nl + (ng + 1);
    ull* g_ls = g_hd + (ng + 1);
    ull* g_keep = g_ls + (ng + 1);
    Info* info = (Info*)(g_keep + (ng + 1));
    std::string err;
    int code = KC_E_NOMEM;
    void* pub_dev = nullptr;
    Info* const pub = (Info*)kc::thread_pinned(sizeof(Info), &pub_dev, &err, &code);
    if (!pub) {
      kc::set_last_error(err);
      return code;
    }
    ScanArrays sa3 = {{t_nl, t_hd, t_ls}, {g_nl, g_hd, g_ls}, {0, 0, 1}, 3};
    ScanArrays sa1 = {{t_keep, nullptr, nullptr}, {g_keep, nullptr, nullptr}, {0, 0, 0}, 1};
    const auto passes = [&] {
      hipLaunchKernelGGL(k_fx_lines, dim3((unsigned)nt), dim3(kTB), 0, st, B, info, t_nl, t_hd,
                         t_ls, t_cls);
      hipLaunchKernelGGL(k_fx_scan_groups, dim3((unsigned)ng), dim3(kScanGroup), 0, st, sa3, nt);
      hipLaunchKernelGGL(k_fx_scan_top, dim3(1), dim3(kScanGroup), 0, st, sa3, ng, info);
      hipLaunchKernelGGL(k_fx_keep_groups, dim3((unsigned)ng), dim3(kScanGroup), 0, st, B, info,
                         t_nl, t_ls, g_nl, g_ls, t_cls, t_keep, g_keep, nt);
      hipLaunchKernelGGL(k_fx_scan_top, dim3(1), dim3(kScanGroup), 0, st, sa1, ng, info);
      hipLaunchKernelGGL(k_fx_write, dim3((unsigned)nt), dim3(kTB), 0, st, B, info, t_nl, t_hd,
                         t_ls, g_nl, g_hd, g_ls, t_keep, g_keep, out_reads, reads_capacity,
                         out_offsets, max_records, ng);
      hipLaunchKernelGGL(k_fx_publish, dim3(1), dim3(64), 0, st, info, g_nl, g_hd, g_keep, ng,
                         (Info*)pub_dev);
      chk(hipGetLastError(), "parse launch");
      chk(hipStreamSynchronize(st), "hipStreamSynchronize");
    };
    hipLaunchKernelGGL(k_fx_ends, dim3(1), dim3(kTB), 0, st, text, n_bytes, a, format, info);
    passes();
    if (pub->missing) {
      // more than kPeekMost line ends at an end of the text: the host looks past them
      // (with the first byte among the last kPeekMost, the last one is too)
      const uint64_t s0 = pub->missing & 1 ? trim(text, kPeekMost, n_bytes, 1, st) : pub->lo - a;
      const uint64_t e0 = s0 >= n_bytes           ? s0
                          : pub->missing & 2 ? trim(text, s0, n_bytes - kPeekMost, -1, st)
                                             : n_bytes - pub->tail;
      if (s0 < e0) {
        Info in = *pub;
        in.lo = a + s0;
        in.hi = a + e0;
        in.missing = 0;
        in.err = ~0ull;
        uint8_t first = 0;
        chk(hipMemcpyAsync(&first, text + s0, 1, hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
        chk(hipStreamSynchronize(st), "hipStreamSynchronize");
        in.first = first;
        in.fasta = format == KC_FASTA || (format == KC_FASTX_AUTO && first == '>');
        chk(hipMemcpyAsync(info, &in, sizeof(in), hipMemcpyHostToDevice, st), "hipMemcpyAsync");
        passes();
      }
    }
    const Info r = *pub;
    if (r.lo >= r.hi) {  // nothing but line ends: no records
      const uint64_t zero = 0;
      chk(hipMemcpyAsync(out_offsets, &zero, 8, hipMemcpyHostToDevice, st), "hipMemcpyAsync");
      chk(hipStreamSynchronize(st), "hipStreamSynchronize");
      return KC_OK;
    }
    if (format == KC_FASTX_AUTO) {
      if (r.first == '@') format = KC_FASTQ;
      else if (r.first == '>') format = KC_FASTA;
      else return bad("the text starts with neither '@' (FASTQ) nor '>' (FASTA)");
    }
    if (format_out) *format_out = format;
    if (format == KC_FASTA && r.first != '>') return bad("FASTA text does not start with '>'");
    const uint64_t lines = r.newlines + 1;  // the trimmed text does not end with a newline
    if (!r.fasta && lines % 4)
      return bad("FASTQ text has " + std::to_string(lines) +
                 " lines, not a whole number of 4-line records");
    const uint64_t R = r.fasta ? r.headers : lines / 4;
    *n_records = R;
    if (R > max_records) {
      kc::set_last_error("out_offsets has room for " + std::to_string(max_records) +
                         " records, the text holds " + std::to_string(R));
      return KC_E_CAPACITY;
    }
    if (r.err != ~0ull) {
      *n_records = 0;
      const uint64_t l = r.err;
      return bad("FASTQ line " + std::to_string(l) + " (counting from 0) should start with '" +
                 ((l & 3) == 0 ? "@" : "+") + "'");
    }
    if (r.keep > reads_capacity) {
      *n_bases = r.keep;
      kc::set_last_error("out_reads has room for " + std::to_string(reads_capacity) +
                         " bytes, the sequences hold " + std::to_string(r.keep));
      return KC_E_CAPACITY;
    }
    if (r.keep && !out_reads) return bad("out_reads is NULL");
    *n_bases = r.keep;
  } catch (const Fail& f) {
    return f.code;
  }
  return KC_OK;
}
