// The input side of the step (Algorithm 1's binarisation of the inputs and Section 3.2,
// footnote 1), for integer features (int8):
//   * the median of every feature over a reference set (the lower middle
//     order statistic, so an element of the column and exact);
//   * median binarisation: bit = (x >= median); the same kernel packs ±1 rows;
//   * the fixed random ±1 expansion layer: bit = (sum_i x_i R[j][i] >= 0),
//     exact in int32, with R drawn from Philox stream 5 (counter layer word
//     2^32 - 1, t = 0): element e = j K_raw + i is bit (e & 127) of block
//     e >> 7.
#include "bmlp_internal.h"
#include "philox.h"

namespace bmlp {
namespace {

constexpr int kStreamExpand = 5;
// The median of F neighbouring features per work-group, from 256-bin
// histograms in LDS, over the rows [split * rows, + rows) of the reference
// set.  With one split the work-group takes the median itself; with several
// (the caller gave scratch memory) it writes its counts, and
// median_merge_kernel adds them up.
//
// What bounds it: a work-group touches one cache line per row and F bytes, and
// a compute unit fills a line in two cycles and adds to 64 LDS counters in
// about 16.  So:
//   * F = 16 where rows can be split, so that a line is touched half as often
//     and every compute unit has rows to count; F = 8 where they cannot,
//     since the features alone must fill the chip then;
//   * a lane loads its row's F bytes at once, and a thread has kMedRows rows
//     in flight (16 waves: enough to cover memory latency);
//   * the histograms are kept 64 / F times, bin-major, one LDS bank per
//     (copy, feature) slot, and at step j lane l counts its byte
//     (l + j) mod 4 of dword (l / 4 + j / 4) mod F / 4 into the copy l / F.
//     So the 64 lanes of every atomic are in 64 different banks, whatever the
//     data (features with few distinct values included);
//   * an atomic's address is one v_perm_b32: byte 0 the slot, byte 1 the
//     value.
// The work-groups of one XCD take neighbouring features of the same rows, so
// a row's cache line is fetched into one or two L2s instead of all eight.
// 60000 x 784 (47 MB): 75.2 us in one part, 27.9 + 4.9 us (merge) in eight.
constexpr int kMedThreads = 1024;
constexpr int kMedRows = 4;      // rows per thread and pass

// where the features of a wave's lane l lie in running order: the value of
// bins 4l .. 4l + 3 at which the count reaches floor((n - 1) / 2) + 1
__device__ __forceinline__ void median_of_bins(const uint32_t (&c)[4], int n, int8_t *out) {
  const int lane = threadIdx.x & 63;
  const uint32_t want = (uint32_t)((n - 1) / 2) + 1u;
  const uint32_t own = c[0] + c[1] + c[2] + c[3];
  uint32_t run = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t v = (uint32_t)__shfl_up((int)run, d, 64);
    if (lane >= d) run += v;
  }
  uint32_t before = run - own;
  if (before < want && run >= want) {
    int v = 4 * lane;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      before += c[q];
      if (before < want) ++v;
      else break;
    }
    *out = (int8_t)(v - 128);
  }
}

template <int F>
__global__ __launch_bounds__(kMedThreads) void feature_median_kernel(const int8_t *__restrict__ x, int n, int K,
                                                                     int8_t *__restrict__ med, int per_xcd,
                                                                     int rows, uint4 *__restrict__ part) {
  constexpr int kDw = F / 4, kCopies = 64 / F;
  __shared__ uint32_t hist[256][64];
  const int tid = threadIdx.x, lane = tid & 63;
  // XCD b % 8 takes the tiles [per_xcd * (b % 8), + per_xcd), one split of
  // the rows after the other, or (per_xcd 0) every eighth split of all tiles
  const int xcd = (int)blockIdx.x & 7, idx = (int)blockIdx.x >> 3, tiles = (K + F - 1) / F;
  const int split = per_xcd ? idx / per_xcd : 8 * (idx / tiles) + xcd;
  const int tile = per_xcd ? per_xcd * xcd + idx % per_xcd : idx % tiles;
  // the last tile starts early enough to stay inside the row (its first
  // features are then counted twice, with the same result)
  const int f0 = max(0, min(tile * F, K - F));
  if (tile * F >= K) return;
  for (int i = tid; i < 256 * 64 / 4; i += kMedThreads) reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const int rot = lane % F, copy0 = lane - rot;
  // byte addresses of the slots within a bin, four steps a dword; the perm
  // selectors [slot byte j, value byte (rot + j) % 4, 0, 0] of step j
  // (0x0C gives a zero byte, 0..3 the second source's bytes, 4..7 the first's)
  uint32_t slots[kDw], sel[4];
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const uint32_t f = 4u * (((uint32_t)rot / 4 + j / 4) % kDw) + ((uint32_t)rot + j) % 4;
    const uint32_t byte = (4u * ((uint32_t)copy0 + f)) << (8 * (j & 3));
    slots[j / 4] = (j & 3) ? slots[j / 4] | byte : byte;
    if (j < 4) sel[j] = 0x0C0C0000u | ((4u + ((uint32_t)rot + j) % 4) << 8) | (uint32_t)j;
  }
  uint8_t *const base = reinterpret_cast<uint8_t *>(hist);
  struct Row {
    uint32_t d[kDw];
  };
  auto count = [&](Row v) {
    // dword rot / 4 first
    if constexpr (kDw == 4) {
      const bool two = (rot & 8) != 0;
      const uint32_t t[4] = {two ? v.d[2] : v.d[0], two ? v.d[3] : v.d[1], two ? v.d[0] : v.d[2], two ? v.d[1] : v.d[3]};
      const bool one = (rot & 4) != 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) v.d[q] = one ? t[(q + 1) & 3] : t[q];
    } else {
      const bool one = (rot & 4) != 0;
      const uint32_t a = v.d[0], b = v.d[1];
      v.d[0] = one ? b : a;
      v.d[1] = one ? a : b;
    }
#pragma unroll
    for (int j = 0; j < F; ++j) {
      // bin: the value + 128
      const uint32_t w = v.d[j / 4] ^ 0x80808080u;
      atomicAdd(reinterpret_cast<uint32_t *>(base + __builtin_amdgcn_perm(w, slots[j / 4], sel[j & 3])), 1u);
    }
  };
  const uint32_t first = (uint32_t)split * (uint32_t)rows, end = min((uint32_t)n, first + (uint32_t)rows);
  uint32_t r = first + (uint32_t)tid;
  if (K >= F) {
    const int8_t *xf = x + f0;
    for (; r + (kMedRows - 1) * kMedThreads < end; r += kMedRows * kMedThreads) {
      Row v[kMedRows];
#pragma unroll
      for (int q = 0; q < kMedRows; ++q) __builtin_memcpy(&v[q], xf + (size_t)(r + q * kMedThreads) * K, F);
#pragma unroll
      for (int q = 0; q < kMedRows; ++q) count(v[q]);
    }
    for (; r < end; r += kMedThreads) {
      Row v;
      __builtin_memcpy(&v, xf + (size_t)r * K, F);
      count(v);
    }
  } else {   // rows of fewer bytes than a load
    for (; r < end; r += kMedThreads)
      for (int f = 0; f < K; ++f) atomicAdd(&hist[(int)x[(size_t)r * K + f] + 128][copy0 + f], 1u);
  }
  __syncthreads();
  // one wave per feature: lane l sums the copies of bins 4l .. 4l + 3
  const int f = tid >> 6;
  static_assert(F <= kMedThreads / 64, "a wave per feature");
  if (f < F && f0 + f < K) {
    uint32_t c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c[q] = 0u;
      // each lane starts at a copy of its own (spreads the banks)
#pragma unroll
      for (int k = 0; k < kCopies; ++k) c[q] += hist[4 * lane + q][((lane + k) % kCopies) * F + f];
    }
    if (part == nullptr)
      median_of_bins(c, n, med + f0 + f);
    else   // the features that the last tile repeats are written twice, with the same counts
      part[((size_t)split * K + f0 + f) * 64 + lane] = make_uint4(c[0], c[1], c[2], c[3]);
  }
}

// The splits' counts [splits][K][256] added up: a wave per feature, a lane
// per four bins.
__global__ __launch_bounds__(256) void median_merge_kernel(const uint4 *__restrict__ part, int splits, int n, int K,
                                                           int8_t *__restrict__ med) {
  const int f = (int)blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (f >= K) return;
  uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll 8
  for (int s = 0; s < splits; ++s) {
    const uint4 v = part[((size_t)s * K + f) * 64 + lane];
    c[0] += v.x;
    c[1] += v.y;
    c[2] += v.z;
    c[3] += v.w;
  }
  median_of_bins(c, n, med + f);
}

// The same where the features alone are several rounds of work-groups for the
// chip: 64 of them per work-group, a feature per lane.  A work-group of 8
// features clears and sums as many counters for an eighth of the features,
// which is most of its time where rows are few.  One histogram per feature,
// bin-major, so that the 64 lanes of an atomic or a read are in 64 banks; a
// wave loads 64 bytes of a row at a time, kWideRows rows in flight.  Its 16 waves then
// take 16 bins each: sums of every feature, and the one whose bins reach the
// middle looks through them.
// A launch counts the threads of a dimension in 32 bits (one past that runs
// only part of its work-groups, without an error): past kWideGrid work-groups the
// grid goes on in y.
constexpr int kWideGrid = 1 << 20;
constexpr int kWideFeat = 64, kWideRows = 8, kWideWaves = kMedThreads / 64, kWideBins = 256 / kWideWaves;

__global__ __launch_bounds__(kMedThreads) void feature_median_wide_kernel(const int8_t *__restrict__ x, int n, int K,
                                                                          int8_t *__restrict__ med) {
  __shared__ uint32_t hist[256][kWideFeat];
  __shared__ uint32_t part[kWideWaves][kWideFeat];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f0 = ((int)blockIdx.y * kWideGrid + (int)blockIdx.x) * kWideFeat, left = K - f0;
  if (left <= 0) return;   // (past the last tile)
  for (int i = tid; i < 256 * kWideFeat / 4; i += kMedThreads)
    reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const int8_t *col = x + f0 + min(lane, left - 1);   // lanes past the last feature count it too, into slots of their own
  uint32_t r = (uint32_t)wave;
  for (; r + (kWideRows - 1) * kWideWaves < (uint32_t)n; r += kWideRows * kWideWaves) {
    int v[kWideRows];
#pragma unroll
    for (int q = 0; q < kWideRows; ++q) v[q] = col[(size_t)(r + q * kWideWaves) * K];
#pragma unroll
    for (int q = 0; q < kWideRows; ++q) atomicAdd(&hist[v[q] + 128][lane], 1u);
  }
  for (; r < (uint32_t)n; r += kWideWaves) atomicAdd(&hist[(int)col[(size_t)r * K] + 128][lane], 1u);
  __syncthreads();
  uint32_t own = 0u;
#pragma unroll
  for (int q = 0; q < kWideBins; ++q) own += hist[kWideBins * wave + q][lane];
  part[wave][lane] = own;
  __syncthreads();
  const uint32_t want = (uint32_t)((n - 1) / 2) + 1u;
  uint32_t before = 0u;
  for (int w = 0; w < wave; ++w) before += part[w][lane];
  if (lane < left && before < want && before + own >= want) {
    int v = kWideBins * wave;
    while ((before += hist[v][lane]) < want) ++v;   // ends inside the wave's bins
    med[f0 + lane] = (int8_t)(v - 128);
  }
}

constexpr int kMedFeatSplit = 16, kMedFeat = 8;

inline int med_tiles(int K, int F) { return (K - 1) / F + 1; }

// Splits of the rows: about two work-groups for each of 256 compute units,
// with at least one pass of rows each.  A multiple of 8 where the
// tiles are too few to share out among the XCDs evenly: each XCD then has rows of
// its own.  (60000 x 784: 8 splits 27.9 us, 16 34.8, 24 34.0, 32 40.9; 10 splits with
// the tiles shared out 32.6, one of the XCDs idle.)
int med_splits(int n, int K) {
  const int tiles = med_tiles(K, kMedFeatSplit), most = (n - 1) / kMedThreads + 1;
  if (tiles > 64 || most < 8) return min(max(1, 512 / tiles), most);
  return 8 * min(64 / tiles, most / 8);
}

// Bit rows from int8 rows: bit = (x >= threshold of the column), the
// thresholds a row of int8 (median binarisation) or, with PM1, 1 everywhere
// (x > 0: packing ±1 rows).
//
// Bound by the read of x.  A lane takes 16 neighbouring columns with one
// 16-byte load (any alignment) and stores their 16 bits; its thresholds stay
// in registers while it walks kBinRows rows, whose loads are all issued
// before the first is used.  Four bytes are compared with two subtractions:
// with x and t biased to unsigned bytes and spread to 16-bit halves, bit 8
// of (x | 0x100) - t is set iff x >= t, and no half borrows from the other.
// A wave covers 64 / lpr rows by lpr lanes each (lpr a power of two, at most
// 64), so that narrow rows do not leave lanes idle.
// 60000 x 784 (47 MB): 103 -> 10.6 us; the kernel before took one byte per
// lane and one 64-bit word per wave.
constexpr int kBinRows = 4;

struct BinLane {
  uint32_t te[4], to[4];   // thresholds of the even and odd bytes, biased, in 16-bit halves
};

// bits 0..3: x >= threshold for the four bytes of w (dword q of the lane's 16)
__device__ __forceinline__ uint32_t ge4(uint32_t w, const BinLane &t, int q) {
  const uint32_t v = w ^ 0x80808080u;
  const uint32_t e = ((v & 0x00FF00FFu) | 0x01000100u) - t.te[q];          // bytes 0, 2 -> bits 8, 24
  const uint32_t o = (((v >> 8) & 0x00FF00FFu) | 0x01000100u) - t.to[q];   // bytes 1, 3 -> bits 8, 24
  const uint32_t m = ((e >> 8) & 0x00010001u) | ((o >> 7) & 0x00020002u);  // bits 0, 1, 16, 17
  return (m | (m >> 14)) & 0xFu;
}

template <bool PM1>
__global__ __launch_bounds__(256) void binarize_kernel(const int8_t *__restrict__ x, int n, int K, int words,
                                                       const int8_t *__restrict__ thr, uint64_t *__restrict__ bits,
                                                       int lpr_log) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lpr = 1 << lpr_log, rpw = 64 >> lpr_log;          // lanes per row, rows per wave
  const int unit = (int)blockIdx.x * lpr + (lane & (lpr - 1));   // 16 columns of the row
  if (unit >= 4 * words) return;
  const int col = 16 * unit;
  uint16_t *out = reinterpret_cast<uint16_t *>(bits) + unit;
  const int row0 = ((int)blockIdx.y * 4 + wave) * (kBinRows * rpw) + (lane >> lpr_log);
  if (K >= 16) {
    // a lane whose columns end past the row loads the row's last 16 and shifts
    // the bits before its own out, which leaves zeros past column K (byte
    // loads there, one after another, took 100 x 1000 5.2 us instead of 3.3)
    const int start = min(col, K - 16), past = min(col - start, 16);
    BinLane t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t w = 0x01010101u;
      if constexpr (!PM1) __builtin_memcpy(&w, thr + start + 4 * q, 4);
      w ^= 0x80808080u;
      t.te[q] = w & 0x00FF00FFu;
      t.to[q] = (w >> 8) & 0x00FF00FFu;
    }
    uint4 v[kBinRows];
#pragma unroll
    for (int i = 0; i < kBinRows; ++i) __builtin_memcpy(&v[i], x + (size_t)min(row0 + i * rpw, n - 1) * K + start, 16);
#pragma unroll
    for (int i = 0; i < kBinRows; ++i) {
      const int row = row0 + i * rpw;
      if (row < n)
        out[(size_t)row * 4 * words] = (uint16_t)((ge4(v[i].x, t, 0) | (ge4(v[i].y, t, 1) << 4) |
                                                   (ge4(v[i].z, t, 2) << 8) | (ge4(v[i].w, t, 3) << 12)) >> past);
    }
  } else {   // rows shorter than a load: bytes, all loads at once (repeats past the row; 1000 x 15: 6.6 -> 3.4 us)
    uint32_t m[kBinRows] = {};
    if (unit == 0) {
      int8_t v[kBinRows][16], t[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        t[c] = 1;
        if constexpr (!PM1) t[c] = thr[min(c, K - 1)];
      }
#pragma unroll
      for (int i = 0; i < kBinRows; ++i)
#pragma unroll
        for (int c = 0; c < 16; ++c) v[i][c] = x[(size_t)min(row0 + i * rpw, n - 1) * K + min(c, K - 1)];
#pragma unroll
      for (int i = 0; i < kBinRows; ++i) {
#pragma unroll
        for (int c = 0; c < 16; ++c) m[i] |= (uint32_t)(v[i][c] >= t[c]) << c;
        m[i] &= (1u << K) - 1u;
      }
    }
#pragma unroll
    for (int i = 0; i < kBinRows; ++i) {
      const int row = row0 + i * rpw;
      if (row < n) out[(size_t)row * 4 * words] = (uint16_t)m[i];
    }
  }
}

// The expansion layer on the int8 matrix cores (v_mfma_i32_32x32x32_i8).
//
// A work-group computes 128 patterns x 128 output columns with four waves of
// 64 x 64, and walks the row tiles blockIdx.y, + gridDim.y, ... of its
// columns.  Bound by the matrix cores' feed: per MFMA a wave spends about four
// vector instructions on operands, so both are made cheaply.
//   * R's weights enter as the bit alone, r = (w + 1) / 2 in {0, 1}: byte b
//     of operand dword s of a 32-bit word is bit 8b + s, (word >> s) &
//     0x01010101, two instructions per four weights straight from R's bits;
//     then sum_i x_i w_i = 2 acc - sum_i x_i, the row sums of x added up
//     (v_dot4_i32_i8) as x is staged.
//   * x is staged through LDS with the bytes of each 32 inputs transposed to
//     match (dword s holds inputs s, s + 8, s + 16, s + 24), 16 v_perm_b32
//     per 32 bytes once for all columns.  Rows are 128 + 16 bytes apart, so
//     that 16-byte reads at one row per lane hit every bank once; the global
//     loads of the next two stages are in flight while one is computed.
//   * rows that end inside a stage (ROW) load the row's last 16 bytes where
//     fewer are left, and put them in place as they are stored: byte loads
//     there, one after another, took 1 x 16 -> 256 7.5 us instead of 4.7.
//   * R's bits for kXChunk inputs of the 128 columns are drawn into LDS as
//     whole Philox blocks; the columns' bit offsets in them are taken out by
//     one v_alignbit_b32 per word read.  They are drawn once per work-group
//     when all inputs fit one chunk.
// Exact: |acc| <= 128 * 65536.
// 10000 x 784 -> 3072: 1342 -> 39 us (the kernel before summed 4 inputs at a
// time with v_dot4_i32_i8, rebuilding the +-1 bytes for every pattern).
typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kXTile = 128;                      // patterns and output columns of a tile
constexpr int kXStage = 128;                     // inputs per LDS stage
constexpr int kXChunk = 1024;                    // inputs whose R bits are in LDS at once
constexpr int kXLd = kXStage + 16;               // bytes between staged rows
constexpr int kXBlocks = kXChunk / 128 + 1;      // Philox blocks covering a chunk of a column
constexpr int kXWords = 4 * kXBlocks + 1;        // words between columns (odd: banks spread)

// byte s of a, b, c, d as one dword, for s = 0..3
__device__ __forceinline__ uint4 transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u);   // a0 b0 a1 b1
  const uint32_t ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u);   // a2 b2 a3 b3
  const uint32_t cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u);
  const uint32_t cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
  return make_uint4(__builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u), __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u),
                    __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u), __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u));
}

// A row's 16 bytes from a place with `left` bytes before the row's end, out of
// what was loaded there: those bytes, or, with fewer than 16 left, the last 16
// of the row.
__device__ __forceinline__ v4u row_end(const v4u &v, int left, int k_raw) {
  const int s = 16 - (k_raw & 15);   // bytes to drop then, the same for all lanes (16: none are loaded so)
  const bool one = (s & 4) != 0, two = (s & 8) != 0;
  const uint32_t a0 = one ? v.y : v.x, a1 = one ? v.z : v.y, a2 = one ? v.w : v.z, a3 = one ? 0u : v.w;
  const uint32_t b0 = two ? a2 : a0, b1 = two ? a3 : a1, b2 = two ? 0u : a2, b3 = two ? 0u : a3;
  const uint32_t r = (uint32_t)(s & 3);
  const v4u e = {__builtin_amdgcn_alignbyte(b1, b0, r), __builtin_amdgcn_alignbyte(b2, b1, r),
                 __builtin_amdgcn_alignbyte(b3, b2, r), __builtin_amdgcn_alignbyte(0u, b3, r)};
  return left >= 16 ? v : left > 0 ? e : (v4u)(0u);
}

// v_writelane_b32 (see the forward kernel)
extern "C" __device__ uint32_t bmlp_input_writelane(uint32_t v, uint32_t lane, uint32_t old)
    __asm("llvm.amdgcn.writelane.i32");

// ROW: whole stages only (kWhole), or rows that end inside a stage, shorter
// than a load (kShort, k_raw < 16) or not (kRagged).
enum { kWhole = 0, kRagged = 1, kShort = 2 };
template <int ROW>
__global__ __launch_bounds__(256, 2) void expand_kernel(const int8_t *__restrict__ x, int n, int k_raw, int k0,
                                                        uint64_t seed, uint32_t *__restrict__ bits, int words32) {
  __shared__ __align__(16) uint8_t sX[2][kXTile * kXLd];
  __shared__ uint32_t sR[kXTile * kXWords];
  __shared__ __align__(16) int32_t sSum[kXTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, lc = lane & 31, lh = lane >> 5;
  const int j0 = (int)blockIdx.x * kXTile;
  const uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32);
  const int ns = (k_raw + kXStage - 1) / kXStage, row_tiles = (n - 1) / kXTile + 1;
  constexpr int kChunkStages = kXChunk / kXStage;

  // R's bits of the inputs i0 .. i0 + kXChunk of every column: the Philox
  // blocks that hold them, block b of column c at words 4b .. 4b + 3
  auto draw = [&](int i0) {
    const int len = min(kXChunk, k_raw - i0);
    for (int t = tid; t < kXTile * kXBlocks; t += 256) {
      const int c = t % kXTile, b = t / kXTile;
      const uint64_t e = (uint64_t)(j0 + c) * (uint64_t)k_raw + (uint64_t)i0;
      if (j0 + c >= k0 || b > (int)(((uint32_t)(e & 127) + (uint32_t)len - 1u) >> 7)) continue;
      const U32x4 v = philox4x32_10((uint32_t)(e >> 7) + (uint32_t)b, 0xFFFFFFFFu, 0u, kStreamExpand, key0, key1);
      uint32_t *d = sR + c * kXWords + 4 * b;
      d[0] = v.x;
      d[1] = v.y;
      d[2] = v.z;
      d[3] = v.w;
    }
  };

  // a thread stages 64 bytes of one row: words 2 (tid & 1), + 1 of the stage
  const int srow = tid >> 1, sbyte = 64 * (tid & 1);
  // The stages of the work-group's row tiles run as one sequence, two of them
  // in registers ahead of the one that is computed: the first stages of a
  // tile are loaded during the last ones of the tile before.
  int rt = (int)blockIdx.y, st = 0;     // computed next
  int lrt = rt, lst = 0;                // loaded next
  int sum = 0;
  v16i acc[2][2];
  // the lane's columns: where their bits start in sR
  int base[2];
  uint32_t sh[2];
  auto load = [&](v4u (&v)[4]) {
    // rows past n repeat the last one; what is loaded past the last tile is not used
    const int8_t *xr = x + (size_t)min(lrt * kXTile + srow, n - 1) * k_raw;
    const int i = lst * kXStage + sbyte;
    if constexpr (ROW != kShort) {   // past the row's end its last 16 bytes (see store)
#pragma unroll
      for (int q = 0; q < 4; ++q) __builtin_memcpy(&v[q], xr + min(i + 16 * q, k_raw - 16), 16);
    } else {   // bytes, all loads at once
      uint32_t w[4] = {0u, 0u, 0u, 0u};
      if (i == 0) {
        uint8_t c[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) c[b] = (uint8_t)xr[min(b, k_raw - 1)];
#pragma unroll
        for (int b = 0; b < 16; ++b) w[b >> 2] |= (b < k_raw ? (uint32_t)c[b] : 0u) << (8 * (b & 3));
      }
      v[0] = (v4u){w[0], w[1], w[2], w[3]};
#pragma unroll
      for (int q = 1; q < 4; ++q) v[q] = (v4u)(0u);
    }
    if (++lst == ns) {
      lst = 0;
      lrt = min(lrt + (int)gridDim.y, row_tiles - 1);
    }
  };
  auto store = [&](const v4u (&v)[4], uint8_t *d) {
    const bool ends = ROW == kRagged && st == ns - 1;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v4u a = v[2 * h], b = v[2 * h + 1];
      if (ends) {   // the row's last stage: what a load took from before its place shifted out, zeros past the row
        a = row_end(a, k_raw - (st * kXStage + sbyte + 32 * h), k_raw);
        b = row_end(b, k_raw - (st * kXStage + sbyte + 32 * h + 16), k_raw);
      }
      const uint32_t d8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int q = 0; q < 8; ++q) sum = __builtin_amdgcn_sdot4((int)d8[q], 0x01010101, sum, false);
      uint4 *o = reinterpret_cast<uint4 *>(d + srow * kXLd + sbyte + 32 * h);
      o[0] = transpose4(d8[0], d8[2], d8[4], d8[6]);
      o[1] = transpose4(d8[1], d8[3], d8[5], d8[7]);
    }
  };

  auto epilogue = [&]() {
    sum += __shfl_xor(sum, 1, 64);
    if ((tid & 1) == 0) sSum[srow] = sum;
    __syncthreads();
    // a_0 = (2 acc >= sum): result element e of lane l is row 8 (e >> 2) +
    // 4 (l >> 5) + (e & 3), column l & 31; ballot k = 16 (2i + j) + e goes to
    // lane k, which stores both rows' 32 bits
    uint32_t blo = 0u, bhi = 0u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int4 s[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] = *reinterpret_cast<const int4 *>(&sSum[wm * 64 + i * 32 + 8 * q + 4 * lh]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint64_t colok = __ballot(j0 + wn * 64 + j * 32 + lc < k0);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int4 sq = s[e >> 2];
          const int se = (e & 3) == 0 ? sq.x : (e & 3) == 1 ? sq.y : (e & 3) == 2 ? sq.z : sq.w;
          const uint64_t bal = __ballot(2 * acc[i][j][e] >= se) & colok;
          const uint32_t k = (uint32_t)((2 * i + j) * 16 + e);
          blo = bmlp_input_writelane((uint32_t)bal, k, blo);
          bhi = bmlp_input_writelane((uint32_t)(bal >> 32), k, bhi);
        }
      }
    }
    const int i = lane >> 5, j = (lane >> 4) & 1, e = lane & 15;
    const int cw = ((j0 + wn * 64) >> 5) + j;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m = rt * kXTile + wm * 64 + i * 32 + 8 * (e >> 2) + (e & 3) + 4 * h;
      if (m < n && cw < words32) bits[(size_t)m * words32 + cw] = h ? bhi : blo;
    }
  };
  auto stage = [&](v4u (&v)[4], uint8_t *t) {
    if (st == 0) {
      sum = 0;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (v16i){};
    }
    if (st % kChunkStages == 0) {
      const int i0 = st * kXStage;
      if (ns > kChunkStages || rt == (int)blockIdx.y) {
        __syncthreads();   // the chunk before is no longer read
        draw(i0);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = wn * 64 + j * 32 + lc;
        const uint32_t off = (uint32_t)((uint64_t)(j0 + c) * (uint64_t)k_raw + (uint64_t)i0) & 127u;
        base[j] = c * kXWords + (int)(off >> 5);
        sh[j] = off & 31u;
      }
    }
    store(v, t);
    __syncthreads();
    load(v);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int w = 2 * ks + lh;   // the lane's 32 inputs of the stage
      uint4 a[2][2];
      uint32_t r[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint4 *p = reinterpret_cast<const uint4 *>(t + (wm * 64 + i * 32 + lc) * kXLd + 32 * w);
        a[i][0] = p[0];
        a[i][1] = p[1];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t *p = sR + base[j] + 4 * (st % kChunkStages) + w;
        r[j] = __builtin_amdgcn_alignbit(p[1], p[0], sh[j]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v4i eb[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) eb[j][q] = (int)((r[j] >> (4 * h + q)) & 0x01010101u);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const v4i ea = {(int)a[i][h].x, (int)a[i][h].y, (int)a[i][h].z, (int)a[i][h].w};
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ea, eb[j], acc[i][j], 0, 0, 0);
        }
      }
    }
    if (++st < ns) return;
    st = 0;
    epilogue();
    rt += (int)gridDim.y;
  };
  v4u v0[4], v1[4];
  load(v0);
  load(v1);
  // counted, and the odd stage after the loop: left from its middle, the
  // compiler copies the stages' registers at its end, after a wait for their
  // loads (10000 x 1024 -> 3072: 44.8 us so, 40.5 now)
  int left = ns * ((row_tiles - rt + (int)gridDim.y - 1) / (int)gridDim.y);
  for (; left >= 2; left -= 2) {
    stage(v0, sX[0]);
    stage(v1, sX[1]);
  }
  if (left) stage(v0, sX[0]);
}

}  // namespace

size_t feature_median_ws_bytes(int n, int K) {
  const int splits = med_splits(n, K);
  return splits > 1 ? (size_t)splits * (size_t)K * 256 * sizeof(uint32_t) : 0;
}

hipError_t launch_feature_median(const int8_t *x, int n, int K, int8_t *med, void *ws, hipStream_t s) {
  if (n <= 0 || K <= 0) return hipSuccess;
  const int splits = ws != nullptr ? med_splits(n, K) : 1;
  if (splits > 1) {
    const int tiles = med_tiles(K, kMedFeatSplit), per_xcd = splits % 8 == 0 ? 0 : (tiles + 7) / 8;   // tiles of each XCD
    const int rows = (n - 1) / splits + 1;
    hipLaunchKernelGGL((feature_median_kernel<kMedFeatSplit>), dim3((per_xcd ? 8 * per_xcd : tiles) * splits), dim3(kMedThreads), 0, s, x, n,
                       K, med, per_xcd, rows, static_cast<uint4 *>(ws));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(median_merge_kernel, dim3((K + 3) / 4), dim3(256), 0, s, static_cast<const uint4 *>(ws), splits, n,
                       K, med);
    return hipGetLastError();
  }
  // Few rows, or features enough to fill the chip 64 at a time.  Work-groups of
  // 8 features -> of 64, us: 256 rows 784 features 4.7 -> 4.0, 1000 rows 5.2 -> 6.7,
  // 10000 x 6000: 39.5 -> 44.7, x 8192: 46.5 -> 44.6, x 16384: 87.6 -> 49.5; one
  // row of 65536: 88.8 -> 6.9.
  if (n <= 256 || K > 8192) {
    const int tiles = med_tiles(K, kWideFeat);
    hipLaunchKernelGGL(feature_median_wide_kernel, dim3(min(tiles, kWideGrid), (tiles - 1) / kWideGrid + 1), dim3(kMedThreads),
                       0, s, x, n, K, med);
    return hipGetLastError();
  }
  const int per_xcd = (med_tiles(K, kMedFeat) + 7) / 8;
  hipLaunchKernelGGL((feature_median_kernel<kMedFeat>), dim3(8 * per_xcd), dim3(kMedThreads), 0, s, x, n, K, med, per_xcd,
                     n, static_cast<uint4 *>(nullptr));
  return hipGetLastError();
}

hipError_t launch_binarize(const int8_t *x, int n, int K, const int8_t *thr, uint64_t *bits, hipStream_t s) {
  if (n <= 0 || K <= 0) return hipSuccess;
  const int words = (K + 63) / 64;
  int lpr_log = 2;   // a row has 4 words units of 16 columns
  while (lpr_log < 6 && (1 << lpr_log) < 4 * words) ++lpr_log;
  const int rows = 4 * kBinRows * (64 >> lpr_log);   // rows of a work-group
  const dim3 grid((4 * words + (1 << lpr_log) - 1) >> lpr_log, (n + rows - 1) / rows);
  if (thr != nullptr)
    hipLaunchKernelGGL((binarize_kernel<false>), grid, dim3(256), 0, s, x, n, K, words, thr, bits, lpr_log);
  else
    hipLaunchKernelGGL((binarize_kernel<true>), grid, dim3(256), 0, s, x, n, K, words, thr, bits, lpr_log);
  return hipGetLastError();
}

hipError_t launch_expand(const int8_t *x, int n, int k_raw, int k0, uint64_t seed, uint64_t *bits, hipStream_t s) {
  if (n <= 0 || k0 <= 0) return hipSuccess;
  if (k_raw <= 0) return hipErrorInvalidValue;
  // Two work-groups for each of 256 compute units, all running at once; past
  // that a work-group takes more row tiles and draws its columns' bits once
  // for all of them.  (10000 x 784 -> 3072: 39.9 us; at most 256 work-groups
  // 54.9, 384 48.1, 640 48.2, 768 43.5, 1024 40.5.)
  const int col_tiles = (k0 + kXTile - 1) / kXTile, row_tiles = (n - 1) / kXTile + 1;
  const dim3 grid(col_tiles, min(row_tiles, max(1, 512 / col_tiles)));
  uint32_t *const out = reinterpret_cast<uint32_t *>(bits);
  const int words32 = 2 * ((k0 + 63) / 64);
  if (k_raw < 16)
    hipLaunchKernelGGL((expand_kernel<kShort>), grid, dim3(256), 0, s, x, n, k_raw, k0, seed, out, words32);
  else if (k_raw % kXStage != 0)
    hipLaunchKernelGGL((expand_kernel<kRagged>), grid, dim3(256), 0, s, x, n, k_raw, k0, seed, out, words32);
  else
    hipLaunchKernelGGL((expand_kernel<kWhole>), grid, dim3(256), 0, s, x, n, k_raw, k0, seed, out, words32);
  return hipGetLastError();
}

}  // namespace bmlp
