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
// The median of kMedFeat neighbouring features per work-group, from 256-bin
// histograms in LDS.
//
// What bounds it: each feature's whole column is counted by one work-group
// (there is no scratch memory to merge partial counts in), so a compute unit
// takes n cache lines, one per row, and the line fills (two cycles each)
// are what is left.  To get there the counting must cost less than that:
//   * a lane loads its row's kMedFeat bytes at once, and a thread has
//     kMedRows rows in flight (16 waves: enough to cover memory latency);
//   * the histograms are kept kMedCopies times, bin-major, one LDS bank per
//     (copy, feature) slot, and lane l counts its bytes in the rotated order
//     l, l + 1, ... (mod kMedFeat) into the copy l / kMedFeat.  So the 64
//     lanes of every atomic are in 64 different banks, whatever the data
//     (features with few distinct values included);
//   * an atomic's address is one v_perm_b32: byte 0 the slot, byte 1 the
//     value.
// The work-groups of one XCD take neighbouring features, so a row's cache
// line is fetched into one or two L2s instead of all eight.
// 60000 x 784 (47 MB): 3810 -> 75 us (the kernel before had a work-group of
// 256 threads per 64 features, one byte load per thread in flight).
constexpr int kMedFeat = 8;
constexpr int kMedCopies = 64 / kMedFeat;
constexpr int kMedThreads = 1024;
constexpr int kMedRows = 8;      // rows per thread and pass

// the 8 bytes at p (any alignment)
__device__ __forceinline__ uint2 load8(const int8_t *p) {
  uint2 v;
  __builtin_memcpy(&v, p, 8);
  return v;
}

__global__ __launch_bounds__(kMedThreads) void feature_median_kernel(const int8_t *__restrict__ x, int n, int K,
                                                                     int8_t *__restrict__ med, int per_xcd) {
  __shared__ uint32_t hist[256][64];
  const int tid = threadIdx.x, lane = tid & 63;
  // XCD b % 8 takes the tiles [per_xcd * (b % 8), + per_xcd)
  const int tile = per_xcd * ((int)blockIdx.x & 7) + ((int)blockIdx.x >> 3);
  // the last tile starts early enough to stay inside the row (its first
  // features are then counted twice, with the same result)
  const int f0 = max(0, min(tile * kMedFeat, K - kMedFeat));
  if (tile * kMedFeat >= K) return;
  for (int i = tid; i < 256 * 64 / 4; i += kMedThreads) reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const int rot = lane % kMedFeat, copy0 = lane - rot;
  uint32_t slot[kMedFeat];   // byte address of the slot within a bin, per step
#pragma unroll
  for (int j = 0; j < kMedFeat; ++j) slot[j] = 4u * (uint32_t)(copy0 + (rot + j) % kMedFeat);
  uint8_t *const base = reinterpret_cast<uint8_t *>(hist);
  auto count = [&](uint2 v) {
    // value + 128 per byte, then the bytes rotated by rot
    uint64_t w = ((uint64_t)(v.y ^ 0x80808080u) << 32) | (v.x ^ 0x80808080u);
    if (rot) w = (w >> (8 * rot)) | (w << (64 - 8 * rot));
    const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
#pragma unroll
    for (int j = 0; j < kMedFeat; ++j) {
      // bytes: [slot, value, 0, 0] (selector 0x0C gives a zero byte, 0 the
      // second source's byte 0, 4 + b the first source's byte b)
      const uint32_t addr = __builtin_amdgcn_perm(j < 4 ? lo : hi, slot[j], 0x0C0C0000u | ((4u + (j & 3)) << 8));
      atomicAdd(reinterpret_cast<uint32_t *>(base + addr), 1u);
    }
  };
  if (K >= kMedFeat) {
    const int8_t *xf = x + f0;
    const uint32_t rows = (uint32_t)n;
    uint32_t r = (uint32_t)tid;
    for (; r + (kMedRows - 1) * kMedThreads < rows; r += kMedRows * kMedThreads) {
      uint2 v[kMedRows];
#pragma unroll
      for (int q = 0; q < kMedRows; ++q) v[q] = load8(xf + (size_t)(r + q * kMedThreads) * K);
#pragma unroll
      for (int q = 0; q < kMedRows; ++q) count(v[q]);
    }
    for (; r < rows; r += kMedThreads) count(load8(xf + (size_t)r * K));
  } else {   // rows of fewer bytes than a load
    for (uint32_t r = (uint32_t)tid; r < (uint32_t)n; r += kMedThreads)
      for (int f = 0; f < K; ++f) atomicAdd(&hist[(int)x[(size_t)r * K + f] + 128][copy0 + f], 1u);
  }
  __syncthreads();
  // one wave per feature: lane l sums the copies of bins 4l .. 4l + 3, the
  // wave scans, and the lane in whose bins the running count reaches
  // floor((n - 1) / 2) + 1 writes the value
  const int f = tid >> 6;
  if (f < kMedFeat && f0 + f < K) {
    const uint32_t want = (uint32_t)((n - 1) / 2) + 1u;
    uint32_t c[4], own = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c[q] = 0u;
      // each lane starts at a copy of its own (spreads the banks)
#pragma unroll
      for (int k = 0; k < kMedCopies; ++k) c[q] += hist[4 * lane + q][((lane + k) % kMedCopies) * kMedFeat + f];
      own += c[q];
    }
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
      med[f0 + f] = (int8_t)(v - 128);
    }
  }
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
// 60000 x 784 (47 MB): 107 -> 12.3 us; the kernel before took one byte per
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
  if (col + 16 <= K) {
    BinLane t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t w = 0x01010101u;
      if constexpr (!PM1) __builtin_memcpy(&w, thr + col + 4 * q, 4);
      w ^= 0x80808080u;
      t.te[q] = w & 0x00FF00FFu;
      t.to[q] = (w >> 8) & 0x00FF00FFu;
    }
    uint4 v[kBinRows];
#pragma unroll
    for (int i = 0; i < kBinRows; ++i) __builtin_memcpy(&v[i], x + (size_t)min(row0 + i * rpw, n - 1) * K + col, 16);
#pragma unroll
    for (int i = 0; i < kBinRows; ++i) {
      const int row = row0 + i * rpw;
      if (row < n)
        out[(size_t)row * 4 * words] = (uint16_t)(ge4(v[i].x, t, 0) | (ge4(v[i].y, t, 1) << 4) |
                                                  (ge4(v[i].z, t, 2) << 8) | (ge4(v[i].w, t, 3) << 12));
    }
  } else {   // the row's end: byte loads, and zeros past column K
    for (int i = 0; i < kBinRows; ++i) {
      const int row = row0 + i * rpw;
      if (row >= n) break;
      uint32_t m = 0u;
      for (int c = 0; c < 16 && col + c < K; ++c)
        m |= (uint32_t)(x[(size_t)row * K + col + c] >= (PM1 ? (int8_t)1 : thr[col + c])) << c;
      out[(size_t)row * 4 * words] = (uint16_t)m;
    }
  }
}

// bits e .. e + 31 of stream 5 (32 consecutive elements; they straddle at
// most two Philox blocks)
__device__ uint32_t expand_bits32(uint64_t e, uint32_t k0, uint32_t k1) {
  const uint32_t blk = (uint32_t)(e >> 7), off = (uint32_t)(e & 127);
  const U32x4 a = philox4x32_10(blk, 0xFFFFFFFFu, 0u, kStreamExpand, k0, k1);
  const uint32_t wi = off >> 5, sh = off & 31;
  const uint32_t lo = pick_word(a, wi);
  uint32_t hi;
  if (wi < 3) {
    hi = pick_word(a, wi + 1);
  } else {
    const U32x4 b = philox4x32_10(blk + 1u, 0xFFFFFFFFu, 0u, kStreamExpand, k0, k1);
    hi = b.x;
  }
  return sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
}

constexpr int kXCols = 64;    // output columns (R rows) per work-group
constexpr int kXRows = 64;    // patterns per pass
constexpr int kXWords = 128;  // R words per column held in LDS (4096 inputs)

// Work-group: 64 output columns j0 .. j0 + 63 and a chunk of patterns.
// The columns' R rows are made once, as bits in LDS (in passes of 4096
// inputs); thread (pattern p, column group g) sums 16 columns with sdot4 on
// 4 int8 inputs and 4 ±1 bytes at a time.
__global__ __launch_bounds__(256) void expand_kernel(const int8_t *__restrict__ x, int n, int k_raw, int k0,
                                                     uint64_t seed, int rows_per_block, uint64_t *__restrict__ bits,
                                                     int words_out) {
  __shared__ uint32_t sR[kXCols][kXWords + 1];
  __shared__ int32_t sZ[kXRows][kXCols + 1];
  const int j0 = blockIdx.x * kXCols;
  const int p0 = blockIdx.y * rows_per_block;
  const int p1 = min(n, p0 + rows_per_block);
  const uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32);
  const int tid = threadIdx.x;
  const int pl = tid >> 2, cg = tid & 3;   // pattern in the pass, group of 16 columns
  for (int q0 = p0; q0 < p1; q0 += kXRows) {
    int32_t z[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) z[c] = 0;
    const int mu = q0 + pl;
    const int8_t *xr = x + (size_t)min(mu, n - 1) * k_raw;
    for (int i0 = 0; i0 < k_raw; i0 += 32 * kXWords) {
      const int nw = min(kXWords, (k_raw - i0 + 31) / 32);
      __syncthreads();   // the previous pass's R words are no longer read
      for (int t = tid; t < kXCols * nw; t += 256) {
        const int c = t / nw, w = t % nw;
        const int j = j0 + c, i = i0 + 32 * w;
        uint32_t r = 0u;
        if (j < k0) {
          r = expand_bits32((uint64_t)j * (uint64_t)k_raw + (uint64_t)i, key0, key1);
          const int valid = min(32, k_raw - i);   // past the row: no input, no weight
          if (valid < 32) r &= (1u << valid) - 1u;
        }
        sR[c][w] = r;
      }
      __syncthreads();
      for (int w = 0; w < nw; ++w) {
        const int i = i0 + 32 * w;
        // 32 inputs as 8 words of 4 int8 (zero past the row)
        int xs[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          uint32_t v = 0u;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int ii = i + 4 * q + b;
            if (ii < k_raw) v |= (uint32_t)(uint8_t)xr[ii] << (8 * b);
          }
          xs[q] = (int)v;
        }
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const uint32_t r = sR[cg * 16 + c][w];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            // the 4 weights of inputs 4q .. 4q + 3 as bytes +1 / -1 (0xFF);
            // inputs past the row are 0, so their weight does not matter
            // bit b of the nibble to bit 0 of byte b (the four shifted
            // copies do not overlap), then 1 -> 0x01 and 0 -> 0xFF
            const uint32_t nib = (r >> (4 * q)) & 0xFu;
            const uint32_t spread = (nib * 0x00204081u) & 0x01010101u;
            const uint32_t wv = ~(spread * 0xFEu);
            z[c] = __builtin_amdgcn_sdot4(xs[q], (int)wv, z[c], false);
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 16; ++c) sZ[pl][cg * 16 + c] = z[c];
    __syncthreads();
    // a_0 = sign(z), sign(0) = +1: one ballot per (pattern, 64 columns)
    const int wave = tid >> 6, lane = tid & 63;
    for (int r = wave; r < kXRows; r += 4) {
      const int m = q0 + r;
      const bool pos = j0 + lane < k0 && sZ[r][lane] >= 0;
      const uint64_t bal = __ballot(pos);
      if (lane == 0 && m < p1) bits[(size_t)m * words_out + (j0 >> 6)] = bal;
    }
  }
}

}  // namespace

hipError_t launch_feature_median(const int8_t *x, int n, int K, int8_t *med, hipStream_t s) {
  if (n <= 0 || K <= 0) return hipSuccess;
  const int per_xcd = ((K + kMedFeat - 1) / kMedFeat + 7) / 8;   // tiles of each XCD
  hipLaunchKernelGGL(feature_median_kernel, dim3(8 * per_xcd), dim3(kMedThreads), 0, s, x, n, K, med, per_xcd);
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
  const int rows_per_block = 256;   // patterns per work-group (R made once per 256 patterns)
  const dim3 grid((k0 + kXCols - 1) / kXCols, (n + rows_per_block - 1) / rows_per_block);
  hipLaunchKernelGGL(expand_kernel, grid, dim3(256), 0, s, x, n, k_raw, k0, seed, rows_per_block, bits,
                     (k0 + 63) / 64);
  return hipGetLastError();
}

}  // namespace bmlp
