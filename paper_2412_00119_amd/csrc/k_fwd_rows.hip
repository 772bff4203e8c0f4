// Hidden-layer forward and local outputs for a handful of patterns
// (Algorithm 1: z = a_{l-1} W_l^T, a_l = sign(z); y_hat = a_l P_l^T), by
// XNOR and popcount: z = K - 2 popcount(a xor w).
//
// Bound by latency: a launch is one read of W_l, spread over as many waves as
// possible, and what a wave does between its loads and its store.  With
// matrix tiles a few patterns fill 32 rows, a 4096-wide layer makes 64
// work-groups, and each waits for its MFMAs and a barrier.  Here a wave takes 8
// rows of W_l, one 8-byte word of each per lane and load (64 words: 4096
// inputs in one round, any row stride), so that every load is issued at once;
// the eight sums are spread over the lanes as they are added up (16 cross-lane
// steps for all eight), and the eight signs are one byte of a_l: no LDS and
// no barrier.
#include "bmlp_internal.h"

namespace bmlp {
namespace {

constexpr int kRows = 8;        // rows of B per wave
constexpr int kRowWaves = 2;    // waves of a work-group

template <int CTRL>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

// NP: patterns, at least M.  The leading arguments are preloaded into scalar
// registers when the wave starts.
template <int NP, bool SLICED>
__global__ __launch_bounds__(64 * kRowWaves) void fwd_rows_kernel(const uint64_t *pA, const uint64_t *pB, int pld,
                                                                  int pK, int pM, int pN, int punits, FwdArgs p) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  FwdSlice S;
  int unit = (int)blockIdx.x * kRowWaves + wave;   // kRows columns of z
  if constexpr (SLICED) {
    const int sli = unit / punits;
    if (sli >= p.nslices) return;
    S = p.sl[sli];
    unit -= sli * punits;
  } else {
    if (unit >= punits) return;
    S = FwdSlice{pA, pB, pld, pK, p.z, p.z32};
  }
  const int n0 = kRows * unit, nw = (S.K + 63) >> 6;
  int cnt[NP][kRows];
#pragma unroll
  for (int m = 0; m < NP; ++m)
#pragma unroll
    for (int r = 0; r < kRows; ++r) cnt[m][r] = 0;
  for (int w = lane; w < nw; w += 64) {
    uint64_t b[kRows], a[NP];
    // columns past N repeat the last row, patterns past M the last one: their
    // sums are not stored
#pragma unroll
    for (int m = 0; m < NP; ++m) a[m] = S.A[(size_t)min(m, pM - 1) * S.ld + w];
#pragma unroll
    for (int r = 0; r < kRows; ++r) b[r] = S.B[(size_t)min(n0 + r, pN - 1) * S.ld + w];
    const int left = S.K - 64 * w;
    const uint64_t valid = left >= 64 ? ~0ull : (1ull << left) - 1ull;   // left >= 1
#pragma unroll
    for (int m = 0; m < NP; ++m)
#pragma unroll
      for (int r = 0; r < kRows; ++r) cnt[m][r] += __popcll((a[m] ^ b[r]) & valid);
  }
  // Sums over the 64 lanes, spread: lane bits 5 and 4 choose four, then two of
  // the eight rows, bit 3 one of two, bits 2..0 just add.  Lane l then holds
  // the sum of row l >> 3.
  int own = 0;   // Z32: the sum of pattern lane & 7
  uint32_t bits[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    int (&v)[kRows] = cnt[m];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)v[k], (uint32_t)v[k + 4], false, false);
      v[k] = (int)((uint32_t)sw[0] + (uint32_t)sw[1]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const auto sw = __builtin_amdgcn_permlane16_swap((uint32_t)v[k], (uint32_t)v[k + 2], false, false);
      v[k] = (int)((uint32_t)sw[0] + (uint32_t)sw[1]);
    }
    const bool up = (lane & 8) != 0;
    const int send = up ? v[0] : v[1], keep = up ? v[1] : v[0];
    int s = keep + __builtin_amdgcn_update_dpp(0, send, 0x140, 0xF, 0xF, false);   // row_mirror
    s = dpp_add<0x141>(s);   // row_half_mirror
    s = dpp_add<0x4E>(s);    // quad_perm [2,3,0,1]
    s = dpp_add<0xB1>(s);    // quad_perm [1,0,3,2]
    const int z = S.K - 2 * s;
    own = (lane & 7) == m ? z : own;
    // rows' signs: bit 8r of the ballot, gathered to bit r
    const uint64_t bal = __ballot(z >= 0 && n0 + (lane >> 3) < pN) & 0x0101010101010101ull;
    bits[m] = (uint32_t)((bal * 0x0102040810204080ull) >> 56);
  }
  if (p.words_out > 0) {
    uint8_t *out = reinterpret_cast<uint8_t *>(p.abits) + unit;
    uint32_t mine = 0u;
#pragma unroll
    for (int m = 0; m < NP; ++m) mine = lane == m ? bits[m] : mine;
    if (lane < pM) out[(size_t)lane * 8 * p.words_out] = (uint8_t)mine;
  } else {
    const int m = lane & 7, col = n0 + (lane >> 3);
    if (m < pM && col < pN) S.z32[(size_t)m * p.ldz + col] = own;
  }
}

}  // namespace

// One-pattern inference over six equal widths and 100 classes, seven launches
// (fwd_small_kernel and the classifier kernel -> this kernel): 256: 29.0 ->
// 27.2 us, 1024: 29.6 -> 29.2, 4096: 32.4 -> 28.4, 8192: 49.0 -> 28.0; four
// patterns, 8192: 49.6 -> 31.4; a launch of 4096 x 4096 takes 5.0 -> 2.6 us.
// Eight patterns took 29.7 -> 32.6 at 1024 and 50.4 -> 46.4 at 8192 (z of
// eight patterns and rows in 64 registers; five to seven were not timed), so
// the line lies at four.
bool fwd_rows_wins(const FwdArgs &a) {
  return a.M <= kFwdRowsMax && ((a.mode == kFwdPlain && a.nslices == 1 && a.words_out > 0) ||
                                (a.mode == kFwdWriteZ32 && a.words_out == 0));
}

// Arguments as launch_fwd_fp4 has checked and completed them.
hipError_t launch_fwd_rows(const FwdArgs &a, hipStream_t s) {
  // with sign bits, also the last word's columns past N (zeros)
  const int units = a.words_out > 0 ? 8 * a.words_out : (a.N + kRows - 1) / kRows;
  const dim3 grid((unsigned)((a.nslices * units + kRowWaves - 1) / kRowWaves));
  const FwdSlice &s0 = a.sl[0];
#define BMLP_ROWS(NP_)                                                                                         \
  do {                                                                                                         \
    if (a.nslices > 1)                                                                                         \
      hipLaunchKernelGGL((fwd_rows_kernel<NP_, true>), grid, dim3(64 * kRowWaves), 0, s, s0.A, s0.B, s0.ld, s0.K, \
                         a.M, a.N, units, a);                                                                  \
    else                                                                                                       \
      hipLaunchKernelGGL((fwd_rows_kernel<NP_, false>), grid, dim3(64 * kRowWaves), 0, s, s0.A, s0.B, s0.ld, s0.K, \
                         a.M, a.N, units, a);                                                                  \
  } while (0)
  if (a.M <= 1)
    BMLP_ROWS(1);
  else if (a.M <= 2)
    BMLP_ROWS(2);
  else
    BMLP_ROWS(4);
#undef BMLP_ROWS
  return hipGetLastError();
}

}  // namespace bmlp
