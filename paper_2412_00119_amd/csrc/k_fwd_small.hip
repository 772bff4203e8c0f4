// Hidden-layer forward (Algorithm 1: z = a_{l-1} W_l^T, a_l = sign(z), and
// Algorithm 2's choice for gamma >= 64) where the tiles of fwd_fp4_kernel are
// too few to fill the chip.
//
// There a launch is bound by the latency of one work-group: first loads, K
// steps one after another, epilogue.  So a work-group here takes a small
// tile, 32 patterns x 64 perceptrons, and its four waves split K: wave w
// takes the chunks w, w + 4, ... of 256 elements over the whole tile, with the
// operand bit rows loaded straight into registers (buffer loads; every load
// of CH chunks is issued before the first MFMA).  No LDS ring and no barrier
// before the partial sums meet in LDS; then each wave finishes 8 rows with one
// lane per column: a row's 64 signs are one ballot and one word of a_l,
// and the 64 perceptrons of a group are the lanes of the wave.
//
// Operands by K class, a_{l-1} as ±1 in every class and W_l as ±1 in class 3
// and the bit alone in classes 0..2 (fp4.h), v_mfma_scale_f32_32x32x64_f8f6f4:
// the accumulators hold z + 2 P_a - n_low (P_a the pattern row's popcount over
// classes 0..2, n_low = K - floor(K / 4)); -2 P_a is added by one fp32 MFMA per
// accumulator.  Every value is an integer below 2^24: exact in fp32.
#include <type_traits>

#include "bmlp_internal.h"
#include "fp4.h"

namespace bmlp {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;      // K groups
constexpr int TM = 32;         // rows of a tile
constexpr int kCols = 64;      // columns of a tile
constexpr int RW = TM / kWaves;   // rows a wave finishes
constexpr int kLdRed = 72;     // floats between rows of the partial sums: rows r and r + 4 half the banks apart

// lane l: A row / B column (l & 31), half (l >> 5) of the 64-element K block;
// result element e of lane l is row 8 (e >> 2) + 4 (l >> 5) + (e & 3), column
// (l & 31).  Block scales: 1 for A, class_scale(s) for B.
__device__ __forceinline__ v16f mfma_class(const uint4 &a, const uint4 &b, v16f c, int s) {
  const v8i av = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
  const v8i bv = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 4, 0, 127, 0, class_scale(s));
}

__device__ __forceinline__ uint4 pm1_operand(const v4u &w, int s) {
  return make_uint4(pm1_class(w.x, s), pm1_class(w.y, s), pm1_class(w.z, s), pm1_class(w.w, s));
}
__device__ __forceinline__ uint4 bit_operand(const v4u &w, int s) {
  return make_uint4(class_bits(w.x, s), class_bits(w.y, s), class_bits(w.z, s), class_bits(w.w, s));
}
__device__ __forceinline__ uint4 bit_operand_masked(const v4u &w, const v4u &v, int s) {
  return make_uint4(class_bits_masked(w.x, v.x, s), class_bits_masked(w.y, v.y, s), class_bits_masked(w.z, v.z, s),
                    class_bits_masked(w.w, v.w, s));
}

// the minimum with the lane that DPP control CTRL pairs this one with
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_min(uint32_t v) {
  return min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false));
}

// v_writelane_b32 (see fwd_fp4_kernel)
extern "C" __device__ uint32_t bmlp_small_writelane(uint32_t v, uint32_t lane, uint32_t old)
    __asm("llvm.amdgcn.writelane.i32");

// The leading arguments are preloaded into scalar registers when the wave
// starts, so that the first loads do not wait for the argument buffer.
// CH: chunks per load round.
template <int CH, bool SLICED>
__global__ __launch_bounds__(64 * kWaves) void fwd_small_kernel(const uint64_t *pA, const uint64_t *pB,
                                                                const int32_t *py, int pld, int pK, int pM, int pN,
                                                                int pnt_m, int pnt_n, int pper, int pmode,
                                                                FwdArgs p) {
  __shared__ float red[kWaves][TM][kLdRed];
  const int tid = threadIdx.x, kg = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lc = lane & 31, lh = lane >> 5;
  FwdSlice S;
  int b = (int)blockIdx.x;
  if constexpr (SLICED) {
    const int tiles = pper ? 8 * pper * pnt_m : pnt_m * pnt_n;
    const int sli = b / tiles;
    S = p.sl[sli];
    b -= sli * tiles;
  } else {
    S = FwdSlice{pA, pB, pld, pK, p.z, p.z32};
  }
  int mt, nt;
  if (pper) {   // XCD x (work-group id mod 8) takes the column tiles x pper ..
    const int idx = b >> 3;
    nt = (b & 7) * pper + idx / pnt_m;
    mt = idx % pnt_m;
    if (nt >= pnt_n) return;
  } else {
    nt = b / pnt_m;
    mt = b % pnt_m;
  }
  const int m0 = mt * TM, n0 = nt * kCols;
  if (p.zero != nullptr && blockIdx.x == 0)   // the step statistics start at zero
    for (int i = tid; i < p.nzero; i += 64 * kWaves) p.zero[i] = 0;

  // the label of the row lane q < RW of this wave looks up below, first: its
  // classifier word (64 columns of rho^{y}) is requested once it is here
  const int mq = m0 + RW * kg + min(lane, RW - 1);   // the lane's row in the epilogue
  int label = 0;
  const bool selects = pmode == kFwdFusedSelect || pmode == kFwdSelectParts;
  if (selects) label = py[min(mq, pM - 1)];

  const uint32_t rowbytes = 8u * (uint32_t)S.ld;
  const __amdgpu_buffer_rsrc_t rsA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(S.A), 0, (int)((uint32_t)pM * rowbytes), kRawRsrcWord3);
  const __amdgpu_buffer_rsrc_t rsB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(S.B), 0, (int)((uint32_t)pN * rowbytes), kRawRsrcWord3);
  // lane (row, half): bytes 32 chunk + 16 half .. of its row; rows past the
  // matrix repeat the last one, bytes past a row are the next row's (masked
  // below) or, past the matrix, zeros
  uint32_t offB[2];
  const uint32_t offA = (uint32_t)min(m0 + lc, pM - 1) * rowbytes + 16u * lh;
#pragma unroll
  for (int j = 0; j < 2; ++j) offB[j] = (uint32_t)min(n0 + 32 * j + lc, pN - 1) * rowbytes + 16u * lh;

  v16f acc[2] = {(v16f){}, (v16f){}};
  int pa = 0;   // P_a over the lane's words

  const int nch = (S.K + 255) / 256, nfull = S.K / 256;
  uint64_t rho = 0ull;
  struct Chunk {
    v4u a, b[2];
  };
  auto load = [&](Chunk &c, int ch) {
    const uint32_t so = 32u * (uint32_t)ch;
    c.a = __builtin_amdgcn_raw_buffer_load_b128(rsA, (int)(offA + so), 0, 0);
#pragma unroll
    for (int j = 0; j < 2; ++j) c.b[j] = __builtin_amdgcn_raw_buffer_load_b128(rsB, (int)(offB[j] + so), 0, 0);
  };
  auto compute = [&](const Chunk &c, int ch) {
    if (ch < nfull) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint4 eb[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) eb[j] = bit_operand(c.b[j], s);
        const uint4 ea = pm1_operand(c.a, s);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = mfma_class(ea, eb[j], acc[j], s);
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) pa += __popc(c.a[d] & kLowClasses);
    } else if (ch < nch) {   // the chunk that holds K's end
      v4u valid;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int nv = S.K - (256 * ch + 128 * lh + 32 * d);
        valid[d] = nv >= 32 ? 0xFFFFFFFFu : nv <= 0 ? 0u : ((1u << nv) - 1u);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint4 eb[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) eb[j] = bit_operand_masked(c.b[j], valid, s);
        const uint4 ea = pm1_operand(c.a, s);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = mfma_class(ea, eb[j], acc[j], s);
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) pa += __popc(c.a[d] & kLowClasses & valid[d]);
    }
  };
  Chunk cur[CH];
  // a chunk past the last one is loaded (zeros, or the next rows' bytes) but
  // not used
#pragma unroll
  for (int u = 0; u < CH; ++u) load(cur[u], kg + kWaves * u);
  if (selects) {
    const int yl = min(max(label, 0), p.c - 1);   // stay inside P on a bad label
    rho = p.P[(size_t)yl * p.ldp + min(n0 >> 6, p.pw_max)];
  }
  for (int ch = kg; ch < nch; ch += kWaves * CH) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      compute(cur[u], ch + kWaves * u);
      // the chunk's registers take its successor of the next round
      if (ch + kWaves * CH < nch) load(cur[u], ch + kWaves * (CH + u));
    }
  }
  // -2 P_a of every row, both halves (k = l >> 5) at once: A = -2 P_a, B = 1
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(-2.f * (float)pa, 1.f, acc[j], 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 16; ++e) red[kg][8 * (e >> 2) + 4 * lh + (e & 3)][32 * j + lc] = acc[j][e];
  }
  __syncthreads();

  // ---- epilogue: rows RW kg .. of the tile, lane = column -----------------------
  const float nlow = (float)(S.K - S.K / 4);
  float z[RW];
#pragma unroll
  for (int q = 0; q < RW; ++q) {
    z[q] = nlow;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) z[q] += red[k][RW * kg + q][lane];
  }
  const int col = n0 + lane;
  const uint64_t colok = __ballot(col < pN);
  if (p.words_out > 0) {   // a_l = sign(z): lane q takes row q's word
    uint32_t lo = 0u, hi = 0u;
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      const uint64_t bal = __ballot(z[q] >= 0.f) & colok;
      lo = bmlp_small_writelane((uint32_t)bal, (uint32_t)q, lo);
      hi = bmlp_small_writelane((uint32_t)(bal >> 32), (uint32_t)q, hi);
    }
    if (lane < RW && mq < pM) p.abits[(size_t)mq * p.words_out + (n0 >> 6)] = (uint64_t)lo | ((uint64_t)hi << 32);
  }
  if (selects) {
    // key of (row, column) as in fwd_fp4_kernel: bits(s) - bits(1.0f) + k with
    // s = -z where rho = +1, else z; below 2^27 exactly for the wrong
    // perceptrons, in the order (|z|, k)
    const uint32_t rlo = (uint32_t)rho, rhi = (uint32_t)(rho >> 32);
    const bool clip = p.zlo > -32767.f || p.zhi < 32767.f;
    const uint32_t kbase = (uint32_t)lane - 0x3F800000u;
    uint32_t keys[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)rlo, q) |
                         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)rhi, q) << 32);
      const float zc = clip ? fminf(fmaxf(z[q], p.zlo), p.zhi) : z[q];
      const float s = __builtin_amdgcn_inverse_ballot_w64(r) ? -zc : zc;
      keys[q] = __float_as_uint(s) + kbase;
    }
    // minimum over the 64 lanes, the eight rows spread over them: lane bits
    // 5, 4 and 3 choose which of two rows a lane keeps, bits 2..0 just reduce
    static_assert(RW == 8, "three lane bits for the rows");
    const int m = m0 + RW * kg + 4 * lh + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1);   // the lane's row then
    const bool writes = (lane & 7) == 0 && m < pM;
    auto lowest = [&](uint32_t (&v)[RW]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const auto sw = __builtin_amdgcn_permlane32_swap(v[k], v[k + 4], false, false);
        v[k] = min((uint32_t)sw[0], (uint32_t)sw[1]);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const auto sw = __builtin_amdgcn_permlane16_swap(v[k], v[k + 2], false, false);
        v[k] = min((uint32_t)sw[0], (uint32_t)sw[1]);
      }
      const bool up = (lane & 8) != 0;
      const uint32_t send = up ? v[0] : v[1], keep = up ? v[1] : v[0];
      uint32_t key = min(keep, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x140, 0xF, 0xF, false));   // row_mirror
      key = dpp_min<0x141>(key);   // row_half_mirror
      key = dpp_min<0x4E>(key);    // quad_perm [2,3,0,1]
      return dpp_min<0xB1>(key);   // quad_perm [1,0,3,2]
    };
    if (pmode == kFwdFusedSelect) {   // the tile is a group
      const uint32_t key = lowest(keys);
      if (writes) p.kstar[(size_t)nt * p.ldk + m] = key >= (1u << 27) ? (int16_t)-1 : (int16_t)(key & 0x3Fu);
    } else {                          // columns [0, end) of one group, [end, 64) of the next
      const int end = p.gamma - n0 % p.gamma;
      uint32_t v[RW];
#pragma unroll
      for (int q = 0; q < RW; ++q) v[q] = lane < end && col < pN ? keys[q] : 0xFFFFFFFFu;
      uint32_t key = lowest(v);
      if (writes) p.part[(size_t)(2 * nt) * pM + m] = key;
      if (end < kCols) {
#pragma unroll
        for (int q = 0; q < RW; ++q) v[q] = lane >= end && col < pN ? keys[q] : 0xFFFFFFFFu;
        key = lowest(v);
        if (writes) p.part[(size_t)(2 * nt + 1) * pM + m] = key;
      }
    }
  } else if (pmode != kFwdPlain && col < pN) {
#pragma unroll
    for (int q = 0; q < RW; ++q) {
      const int m = m0 + RW * kg + q;
      if (m >= pM) break;
      if (pmode == kFwdWriteZ32)
        S.z32[(size_t)m * p.ldz + col] = (int)z[q];
      else
        S.z[(size_t)m * p.ldz + col] = (int16_t)(int)z[q];
    }
  }
}

template <int CH>
void launch_shape(bool sliced, dim3 grid, int nt_m, int nt_n, int per, const FwdArgs &a, hipStream_t s) {
  const FwdSlice &s0 = a.sl[0];
#define BMLP_SMALL_ARGS s0.A, s0.B, a.y, s0.ld, s0.K, a.M, a.N, nt_m, nt_n, per, a.mode, a
  if (sliced)
    hipLaunchKernelGGL((fwd_small_kernel<CH, true>), grid, dim3(64 * kWaves), 0, s, BMLP_SMALL_ARGS);
  else
    hipLaunchKernelGGL((fwd_small_kernel<CH, false>), grid, dim3(64 * kWaves), 0, s, BMLP_SMALL_ARGS);
#undef BMLP_SMALL_ARGS
}

}  // namespace

// Two work-groups per compute unit, up to which every first load is in
// flight at once.  Per launch, inference over equal widths (us including the
// dependent launch; 128 x 128 tiles, 64 x 128 tiles of fwd_fp4_kernel -> this kernel): 8 x
// 4096: 8.6, 6.5 -> 5.1; 256 x 1024: 5.6, 4.6 -> 3.8; 512 x 2048 (512 tiles): 6.6,
// 5.3 -> 5.3; past 512 tiles 640 x 2048: 6.7, 5.4 -> 6.0, 512 x 4096: 9.0, 7.1
// -> 10.4.  With few chunks, half as many tiles more are about even (training
// step of six layers, 64 x 128 tiles -> this kernel: 1536 x 1024 (768 tiles)
// 48.9 -> 49.2, 3072 x 512 78.9 -> 74.1, 6144 x 256 102.9 -> 101.4; inference 26.8 ->
// 29.2, 24.1 -> 26.9, 26.3 -> 25.2).
bool fwd_small_wins(const FwdArgs &a) {
  const long long tiles = (long long)a.nslices * ((a.M + TM - 1) / TM) * ((a.N + kCols - 1) / kCols);
  int kmax = 0;
  for (int i = 0; i < a.nslices; ++i) kmax = a.sl[i].K > kmax ? a.sl[i].K : kmax;
  return tiles <= (kmax <= 256 * kWaves ? 768 : 512);
}

// Arguments as launch_fwd_fp4 has checked and completed them.
hipError_t launch_fwd_small(const FwdArgs &a, hipStream_t s) {
  const int nt_m = (a.M + TM - 1) / TM, nt_n = (a.N + kCols - 1) / kCols;
  // each XCD reads its own slice of B's rows, unless that would leave XCDs
  // with much less work than others
  const int per = nt_n % 8 == 0 || nt_n >= 24 ? (nt_n + 7) / 8 : 0;
  const dim3 grid((unsigned)a.nslices * (unsigned)(per ? 8 * per * nt_m : nt_m * nt_n));
  int kmax = 0;
  for (int i = 0; i < a.nslices; ++i) kmax = a.sl[i].K > kmax ? a.sl[i].K : kmax;
  const bool sliced = a.nslices > 1;
  const int per_wave = ((kmax + 255) / 256 + kWaves - 1) / kWaves;   // chunks of a wave
  if (per_wave <= 1)
    launch_shape<1>(sliced, grid, nt_m, nt_n, per, a, s);
  else if (per_wave <= 2)
    launch_shape<2>(sliced, grid, nt_m, nt_n, per, a, s);
  else
    launch_shape<4>(sliced, grid, nt_m, nt_n, per, a, s);
  return hipGetLastError();
}

}  // namespace bmlp
