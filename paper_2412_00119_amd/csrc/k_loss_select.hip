// Local error signal and perceptron selection (Algorithm 1 01-loss and
// robustness test, Eq. 1; Algorithm 2 easiest-perceptron choice).
//
// Error signal, one wave per pattern: given y_hat, the first argmax and the
// two largest values (tau = top1 - top2, 0 on a tie), err = (pred != y) and
// upd = err or tau < ceil(r K_l).
// Selection, for every pattern and every group of gamma perceptrons
// (contiguous, or consecutive in the reshuffle variant's per-step order): the
// one with the largest negative stability delta_k = z_k rho^{y}_k, i.e. the
// smallest |z_k| among those whose sign disagrees with rho^{y}_k, lowest k on
// ties; delta = 0 is not eligible.  The update keeps only the patterns in M.
#include <limits.h>

#include "bmlp_internal.h"
#include "gather.h"
#include "philox.h"

namespace bmlp {
namespace {

struct Top2 {
  int v1, i1, v2;
};

__device__ __forceinline__ Top2 merge(Top2 a, Top2 b) {
  Top2 r;
  if (a.v1 > b.v1 || (a.v1 == b.v1 && a.i1 < b.i1)) {
    r.v1 = a.v1;
    r.i1 = a.i1;
  } else {
    r.v1 = b.v1;
    r.i1 = b.i1;
  }
  // second largest value of the union of the two multisets
  r.v2 = max(min(a.v1, b.v1), max(a.v2, b.v2));
  return r;
}

__device__ __forceinline__ Top2 wave_top2(const int32_t *row, int c, int lane) {
  Top2 t{INT_MIN, INT_MAX, INT_MIN};
  for (int cl = lane; cl < c; cl += 64) {
    const int v = row[cl];
    if (v > t.v1) {
      t.v2 = t.v1;
      t.v1 = v;
      t.i1 = cl;
    } else if (v > t.v2) {
      t.v2 = v;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Top2 o;
    o.v1 = __shfl_xor(t.v1, off, 64);
    o.i1 = __shfl_xor(t.i1, off, 64);
    o.v2 = __shfl_xor(t.v2, off, 64);
    t = merge(t, o);
  }
  return t;
}

// The first sel_blocks work-groups select, the others (when y_hat is given)
// take the error signal of four patterns each.
//
// Selection: lpi = 2^lpi_log neighbouring lanes share a (pattern, group) item,
// lane s taking the group's members s, s + lpi, ..., then merge their keys.
// It is bound by the latency of its loads (z and the rho words), so a lane's
// walk is short (about 8 to 16 members) and its loads are independent; the
// items of a work-group are neighbouring groups of one pattern, so that the
// lines of z are used whole.  With one lane per item and gamma dependent
// steps it took 29 us (100 patterns, 5 groups of 105) and 20 us (500
// patterns, 25 groups of 81); now 5.0 and 5.3 us.  (On the matrix cores such
// groups, contiguous and above 64, now come here only where their keys do not
// fit the z scratch; groups below 64 and reshuffled ones always do.)
constexpr int kSelThreads = 256;

template <bool PERM>
__global__ __launch_bounds__(kSelThreads) void loss_select_kernel(LossSelectArgs p, int sel_blocks, int lpi_log) {
  if ((int)blockIdx.x < sel_blocks) {
    const long long t = (long long)blockIdx.x * kSelThreads + threadIdx.x;
    const long long item = t >> lpi_log;
    const int lpi = 1 << lpi_log, sub = (int)threadIdx.x & (lpi - 1);
    const bool on = item < (long long)p.n * p.groups;
    const int mu = on ? (int)(item / p.groups) : 0, g = on ? (int)(item % p.groups) : 0;
    const int yl = min(max(p.y[mu], 0), p.c - 1);      // stay inside P on a bad label
    const int16_t *zr = p.z + (size_t)mu * p.ldz;
    const uint32_t *rho = reinterpret_cast<const uint32_t *>(p.P + (size_t)yl * p.words_out);
    const int k0 = g * p.gamma;
    // key: |z| then k (both below 2^15); best is the member's place in the group
    uint32_t bestkey = 0xFFFFFFFFu;
    int best = -1;
#pragma unroll 4
    for (int e = sub; e < p.gamma; e += lpi) {
      const int k = PERM ? p.perm[k0 + e] : k0 + e;
      const int zz = min(max((int)zr[k], p.zlo), p.zhi);   // z as the selection sees it
      const bool rpos = (rho[k >> 5] >> (k & 31)) & 1u;
      const bool wrong = rpos ? (zz < 0) : (zz > 0);
      const uint32_t key = wrong ? ((uint32_t)(zz < 0 ? -zz : zz) << 15) | (uint32_t)k : 0xFFFFFFFFu;
      if (key < bestkey) {
        bestkey = key;
        best = e;
      }
    }
    for (int d = lpi >> 1; d >= 1; d >>= 1) {
      const uint32_t ok = (uint32_t)__shfl_xor((int)bestkey, d, 64);
      const int ob = __shfl_xor(best, d, 64);
      if (ok < bestkey) {
        bestkey = ok;
        best = ob;
      }
    }
    if (on && sub == 0) p.kstar[(size_t)g * p.ldk + mu] = (int16_t)best;
    return;
  }
  __shared__ int cnt[2];
  if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int mu = ((int)blockIdx.x - sel_blocks) * 4 + ((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (mu < p.n) {
    const Top2 t = wave_top2(p.yhat + (size_t)mu * p.c, p.c, lane);
    const bool err = t.i1 != p.y[mu];
    const bool upd = err || (t.v1 - t.v2) < p.thr;
    if (lane == 0) {
      p.err[mu] = err ? 1 : 0;
      p.upd[mu] = upd ? 1 : 0;
      if (err) atomicAdd(&cnt[0], 1);
      if (upd) atomicAdd(&cnt[1], 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {   // one global atomic per counter and work-group
    if (cnt[0]) atomicAdd(p.stats + 0, cnt[0]);
    if (cnt[1]) atomicAdd(p.stats + 1, cnt[1]);
  }
}

__global__ __launch_bounds__(256) void eval_count_kernel(const int32_t *yhat, int c, const int32_t *y,
                                                         int n, int32_t *correct, uint8_t *flag, int thr) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  const int mu = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (mu < n) {
    const Top2 t = wave_top2(yhat + (size_t)mu * c, c, lane);
    const bool ok = t.i1 == y[mu];
    if (lane == 0) {
      if (flag != nullptr)
        flag[mu] = (uint8_t)((ok ? 1 : 0) | ((t.v1 - t.v2) >= thr ? 2 : 0));
      else if (ok)
        atomicAdd(&cnt, 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && cnt) atomicAdd(correct, cnt);
}

// Correct predictions of every layer and early exits (one thread per pattern):
// a pattern leaves at the first layer whose flag has bit 1 (margin reached),
// else at the last.  Counts are ballots, gathered per work-group in LDS, then
// one atomic per nonzero counter: atomics on one address run one after
// the other, so the counts are made here, by few large work-groups, and not
// by the classifiers' (one per 16 patterns and layer; eval of 10000 patterns
// over three 256-wide layers, 10 classes: 37.9 -> 22.0 us).
constexpr int kExitThreads = 1024;

__global__ __launch_bounds__(kExitThreads) void exit_count_kernel(const uint8_t *flags, int ldf, int L, int n,
                                                                  int32_t *counts) {
  __shared__ int cnt[3 * BMLP_MAX_LAYERS];
  for (int i = threadIdx.x; i < 3 * L; i += kExitThreads) cnt[i] = 0;
  __syncthreads();
  const int mu = blockIdx.x * kExitThreads + threadIdx.x, lane = threadIdx.x & 63;
  bool left = mu >= n;   // a thread past the patterns has none to count
  const int muc = min(mu, n - 1);
  for (int l = 0; l < L; ++l) {
    const uint8_t f = mu < n ? flags[(size_t)l * ldf + muc] : (uint8_t)0;
    const bool leaves = !left && ((f & 2) || l == L - 1);
    left |= leaves;
    const int c0 = __popcll(__ballot(f & 1)), c1 = __popcll(__ballot(leaves)), c2 = __popcll(__ballot(leaves && (f & 1)));
    if (lane < 3) {
      const int v = lane == 0 ? c0 : lane == 1 ? c1 : c2;
      if (v) atomicAdd(&cnt[3 * l + lane], v);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 3 * L; i += kExitThreads)
    if (cnt[i]) atomicAdd(counts + i, cnt[i]);
}

__global__ __launch_bounds__(256) void gather_batch_kernel(GatherArgs a) {
  gather_item(a, blockIdx.x * 256u + threadIdx.x);
}

// The reshuffle variant's group order: perceptron k's key is word (k & 3)
// of stream-6 block k >> 2, and its position is its rank among all K keys
// (ties by index).  One thread per perceptron counts the keys below its
// own, with the keys staged through LDS kPermChunk at a time; every block
// makes each chunk's keys itself (a few Philox blocks per thread).
constexpr int kPermThreads = 256;
constexpr int kPermChunk = 2048;

__device__ __forceinline__ uint32_t word_of(const U32x4 &w, int i) {
  return i == 0 ? w.x : i == 1 ? w.y : i == 2 ? w.z : w.w;
}

__global__ __launch_bounds__(kPermThreads) void group_perm_kernel(PermBatch p) {
  __shared__ uint4 keys[kPermChunk / 4];
  int li = 0;
#pragma unroll 1
  for (int i = 1; i < p.nl; ++i)
    if ((int)blockIdx.x >= p.L[i].block0) li = i;
  const PermLayer &q = p.L[li];
  const int k = ((int)blockIdx.x - q.block0) * kPermThreads + (int)threadIdx.x;
  const bool on = k < q.k;
  uint32_t mine = 0;
  if (on) mine = word_of(philox4x32_10((uint32_t)k >> 2, q.ctr1, p.step, kStreamGroups, p.key0, p.key1), k & 3);
  int rank = 0;
#pragma unroll 1
  for (int j0 = 0; j0 < q.k; j0 += kPermChunk) {
    const int nj = min(kPermChunk, q.k - j0);
    __syncthreads();   // the previous chunk has been read
    for (int b = threadIdx.x; b < (nj + 3) / 4; b += kPermThreads) {
      const U32x4 w = philox4x32_10((uint32_t)(j0 / 4 + b), q.ctr1, p.step, kStreamGroups, p.key0, p.key1);
      keys[b] = make_uint4(w.x, w.y, w.z, w.w);
    }
    __syncthreads();
    if (on) {
      // keys of indices below k count on ties, the others only when smaller
      int j = 0;
#pragma unroll 4
      for (; j + 4 <= nj; j += 4) {
        const uint4 v = keys[j / 4];
        const int jj = j0 + j;
        rank += (v.x < mine) | ((v.x == mine) & (jj < k));
        rank += (v.y < mine) | ((v.y == mine) & (jj + 1 < k));
        rank += (v.z < mine) | ((v.z == mine) & (jj + 2 < k));
        rank += (v.w < mine) | ((v.w == mine) & (jj + 3 < k));
      }
      const uint32_t *tail = reinterpret_cast<const uint32_t *>(keys);
      for (; j < nj; ++j) rank += (tail[j] < mine) | ((tail[j] == mine) & (j0 + j < k));
    }
  }
  if (on) q.perm[rank] = k;
}

}  // namespace

hipError_t launch_loss_select(const LossSelectArgs &a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (a.gamma < 1 || a.groups < 1) return hipErrorInvalidValue;
  int lpi_log = 0;   // at most 16 members per lane while lanes last
  while (lpi_log < 6 && (a.gamma >> lpi_log) > 16) ++lpi_log;
  const long long lanes = ((long long)a.n * a.groups) << lpi_log;
  const int sel_blocks = (int)((lanes + kSelThreads - 1) / kSelThreads);
  const dim3 grid(sel_blocks + (a.yhat != nullptr ? (a.n + 3) / 4 : 0));
  if (a.perm != nullptr)
    hipLaunchKernelGGL((loss_select_kernel<true>), grid, dim3(kSelThreads), 0, s, a, sel_blocks, lpi_log);
  else
    hipLaunchKernelGGL((loss_select_kernel<false>), grid, dim3(kSelThreads), 0, s, a, sel_blocks, lpi_log);
  return hipGetLastError();
}

hipError_t launch_group_perm(PermBatch &b, hipStream_t s) {
  if (b.nl < 1 || b.nl > 8) return hipErrorInvalidValue;
  int blocks = 0;
  for (int i = 0; i < b.nl; ++i) {
    if (b.L[i].k < 1 || b.L[i].perm == nullptr) return hipErrorInvalidValue;
    b.L[i].block0 = blocks;
    blocks += (b.L[i].k + kPermThreads - 1) / kPermThreads;
  }
  hipLaunchKernelGGL(group_perm_kernel, dim3(blocks), dim3(kPermThreads), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_eval_count(const int32_t *yhat, int c, const int32_t *y, int n, int32_t *correct,
                             uint8_t *flag, int thr, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(eval_count_kernel, dim3((n + 3) / 4), dim3(256), 0, s, yhat, c, y, n, correct, flag, thr);
  return hipGetLastError();
}

hipError_t launch_exit_count(const uint8_t *flags, int ldf, int L, int n, int32_t *counts, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (L < 1 || L > BMLP_MAX_LAYERS) return hipErrorInvalidValue;
  hipLaunchKernelGGL(exit_count_kernel, dim3((n + kExitThreads - 1) / kExitThreads), dim3(kExitThreads), 0, s, flags, ldf, L, n, counts);
  return hipGetLastError();
}

hipError_t launch_gather_batch(const GatherArgs &a, hipStream_t s) {
  const long long total = gather_items(a);
  if (total <= 0) return hipSuccess;
  if (a.n_all < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_batch_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace bmlp
