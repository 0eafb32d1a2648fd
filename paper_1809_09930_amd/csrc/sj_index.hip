// Grid index build on the device (Section 3.2.1 grid index, Section 4.1
// indexing k of the n dimensions, Section 4.2 variance reorder):
//   ingest/validate -> per-dimension min/max, sample variance -> cell keys
//   over the first k reordered dimensions -> radix sort by key -> gather the
//   points in cell order (reordered, zero-padded rows) -> compact the
//   non-empty cells -> adjacent cells by binary search in an LDS-staged key
//   table -> candidate runs -> work units for the distance kernels.
#include "sj_index.hpp"
#include "sj_launch.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <vector>

namespace sj {

namespace {

// ---------------------------------------------------------------------------
// a1: per-dimension min/max of the caller's rows and a non-finite flag.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_minmax(const float *__restrict__ P, uint64_t total,
                                                   uint32_t d, uint32_t *__restrict__ gmin,
                                                   uint32_t *__restrict__ gmax,
                                                   uint32_t *__restrict__ bad) {
  __shared__ uint32_t smin[SJ_MAX_DIM], smax[SJ_MAX_DIM];
  __shared__ uint32_t sbad;
  for (uint32_t t = threadIdx.x; t < d; t += kBlock) {
    smin[t] = 0xffffffffu;
    smax[t] = 0u;
  }
  if (threadIdx.x == 0) sbad = 0;
  __syncthreads();
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const uint32_t step = (uint32_t)(stride % d);
  uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  uint32_t t = (uint32_t)(e % d);
  uint32_t lmin = 0xffffffffu, lmax = 0u;
  uint32_t lt = t;  // dimension the local min/max belongs to (only when step == 0)
  for (; e < total; e += stride) {
    const float v = P[e];
    if (!__builtin_isfinite(v)) {
      sbad = 1;
    } else {
      const uint32_t u = float_to_ordered(v);
      if (step == 0) {
        lmin = min(lmin, u);
        lmax = max(lmax, u);
      } else {
        atomicMin(&smin[t], u);
        atomicMax(&smax[t], u);
      }
    }
    t += step;
    if (t >= d) t -= d;
  }
  if (step == 0 && lmax != 0u) {
    atomicMin(&smin[lt], lmin);
    atomicMax(&smax[lt], lmax);
  }
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < d; q += kBlock) {
    if (smax[q] != 0u) {
      atomicMin(&gmin[q], smin[q]);
      atomicMax(&gmax[q], smax[q]);
    }
  }
  if (threadIdx.x == 0 && sbad) atomicOr(bad, 1u);
}

__global__ void k_init_minmax(uint32_t *gmin, uint32_t *gmax, uint32_t *bad, uint32_t d) {
  for (uint32_t t = threadIdx.x; t < d; t += blockDim.x) {
    gmin[t] = 0xffffffffu;
    gmax[t] = 0u;
  }
  if (threadIdx.x == 0) *bad = 0u;
}

// ---------------------------------------------------------------------------
// a2: variance of every dimension over a strided sample (one workgroup per
// dimension, fixed-order reductions: deterministic).
// ---------------------------------------------------------------------------
__device__ double block_sum_f64(double v) {
  __shared__ double red[kBlock];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  double r = red[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(kBlock) void k_variance(const float *__restrict__ P, uint32_t d,
                                                     uint64_t stride, uint64_t m,
                                                     double *__restrict__ var) {
  const uint32_t t = blockIdx.x;
  double s = 0.0;
  for (uint64_t i = threadIdx.x; i < m; i += kBlock) s += (double)P[i * stride * d + t];
  const double mean = block_sum_f64(s) / (double)m;
  double q = 0.0;
  for (uint64_t i = threadIdx.x; i < m; i += kBlock) {
    const double x = (double)P[i * stride * d + t] - mean;
    q += x * x;
  }
  const double ss = block_sum_f64(q);
  if (threadIdx.x == 0) {
    var[t] = m > 1 ? ss / (double)(m - 1) : 0.0;
    var[d + t] = mean;
  }
}

// ---------------------------------------------------------------------------
// a3: linearised cell key over the first k reordered dimensions.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t sort_key(const float *__restrict__ x, const KeyParams &kp,
                                             uint32_t pid) {
  uint64_t key = 0;
  for (uint32_t r = 0; r < kp.k; ++r) {
    const double xv = (double)x[kp.dim[r]];
    double c = floor((xv - kp.org[r]) / kp.w);
    c = c < 0.0 ? 0.0 : c;
    uint64_t ci = (uint64_t)c;
    ci = ci > kp.cmax[r] ? kp.cmax[r] : ci;
    key += ci * kp.mult[r];
  }
  uint64_t fine = pid;
  if (kp.fm) {
    uint32_t f[kFineMaxDims];
    const uint32_t fmax = (1u << kp.fb) - 1u;
    for (uint32_t r = 0; r < kp.fm; ++r) {
      double v = ((double)x[kp.fdim[r]] - kp.forg[r]) * kp.fscale[r];
      v = v < 0.0 ? 0.0 : v;
      uint32_t q = (uint32_t)v;
      f[r] = q > fmax ? fmax : q;
    }
    for (int b = (int)kp.fb - 1; b >= 0; --b)
      for (uint32_t r = 0; r < kp.fm; ++r) fine = (fine << 1) | ((f[r] >> b) & 1u);
  }
  return (key << (kp.fm * kp.fb + kp.pb)) | fine;
}

__global__ __launch_bounds__(kBlock) void k_cellkey(const float *__restrict__ P, uint64_t n,
                                                    uint32_t d, KeyParams kp,
                                                    const uint8_t *__restrict__ pid,
                                                    uint64_t *__restrict__ keys,
                                                    uint32_t *__restrict__ ids) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  keys[i] = sort_key(P + i * d, kp, pid ? pid[i] : 0u);
  ids[i] = (uint32_t)i;
}

// Nearest of the kPivots pivot points, in FP32 (any choice is a valid order).
// Without it the in-cell order of clustered data above 24 dimensions mixes the
// clusters: the Morton code sees only the dimensions of largest variance,
// where the clusters overlap most.  The pivots' coordinates are wave-uniform
// scalar loads; a lane holds one point's 64 sums.
__global__ __launch_bounds__(kBlock) void k_pivot_table(const float *__restrict__ P,
                                                        uint64_t stride, uint32_t d,
                                                        float *__restrict__ table) {
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  if (e < kPivots * d) table[e] = P[(uint64_t)(e % kPivots) * stride * d + e / kPivots];
}

// Half of the pivots at equal distances in the sample, then the other half one by
// one, each the sample's farthest row from those before: rows at equal distances
// alone miss one of 20 clusters in half of all sets, and its points then share
// other clusters' query blocks (a quarter to a third of all blocks, which pass
// every candidate's group test).  One workgroup, a thread per sampled row; bound by
// reading the sample ([d][kPickSample]) 33 times from L2, 0.1 to 0.2 ms.
__global__ __launch_bounds__(kBlock) void k_pick_sample(const float *__restrict__ P,
                                                        uint64_t stride, uint32_t d,
                                                        float *__restrict__ sample) {
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= kPickSample * d) return;
  const uint32_t i = e / d, t = e - i * d;
  sample[t * kPickSample + i] = P[(uint64_t)i * stride * d + t];
}

__global__ __launch_bounds__(kPickSample) void k_pivot_pick(const float *__restrict__ sample,
                                                            uint32_t d,
                                                            float *__restrict__ table) {
  constexpr uint32_t kFirst = kPivots / 2, kW = kPickSample / kWave;
  __shared__ float row[SJ_MAX_DIM][kFirst];
  __shared__ uint64_t best[kW];
  const uint32_t i = threadIdx.x;
  for (uint32_t e = i; e < d * kFirst; e += kPickSample) {
    const uint32_t t = e / kFirst, j = e % kFirst;
    const float x = sample[t * kPickSample + j * (kPickSample / kFirst)];
    row[t][j] = x;
    table[t * kPivots + j] = x;
  }
  __syncthreads();
  float near[kFirst];
#pragma unroll
  for (uint32_t j = 0; j < kFirst; ++j) near[j] = 0.0f;
  for (uint32_t t = 0; t < d; ++t) {
    const float x = sample[t * kPickSample + i];
#pragma unroll
    for (uint32_t j = 0; j < kFirst; ++j) {
      const float e = x - row[t][j];
      near[j] = __builtin_fmaf(e, e, near[j]);
    }
  }
  float dist = near[0];
#pragma unroll
  for (uint32_t j = 1; j < kFirst; ++j) dist = __builtin_fminf(dist, near[j]);
  for (uint32_t j = kFirst; j < kPivots; ++j) {
    // (non-negative floats compare like their bits)
    uint64_t b = ((uint64_t)__builtin_bit_cast(uint32_t, dist) << 32) | i;
    for (int off = 32; off > 0; off >>= 1) {
      const uint64_t o = __shfl_xor(b, off);
      b = o > b ? o : b;
    }
    if (lane_id() == 0) best[i / kWave] = b;
    __syncthreads();
    b = best[0];
    for (uint32_t w = 1; w < kW; ++w) b = best[w] > b ? best[w] : b;
    const uint32_t pick = (uint32_t)b;
    if (i < d) {
      const float x = sample[i * kPickSample + pick];
      row[i][0] = x;
      table[i * kPivots + j] = x;
    }
    __syncthreads();
    float e2 = 0.0f;
#pragma unroll 8
    for (uint32_t t = 0; t < d; ++t) {
      const float e = sample[t * kPickSample + i] - row[t][0];
      e2 = __builtin_fmaf(e, e, e2);
    }
    dist = __builtin_fminf(dist, e2);
    // (row is written again after the next barrier)
  }
}

__global__ __launch_bounds__(kBlock) void k_nearest_pivot(const float *__restrict__ P, uint64_t n,
                                                          uint32_t d,
                                                          const float *__restrict__ table,
                                                          uint8_t *__restrict__ pid) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  float s[kPivots];
#pragma unroll
  for (uint32_t j = 0; j < kPivots; ++j) s[j] = 0.0f;
  for_row(P, n, d, [&](uint32_t t, float x) {
    const float *q = table + t * kPivots;
#pragma unroll
    for (uint32_t j = 0; j < kPivots; ++j) {
      const float e = x - q[j];
      s[j] = __builtin_fmaf(e, e, s[j]);
    }
  });
  if (i >= n) return;
  uint32_t best = 0;
  float b = s[0];
#pragma unroll
  for (uint32_t j = 1; j < kPivots; ++j)
    if (s[j] < b) {
      b = s[j];
      best = j;
    }
  pid[i] = (uint8_t)best;
}

// One workgroup per pivot: 256 sampled rows at a time, thread t sums dimension t
// of those that are the pivot's.
static_assert(SJ_MAX_DIM <= kBlock, "a thread per dimension");
__global__ __launch_bounds__(kBlock) void k_pivot_means(const float *__restrict__ P, uint64_t m,
                                                        uint64_t stride, uint32_t d,
                                                        const uint8_t *__restrict__ pid,
                                                        float *__restrict__ out) {
  __shared__ uint64_t mine[kWavesPerBlock];
  const uint32_t b = blockIdx.x, t = threadIdx.x;
  float sum = 0.0f;
  uint32_t cnt = 0;
  for (uint64_t base = 0; base < m; base += kBlock) {
    const uint64_t i = base + t;
    const uint64_t hit = ballot(i < m && pid[i * stride] == b);
    if (lane_id() == 0) mine[t / kWave] = hit;
    __syncthreads();
    for (uint32_t w = 0; w < (uint32_t)kWavesPerBlock; ++w)
      for (uint64_t x = mine[w]; x; x &= x - 1) {
        const uint64_t row = (base + w * kWave + (uint32_t)__builtin_ctzll(x)) * stride;
        if (t < d) sum += P[row * d + t];
        ++cnt;
      }
    __syncthreads();
  }
  if (t < d) out[(uint64_t)b * (d + 1) + t] = cnt ? sum / (float)cnt : 0.0f;
  if (t == 0) out[(uint64_t)b * (d + 1) + d] = (float)cnt;
}

__global__ __launch_bounds__(kBlock) void k_pivot_order(const uint8_t *__restrict__ pid, uint64_t n,
                                                        const uint32_t *__restrict__ orig_id,
                                                        uint8_t *__restrict__ out) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p < n) out[p] = pid[orig_id[p]];
}

// Keys of query points in the grid of an indexed set E (the general join
// Q join_eps E of Section 3.1).  A query with some coordinate more than
// two cell widths outside E's range [lo_t, hi_t] (lo = lo_t - 2w and
// hi = hi_t + 2w here, caller's dimension order) is farther than eps from
// every point of E: it gets far_key, which sorts after every cell key, and
// is counted in *n_far.  The others are clamped into E's grid like E's own
// points; a clamped query searches cells that include all of its true
// neighbour cells.
__global__ __launch_bounds__(kBlock) void k_query_keys(const float *__restrict__ Q, uint64_t m,
                                                       uint32_t d, KeyParams kp,
                                                       const uint8_t *__restrict__ pid,
                                                       const double *__restrict__ lo,
                                                       const double *__restrict__ hi,
                                                       uint64_t far_key,
                                                       uint64_t *__restrict__ keys,
                                                       uint32_t *__restrict__ ids,
                                                       unsigned long long *__restrict__ n_far) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  bool far = false;
  if (i < m) {
    const float *x = Q + i * d;
    for (uint32_t t = 0; t < d; ++t) {
      const double v = (double)x[t];
      far = far || v < lo[t] || v > hi[t];
    }
    keys[i] = far ? far_key : sort_key(x, kp, pid ? pid[i] : 0u);
    ids[i] = (uint32_t)i;
  }
  const uint64_t fm = ballot(far);
  if (lane_id() == 0 && fm) atomicAdd(n_far, (unsigned long long)__builtin_popcountll(fm));
}

// ---------------------------------------------------------------------------
// a4: gather rows in cell order: X[p][r] = P[id_p][perm[r]], zero padded.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_gather(const float *__restrict__ P, uint64_t n,
                                                   uint32_t d, uint32_t dp,
                                                   const uint32_t *__restrict__ perm,
                                                   const uint32_t *__restrict__ sorted_ids,
                                                   float *__restrict__ X,
                                                   uint32_t *__restrict__ orig_id,
                                                   uint32_t *__restrict__ pos_of) {
  // grid-stride: n * dp elements may exceed the 2^32 work-items of a dispatch
  const uint64_t total = n * dp;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t p = e / dp;
    const uint32_t r = (uint32_t)(e - p * dp);
    const uint32_t id = sorted_ids[p];
    X[e] = r < d ? P[(uint64_t)id * d + perm[r]] : 0.0f;
    if (r == 0) {
      orig_id[p] = id;
      pos_of[id] = (uint32_t)p;
    }
  }
}

// ---------------------------------------------------------------------------
// a5: compaction of the non-empty cells.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_cell_flags(const uint64_t *__restrict__ keys,
                                                       uint64_t n, uint32_t sh,
                                                       uint32_t *__restrict__ flag) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n) return;
  flag[p] = (p == 0 || (keys[p] >> sh) != (keys[p - 1] >> sh)) ? 1u : 0u;
}

__global__ __launch_bounds__(kBlock) void k_cell_write(const uint64_t *__restrict__ keys,
                                                       uint64_t n, uint32_t sh,
                                                       const uint32_t *__restrict__ cidx,
                                                       uint64_t *__restrict__ cell_key,
                                                       uint32_t *__restrict__ cell_start) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n) return;
  const bool first = (p == 0 || (keys[p] >> sh) != (keys[p - 1] >> sh));
  if (first) {
    cell_key[cidx[p]] = keys[p] >> sh;
    cell_start[cidx[p]] = (uint32_t)p;
  }
  // cell index of p is cidx[p] when p starts a cell, else cidx[p] - 1
  if (p == n - 1) cell_start[cidx[p] + (first ? 1u : 0u)] = (uint32_t)n;
}

// ---------------------------------------------------------------------------
// a6: adjacent non-empty cells (Section 3.2.1: only the 3^k cells around a
// query cell can hold its neighbours; Section 5.5: each is found by binary
// search over the non-empty cell ids).  One wave per query cell, 64 offsets
// per step; the cell-key table is staged in LDS, whole when it fits, else
// as a fence of every stride-th key that narrows the search to a short
// stretch of the table in global memory.  The searches wait on dependent
// loads, so a workgroup of 16 waves shares one fence: two of them fill a CU
// with 32 waves where workgroups of 4 waves would leave it at 8.
// ---------------------------------------------------------------------------
constexpr int kFenceMax = 8192;  // 64 KiB of u64 keys in LDS
constexpr int kNbrBlock = 1024;
constexpr int kNbrWaves = kNbrBlock / kWave;

// First table position whose key is >= key (ncell if none).  The fence
// holds cell_key[f * fstride]; when fstride is 1 it is the whole table.
__device__ __forceinline__ uint64_t lower_bound_cell(uint64_t key,
                                                    const uint64_t *__restrict__ fence,
                                                    uint32_t nfence, uint32_t fstride,
                                                    const uint64_t *__restrict__ cell_key,
                                                    uint64_t ncell) {
  uint32_t lo = 0, hi = nfence;  // first fence entry >= key
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (fence[mid] < key) lo = mid + 1; else hi = mid;
  }
  if (fstride == 1 || lo == 0) return (uint64_t)lo * fstride;
  // cell_key[(lo-1) fstride] < key <= cell_key[lo fstride] (or the end)
  uint64_t a = (uint64_t)(lo - 1) * fstride + 1, b = (uint64_t)lo * fstride;
  if (b > ncell) b = ncell;
  while (a < b) {
    const uint64_t mid = (a + b) >> 1;
    if (cell_key[mid] < key) a = mid + 1; else b = mid;
  }
  return a;
}

// Query cells are qkey[0 .. nq) (the table itself in a self-join); the
// table is cell_key[0 .. ncell) with its cell_start.  The 3^k offsets are
// taken in groups of three that differ only in the last indexed dimension,
// the least significant digit of the key (multiplier 1): their keys are
// consecutive, so one search finds the position of the smallest and the
// other two are the entries after it.  Each lane takes one group; groups
// and the cells inside a group come in ascending key order, so the
// neighbour list of a cell is written sorted.
__global__ __launch_bounds__(kNbrBlock) void k_neighbors(
    int pass, const uint64_t *__restrict__ qkey, uint64_t nq,
    const uint64_t *__restrict__ cell_key, const uint32_t *__restrict__ cell_start,
    uint64_t ncell, NbrParams np, uint32_t *__restrict__ nbr_count,
    uint64_t *__restrict__ cand_sum, const uint32_t *__restrict__ nbr_off,
    uint32_t *__restrict__ nbr_cell) {
  __shared__ uint64_t fence[kFenceMax];
  for (uint32_t i = threadIdx.x; i < np.nfence; i += kNbrBlock)
    fence[i] = cell_key[(uint64_t)i * np.fstride];
  __syncthreads();
  const uint32_t l = lane_id();
  const uint64_t wid = (uint64_t)blockIdx.x * kNbrWaves + threadIdx.x / kWave;
  const uint64_t nw = (uint64_t)gridDim.x * kNbrWaves;
  const uint32_t kl = np.k - 1;                   // the last indexed dimension
  const uint32_t ng = (uint32_t)(np.n_off / 3);  // 3^(k-1) <= 3^15 groups
  for (uint64_t A = wid; A < nq; A += nw) {
    const uint64_t keyA = qkey[A];
    int64_t cA[kKeyMaxDims];
    for (uint32_t r = 0; r < np.k; ++r) cA[r] = (int64_t)((keyA / np.mult[r]) % np.m[r]);
    const bool lo_ok = cA[kl] >= 1;                       // the cell below exists
    const bool hi_ok = cA[kl] + 1 < (int64_t)np.m[kl];  // the cell above exists
    uint32_t count = 0, wpos = (pass == 1) ? nbr_off[A] : 0u;
    uint64_t csum = 0;
    for (uint32_t base = 0; base < ng; base += kWave) {
      const uint32_t g = base + l;
      bool ok = g < ng;
      uint64_t keyB = keyA;  // the group's key with the last digit of A
      uint32_t rem = g;
      for (int r = (int)kl - 1; r >= 0; --r) {  // dimension 0 is the most significant digit
        const int64_t delta = (int64_t)(rem % 3u) - 1;
        rem /= 3u;
        const int64_t c = cA[r] + delta;
        ok = ok && c >= 0 && c < (int64_t)np.m[r];
        keyB += (uint64_t)delta * np.mult[r];
      }
      // keys keyB - 1, keyB, keyB + 1 (those inside the grid), ascending
      int64_t Bx[3] = {-1, -1, -1};
      if (ok) {
        const uint64_t first = lo_ok ? keyB - 1 : keyB;
        uint64_t q = lower_bound_cell(first, fence, np.nfence, np.fstride, cell_key, ncell);
        for (uint32_t t = 0; t < 3; ++t) {
          const uint64_t kk = keyB + t - 1;
          if ((t == 0 && !lo_ok) || (t == 2 && !hi_ok)) continue;
          // q is the first position with key >= kk
          if (q < ncell && (np.fstride == 1 ? fence[q] : cell_key[q]) == kk) Bx[t] = (int64_t)q++;
        }
      }
      const uint64_t m0 = ballot(Bx[0] >= 0), m1 = ballot(Bx[1] >= 0), m2 = ballot(Bx[2] >= 0);
      const uint32_t found = (uint32_t)(__builtin_popcountll(m0) + __builtin_popcountll(m1) +
                                        __builtin_popcountll(m2));
      if (pass == 0) {
        count += found;
        for (uint32_t t = 0; t < 3; ++t)
          if (Bx[t] >= 0) csum += (uint64_t)(cell_start[Bx[t] + 1] - cell_start[Bx[t]]);
      } else {
        uint32_t w = wpos + lanes_below(m0) + lanes_below(m1) + lanes_below(m2);
        for (uint32_t t = 0; t < 3; ++t)
          if (Bx[t] >= 0) nbr_cell[w++] = (uint32_t)Bx[t];
        wpos += found;
      }
    }
    if (pass == 0) {
      // wave-wide sum of the candidate counts
      for (int off = 32; off > 0; off >>= 1) csum += __shfl_xor(csum, off);
      if (l == 0) {
        nbr_count[A] = count;
        cand_sum[A] = csum;
      }
    }
  }
}

// Candidate runs: maximal stretches of consecutive cell indices in A's
// (sorted) neighbour list, as position ranges.  sym = 1 keeps only B >= A.
// G lanes per cell take G list entries per step: an entry starts a run when its
// predecessor in the list is not the cell before it, and ends one likewise, and
// the i-th start and the i-th end are of the same run.  (One lane per cell walked
// lists of up to thousands of entries by dependent loads: 10.1 ms of the 2M x 16
// exponential join, whose cells have hundreds of neighbours, for four launches;
// now 0.36 ms.)
template <int G>
__global__ __launch_bounds__(kBlock) void k_runs(int pass, int sym, uint64_t ncell,
                                                 const uint32_t *__restrict__ cell_start,
                                                 const uint32_t *__restrict__ nbr_off,
                                                 const uint32_t *__restrict__ nbr_cell,
                                                 uint32_t *__restrict__ run_count,
                                                 const uint32_t *__restrict__ run_off,
                                                 uint2 *__restrict__ runs) {
  const uint32_t l = threadIdx.x % G;
  const uint32_t shift = lane_id() - l;  // this group's lanes in a wave's ballot
  const uint64_t mask = (G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull) << shift;
  const uint64_t below = mask & ((1ull << lane_id()) - 1ull);
  // (A0: the wave's first list)
  for (uint64_t A0 = ((uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~63u)) / G; A0 < ncell;
       A0 += (uint64_t)gridDim.x * (kBlock / G)) {
    const uint64_t A = A0 + lane_id() / G;
    const bool live = A < ncell;
    const uint32_t b0 = live ? nbr_off[A] : 0u, b1 = live ? nbr_off[A + 1] : 0u;
    const uint32_t w = pass && live ? run_off[A] : 0u;
    uint32_t ns = 0, ne = 0;  // starts and ends so far
    const uint32_t steps = list_steps(b0, b1, G);
    for (uint32_t t = 0; ballot(t < steps) != 0; ++t) {
      uint32_t i;
      const bool in = list_entry(b0, b1, t, G, l, &i);
      const uint32_t B = in ? nbr_cell[i] : 0u;
      const bool ok = in && !(sym && B < A);
      const uint32_t prev = ok && i > b0 ? nbr_cell[i - 1] : 0xffffffffu;
      const uint32_t next = ok && b1 - i > 1 ? nbr_cell[i + 1] : 0xffffffffu;
      const bool start = ok && (prev == 0xffffffffu || prev + 1 != B || (sym && prev < A));
      const bool end = ok && (next == 0xffffffffu || next != B + 1);
      const uint64_t ms = ballot(start), me = ballot(end);
      if (pass) {
        if (start) runs[w + ns + (uint32_t)__builtin_popcountll(ms & below)].x = cell_start[B];
        if (end) runs[w + ne + (uint32_t)__builtin_popcountll(me & below)].y = cell_start[B + 1];
      }
      ns += (uint32_t)__builtin_popcountll(ms & mask);
      ne += (uint32_t)__builtin_popcountll(me & mask);
    }
    if (!pass && live && l == 0) run_count[A] = ns;
  }
}

// Union of the candidate runs of each group of consecutive cells
// [gfirst[g], gfirst[g + 1]) (at most kGroupMaxCells cells): the cells' run
// lists, each sorted and disjoint, merged in position order with
// overlapping or touching ranges joined, so that no candidate appears
// twice.  pass 0 counts the group's runs, pass 1 writes them at goff[g].
__global__ __launch_bounds__(kBlock) void k_group_runs(int pass, uint64_t ngroup,
                                                       const uint32_t *__restrict__ gfirst,
                                                       const uint32_t *__restrict__ run_off,
                                                       const uint2 *__restrict__ runs,
                                                       uint32_t *__restrict__ gcount,
                                                       const uint32_t *__restrict__ goff,
                                                       uint2 *__restrict__ gruns) {
  const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= ngroup) return;
  const uint32_t a0 = gfirst[g], na = gfirst[g + 1] - a0;
  uint32_t at[kGroupMaxCells], end[kGroupMaxCells];
  for (uint32_t i = 0; i < kGroupMaxCells; ++i) {
    at[i] = i < na ? run_off[a0 + i] : 0u;
    end[i] = i < na ? run_off[a0 + i + 1] : 0u;
  }
  uint32_t cnt = 0, w = pass ? goff[g] : 0u;
  bool have = false;
  uint2 cur = make_uint2(0u, 0u);
  for (;;) {
    int best = -1;
    uint32_t bx = 0xffffffffu;
    for (uint32_t i = 0; i < kGroupMaxCells; ++i)
      if (at[i] < end[i] && runs[at[i]].x < bx) {
        bx = runs[at[i]].x;
        best = (int)i;
      }
    if (best < 0) break;
    const uint2 r = runs[at[best]++];
    if (have && r.x <= cur.y) {
      cur.y = r.y > cur.y ? r.y : cur.y;
    } else {
      if (have) {
        if (pass) gruns[w + cnt] = cur;
        ++cnt;
      }
      cur = r;
      have = true;
    }
  }
  if (have) {
    if (pass) gruns[w + cnt] = cur;
    ++cnt;
  }
  if (!pass) gcount[g] = cnt;
}

// Work units (see WorkUnit).  Query slots of cell A are [qa, qb): positions
// in contiguous mode, indices into the sorted query list in list mode.
// In symmetric mode the first run of A starts at A itself and each query
// block only looks at candidates from its own first query onwards.
__device__ __forceinline__ void cell_query_slots(uint64_t A, const uint32_t *__restrict__ cell_start,
                                                 const uint32_t *__restrict__ qlist, uint64_t nq,
                                                 uint32_t *qa, uint32_t *qb) {
  const uint32_t s = cell_start[A], e = cell_start[A + 1];
  if (!qlist) {
    *qa = s;
    *qb = e;
    return;
  }
  uint64_t lo = 0, hi = nq;
  while (lo < hi) { uint64_t m = (lo + hi) >> 1; if (qlist[m] < s) lo = m + 1; else hi = m; }
  *qa = (uint32_t)lo;
  hi = nq;
  while (lo < hi) { uint64_t m = (lo + hi) >> 1; if (qlist[m] < e) lo = m + 1; else hi = m; }
  *qb = (uint32_t)lo;
}

// Per cell (or, without nqb, per query block with runs of its own): its number
// of query blocks, the total length of its runs and, per run, the length of the
// cell's runs before it (below 2^32: the runs are disjoint).  G lanes per list
// (the 2M x 16 exponential join: 1.10 ms with one lane per cell, 0.18 ms now, for
// three launches).
template <int G>
__global__ __launch_bounds__(kBlock) void k_wu_cells(
    uint64_t nlist, uint32_t tq, const uint32_t *__restrict__ cell_start,
    const uint32_t *__restrict__ qlist, uint64_t nq, const uint32_t *__restrict__ run_off,
    const uint2 *__restrict__ runs, uint32_t *__restrict__ nqb, uint64_t *__restrict__ run_total,
    uint32_t *__restrict__ before) {
  const uint32_t l = threadIdx.x % G;
  for (uint64_t A0 = ((uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~63u)) / G; A0 < nlist;
       A0 += (uint64_t)gridDim.x * (kBlock / G)) {
    const uint64_t A = A0 + lane_id() / G;
    const bool live = A < nlist;
    const uint32_t r0 = live ? run_off[A] : 0u, r1 = live ? run_off[A + 1] : 0u;
    uint32_t total = 0;
    const uint32_t steps = list_steps(r0, r1, G);
    for (uint32_t t = 0; ballot(t < steps) != 0; ++t) {
      uint32_t r;
      const bool in = list_entry(r0, r1, t, G, l, &r);
      const uint2 x = in ? runs[r] : make_uint2(0u, 0u);
      const uint32_t len = x.y - x.x;
      uint32_t inc = len;
#pragma unroll
      for (int off = 1; off < G; off <<= 1) {
        const uint32_t u = __shfl_up(inc, off, G);
        if (l >= (uint32_t)off) inc += u;
      }
      if (in) before[r] = total + inc - len;
      total += __shfl(inc, G - 1, G);
    }
    if (!live || l != 0) continue;
    if (nqb) {
      uint32_t qa, qb;
      cell_query_slots(A, cell_start, qlist, nq, &qa, &qb);
      nqb[A] = (qb - qa + tq - 1) / tq;
    }
    run_total[A] = total;
  }
}

// Query block t: its cell (binary search over the scanned block counts),
// slot range and candidate count.
__device__ __forceinline__ QBlock query_block(uint64_t t, int sym, uint64_t ncell, uint32_t tq,
                                              const uint32_t *__restrict__ cell_start,
                                              const uint32_t *__restrict__ qlist, uint64_t nq,
                                              const uint32_t *__restrict__ qb_off,
                                              const uint32_t *__restrict__ run_off,
                                              const uint2 *__restrict__ runs,
                                              const uint64_t *__restrict__ run_total,
                                              int per_block) {
  uint64_t lo = 0, hi = ncell;  // last cell with qb_off[A] <= t
  while (hi - lo > 1) {
    const uint64_t m = (lo + hi) >> 1;
    if (qb_off[m] <= t) lo = m; else hi = m;
  }
  // cells without query blocks share their offset with the next cell, so
  // the last cell whose offset is <= t is the one that owns block t
  QBlock b;
  b.A = (uint32_t)lo;
  uint32_t qa, qe;
  cell_query_slots(lo, cell_start, qlist, nq, &qa, &qe);
  b.q0 = qa + (uint32_t)(t - qb_off[lo]) * tq;
  b.q1 = min(b.q0 + tq, qe);
  if (per_block) {  // the block's own runs (SORTIDU ranges), already cut at q0
    b.r0 = run_off[t];
    b.r1 = run_off[t + 1];
    b.skip = 0u;
    b.L = run_total[t];
    return b;
  }
  b.r0 = run_off[lo];
  b.r1 = run_off[lo + 1];
  // a symmetric block starts at its first query's position (in list mode
  // the list holds whole cells, so that position is qlist[q0])
  b.skip = sym ? ((qlist ? qlist[b.q0] : b.q0) - runs[b.r0].x) : 0u;
  b.L = run_total[lo] - b.skip;
  return b;
}

// Stretches of a block's candidates: cut at multiples of tc of the position that a
// candidate has if the runs follow each other without gaps.  Blocks then share
// their cuts, and units in stretch order read the same candidates at a time.  (Cut
// from each block's own first candidate, the units in flight read a window of
// 500k candidates, far more than an L2 holds: the 2M x 16 FP32 join fetched 0.50
// TB at 4.8 TB/s.  Whole passes: 2M x 16 FP32 114 to 108 ms, FP16 69 to 63, 2M x 64
// BF16 229 to 215.)
// Blocks of less than kSharedCuts stretches keep cuts from their first candidate
// (shared ones give them up to a unit more each, of less work: 5M x 18 42.5 ms
// against 40.0).
constexpr uint32_t kSharedCuts = 8;
__device__ __forceinline__ uint64_t block_origin(const QBlock &b, const uint2 *__restrict__ runs,
                                                 uint32_t tc) {
  return b.L >= (uint64_t)kSharedCuts * tc ? (uint64_t)runs[b.r0].x + b.skip : 0ull;
}
__device__ __forceinline__ void block_stretches(const QBlock &b, uint64_t v0, uint32_t tc,
                                                uint32_t *first, uint32_t *count) {
  *first = *count = 0u;
  if (!b.L) return;
  *first = (uint32_t)(v0 / tc);
  *count = (uint32_t)((v0 + b.L - 1) / tc) - *first + 1u;
}

__global__ __launch_bounds__(kBlock) void k_wu_count(
    uint64_t nqb_total, int sym, uint64_t ncell, uint32_t tq, uint32_t tc,
    const uint32_t *__restrict__ cell_start, const uint32_t *__restrict__ qlist, uint64_t nq,
    const uint32_t *__restrict__ qb_off, const uint32_t *__restrict__ run_off,
    const uint2 *__restrict__ runs, const uint64_t *__restrict__ run_total,
    uint32_t *__restrict__ units, uint64_t *__restrict__ eval, QBlock *__restrict__ blocks,
    int per_block) {
  const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= nqb_total) return;
  const QBlock b = query_block(t, sym, ncell, tq, cell_start, qlist, nq, qb_off, run_off, runs,
                               run_total, per_block);
  blocks[t] = b;
  uint32_t first, count;
  block_stretches(b, block_origin(b, runs, tc), tc, &first, &count);
  units[t] = count;
  eval[t] = (uint64_t)(b.q1 - b.q0) * b.L;
}

// One lane per work unit: its block (the last one with unit_off <= w: blocks
// without units share their offset with the next), and by binary search over the
// block's runs where its stretch of tc candidates begins and ends.  (One lane
// per block walked the runs for all of its units in turn: 3.5 ms of the 2M x 16
// exponential join for three launches; now 0.2 ms.)
__global__ __launch_bounds__(kBlock) void k_wu_fill(
    uint64_t n_wu, uint64_t nqb_total, uint32_t tc, const QBlock *__restrict__ blocks,
    const uint2 *__restrict__ runs, const uint32_t *__restrict__ before,
    const uint32_t *__restrict__ unit_off, WorkUnit *__restrict__ wu,
    uint64_t *__restrict__ order_key) {
  const uint64_t w = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (w >= n_wu) return;
  uint64_t lo = 0, hi = nqb_total;
  while (hi - lo > 1) {
    const uint64_t m = (lo + hi) >> 1;
    if (unit_off[m] <= w) lo = m; else hi = m;
  }
  const QBlock b = blocks[lo];
  uint32_t first, count;
  const uint64_t v0 = block_origin(b, runs, tc), v1 = v0 + b.L;
  block_stretches(b, v0, tc, &first, &count);
  const uint32_t u = first + (uint32_t)(w - unit_off[lo]);  // the stretch
  // candidates [o0, o1) of the runs, counted from the first run's start
  const uint64_t cut0 = (uint64_t)u * tc, cut1 = cut0 + tc;
  const uint32_t o0 = b.skip + (uint32_t)((cut0 > v0 ? cut0 : v0) - v0);
  const uint32_t o1 = b.skip + (uint32_t)((cut1 < v1 ? cut1 : v1) - v0);
  auto run_of = [&](uint32_t o, uint32_t first) {  // the run holding candidate o
    uint32_t x = first, y = b.r1;
    while (y - x > 1) {
      const uint32_t m = x + (y - x) / 2;
      if (before[m] <= o) x = m; else y = m;
    }
    return x;
  };
  WorkUnit x;
  x.q0 = b.q0;
  x.q1 = b.q1;
  x.cell = b.A;
  x.pad = 0;
  x.run_first = run_of(o0, b.r0);
  x.c_begin = runs[x.run_first].x + (o0 - before[x.run_first]);
  x.run_last = run_of(o1 - 1, x.run_first);
  x.c_end = runs[x.run_last].x + (o1 - before[x.run_last]);
  // optional order key: stretch, then unit index
  if (order_key) order_key[w] = ((uint64_t)u << 32) | w;
  wu[w] = x;
}

// SORTIDU for blocks of queries (see launch_qb_ranges).  The window around
// the block's u-range [umin, umax] is widened by eps (1 + 2^-16) plus a
// relative 2^-40: a candidate outside it is farther than eps (1 + 2^-16)
// from every query of the block along u alone, so its canonical FP64 sum
// exceeds eps^2 and no pair is lost.  The window is quantised like the sort
// key, so the search runs over the sorted keys of each adjacent cell.
__device__ __forceinline__ uint32_t quantise_u(double v, const USearch &us) {
  double q = (v - us.org) * us.scale;
  q = q < 0.0 ? 0.0 : q;
  q = q > (double)us.fmax ? (double)us.fmax : q;
  return (uint32_t)q;
}

__global__ __launch_bounds__(kBlock) void k_qb_ranges(
    int pass, int sym, uint64_t nqb_total, uint64_t ncell, uint32_t tq,
    const uint32_t *__restrict__ cell_start, const uint32_t *__restrict__ qb_off,
    const uint32_t *__restrict__ nbr_off, const uint32_t *__restrict__ nbr_cell,
    const uint32_t *__restrict__ ecell_start, const uint64_t *__restrict__ ekey,
    const float *__restrict__ Xq, USearch us, uint32_t *__restrict__ rcount,
    uint64_t *__restrict__ rlen, const uint32_t *__restrict__ roff, uint2 *__restrict__ ranges) {
  const uint32_t l = lane_id();
  const uint64_t nw = (uint64_t)gridDim.x * kWavesPerBlock;
  for (uint64_t t = (uint64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; t < nqb_total;
       t += nw) {
    // the block: its cell A (last cell with qb_off[A] <= t) and slots
    uint64_t lo = 0, hi = ncell;
    while (hi - lo > 1) {
      const uint64_t m = (lo + hi) >> 1;
      if (qb_off[m] <= t) lo = m; else hi = m;
    }
    const uint32_t A = (uint32_t)lo;
    const uint32_t q0 = cell_start[A] + (uint32_t)(t - qb_off[A]) * tq;
    const uint32_t q1 = min(q0 + tq, cell_start[A + 1]);
    // the queries' u-range
    float umin = __builtin_inff(), umax = -__builtin_inff();
    for (uint32_t q = q0 + l; q < q1; q += kWave) {
      const float u = Xq[(uint64_t)q * us.dp + us.ur];
      umin = fminf(umin, u);
      umax = fmaxf(umax, u);
    }
    for (int off = 32; off > 0; off >>= 1) {
      umin = fminf(umin, __shfl_xor(umin, off));
      umax = fmaxf(umax, __shfl_xor(umax, off));
    }
    const double dl = (double)umin, dh = (double)umax;
    const double wl = us.eps * (1.0 + 0x1p-16) + (__builtin_fabs(dl) + us.eps) * 0x1p-40;
    const double wh = us.eps * (1.0 + 0x1p-16) + (__builtin_fabs(dh) + us.eps) * 0x1p-40;
    const uint64_t flo = quantise_u(dl - wl, us), fhi = quantise_u(dh + wh, us);
    // adjacent cells, 64 at a time: each lane searches one cell, then the
    // wave merges the lanes' ranges in cell order
    const uint32_t b0 = nbr_off[A], b1 = nbr_off[A + 1];
    uint32_t cnt = 0, oc0 = 0, oc1 = 0;
    uint64_t len = 0;
    bool open = false;
    const uint32_t wbase = pass ? roff[t] : 0u;
    for (uint32_t base = b0; base < b1; base += kWave) {
      const uint32_t i = base + l;
      uint32_t c0 = 0, c1 = 0;
      if (i < b1) {
        const uint32_t B = nbr_cell[i];
        if (!(sym && B < A)) {
          const uint32_t cs = ecell_start[B], ce = ecell_start[B + 1];
          uint32_t a = cs, b = ce;  // first position with u-part >= flo
          while (a < b) {
            const uint32_t m = (a + b) >> 1;
            if ((ekey[m] & us.fmask) < flo) a = m + 1; else b = m;
          }
          c0 = a;
          b = ce;  // first position with u-part > fhi
          while (a < b) {
            const uint32_t m = (a + b) >> 1;
            if ((ekey[m] & us.fmask) <= fhi) a = m + 1; else b = m;
          }
          c1 = a;
          if (sym && B == A && c0 < q0) c0 = q0;
        }
      }
      const uint32_t nl = min((uint32_t)kWave, b1 - base);
      for (uint32_t j = 0; j < nl; ++j) {
        const uint32_t x0 = (uint32_t)__builtin_amdgcn_readlane((int)c0, (int)j);
        const uint32_t x1 = (uint32_t)__builtin_amdgcn_readlane((int)c1, (int)j);
        if (x1 <= x0) continue;
        if (open && x0 == oc1) {
          oc1 = x1;
          continue;
        }
        if (open) {
          if (pass && l == 0) ranges[wbase + cnt] = make_uint2(oc0, oc1);
          len += oc1 - oc0;
          ++cnt;
        }
        open = true;
        oc0 = x0;
        oc1 = x1;
      }
    }
    if (open) {
      if (pass && l == 0) ranges[wbase + cnt] = make_uint2(oc0, oc1);
      len += oc1 - oc0;
      ++cnt;
    }
    if (!pass && l == 0) {
      rcount[t] = cnt;
      rlen[t] = len;
    }
  }
}

// dst[i] = src[low 32 bits of keys[i]]
__global__ __launch_bounds__(kBlock) void k_gather_wu(const WorkUnit *__restrict__ src,
                                                      const uint64_t *__restrict__ keys,
                                                      uint64_t n, WorkUnit *__restrict__ dst) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  dst[i] = src[(uint32_t)keys[i]];
}

// out[A] = (query slots of cell A's units of tq queries) * cand_sum[A]: the
// lane work of A's units, idle slots included
__global__ void k_cell_slot_work(uint64_t ncell, const uint32_t *__restrict__ cell_start,
                                 const uint64_t *__restrict__ cand_sum, uint32_t tq,
                                 uint64_t *__restrict__ out) {
  const uint64_t A = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (A >= ncell) return;
  const uint64_t m = cell_start[A + 1] - cell_start[A];
  out[A] = (m + tq - 1) / tq * tq * cand_sum[A];
}

__global__ void k_cell_products(uint64_t ncell, const uint32_t *__restrict__ cell_start,
                                const uint64_t *__restrict__ cand_sum, uint64_t *__restrict__ out) {
  const uint64_t A = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (A >= ncell) return;
  out[A] = (uint64_t)(cell_start[A + 1] - cell_start[A]) * cand_sum[A];
}

inline uint32_t blocks_for(uint64_t n) { return (uint32_t)((n + kBlock - 1) / kBlock); }
// Pairs per row of sorted keys (row = key >> 32): counts[i] += the number
// of keys of row i.  Each wave adds one count per row it holds: the lane
// that starts a run of equal rows inside the wave adds the run's length.
// Grid-stride over 64-key segments, one per wave and step (count may exceed
// the 2^32 work-items of one dispatch).
__global__ __launch_bounds__(kBlock) void k_row_counts(const uint64_t *__restrict__ keys,
                                                       uint64_t count,
                                                       unsigned long long *__restrict__ counts) {
  const uint32_t l = lane_id();
  const uint64_t step = (uint64_t)gridDim.x * kBlock;
  for (uint64_t e0 = (uint64_t)blockIdx.x * kBlock + (threadIdx.x & ~(uint32_t)(kWave - 1));
       e0 < count; e0 += step) {
    const uint64_t e = e0 + l;
    const bool live = e < count;
    const uint64_t row = live ? keys[e] >> 32 : 0;
    const bool head = live && (l == 0 || (keys[e - 1] >> 32) != row);
    const uint64_t heads = ballot(head);
    const uint64_t lives = ballot(live);
    if (head) {
      // the run ends at the next head above this lane, or at the last live lane
      const uint64_t above = heads & ~((2ull << l) - 1ull);
      const uint32_t end = above ? (uint32_t)__builtin_ctzll(above)
                                 : (uint32_t)(64 - __builtin_clzll(lives));
      atomicAdd(&counts[row], (unsigned long long)(end - l));
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
void launch_minmax(const float *P, uint64_t n, uint32_t d, uint32_t *gmin, uint32_t *gmax,
                   uint32_t *bad, hipStream_t s) {
  hipLaunchKernelGGL(k_init_minmax, dim3(1), dim3(kBlock), 0, s, gmin, gmax, bad, d);
  SJ_HIP(hipGetLastError());
  const uint64_t total = n * d;
  if (total == 0) return;
  uint32_t grid = (uint32_t)std::min<uint64_t>((total + kBlock - 1) / kBlock, 1024);
  // a stride of whole rows keeps a thread in one dimension (step == 0), its
  // extremes in registers instead of two LDS atomics per coordinate
  const uint32_t rows = d / std::gcd(d, (uint32_t)kBlock);
  if (grid > rows) grid -= grid % rows;
  hipLaunchKernelGGL(k_minmax, dim3(grid), dim3(kBlock), 0, s, P, total, d, gmin, gmax, bad);
  SJ_HIP(hipGetLastError());
}

void launch_variance(const float *P, uint32_t d, uint64_t stride, uint64_t m, double *var,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_variance, dim3(d), dim3(kBlock), 0, s, P, d, stride, m, var);
  SJ_HIP(hipGetLastError());
}

void launch_cellkey(const float *P, uint64_t n, uint32_t d, const KeyParams &kp,
                    const uint8_t *pid, uint64_t *keys, uint32_t *ids, hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_cellkey, dim3(blocks_for(n)), dim3(kBlock), 0, s, P, n, d, kp, pid, keys,
                     ids);
  SJ_HIP(hipGetLastError());
}

void launch_pivot_table(const float *P, uint64_t stride, uint32_t d, float *table, hipStream_t s) {
  hipLaunchKernelGGL(k_pivot_table, dim3(blocks_for(kPivots * d)), dim3(kBlock), 0, s, P, stride, d,
                     table);
  SJ_HIP(hipGetLastError());
}

void launch_pivot_pick(const float *P, uint64_t n, uint32_t d, float *sample, float *table,
                       hipStream_t s) {
  if (n < kPickSample || d > SJ_MAX_DIM) fail(SJ_ERR_INVALID_ARG, "too few rows to pick pivots");
  hipLaunchKernelGGL(k_pick_sample, dim3(blocks_for(kPickSample * d)), dim3(kBlock), 0, s, P,
                     n / kPickSample, d, sample);
  SJ_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_pivot_pick, dim3(1), dim3(kPickSample), 0, s, sample, d, table);
  SJ_HIP(hipGetLastError());
}

void launch_nearest_pivot(const float *P, uint64_t n, uint32_t d, const float *table, uint8_t *pid,
                          hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_nearest_pivot, dim3(blocks_for(n)), dim3(kBlock), 0, s, P, n, d, table, pid);
  SJ_HIP(hipGetLastError());
}

void launch_pivot_means(const float *P, uint64_t n, uint32_t d, const uint8_t *pid, float *out,
                        hipStream_t s) {
  if (!n) return;
  const uint64_t stride = std::max<uint64_t>(1, n / kPivotSample), m = n / stride;
  hipLaunchKernelGGL(k_pivot_means, dim3(kPivots), dim3(kBlock), 0, s, P, m, stride, d, pid, out);
  SJ_HIP(hipGetLastError());
}

void launch_pivot_order(const uint8_t *pid, uint64_t n, const uint32_t *orig_id, uint8_t *out,
                        hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_pivot_order, dim3(blocks_for(n)), dim3(kBlock), 0, s, pid, n, orig_id, out);
  SJ_HIP(hipGetLastError());
}

void launch_query_keys(const float *Q, uint64_t m, uint32_t d, const KeyParams &kp,
                       const uint8_t *pid, const double *lo, const double *hi, uint64_t far_key,
                       uint64_t *keys, uint32_t *ids, unsigned long long *n_far, hipStream_t s) {
  if (!m) return;
  hipLaunchKernelGGL(k_query_keys, dim3(blocks_for(m)), dim3(kBlock), 0, s, Q, m, d, kp, pid, lo,
                     hi, far_key, keys, ids, n_far);
  SJ_HIP(hipGetLastError());
}

void launch_gather(const float *P, uint64_t n, uint32_t d, uint32_t dp, const uint32_t *perm,
                   const uint32_t *sorted_ids, float *X, uint32_t *orig_id, uint32_t *pos_of,
                   hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_gather, dim3(stride_blocks(n * dp)), dim3(kBlock), 0, s, P, n, d, dp, perm,
                     sorted_ids, X, orig_id, pos_of);
  SJ_HIP(hipGetLastError());
}

void launch_compact(const uint64_t *keys, uint64_t n, uint32_t fine_shift, uint32_t *flag_tmp,
                    uint32_t *d_ncell, uint64_t *cell_key, uint32_t *cell_start, void *scan_tmp,
                    hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_cell_flags, dim3(blocks_for(n)), dim3(kBlock), 0, s, keys, n, fine_shift,
                     flag_tmp);
  SJ_HIP(hipGetLastError());
  exclusive_scan_u32(flag_tmp, flag_tmp, n, d_ncell, scan_tmp, s);
  hipLaunchKernelGGL(k_cell_write, dim3(blocks_for(n)), dim3(kBlock), 0, s, keys, n, fine_shift,
                     flag_tmp, cell_key, cell_start);
  SJ_HIP(hipGetLastError());
}

void launch_neighbors(int pass, const uint64_t *qkey, uint64_t nq, const uint64_t *cell_key,
                      const uint32_t *cell_start, uint64_t ncell, const NbrParams &np,
                      uint32_t *nbr_count, uint64_t *cand_sum, const uint32_t *nbr_off,
                      uint32_t *nbr_cell, hipStream_t s) {
  if (!nq || !ncell) return;
  const uint64_t waves = nq;
  uint32_t grid = (uint32_t)std::min<uint64_t>((waves + kNbrWaves - 1) / kNbrWaves, 1024);
  hipLaunchKernelGGL(k_neighbors, dim3(grid), dim3(kNbrBlock), 0, s, pass, qkey, nq, cell_key,
                     cell_start, ncell, np, nbr_count, cand_sum, nbr_off, nbr_cell);
  SJ_HIP(hipGetLastError());
}

// Lanes per list of the kernels above: a wave for long lists, 8 lanes for lists
// of a few entries, where a wave per list would leave most lanes idle (both forms
// take one step per list up to 8 entries; from 16 on the wave takes half as many
// or fewer).  Strided launches: 64 lanes for each of 2^26 lists pass what a dispatch
// holds.
constexpr uint64_t kLongLists = 16;  // entries per list, on average

void launch_runs(int pass, int sym, uint64_t ncell, uint64_t n_nbr, const uint32_t *cell_start,
                 const uint32_t *nbr_off, const uint32_t *nbr_cell, uint32_t *run_count,
                 const uint32_t *run_off, uint2 *runs, hipStream_t s) {
  if (!ncell) return;
  if (n_nbr >= kLongLists * ncell)
    hipLaunchKernelGGL(k_runs<64>, dim3(stride_blocks(ncell * 64)), dim3(kBlock), 0, s, pass, sym,
                       ncell, cell_start, nbr_off, nbr_cell, run_count, run_off, runs);
  else
    hipLaunchKernelGGL(k_runs<8>, dim3(stride_blocks(ncell * 8)), dim3(kBlock), 0, s, pass, sym,
                       ncell, cell_start, nbr_off, nbr_cell, run_count, run_off, runs);
  SJ_HIP(hipGetLastError());
}

void launch_group_runs(int pass, uint64_t ngroup, const uint32_t *gfirst, const uint32_t *run_off,
                       const uint2 *runs, uint32_t *gcount, const uint32_t *goff, uint2 *gruns,
                       hipStream_t s) {
  if (!ngroup) return;
  hipLaunchKernelGGL(k_group_runs, dim3(blocks_for(ngroup)), dim3(kBlock), 0, s, pass, ngroup,
                     gfirst, run_off, runs, gcount, goff, gruns);
  SJ_HIP(hipGetLastError());
}

void launch_wu_cells(uint64_t nlist, uint64_t n_runs, uint32_t tq, const uint32_t *cell_start,
                     const uint32_t *qlist, uint64_t nq, const uint32_t *run_off,
                     const uint2 *runs, uint32_t *nqb, uint64_t *run_total, uint32_t *before,
                     hipStream_t s) {
  if (!nlist) return;
  if (n_runs >= kLongLists * nlist)
    hipLaunchKernelGGL(k_wu_cells<64>, dim3(stride_blocks(nlist * 64)), dim3(kBlock), 0, s, nlist, tq,
                       cell_start, qlist, nq, run_off, runs, nqb, run_total, before);
  else
    hipLaunchKernelGGL(k_wu_cells<8>, dim3(stride_blocks(nlist * 8)), dim3(kBlock), 0, s, nlist, tq,
                       cell_start, qlist, nq, run_off, runs, nqb, run_total, before);
  SJ_HIP(hipGetLastError());
}

void launch_wu_count(uint64_t nqb_total, int sym, uint64_t ncell, uint32_t tq, uint32_t tc,
                     const uint32_t *cell_start, const uint32_t *qlist, uint64_t nq,
                     const uint32_t *qb_off, const uint32_t *run_off, const uint2 *runs,
                     const uint64_t *run_total, uint32_t *units, uint64_t *eval, QBlock *blocks,
                     hipStream_t s, int per_block) {
  if (!nqb_total) return;
  hipLaunchKernelGGL(k_wu_count, dim3(blocks_for(nqb_total)), dim3(kBlock), 0, s, nqb_total, sym,
                     ncell, tq, tc, cell_start, qlist, nq, qb_off, run_off, runs, run_total, units,
                     eval, blocks, per_block);
  SJ_HIP(hipGetLastError());
}

void launch_wu_fill(uint64_t n_wu, uint64_t nqb_total, uint32_t tc, const QBlock *blocks,
                    const uint2 *runs, const uint32_t *before, const uint32_t *unit_off,
                    WorkUnit *wu, uint64_t *order_key, hipStream_t s) {
  if (!n_wu) return;
  hipLaunchKernelGGL(k_wu_fill, dim3(blocks_for(n_wu)), dim3(kBlock), 0, s, n_wu, nqb_total, tc,
                     blocks, runs, before, unit_off, wu, order_key);
  SJ_HIP(hipGetLastError());
}

void launch_qb_ranges(int pass, int sym, uint64_t nqb_total, uint64_t ncell, uint32_t tq,
                      const uint32_t *cell_start, const uint32_t *qb_off,
                      const uint32_t *nbr_off, const uint32_t *nbr_cell,
                      const uint32_t *ecell_start, const uint64_t *ekey, const float *Xq,
                      const USearch &us, uint32_t *rcount, uint64_t *rlen,
                      const uint32_t *roff, uint2 *ranges, hipStream_t s) {
  if (!nqb_total) return;
  const uint32_t grid = (uint32_t)std::min<uint64_t>((nqb_total + kWavesPerBlock - 1) /
                                                     kWavesPerBlock, 1u << 16);
  hipLaunchKernelGGL(k_qb_ranges, dim3(grid), dim3(kBlock), 0, s, pass, sym, nqb_total, ncell,
                     tq, cell_start, qb_off, nbr_off, nbr_cell, ecell_start, ekey, Xq, us,
                     rcount, rlen, roff, ranges);
  SJ_HIP(hipGetLastError());
}

void launch_gather_wu(const WorkUnit *src, const uint64_t *keys, uint64_t n, WorkUnit *dst,
                      hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_gather_wu, dim3(blocks_for(n)), dim3(kBlock), 0, s, src, keys, n, dst);
  SJ_HIP(hipGetLastError());
}

void launch_cell_products(uint64_t ncell, const uint32_t *cell_start, const uint64_t *cand_sum,
                          uint64_t *out, hipStream_t s) {
  if (!ncell) return;
  hipLaunchKernelGGL(k_cell_products, dim3(blocks_for(ncell)), dim3(kBlock), 0, s, ncell,
                     cell_start, cand_sum, out);
  SJ_HIP(hipGetLastError());
}

void launch_cell_slot_work(uint64_t ncell, const uint32_t *cell_start, const uint64_t *cand_sum,
                           uint32_t tq, uint64_t *out, hipStream_t s) {
  if (!ncell) return;
  hipLaunchKernelGGL(k_cell_slot_work, dim3(blocks_for(ncell)), dim3(kBlock), 0, s, ncell,
                     cell_start, cand_sum, tq, out);
  SJ_HIP(hipGetLastError());
}

void launch_row_counts(const uint64_t *keys, uint64_t count, unsigned long long *counts,
                       hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_row_counts, dim3(stride_blocks(count)), dim3(kBlock), 0, s, keys, count,
                     counts);
  SJ_HIP(hipGetLastError());
}

}  // namespace sj
