// Matrix-core distance filter of the self-join on gfx950: 16-bit operands,
// FP32 accumulation, rigorous error band, FP64 recheck of the band.
//
// Form.  With a fixed centre c, every point is stored as x~ = Q(x - c) in
// FP16 or BF16 (Q = round to nearest; magnitudes below the format's
// smallest normal are flushed to 0).  For a query row b and a candidate
// column a one 32x32 MFMA tile computes
//     D = -Thi(b) - 2 b~ . a~
// with the query's threshold as the row's initial accumulator, and the pair
// is rejected when D > -fl32(n_a), n_a = |a~|^2 in FP64.  The operands are laid
// out K-contiguous and zero-padded to K: query rows [-2 b~ | 0], candidate
// columns [a~ | 0]; scaling by -2 is exact.
//
// Band.  Per query b the FP64 preparation below gives thresholds
// Thi(b) >= n_a - 2 b~ . a~, up to every rounding of the tile, for every
// candidate the canonical predicate accepts, and Tlo(b) such that a value at or
// below it proves acceptance (derivation in k_mfma_thresholds).  Above Thi
// rejects, at or below Tlo accepts, the rest is rechecked with the canonical
// FP64 predicate, so the pair set is exact.
//
// Tiles.  32 queries by 32 consecutive (or gathered) candidates; a wave holds
// QB query blocks (A operands and thresholds in registers) and streams
// candidate blocks (B operands).  Each lane's 16 accumulators share one
// candidate column, so "any pair of this lane below its threshold" is one min
// over 16 values (v_min3) and one compare; only tiles with a hit enter the
// per-element path (tile_masks, emit_hits in sj_tile.hpp).
#include "sj_internal.hpp"
#include "sj_launch.hpp"
#include "sj_mfma.hpp"
#include "sj_mx32.hpp"
#include "sj_tile.hpp"

#include <algorithm>
#include <cfloat>

namespace sj {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int FMT>
struct Fmt;
template <>
struct Fmt<kFmtF16> {
  typedef _Float16 T;
  typedef half8 V8;
  __device__ static float16v mfma(V8 a, V8 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Fmt<kFmtBF16> {
  typedef __bf16 T;
  typedef bf16x8 V8;
  __device__ static float16v mfma(V8 a, V8 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

// Round to the 16-bit format, flushing magnitudes below its smallest
// normal to zero (the error bound budgets for that flush).
template <int FMT>
__device__ __forceinline__ typename Fmt<FMT>::T quantise(double v) {
  const double tiny = FMT == kFmtF16 ? 6.103515625e-05 /* 2^-14 */ : 1.1754943508222875e-38;
  if (__builtin_fabs(v) < tiny) return (typename Fmt<FMT>::T)0.0f;
  // double -> float is exact for the values used here (v is a float
  // difference or a residual of a float-sized sum); float -> 16 bit rounds
  return (typename Fmt<FMT>::T)(float)v;
}

// ---------------------------------------------------------------------------
// Preparation, pass 1: quantised rows, norms and the global maxima.
// ---------------------------------------------------------------------------
// One centred, quantised coordinate (the same value wherever it is needed).
template <int FMT>
__device__ __forceinline__ typename Fmt<FMT>::T prep_coord(float x, float c) {
  const float diff = x - c;  // rounded to FP32: budgeted
  return quantise<FMT>((double)diff);
}

// The operand rows: 8 consecutive K slots per thread, so that the 16-byte
// stores of XA and XB are contiguous across the lanes.  Candidates XA [x~ | 0],
// the tiles' columns; queries XB [-2 x~ | 0], their rows (scaling by -2 is exact);
// padding is zero.
template <int FMT>
__global__ __launch_bounds__(kBlock) void k_mfma_prep(
    const float *__restrict__ X, uint64_t n, uint64_t n_pad, uint32_t d, uint32_t dp,
    uint32_t kp, const float *__restrict__ centre, typename Fmt<FMT>::T *__restrict__ XA,
    typename Fmt<FMT>::T *__restrict__ XB) {
  typedef typename Fmt<FMT>::T T;
  typedef typename Fmt<FMT>::V8 V8;
  const uint32_t kv = kp / 8;  // vectors per row
  const uint64_t total = n_pad * kv;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t p = e / kv;
    const uint32_t k0 = (uint32_t)(e - p * kv) * 8u;
    V8 a, b;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t t = k0 + (uint32_t)j;
      const T q = p < n && t < d ? prep_coord<FMT>(X[p * dp + t], centre[t]) : (T)0.0f;
      a[j] = q;
      b[j] = (T)(-2.0f * (float)q);  // exact
    }
    reinterpret_cast<V8 *>(XA)[e] = a;
    reinterpret_cast<V8 *>(XB)[e] = b;
  }
}

// Per point, in dimension order: the quantised norm |x~|^2 and the distance
// from the centre, both in FP64.  cn is what a tile element must stay below to
// be a hit: the float above -fl32(norm); that rounding is the "fold" error of
// the bound.  Padding rows get -inf (never a hit).  Each lane reads its own row
// as 16-byte vectors.
template <int FMT>
__global__ __launch_bounds__(kBlock) void k_mfma_norms(
    const float *__restrict__ X, uint64_t n, uint64_t n_pad, uint32_t d, uint32_t dp,
    const float *__restrict__ centre, float *__restrict__ cn, double *__restrict__ norm2,
    double *__restrict__ dist_c, double *__restrict__ fold_err) {
  typedef typename Fmt<FMT>::T T;
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n_pad) return;
  if (p >= n) {
    cn[p] = -__builtin_inff();
    return;
  }
  const float4 *x4 = reinterpret_cast<const float4 *>(X + p * dp);  // dp: a multiple of 8
  double nn = 0.0, dc = 0.0;
  for (uint32_t t0 = 0; t0 < d; t0 += 4) {
    const float4 v = x4[t0 / 4];
    const float xv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t = t0 + (uint32_t)j;
      if (t < d) {
        const T q = prep_coord<FMT>(xv[j], centre[t]);
        const double qd = (double)(float)q;
        nn += qd * qd;
        const double e = (double)xv[j] - (double)centre[t];
        dc += e * e;
      }
    }
  }
  const float h = (float)nn;
  cn[p] = strict(-h);
  norm2[p] = nn;
  dist_c[p] = __builtin_sqrt(dc);
  fold_err[p] = __builtin_fabs(nn - (double)h);
}

// Maxima of |x - c|, |x~|, n and the fold residual over all points.
// Non-negative doubles compare like their bit patterns.
__global__ __launch_bounds__(kBlock) void k_mfma_maxima(uint64_t n, const double *__restrict__ norm2,
                                                        const double *__restrict__ dist_c,
                                                        const double *__restrict__ fold_err,
                                                        unsigned long long *__restrict__ maxima) {
  __shared__ unsigned long long red[4][kWavesPerBlock];
  unsigned long long m[4] = {0, 0, 0, 0};
  for (uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x; p < n;
       p += (uint64_t)gridDim.x * kBlock) {
    const double v[4] = {dist_c[p], __builtin_sqrt(norm2[p]), norm2[p], fold_err[p]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned long long b = __builtin_bit_cast(unsigned long long, v[i]);
      m[i] = b > m[i] ? b : m[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long o = __shfl_xor(m[i], off);
      m[i] = o > m[i] ? o : m[i];
    }
    if (lane_id() == 0) red[i][threadIdx.x / kWave] = m[i];
  }
  __syncthreads();
  // one atomic per value and workgroup: with one per wave of 1024 workgroups the
  // atomics on four addresses took 0.14 to 0.19 ms at any size
  if (threadIdx.x < 4) {
    unsigned long long b = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
      const unsigned long long o = red[threadIdx.x][w];
      b = o > b ? o : b;
    }
    atomicMax(&maxima[threadIdx.x], b);
  }
}

// ---------------------------------------------------------------------------
// Preparation, pass 2: per-query thresholds.
//
// Notation for a query b and any candidate a:
//   S    exact squared distance of the FP32 points, S64 its canonical FP64
//        value; canonical acceptance is S64 <= eps2, and
//        S64 <= eps2 implies S <= s_hi = eps2/(1-g64), while
//        S <= s_lo = eps2/(1+g64) implies S64 <= eps2 (g64 = gamma_{d+2}(2^-53)).
//   S_q  squared distance of the quantised points a~, b~.
//   Each coordinate error |x~ - (x-c)| <= u|x-c| + eta, u = (1+2^-24)(1+u16)-1
//   (u16 = 2^-11 FP16, 2^-8 BF16; eta = the flush threshold), hence by the
//   triangle inequality |sqrt(S_q) - sqrt(S)| <= Delta_b =
//   u (|b-c| + R) + 2 eta sqrt(d), R = max over points of |x-c|.
//   D = -Thi - 2 b~.a~ up to gamma_{K+4}(2^-23) (|Thi| + 2 |b~| Rq): the MFMA
//   starts from Thi and adds K exact products in FP32 in any order, even with
//   truncating adds.  With the rounding of n_a (F) and of the accept test's
//   addition, everything stays within
//     E' = gamma_{K+4}(2^-23) (1.01 (hi_root^2 + n_b) + N + F + 2 |b~| Rq) + F + 2^-120
//   (N, Rq, F = maxima of n_a, |a~| and |n_a - fl32(n_a)|; |Thi| <= hi_root^2 +
//   n_b up to the last percent), and S_q = n_a - 2 a~.b~ + n_b.
//   (Thi is at most FLT_MAX, so that a tile starts from finite values: every pair
//   has n_a - 2 b~.a~ <= 3 N, and N is below 2e30.)
// Then
//   Thi(b) = (sqrt(s_hi) + Delta_b)^2 - n_b + E'   (canonical accept => a hit)
//   Tlo(b) = (max(0, sqrt(s_lo) - Delta_b))^2 - n_b - E'   (at or below: accept)
// evaluated in FP64 with a relative margin and rounded outward to FP32.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_mfma_thresholds(
    uint64_t n, uint64_t n_pad, MfmaBand band, const double *__restrict__ norm2,
    const double *__restrict__ dist_c, const unsigned long long *__restrict__ maxima,
    float *__restrict__ thi, float *__restrict__ tlo) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n_pad) return;
  if (p >= n) {
    thi[p] = -__builtin_inff();
    tlo[p] = -__builtin_inff();
    return;
  }
  const double R = __builtin_bit_cast(double, (uint64_t)maxima[0]);
  const double Rq = __builtin_bit_cast(double, (uint64_t)maxima[1]);
  const double N = __builtin_bit_cast(double, (uint64_t)maxima[2]);
  const double F = __builtin_bit_cast(double, (uint64_t)maxima[3]);
  const double nb = norm2[p];
  const double bq = __builtin_sqrt(nb);
  const double delta = band.u * (dist_c[p] + R) + band.eta_term;
  const double m = 0x1p-45;
  const double hi_root = __builtin_sqrt(band.s_hi) * (1.0 + m) + delta;
  const double E = band.gamma_acc * (1.01 * (hi_root * hi_root + nb) + N + F + 2.0 * bq * Rq) + F +
                   0x1p-120;
  const double thi_v = (hi_root * hi_root - nb + E) + m * (hi_root * hi_root + nb + E);
  double lo_root = __builtin_sqrt(band.s_lo) * (1.0 - m) - delta;
  double tlo_v;
  if (lo_root <= 0.0) {
    tlo_v = -__builtin_inf();
  } else {
    tlo_v = (lo_root * lo_root - nb - E) - m * (lo_root * lo_root + nb + E);
  }
  thi[p] = __builtin_fminf(round_up_f32(thi_v), FLT_MAX);
  tlo[p] = round_down_f32(tlo_v);
}

// Hit modes of the join kernels: kHitsRare tests the minimum of each tile
// first and builds the hit masks only of tiles with a hit; kHitsFrequent goes
// straight to the masks.
constexpr int kHitsRare = 0;
constexpr int kHitsFrequent = 1;

// The queries of a unit or a part of one: operands and initial accumulators in
// registers, positions and accept margins in LDS tables of 32 QB entries.
template <int KP, int FMT, int QB>
struct Queries {
  typedef typename Fmt<FMT>::V8 V8;
  V8 A[QB][KP / 16];
  float16v c0[QB];       // (where they stay in registers)
  const float *cinit;    // and the values that they come from
  const float *delta;    // Thi - Tlo, rounded up
  const uint32_t *qpos;  // positions (0xffffffff: no query)
};

// Loads the queries at slots [q0, q1) of v into q; cinit / delta / qpos: this
// wave's LDS tables.
template <int KP, int FMT, int QB>
__device__ __forceinline__ void load_queries(const MfmaView &v, uint32_t q0, uint32_t q1,
                                             float *cinit, float *delta, uint32_t *qpos,
                                             Queries<KP, FMT, QB> &q) {
  typedef typename Fmt<FMT>::V8 V8;
  constexpr int KS = KP / 16, RV = KP / 8;
  const V8 *__restrict__ XB = static_cast<const V8 *>(v.XB);
  const uint32_t l = lane_id(), half = l >> 5, col = l & 31;
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const uint32_t idx = (uint32_t)j * 32 + col;
    const uint32_t slot = q0 + idx;
    const bool live = slot < q1;
    const uint32_t p = live ? (v.qlist ? v.qlist[slot] : slot) : 0u;
    const float hi = v.thi[p], lo = v.tlo[p];
    if (half == 0) {
      cinit[idx] = live ? -hi : __builtin_inff();
      delta[idx] = live ? round_up_f32((double)hi - (double)lo) : 0.0f;
      qpos[idx] = live ? p : 0xffffffffu;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q.A[j][ks] = XB[(uint64_t)p * RV + ks * 2 + half];
  }
  __builtin_amdgcn_wave_barrier();  // the tables belong to this wave
#pragma unroll
  for (int j = 0; j < QB; ++j) q.c0[j] = rows_init(cinit + j * 32, half);
  q.cinit = cinit;
  q.delta = delta;
  q.qpos = qpos;
}

// The QB tiles of one 32-candidate block: operands b, reject value nn and
// position cp of each lane's candidate.  A tile's products are issued before the
// minima of the one ahead of it, so that a wave keeps the matrix unit busy by
// itself.
template <int KP, int FMT, int QB, int HM>
__device__ __forceinline__ void tiles(const Queries<KP, FMT, QB> &q,
                                      const typename Fmt<FMT>::V8 (&b)[KP / 16], float nn,
                                      uint32_t cp, uint32_t half, const KeyForm &kf, Stage &st,
                                      BandSink &bs, uint64_t *__restrict__ out, uint64_t capacity,
                                      unsigned long long *__restrict__ cursor) {
  static_assert(QB <= 4, "64 hit bits per lane");
  auto product = [&](int j) __attribute__((always_inline)) {
    float16v acc = q.c0[j];
#pragma unroll
    for (int ks = 0; ks < KP / 16; ++ks) acc = Fmt<FMT>::mfma(q.A[j][ks], b[ks], acc);
    return acc;
  };
  uint64_t hits = 0, within = 0;
  float16v acc = product(0);
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    float16v next = acc;
    __builtin_amdgcn_sched_barrier(0);
    if (j + 1 < QB) next = product(j + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (HM == kHitsFrequent || ballot(min16(acc, __builtin_inff()) < nn) != 0) {
      uint32_t h, a;
      tile_masks<true>(acc, nn, nn, q.delta + j * 32, half, h, a);
      hits |= (uint64_t)h << (16 * j);
      within |= (uint64_t)a << (16 * j);
    }
    acc = next;
  }
  if (QB > 1 && HM != kHitsFrequent && ballot(hits != 0) == 0) return;
  emit_hits<true>(hits, within, q.qpos, half, cp, nn, kf, st, bs, out, capacity, cursor);
}

// The same with the initial accumulators read from LDS: q.c0 holds those of the
// block, and each tile's are loaded again once its elements are done with, so that
// they are there for the next block.
template <int KP, int FMT, int QB, int HM>
__device__ __forceinline__ void tiles_reload(Queries<KP, FMT, QB> &q,
                                             const typename Fmt<FMT>::V8 (&b)[KP / 16], float nn,
                                             uint32_t cp, uint32_t half, const KeyForm &kf,
                                             Stage &st, BandSink &bs, uint64_t *__restrict__ out,
                                             uint64_t capacity,
                                             unsigned long long *__restrict__ cursor) {
  static_assert(QB <= 4, "64 hit bits per lane");
  uint64_t hits = 0, within = 0;
#pragma unroll
  for (int j = 0; j < QB; ++j)
#pragma unroll
    for (int ks = 0; ks < KP / 16; ++ks) q.c0[j] = Fmt<FMT>::mfma(q.A[j][ks], b[ks], q.c0[j]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    if (HM == kHitsFrequent || ballot(min16(q.c0[j], __builtin_inff()) < nn) != 0) {
      uint32_t h, a;
      tile_masks<true>(q.c0[j], nn, nn, q.delta + j * 32, half, h, a);
      hits |= (uint64_t)h << (16 * j);
      within |= (uint64_t)a << (16 * j);
    }
    q.c0[j] = rows_init(q.cinit + j * 32, half);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (QB > 1 && HM != kHitsFrequent && ballot(hits != 0) == 0) return;
  emit_hits<true>(hits, within, q.qpos, half, cp, nn, kf, st, bs, out, capacity, cursor);
}

__device__ __forceinline__ KeyForm key_form(const MfmaView &v) {
  return KeyForm{v.key_hi, v.pshift, v.symmetric != 0};
}

// One work unit of the matrix-core filter on one wave: 32 QB queries against
// the candidate blocks of the unit's runs, read from memory.  The next block's
// operands are in flight during the current block's tiles; their loads are
// unconditional (past the last block they repeat it), as under a branch the
// compiler copies their results at its end, and so waits for them there.
template <int KP, int FMT, int QB, int HM = kHitsRare>
__device__ __forceinline__ void mfma_unit(const MfmaView &v, const WorkUnit &wu, Stage &st,
                                          BandSink &bs, float *cinit, float *delta, uint32_t *qpos,
                                          uint64_t *__restrict__ out, uint64_t capacity,
                                          unsigned long long *__restrict__ cursor) {
  typedef typename Fmt<FMT>::V8 V8;
  constexpr int KS = KP / 16, RV = KP / 8;
  const V8 *__restrict__ XA = static_cast<const V8 *>(v.XA);
  const uint32_t l = lane_id(), half = l >> 5, col = l & 31;
  // candidate blocks, run by run; rows past the end of a run (at most 31,
  // inside the padded arrays) get a reject value nothing passes
  uint32_t r = wu.run_first, c = wu.c_begin;
  uint32_t ce = (r == wu.run_last) ? wu.c_end : scalar_run(v.runs, r).y;
  auto normalise = [&]() __attribute__((always_inline)) {
    while (c >= ce && r < wu.run_last) {
      const uint2 run = scalar_run(v.runs, ++r);
      c = run.x;
      ce = (r == wu.run_last) ? wu.c_end : run.y;
    }
  };
  normalise();
  if (c >= ce) return;
  struct Block {
    V8 b[KS];
    float nn;
    uint32_t cp, end;  // position, and where the run ends (0: no block)
    // (selected at its use: earlier it would wait for the loads)
    __device__ float reject() const { return cp < end ? nn : -__builtin_inff(); }
  };
  uint32_t last_c = c;
  auto load = [&](Block &k) __attribute__((always_inline)) {
    const bool more = c < ce;
    const uint32_t at = more ? c : last_c;
    k.cp = at + col;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k.b[ks] = XA[(uint64_t)k.cp * RV + ks * 2 + half];
    k.nn = v.cn[k.cp];
    k.end = more ? ce : 0u;
    __builtin_amdgcn_sched_barrier(0);  // issued here, ahead of the tiles
    last_c = at;
    if (more) {
      c += 32;
      normalise();
    }
    return more;
  };
  Queries<KP, FMT, QB> q;
  load_queries<KP, FMT, QB>(v, wu.q0, wu.q1, cinit, delta, qpos, q);
  wait_loads();
  const KeyForm kf = key_form(v);
  Block b0, b1;
  bool more = load(b0);
  for (;;) {
    more = load(b1);
    tiles<KP, FMT, QB, HM>(q, b0.b, b0.reject(), b0.cp, half, kf, st, bs, out, capacity, cursor);
    if (!more) break;
    more = load(b0);
    tiles<KP, FMT, QB, HM>(q, b1.b, b1.reject(), b1.cp, half, kf, st, bs, out, capacity, cursor);
    if (!more) break;
  }
  __builtin_amdgcn_wave_barrier();  // the tables are rewritten by the next unit
}

// Per-wave form for indexes with small cells: every wave takes a work unit
// of its own (32 * SJ_WAVE_QB queries of one cell) and streams that unit's
// candidates itself, so cells much smaller than a workgroup's 256 queries do
// not leave most matrix rows empty.
#ifndef SJ_WAVE_QB
#define SJ_WAVE_QB 1
#endif
template <int KP, int FMT, int HM>
__global__ __launch_bounds__(kBlock) void k_join_mfma_wave(MfmaView v,
                                                           const WorkUnit *__restrict__ wus,
                                                           uint64_t n_wu, uint64_t *__restrict__ out,
                                                           uint64_t capacity,
                                                           unsigned long long *__restrict__ cursor) {
  __shared__ uint64_t stage_mem[kWavesPerBlock][kStage];
  __shared__ uint64_t band_mem[kWavesPerBlock][kBandStage];
  __shared__ __align__(16) float cinit[kWavesPerBlock][32 * SJ_WAVE_QB];
  __shared__ __align__(16) float delta[kWavesPerBlock][32 * SJ_WAVE_QB];
  __shared__ uint32_t qpos[kWavesPerBlock][32 * SJ_WAVE_QB];
  const uint32_t w = uniform_u32(threadIdx.x / kWave);
  const uint64_t u = (uint64_t)blockIdx.x * kWavesPerBlock + w;
  if (u >= n_wu) return;  // whole wave leaves; no workgroup barrier follows
  const WorkUnit wu = wus[u];
  Stage st{&stage_mem[w][0], 0u, kStage};
  BandSink bs{v.band, v.band_cap, v.band_cursor, Stage{&band_mem[w][0], 0u, kBandStage}};
  mfma_unit<KP, FMT, SJ_WAVE_QB, HM>(v, wu, st, bs, cinit[w], delta[w], qpos[w], out, capacity,
                                     cursor);
  flush(st, out, capacity, cursor);
  flush(bs.st, bs.buf, bs.cap, bs.cursor);
}

// Workgroup-cooperative form of the same filter for a single join: the waves
// of a workgroup own the 256 query rows of one work unit, 32 QB each, and
// share every candidate chunk of kChunk rows, which is fetched from memory
// once into a double-buffered LDS stage (global -> registers during the
// MFMAs of the previous chunk -> LDS) instead of once per wave.
constexpr int kChunk = 64;  // candidate rows per LDS stage (2 MFMA column blocks)
// LDS row stride of a staged chunk, in 16-byte vectors.  Lanes read the
// same vector of 32 consecutive rows; with an odd stride (RV is even) the
// reads of 8 consecutive rows fall in different bank groups.
constexpr int lds_row_vectors(int rv) { return rv >= 4 ? rv + 1 : rv; }
// Query blocks per wave: four where two waves per SIMD still hold them (each
// operand read from LDS then serves four products, and the chunk four tiles of
// products without a wait).  Bound by the card's power on the matrix unit at K 64
// (2M x 64 BF16 join, 1.17 PFLOP/s); measured there: 231 to 250 ms with two
// blocks per wave, 223 to 233 with four (226 to 238 with candidates as rows).
constexpr uint32_t kUnitQueries = 256;
template <int KP>
constexpr int wg_qb = KP <= 64 ? 4 : 2;

// Where three waves per SIMD fit once the initial accumulators leave the registers
// (K 80: 184 to 152, K 96: 200 to 164 of them; at K 112 and 128 LDS holds two either
// way).  Joins with the accumulators kept and reloaded: 515k x 90 mixture FP16 27.0
// and 25.0 ms, BF16 28.1 and 25.9, 400k x 70 uniform BF16 18.1 and 16.3, 400k x 96
// FP16 17.3 and 16.0 (400k x 110: 19.3 and 19.5).
template <int KP>
constexpr bool kReloadRows = KP > 64 && KP <= 96;

template <int QB>
constexpr int wg_threads = (int)kUnitQueries / (32 * QB) * kWave;

template <int KP, int FMT, int QB, int HM>
__global__ __launch_bounds__(wg_threads<QB>) void k_join_mfma_wg(
    MfmaView v, const WorkUnit *__restrict__ wus, uint64_t n_wu, uint64_t *__restrict__ out,
    uint64_t capacity, unsigned long long *__restrict__ cursor) {
  typedef typename Fmt<FMT>::V8 V8;
  constexpr int NT = wg_threads<QB>, NW = NT / kWave;
  constexpr int KS = KP / 16;                     // MFMA K steps
  constexpr int RV = KP / 8;                      // 8-element vectors per row
  constexpr int CHUNK_VECS = kChunk * RV;         // vectors per LDS stage
  constexpr int PER_THREAD = (CHUNK_VECS + NT - 1) / NT;
  __shared__ uint64_t stage_mem[NW][kStage];
  constexpr int RS = lds_row_vectors(RV);
  __shared__ V8 tile[2][kChunk * RS];
  __shared__ float tile_n[2][kChunk];  // reject values of the chunk
  __shared__ uint64_t band_mem[NW][kBandStage];
  __shared__ __align__(16) float cinit[NW][32 * QB];
  __shared__ __align__(16) float delta[NW][32 * QB];
  __shared__ uint32_t qpos[NW][32 * QB];
  const uint64_t u = blockIdx.x;
  if (u >= n_wu) return;  // whole workgroup leaves together
  const WorkUnit wu = wus[u];
  const uint32_t w = uniform_u32(threadIdx.x / kWave);
  const uint32_t l = lane_id();
  const uint32_t half = l >> 5, col = l & 31;
  const V8 *__restrict__ XA = static_cast<const V8 *>(v.XA);

  // chunk walk (uniform over the workgroup)
  uint32_t r = wu.run_first, c = wu.c_begin;
  uint32_t ce = (r == wu.run_last) ? wu.c_end : scalar_run(v.runs, r).y;
  auto normalise = [&]() __attribute__((always_inline)) {
    while (c >= ce && r < wu.run_last) {
      const uint2 run = scalar_run(v.runs, ++r);
      c = run.x;
      ce = (r == wu.run_last) ? wu.c_end : run.y;
    }
  };
  normalise();
  if (c >= ce) return;  // empty unit (uniform)
  V8 pre[PER_THREAD];
  float pre_n;
  uint32_t pre_rows;
  // (loads without a branch: its end would wait for them)
  auto fetch = [&](uint32_t base, uint32_t end) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const uint32_t e = threadIdx.x + (uint32_t)i * NT;
      pre[i] = XA[(uint64_t)base * RV + (e < (uint32_t)CHUNK_VECS ? e : 0u)];
    }
    pre_n = v.cn[base + threadIdx.x % kChunk];
    pre_rows = end - base;
    __builtin_amdgcn_sched_barrier(0);  // issued here, ahead of the tiles
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const uint32_t e = threadIdx.x + (uint32_t)i * NT;
      if (e < (uint32_t)CHUNK_VECS) tile[buf][(e / RV) * RS + e % RV] = pre[i];
    }
    if (threadIdx.x < (uint32_t)kChunk)  // rows past the run's end never hit
      tile_n[buf][threadIdx.x] = threadIdx.x < pre_rows ? pre_n : -__builtin_inff();
  };
  fetch(c, ce);
  // this wave's query rows
  Queries<KP, FMT, QB> q;
  load_queries<KP, FMT, QB>(v, wu.q0 + w * QB * 32, wu.q1, cinit[w], delta[w], qpos[w], q);
  const KeyForm kf = key_form(v);
  Stage st{&stage_mem[w][0], 0u, kStage};
  BandSink bs{v.band, v.band_cap, v.band_cursor, Stage{&band_mem[w][0], 0u, kBandStage}};
  wait_loads();
  store(0);
  __syncthreads();
  int cur = 0;
  for (;;) {
    const uint32_t cc = c;
    c += kChunk;
    normalise();
    const bool more = c < ce;
    fetch(more ? c : cc, more ? ce : cc);
    V8 b[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) b[ks] = tile[cur][col * RS + ks * 2 + half];
    float nn = tile_n[cur][col];
#pragma nounroll
    for (uint32_t blk = 0; blk < 2; ++blk) {
      V8 b2[KS];  // the second block's operands, on their way during the first one's tiles
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) b2[ks] = tile[cur][(32 + col) * RS + ks * 2 + half];
      const float nn2 = tile_n[cur][32 + col];
      if constexpr (kReloadRows<KP>)
        tiles_reload<KP, FMT, QB, HM>(q, b, nn, cc + blk * 32 + col, half, kf, st, bs, out,
                                      capacity, cursor);
      else
        tiles<KP, FMT, QB, HM>(q, b, nn, cc + blk * 32 + col, half, kf, st, bs, out, capacity,
                               cursor);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) b[ks] = b2[ks];
      nn = nn2;
    }
    if (!more) break;
    store(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
  flush(bs.st, bs.buf, bs.cap, bs.cursor);
  flush(st, out, capacity, cursor);
}

// Deferred FP64 recheck of the band pairs of a launch: one pair per lane,
// all lanes busy, instead of the few band lanes of one tile element at a
// time.  Accepted pairs are staged and appended like the join's own.
constexpr int kRecheckUnroll = 8;
constexpr int kRecheckBlocksPerCu = 8;

// Appends the pairs of one batch of rechecks (lane: pair q, c, accepted or
// not; both orders in a symmetric join).
__device__ __forceinline__ void emit_rechecked(const MfmaView &v, bool ok, uint32_t q, uint32_t c,
                                               Stage &st, uint64_t *__restrict__ out,
                                               uint64_t capacity,
                                               unsigned long long *__restrict__ cursor) {
  const uint64_t am = ballot(ok);
  if (am == 0) return;
  const bool two = ok && v.symmetric != 0 && q != c;
  const uint64_t m2 = ballot(two);
  const uint32_t n = (uint32_t)(__builtin_popcountll(am) + __builtin_popcountll(m2));
  if (st.cnt + n > (uint32_t)kStage) flush(st, out, capacity, cursor);
  const uint32_t off = st.cnt + lanes_below(am) + lanes_below(m2);
  if (ok) {
    st.buf[off] = v.key_hi | ((uint64_t)q << v.pshift) | c;
    if (two) st.buf[off + 1] = v.key_hi | ((uint64_t)c << v.pshift) | q;
  }
  st.cnt += n;
}

// Rows of up to DPM padded dimensions, NP pairs per batch, one wave per
// workgroup.  The wave first copies the two rows of each of its pairs into
// LDS, 16 bytes per lane and whole row segments per instruction (a row costs
// a few cache-line requests instead of one per dimension and lane); each of
// the first NP lanes then evaluates its pair from LDS in the caller's
// dimension order.  Rows are DPM + 1 floats apart, so the lanes' reads of
// one dimension fall in different banks.  Above 64 padded dimensions a batch
// holds 32 pairs, so that four waves fit a CU's LDS.
template <int DPM, int NP>
__global__ __launch_bounds__(kWave) void k_band_recheck_staged(
    MfmaView v, const unsigned long long *__restrict__ band_count, uint64_t *__restrict__ out,
    uint64_t capacity, unsigned long long *__restrict__ cursor,
    unsigned long long *__restrict__ rechecks) {
  static_assert(NP == kWave || NP == kWave / 2, "one or half a pair per lane");
  constexpr int kRow = DPM + 1;
  constexpr int kVecs = 2 * NP * DPM / 4 / kWave;  // 16-byte loads per lane and batch
  __shared__ float rows[2][NP][kRow];
  __shared__ uint32_t pos[2][NP];
  __shared__ uint64_t stage_mem[kStage];
  __shared__ uint16_t perm[SJ_MAX_DIM];
  const uint32_t l = threadIdx.x;
  for (uint32_t t = l; t < v.d; t += kWave) perm[t] = v.inv_perm[t];
  Stage st{stage_mem, 0u, kStage};
  const uint64_t total = *band_count;
  const uint64_t count = total < v.band_cap ? total : v.band_cap;
  const uint32_t dv = v.dp / 4;  // 16-byte vectors per row (dp <= DPM, a multiple of 8)
  for (uint64_t base = (uint64_t)blockIdx.x * NP; base < count;
       base += (uint64_t)gridDim.x * NP) {
    const uint64_t i = base + l;
    const bool live = l < (uint32_t)NP && i < count;
    uint32_t q = 0, c = 0;  // slots past the end stage row 0 and drop it
    if (live) {
      const uint64_t key = v.band[i];
      q = (uint32_t)(key >> 32);
      c = (uint32_t)key;
    }
    if (l < (uint32_t)NP) {
      pos[0][l] = q;
      pos[1][l] = c;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
      // vector e of the batch's 2 x NP rows of DPM / 4 vectors
      const uint32_t e = (uint32_t)k * kWave + l;
      const uint32_t row = e / (DPM / 4), col = e % (DPM / 4);
      const uint32_t side = row / NP, slot = row % NP;
      if (col < dv) {
        const float *src = side ? v.X : v.Xq;
        const float4 x =
            *reinterpret_cast<const float4 *>(src + (uint64_t)pos[side][slot] * v.dp + col * 4);
        float *dst = &rows[side][slot][col * 4];
        dst[0] = x.x;
        dst[1] = x.y;
        dst[2] = x.z;
        dst[3] = x.w;
      }
    }
    __syncthreads();
    const uint32_t lr = l < (uint32_t)NP ? l : 0u;  // the row a lane evaluates
    const bool ok = live && canonical_within_body<kRecheckUnroll>(&rows[0][lr][0], 0,
                                                                 &rows[1][lr][0], 0, perm, v.d, 0,
                                                                 v.eps2);
    __syncthreads();  // the rows are overwritten by the next batch
    emit_rechecked(v, ok, q, c, st, out, capacity, cursor);
  }
  flush(st, out, capacity, cursor);
  if (blockIdx.x == 0 && l == 0 && count) atomicAdd(rechecks, (unsigned long long)count);
}

// query column blocks per wave of the persistent batched kernel
// Query blocks per wave: the candidate stream from L2 bounds this kernel, and a
// block of candidates serves QB tiles (graph of the 256 jobs with 1, 2 and 4:
// 114, 83 and 76 ms; 150 clustered jobs of up to 100k x 64: 37, 32 and 29 ms).
#ifndef SJ_BATCH_QB
#define SJ_BATCH_QB 4
#endif

// Many independent joins in one persistent launch.  Every wave takes
// `grab` work units at a time from a global queue shared by all jobs and
// runs each with the instantiation of its job's K padding and format.  A
// wave leaves once the queue is exhausted, so the grid drains by itself.
template <int KP, int FMT>
__device__ __forceinline__ void batched_dispatch(const MfmaView &v, const WorkUnit &wu, Stage &st,
                                                 BandSink &bs, float *tab,
                                                 uint64_t *__restrict__ out, uint64_t capacity,
                                                 unsigned long long *__restrict__ cursor) {
  mfma_unit<KP, FMT, SJ_BATCH_QB>(v, wu, st, bs, tab, tab + 32 * SJ_BATCH_QB,
                                  reinterpret_cast<uint32_t *>(tab + 64 * SJ_BATCH_QB), out,
                                  capacity, cursor);
}

__global__ __launch_bounds__(kBlock) void k_join_batched(
    const BatchJob *__restrict__ jobs, const WorkUnit *__restrict__ wus, uint64_t n_wu,
    uint32_t grab, unsigned int *__restrict__ queue, uint64_t *__restrict__ out,
    const unsigned long long *__restrict__ capacity_p, unsigned long long *__restrict__ cursor,
    uint64_t *__restrict__ band, uint64_t band_cap, unsigned long long *__restrict__ band_cursor) {
  __shared__ uint64_t stage_mem[kWavesPerBlock][kStage];
  __shared__ uint64_t band_mem[kWavesPerBlock][kBandStage];
  const uint32_t w = uniform_u32(threadIdx.x / kWave);
  __shared__ __align__(16) float tables[kWavesPerBlock][96 * SJ_BATCH_QB];
  float *tab = &tables[w][0];
  Stage st{&stage_mem[w][0], 0u, kStage};
  BandSink bs{band, band_cap, band_cursor, Stage{&band_mem[w][0], 0u, kBandStage}};
  const uint64_t capacity = *capacity_p;
  for (;;) {
    unsigned int u0 = 0;
    if (lane_id() == 0) u0 = atomicAdd(queue, grab);
    u0 = uniform_u32(__shfl(u0, 0));
    if ((uint64_t)u0 >= n_wu) break;
    const uint64_t u1 = (uint64_t)u0 + grab < n_wu ? (uint64_t)u0 + grab : n_wu;
    for (uint64_t u = u0; u < u1; ++u) {
      const WorkUnit wu = wus[u];
      const uint32_t job = wu.pad;
      MfmaView v = jobs[job].view;
      v.key_hi = (uint64_t)job << 40;
      switch (jobs[job].variant) {
        case 0: batched_dispatch<16, kFmtF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 1: batched_dispatch<32, kFmtF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 2: batched_dispatch<48, kFmtF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 3: batched_dispatch<64, kFmtF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 4: batched_dispatch<80, kFmtF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 5: batched_dispatch<16, kFmtBF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 6: batched_dispatch<32, kFmtBF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 7: batched_dispatch<48, kFmtBF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 8: batched_dispatch<64, kFmtBF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        case 9: batched_dispatch<80, kFmtBF16>(v, wu, st, bs, tab, out, capacity, cursor); break;
        default: break;
      }
    }
  }
  flush(st, out, capacity, cursor);
  flush(bs.st, bs.buf, bs.cap, bs.cursor);
}

// Deferred recheck of a batched launch's band pairs (job << 40 | pos_q << 20
// | pos_c), one per lane, each with its own job's rows.
__global__ __launch_bounds__(kBlock) void k_band_recheck_batched(
    const BatchJob *__restrict__ jobs, const uint64_t *__restrict__ band,
    const unsigned long long *__restrict__ band_count, uint64_t band_cap,
    uint64_t *__restrict__ out, const unsigned long long *__restrict__ capacity_p,
    unsigned long long *__restrict__ cursor, unsigned long long *__restrict__ rechecks) {
  __shared__ uint64_t stage_mem[kWavesPerBlock][kStage];
  const uint32_t w = uniform_u32(threadIdx.x / kWave);
  Stage st{&stage_mem[w][0], 0u, kStage};
  const uint64_t capacity = *capacity_p;
  const uint64_t total = *band_count;
  const uint64_t count = total < band_cap ? total : band_cap;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  constexpr uint64_t kMask = (1ull << 20) - 1ull;
  for (uint64_t base = (uint64_t)blockIdx.x * kBlock + (uint64_t)w * kWave; base < count;
       base += stride) {
    const uint64_t i = base + lane_id();
    bool ok = false, two = false;
    uint64_t key = 0, rkey = 0;
    if (i < count) {
      key = band[i];
      const uint32_t job = (uint32_t)(key >> 40);
      const uint32_t q = (uint32_t)((key >> 20) & kMask), c = (uint32_t)(key & kMask);
      const MfmaView &v = jobs[job].view;
      ok = canonical_within_body<kRecheckUnroll>(v.Xq, q, v.X, c, v.inv_perm, v.d, v.dp, v.eps2);
      two = ok && v.symmetric && q != c;
      rkey = ((uint64_t)job << 40) | ((uint64_t)c << 20) | q;
    }
    const uint64_t am = ballot(ok);
    if (am == 0) continue;
    const uint64_t m2 = ballot(two);
    const uint32_t n = (uint32_t)(__builtin_popcountll(am) + __builtin_popcountll(m2));
    if (st.cnt + n > (uint32_t)kStage) flush(st, out, capacity, cursor);
    const uint32_t off = st.cnt + lanes_below(am) + lanes_below(m2);
    if (ok) {
      st.buf[off] = key;
      if (two) st.buf[off + 1] = rkey;
    }
    st.cnt += n;
  }
  flush(st, out, capacity, cursor);
  if (blockIdx.x == 0 && threadIdx.x == 0 && count) atomicAdd(rechecks, (unsigned long long)count);
}

// Batched keys job << 40 | pos_q << 20 | pos_c -> job << 40 | id_q << 20 | id_c,
// for the first min(*count, capacity) keys.
__global__ __launch_bounds__(kBlock) void k_pos_to_id_batched(
    uint64_t *__restrict__ keys, const unsigned long long *__restrict__ count,
    const unsigned long long *__restrict__ capacity_p, const BatchJob *__restrict__ jobs) {
  const unsigned long long cap = *capacity_p;
  const uint64_t total = *count < cap ? *count : cap;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t k = keys[e];
    const uint32_t job = (uint32_t)(k >> 40);
    const uint32_t *oid = jobs[job].orig_id;
    const uint32_t q = (uint32_t)(k >> 20) & 0xfffffu, c = (uint32_t)k & 0xfffffu;
    keys[e] = ((uint64_t)job << 40) | ((uint64_t)oid[q] << 20) | oid[c];
  }
}

// First and last+1 slot of every job in the sorted batched keys.
__global__ __launch_bounds__(kBlock) void k_job_bounds(
    const uint64_t *__restrict__ keys, const unsigned long long *__restrict__ count,
    const unsigned long long *__restrict__ capacity_p, unsigned long long *__restrict__ first,
    unsigned long long *__restrict__ last) {
  const unsigned long long cap = *capacity_p;
  const uint64_t total = *count < cap ? *count : cap;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint32_t job = (uint32_t)(keys[e] >> 40);
    if (e == 0 || (uint32_t)(keys[e - 1] >> 40) != job) first[job] = e;
    if (e + 1 == total || (uint32_t)(keys[e + 1] >> 40) != job) last[job] = e + 1;
  }
}

// Keys of cell-order positions (q << 32 | c) -> keys of caller indices
// (query positions through qid, candidate positions through orig_id).
__global__ __launch_bounds__(kBlock) void k_pos_to_id(uint64_t *__restrict__ keys, uint64_t count,
                                                      const uint32_t *__restrict__ qid,
                                                      const uint32_t *__restrict__ orig_id) {
  // grid-stride: count may exceed the 2^32 work-items of one dispatch
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < count;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t k = keys[e];
    keys[e] = ((uint64_t)qid[(uint32_t)(k >> 32)] << 32) | orig_id[(uint32_t)k];
  }
}

template <int KP, int FMT>
void launch_kp(const MfmaLaunch &a, hipStream_t s) {
  constexpr int QB = wg_qb<KP>;
  const MfmaView v = a.view;
  // one wave per work unit, or one workgroup
  for_unit_launches(a.n_wu, a.per_wave ? kWave : wg_threads<QB>, [&](uint64_t u, uint64_t n) {
    const WorkUnit *wu = a.wu + u;
    const uint32_t grid = (uint32_t)((n + kWavesPerBlock - 1) / kWavesPerBlock);
    if (a.per_wave && a.hits_frequent)
      hipLaunchKernelGGL((k_join_mfma_wave<KP, FMT, kHitsFrequent>), dim3(grid), dim3(kBlock), 0,
                         s, v, wu, n, a.out, a.capacity, a.cursor);
    else if (a.per_wave)
      hipLaunchKernelGGL((k_join_mfma_wave<KP, FMT, kHitsRare>), dim3(grid), dim3(kBlock), 0, s,
                         v, wu, n, a.out, a.capacity, a.cursor);
    else if (a.hits_frequent)
      hipLaunchKernelGGL((k_join_mfma_wg<KP, FMT, QB, kHitsFrequent>), dim3((uint32_t)n),
                         dim3(wg_threads<QB>), 0, s, v, wu, n, a.out, a.capacity, a.cursor);
    else
      hipLaunchKernelGGL((k_join_mfma_wg<KP, FMT, QB, kHitsRare>), dim3((uint32_t)n),
                         dim3(wg_threads<QB>), 0, s, v, wu, n, a.out, a.capacity, a.cursor);
    SJ_HIP(hipGetLastError());
  });
}

template <int FMT>
void launch_fmt(const MfmaLaunch &a, hipStream_t s) {
  switch (a.kp) {
    case 16: launch_kp<16, FMT>(a, s); break;
    case 32: launch_kp<32, FMT>(a, s); break;
    case 48: launch_kp<48, FMT>(a, s); break;
    case 64: launch_kp<64, FMT>(a, s); break;
    case 80: launch_kp<80, FMT>(a, s); break;
    case 96: launch_kp<96, FMT>(a, s); break;
    case 112: launch_kp<112, FMT>(a, s); break;
    case 128: launch_kp<128, FMT>(a, s); break;
    default: fail(SJ_ERR_INVALID_ARG, "unsupported MFMA K padding");
  }
}

}  // namespace

uint32_t mfma_kp(uint32_t d) { return (d + 15) / 16 * 16; }

int mfma_qb(uint32_t) { return SJ_BATCH_QB; }

uint32_t mfma_wave_queries() { return 32u * SJ_WAVE_QB; }

uint32_t mfma_wg_queries(uint32_t) { return kUnitQueries; }

void launch_mfma_prep(int fmt, const float *X, uint64_t n, uint64_t n_pad, uint32_t d, uint32_t dp,
                      uint32_t kp, const float *centre, void *XA, void *XB, float *cn,
                      double *norm2, double *dist_c, double *fold_err,
                      unsigned long long *maxima, hipStream_t s) {
  const uint32_t grid = (uint32_t)((n_pad + kBlock - 1) / kBlock);
  if (!grid) return;
  const uint32_t grid_rows =
      (uint32_t)std::min<uint64_t>((n_pad * (kp / 8) + kBlock - 1) / kBlock, 1u << 20);
  if (fmt == kFmtF16) {
    hipLaunchKernelGGL(k_mfma_prep<kFmtF16>, dim3(grid_rows), dim3(kBlock), 0, s, X, n, n_pad, d,
                       dp, kp, centre, (_Float16 *)XA, (_Float16 *)XB);
    hipLaunchKernelGGL(k_mfma_norms<kFmtF16>, dim3(grid), dim3(kBlock), 0, s, X, n, n_pad, d, dp,
                       centre, cn, norm2, dist_c, fold_err);
  } else {
    hipLaunchKernelGGL(k_mfma_prep<kFmtBF16>, dim3(grid_rows), dim3(kBlock), 0, s, X, n, n_pad,
                       d, dp, kp, centre, (__bf16 *)XA, (__bf16 *)XB);
    hipLaunchKernelGGL(k_mfma_norms<kFmtBF16>, dim3(grid), dim3(kBlock), 0, s, X, n, n_pad, d, dp,
                       centre, cn, norm2, dist_c, fold_err);
  }
  SJ_HIP(hipGetLastError());
  SJ_HIP(hipMemsetAsync(maxima, 0, 4 * sizeof(unsigned long long), s));
  const uint32_t g2 = (uint32_t)std::min<uint64_t>((n + kBlock - 1) / kBlock, 512);
  if (g2) {
    hipLaunchKernelGGL(k_mfma_maxima, dim3(g2), dim3(kBlock), 0, s, n, norm2, dist_c, fold_err,
                       maxima);
    SJ_HIP(hipGetLastError());
  }
}

void launch_mfma_thresholds(uint64_t n, uint64_t n_pad, const MfmaBand &band, const double *norm2,
                            const double *dist_c, const unsigned long long *maxima, float *thi,
                            float *tlo, hipStream_t s) {
  const uint32_t grid = (uint32_t)((n_pad + kBlock - 1) / kBlock);
  if (!grid) return;
  hipLaunchKernelGGL(k_mfma_thresholds, dim3(grid), dim3(kBlock), 0, s, n, n_pad, band, norm2,
                     dist_c, maxima, thi, tlo);
  SJ_HIP(hipGetLastError());
}

void launch_pos_to_id(uint64_t *keys, uint64_t count, const uint32_t *qid,
                      const uint32_t *orig_id, hipStream_t s) {
  if (!count) return;
  const uint32_t grid = (uint32_t)std::min<uint64_t>((count + kBlock - 1) / kBlock, 1u << 20);
  hipLaunchKernelGGL(k_pos_to_id, dim3(grid), dim3(kBlock), 0, s, keys, count, qid, orig_id);
  SJ_HIP(hipGetLastError());
}

int batched_variant(uint32_t kp, int fmt) {
  int base = fmt == kFmtF16 ? 0 : 5;
  switch (kp) {
    case 16: return base + 0;
    case 32: return base + 1;
    case 48: return base + 2;
    case 64: return base + 3;
    case 80: return base + 4;
    default: return -1;
  }
}

int batched_blocks_per_cu() {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_join_batched, kBlock, 0) !=
      hipSuccess) {
    (void)hipGetLastError();
    blocks = 2;
  }
  return blocks > 0 ? blocks : 1;
}

void launch_join_batched(const BatchJob *jobs, const WorkUnit *wus, uint64_t n_wu, uint32_t grab,
                         unsigned int *queue, uint64_t *out, const unsigned long long *capacity,
                         unsigned long long *cursor, uint32_t grid, uint64_t *band,
                         uint64_t band_cap, unsigned long long *band_cursor, hipStream_t s) {
  hipLaunchKernelGGL(k_join_batched, dim3(grid), dim3(kBlock), 0, s, jobs, wus, n_wu, grab, queue,
                     out, capacity, cursor, band, band_cap, band_cursor);
  SJ_HIP(hipGetLastError());
}

void launch_band_recheck_batched(const BatchJob *jobs, const uint64_t *band,
                                 const unsigned long long *band_count, uint64_t band_cap,
                                 uint64_t *out, const unsigned long long *capacity,
                                 unsigned long long *cursor, unsigned long long *rechecks,
                                 uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_band_recheck_batched, dim3(grid), dim3(kBlock), 0, s, jobs, band,
                     band_count, band_cap, out, capacity, cursor, rechecks);
  SJ_HIP(hipGetLastError());
}

void launch_pos_to_id_batched(uint64_t *keys, const unsigned long long *count,
                              const unsigned long long *capacity, const BatchJob *jobs,
                              uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_pos_to_id_batched, dim3(grid), dim3(kBlock), 0, s, keys, count, capacity,
                     jobs);
  SJ_HIP(hipGetLastError());
}

void launch_job_bounds(const uint64_t *keys, const unsigned long long *count,
                       const unsigned long long *capacity, unsigned long long *first,
                       unsigned long long *last, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_job_bounds, dim3(grid), dim3(kBlock), 0, s, keys, count, capacity, first,
                     last);
  SJ_HIP(hipGetLastError());
}

void launch_band_recheck(const MfmaView &v, uint64_t *out, uint64_t capacity,
                         unsigned long long *cursor, unsigned long long *rechecks, hipStream_t s) {
  int dev = 0, cus = 256;
  SJ_HIP(hipGetDevice(&dev));
  SJ_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const dim3 grid((uint32_t)cus * kRecheckBlocksPerCu);
  if (v.dp <= 32)
    hipLaunchKernelGGL((k_band_recheck_staged<32, kWave>), grid, dim3(kWave), 0, s, v,
                       v.band_cursor, out, capacity, cursor, rechecks);
  else if (v.dp <= 64)
    hipLaunchKernelGGL((k_band_recheck_staged<64, kWave>), grid, dim3(kWave), 0, s, v,
                       v.band_cursor, out, capacity, cursor, rechecks);
  else  // 32 pairs per batch: 33 KB of rows, four waves per CU
    hipLaunchKernelGGL((k_band_recheck_staged<SJ_MAX_DIM, kWave / 2>), grid, dim3(kWave), 0, s, v,
                       v.band_cursor, out, capacity, cursor, rechecks);
  SJ_HIP(hipGetLastError());
}

void launch_join_mfma(const MfmaLaunch &a, hipStream_t s) {
  if (a.box && !a.per_wave && a.kp <= 32) return launch_join_box16(a, s);
  if (a.fmt == kFmtF16) launch_fmt<kFmtF16>(a, s);
  else launch_fmt<kFmtBF16>(a, s);
}

}  // namespace sj
