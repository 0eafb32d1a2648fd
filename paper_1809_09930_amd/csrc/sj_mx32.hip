// FP32 distance filter of the self-join on the matrix cores of gfx950.
//
// Form.  Points are taken relative to a centre c of the indexed set (the
// sample mean) and scaled by a power of two, x~ = sc fl32(x - c) with all
// |x~| <= 2^14, and every x~ is split into two FP16 numbers x1 + x2 (11 bits
// each, the second one signed).  With queries as rows and candidates as
// columns a 32x32 tile accumulates in FP32
//     D = -Thi(q) - 2 q~ . a~
// from the three products q1a1, q1a2, q2a1 (the fourth is below 2^-22 of
// |q||a|): three v_mfma_f32_32x32x16_f16 per 16 dimensions, 96 matrix cycles
// where 16 dimensions of v_mfma_f32_32x32x2_f32 take 512, three BF16 parts (six
// products) 192.  D > -|a~|^2 (1 - kappa) rejects the pair.  Every other pair is
// decided by the canonical FP64 predicate (deferred recheck), except where the
// vector norm form would be the alternative (up to 16 dimensions, eps not small
// against the norms): there D + (Thi - Tlo)(q) <= -|a~|^2 (1 + ...) accepts it
// first.  The pair set is exact either way.
//
// Error.  With S~ the squared distance of the exact x~, |sqrt S~ - sqrt S| <=
// u (|q~| + |a~|) (u = 2^-24: the rounded subtraction; S scaled by sc^2), and
// S <= s_hi for every pair the canonical predicate accepts, hence
//     S~ <= s_hi + u' (s_hi + 2 |q~|^2 + 2 |a~|^2).
// The split leaves at most 2^-22 |x~| + 2^-25 per coordinate (FP16 subnormals
// are kept by the conversions and by the MFMA) and drops q2a2, together at most
// 1.5 2^-21 (|q~|^2 + |a~|^2) + 2^-22 (...) + tiny / 2, and the FP32 accumulation
// of m exact products, in any order and even with truncating adds, at most
// gamma_m(2^-23) (|Thi| + |q~|^2 + |a~|^2).  With kappa the sum of these
// coefficients (mx32_kappa),
//     Thi = s_hi - |q~|^2 + 2.1 kappa (|q~|^2 + s_hi) + tiny
// and the factors on |a~|^2 cover them all, each rounded outward; Tlo is the
// mirror image with s_lo.
// Measured distance error against binary64 (rms over pairs at eps, in units
// of the data; the vector norm form these joins took before in brackets):
// uniform 8-D 4.7e-8 (1.3e-7), uniform 16-D 8.8e-8 (3.5e-7), mixture 14-D
// 1.4e-7 (3.2e-7), exponential 16-D 1.52e-9 (1.62e-9).  Where the joins took the
// vector difference form (uniform 64-D 6.2e-7, here 5.5e-7; mixture 90-D
// 4.3e-7, here 7.4e-7) no pair is accepted on this estimate: what the FP32 sum
// used to accept is now decided in FP64.
// Measured joins, vector forms before and this: uniform 2M x 16 at S_D 64 505
// and 101 ms, exponential 2M x 16 at eps 0.03 151 and 30 ms, mixture 515k x 90
// 253 and 14.5 ms, mixture 301k x 37 in result batches 177 and 10 ms.  A large
// product of FP16 operands reaches about 1.3 PFLOP/s on this card (power), so the
// leading products of the 2M x 16 join (0.43 of 2e12 pairs after the box test, 28
// TFLOP) would take 21 ms.  Vector issue is 0.38 there and the matrix units are busy
// 0.14 of the time: two waves per SIMD wait for gathered rows and LDS.
//
// Candidates reach a tile only after a test against all of the unit's queries
// at once (a bound on the distance, so no pair is lost):
//   up to 24 padded dimensions, the distance from the bounding box of the
//   queries over the first 8 dimensions (k_join_box);
//   above, the distance from the centres of groups of queries in a projection,
//   itself a matrix product (k_join_fp32_mxg).
#include "sj_mx32.hpp"

#include <algorithm>
#include <cmath>

#include "sj_launch.hpp"
#include "sj_tile.hpp"

namespace sj {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int FMT>
struct Mat;
template <>
struct Mat<kFmtF16> {
  typedef half8 V8;
  __device__ static float16v mfma(half8 a, half8 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mat<kFmtBF16> {
  typedef bf16x8 V8;
  __device__ static float16v mfma(bf16x8 a, bf16x8 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
__device__ __forceinline__ float16v mfma(half8 a, half8 b, float16v c) {
  return Mat<kFmtF16>::mfma(a, b, c);
}

// x = a + b up to 2^-22 |x| + 2^-25
__device__ __forceinline__ void split2(float x, _Float16 &a, _Float16 &b) {
  a = (_Float16)x;
  b = (_Float16)(x - (float)a);
}

// ---------------------------------------------------------------------------
// Index build: the candidates' split rows [x1 | x2] of 2 K FP16 numbers, eight
// consecutive ones of a part per thread, rows n .. n_pad - 1 zero.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_mx32_split(const float *__restrict__ X, uint64_t n,
                                                       uint64_t n_pad, uint32_t dp, uint32_t K,
                                                       const float *__restrict__ ctr, float sc,
                                                       half8 *__restrict__ XS) {
  const uint32_t kv = K / 8;  // vectors of one part
  const uint64_t total = n_pad * kv;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t p = e / kv;
    const uint32_t v = (uint32_t)(e - p * kv), t0 = v * 8;
    half8 a = {}, b = {};
    if (p < n && t0 < dp) {  // dp is a multiple of 8
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        _Float16 s1, s2;
        split2(sc * (X[p * dp + t0 + i] - ctr[t0 + i]), s1, s2);
        a[i] = s1;
        b[i] = s2;
      }
    }
    half8 *dst = XS + p * (2 * kv) + v;
    dst[0] = a;
    dst[kv] = b;
  }
}

// Per candidate nn, what a tile element must stay below to be a hit: the float
// above -|a~|^2 (1 - kappa) rounded up.  Rows n .. n_pad - 1 get -inf (never a hit).
__global__ __launch_bounds__(kBlock) void k_mx32_norms(const float *__restrict__ X, uint64_t n,
                                                       uint64_t n_pad, uint32_t dp,
                                                       const float *__restrict__ ctr, float sc,
                                                       double kappa,
                                                       float *__restrict__ nn) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n_pad) return;
  if (p >= n) {
    nn[p] = -__builtin_inff();
    return;
  }
  const f32x4 *x4 = reinterpret_cast<const f32x4 *>(X + p * dp);
  double s = 0.0;
  for (uint32_t t4 = 0; t4 < dp / 4; ++t4) {
    const f32x4 x = x4[t4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float y = sc * (x[i] - ctr[4 * t4 + i]);
      s += (double)y * (double)y;
    }
  }
  nn[p] = strict(round_up_f32(-s * (1.0 - kappa)));
}

// Projected rows y = 2^-4 V x~ in FP16 (|V x~| <= |x~| < 2^18), the reject value
// pn of the group test and the error radius ye of a query (see k_join_fp32_mxg).
// The directions are wave-uniform scalar loads; a lane holds one point's 32 sums.
constexpr double kEta = 0x1p-11 + 0x1p-13;
__global__ __launch_bounds__(kBlock) void k_mx32_project(
    const float *__restrict__ X, uint64_t n, uint64_t n_pad, uint32_t dp,
    const float *__restrict__ dirs, const float *__restrict__ ctr, float sc,
    half8 *__restrict__ ys, float *__restrict__ pn, float *__restrict__ ye) {
  const uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  float y[kMx32Dirs];
#pragma unroll
  for (uint32_t j = 0; j < kMx32Dirs; ++j) y[j] = 0.0f;
  double s = 0.0;
  for_row(X, n, dp, [&](uint32_t t, float xt) {
    const float x = p < n ? sc * (xt - ctr[t]) : 0.0f;
    s += (double)x * (double)x;
#pragma unroll
    for (uint32_t j = 0; j < kMx32Dirs; ++j)
      y[j] = __builtin_fmaf(x, dirs[t * kMx32Dirs + j], y[j]);
  });
  if (p >= n_pad) return;
  double s1 = 0.0;
#pragma unroll
  for (uint32_t g = 0; g < kMx32Dirs / 8; ++g) {
    half8 h;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h[i] = (_Float16)(0x1p-4f * y[8 * g + i]);
      s1 += (double)(float)h[i] * (double)(float)h[i];
    }
    ys[p * (kMx32Dirs / 8) + g] = h;
  }
  s *= 0x1p-8;
  pn[p] = p < n ? round_up_f32(-(s1 * (1.0 - 0x1p-13) - s * (kEta + kEta * kEta)))
                : -__builtin_inff();
  ye[p] = round_up_f32(__builtin_sqrt(s) * kEta * (1.0 + 0x1p-20));
}

// The first 8 dimensions of the cell-ordered rows as two planes of 16-byte
// vectors, so that the box test's loads are contiguous across the lanes: read
// from the rows themselves every lane touched a cache line of its own, twice,
// and the vector cache (busy 62 % of the 2M x 16 FP32 join) set the pace.
__global__ __launch_bounds__(kBlock) void k_box_rows(const float *__restrict__ X, uint64_t n,
                                                     uint32_t dp, f32x4 *__restrict__ box0,
                                                     f32x4 *__restrict__ box1) {
  for (uint64_t p = (uint64_t)blockIdx.x * kBlock + threadIdx.x; p < n;
       p += (uint64_t)gridDim.x * kBlock) {
    const f32x4 *x = reinterpret_cast<const f32x4 *>(X + p * dp);
    box0[p] = x[0];
    box1[p] = x[1];
  }
}

// ---------------------------------------------------------------------------
// Shared by the join kernels
// ---------------------------------------------------------------------------
// One query row's slice of 16 dimensions (8 per half-wave): centred, scaled by
// -2 sc (exact) and split; *n += its part of |q~|^2.
__device__ __forceinline__ void query_slice(const float *__restrict__ row, const Mx32View &v,
                                            uint32_t t0, bool live, half8 &a1, half8 &a2,
                                            double &n) {
  f32x4 x[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  if (live && t0 < v.m.dp) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      x[h] = (*reinterpret_cast<const f32x4 *>(row + t0 + 4 * h) -
              *reinterpret_cast<const f32x4 *>(v.ctr + t0 + 4 * h)) *
             v.sc;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float y = x[i / 4][i % 4];
    n += (double)y * (double)y;
    _Float16 s1, s2;
    split2(-2.0f * y, s1, s2);
    a1[i] = s1;
    a2[i] = s2;
  }
}

// -Thi of the leading product; -Thi and Thi - Tlo of a query with |q~|^2 = n
__device__ __forceinline__ float lead_bound(const Mx32View &v, double lead_kappa, double n) {
  return -round_up_f32(v.s_hi - n + 2.1 * lead_kappa * (n + v.s_hi) + v.tiny);
}
__device__ __forceinline__ void query_bounds(const Mx32View &v, double n, float &cinit,
                                             float &delta) {
  const double k2 = 2.1 * v.kappa;
  const float thi = round_up_f32(v.s_hi - n + k2 * (n + v.s_hi) + v.tiny);
  const double tlo = v.s_lo - n - k2 * (n + v.s_lo) - v.tiny;
  cinit = -thi;
  delta = round_up_f32((double)thi - tlo);
}

// ---------------------------------------------------------------------------
// Candidates tested against the query box: one wave per work unit of 32 QB
// queries (or per part of one), no barriers.  Also the form of the 16-bit
// filters' workgroup units at low selectivity (PARTS = 1: one product of 16-bit
// operands prepared by the index, thresholds of k_mfma_thresholds).  The wave
// alternates two phases.  In the first it tests windows of 64 candidates
// against the box of its queries (vector ALU; four windows in flight) until
// kBatch survivors' positions wait in a ring in LDS; in the second it gathers
// the rows of 32 of them at a time (through LDS into the B operands), in flight
// during the tiles of the two blocks before them.  Long phases let the two
// waves of a SIMD be in different ones: with a test between any two blocks both
// units idled most of the time.  A gathered block serves as many query blocks
// as the registers of two waves per SIMD hold: 8 with one product (4 at K 32),
// 4 with three (2 at K 32).
//
// With one product bound by instruction issue (0.68 of the vector ALU's at 2M x 16
// FP16): 8 minima per tile, 27 instructions per 64 candidates tested.  Measured,
// whole pass of the 2M x 16 uniform join at 64 neighbours: FP16 105 ms with
// workgroups of four waves, candidates as rows and a product's minima right
// behind it, 77 ms with one wave per workgroup and queries as rows, 69 ms with
// products issued ahead; FP32 141 to 130 ms.  With kLead an FP32 tile is the leading
// product alone, and the second parts (queries' in LDS, candidates' in the gathered
// rows) come in for the tiles that pass: the registers then hold 8 query blocks (4 at
// K 32), and half as many candidates are tested and gathered: the join kernels of
// 2M x 16 uniform 124 to 105 ms, 2M x 16 exponential at eps 0.03 41 to 31 ms, 400k x
// 20 uniform 22.6 to 14.5 ms.  (With 4 query blocks the leading product alone gave
// nothing: 122 to 121 ms; nor did rows further ahead: 3, 4 and 6 blocks 123, 128
// and 133 ms.)
// ---------------------------------------------------------------------------
constexpr int kBoxDims = 8;
constexpr uint32_t kBatch = 512;
constexpr int kWindows = 4;
constexpr uint32_t kRingW = 1024;  // >= kBatch - 1 pending + 2 kWindows windows of 64

template <int FMT, int PARTS, int K, int QB, bool kLead>
__global__ __launch_bounds__(kWave) void k_join_box(Mx32View v, const WorkUnit *__restrict__ wus,
                                                     uint32_t parts_per_unit,
                                                     uint64_t *__restrict__ out, uint64_t capacity,
                                                     unsigned long long *__restrict__ cursor) {
  typedef typename Mat<FMT>::V8 V8;
  constexpr int KS = K / 16;
  constexpr int RV = PARTS * (K / 8);  // 16-byte vectors per candidate row
  constexpr bool kTwo = PARTS == 2 && K > 16;  // a second accumulator for the small products
  constexpr bool kAccept = PARTS == 1 || K <= 16;
  static_assert(PARTS == 2 || !kLead, "a second part to leave out");
  // kLead: 20 KB in all, so that a CU holds eight waves
  constexpr int kStageN = kLead ? 256 : kStage, kBandN = kLead ? 96 : kBandStage;
  __shared__ uint64_t stage_mem[kAccept ? kStageN : 1];
  __shared__ uint64_t band_mem[kBandN];
  __shared__ __align__(16) uint32_t ring_mem[kRingW];
  __shared__ float ring_n_mem[kLead ? 1 : kRingW];
  __shared__ V8 a2_mem[kLead ? QB * KS * kWave : 1];
  __shared__ float box_mem[kLead ? 2 * kBoxDims : 1];
  static_assert(!kLead || kRingW >= QB * 32, "the ring holds the leading thresholds at first");
  __shared__ V8 rows_mem[32 * RV];
  __shared__ __align__(16) float cinit_mem[QB * 32];
  __shared__ __align__(16) float delta_mem[QB * 32];
  __shared__ uint32_t qpos_mem[QB * 32];
  const MfmaView &m = v.m;
  WorkUnit wu = wus[blockIdx.x / parts_per_unit];
  wu.q0 += (blockIdx.x % parts_per_unit) * (32u * QB);
  if (wu.q0 >= wu.q1) return;
  if (wu.q1 - wu.q0 > 32u * QB) wu.q1 = wu.q0 + 32u * QB;
  const uint32_t l = lane_id();
  const uint32_t half = l >> 5, col = l & 31;
  const uint32_t dp = m.dp;
  const uint32_t nq = wu.q1 - wu.q0;  // 1 .. 32 QB
  uint32_t *ring = ring_mem;
  float *ring_n = ring_n_mem;

  V8 A1[QB][KS], A2[PARTS == 2 && !kLead ? QB : 1][KS];
  float *const lead_mem = reinterpret_cast<float *>(ring_mem);
  float blo[kBoxDims], bhi[kBoxDims];
#pragma unroll
  for (int t = 0; t < kBoxDims; ++t) {
    blo[t] = __builtin_inff();
    bhi[t] = -__builtin_inff();
  }
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const uint32_t idx = (uint32_t)j * 32 + col;
    const bool live = idx < nq;
    const uint32_t slot = wu.q0 + idx;
    const uint32_t p = live ? (m.qlist ? m.qlist[slot] : slot) : 0u;
    const float *row = m.Xq + (uint64_t)p * dp;
    float ci, de, li = 0.0f;
    if constexpr (PARTS == 2) {
      double n = 0.0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        V8 second;
        query_slice(row, v, (uint32_t)ks * 16 + half * 8, live, A1[j][ks], second, n);
        if constexpr (kLead) a2_mem[(j * KS + ks) * kWave + l] = second;
        else A2[j][ks] = second;
      }
      n += __shfl_xor(n, 32);
      query_bounds(v, n, ci, de);
      if (kLead) li = lead_bound(v, v.lead_kappa, n);
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        A1[j][ks] = static_cast<const V8 *>(m.XB)[(uint64_t)p * RV + ks * 2 + half];
      ci = -m.thi[p];
      de = round_up_f32((double)m.thi[p] - (double)m.tlo[p]);
    }
    if (half == 0) {
      cinit_mem[idx] = live ? ci : __builtin_inff();
      if (kLead) lead_mem[idx] = live ? li : __builtin_inff();
      delta_mem[idx] = live ? de : 0.0f;
      qpos_mem[idx] = live ? p : 0xffffffffu;
    }
#pragma unroll
    for (int t4 = 0; t4 < kBoxDims / 4; ++t4) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(row + 4 * t4);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (live) {
          blo[4 * t4 + i] = __builtin_fminf(blo[4 * t4 + i], x[i]);
          bhi[4 * t4 + i] = __builtin_fmaxf(bhi[4 * t4 + i], x[i]);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < kBoxDims; ++t) {
    float a = blo[t], b = bhi[t];
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
      a = __builtin_fminf(a, __shfl_xor(a, off));
      b = __builtin_fmaxf(b, __shfl_xor(b, off));
    }
    // (kept in vector registers: an instruction reads one scalar register; with
    // kLead they are read again from LDS ahead of each test phase)
    blo[t] = a;
    bhi[t] = b;
    if (kLead && l == 0) {
      box_mem[t] = a;
      box_mem[kBoxDims + t] = b;
    }
  }
  __builtin_amdgcn_wave_barrier();
  float16v c0[QB];
#pragma unroll
  for (int j = 0; j < QB; ++j) c0[j] = rows_init(&(kLead ? lead_mem : cinit_mem)[j * 32], half);

  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the ring follows in the same memory
  Stage st{&stage_mem[0], 0u, kStageN};
  BandSink bs{m.band, m.band_cap, m.band_cursor, Stage{&band_mem[0], 0u, kBandN}};
  uint64_t n_skip = 0;
  const KeyForm kf{m.key_hi, m.pshift, m.symmetric != 0};

  // candidate windows of up to 64 positions of one run
  uint32_t r = wu.run_first, c = wu.c_begin;
  uint32_t ce = (r == wu.run_last) ? wu.c_end : scalar_run(m.runs, r).y;
  auto normalise = [&]() {
    while (c >= ce && r < wu.run_last) {
      const uint2 run = scalar_run(m.runs, ++r);
      c = run.x;
      ce = (r == wu.run_last) ? wu.c_end : run.y;
    }
  };
  normalise();
  struct Window {
    uint32_t c, n;  // first position, length (0: the stream is done)
    f32x4 x0, x1;   // this lane's candidate: its first 8 dimensions
    float nn;       // and its reject value (kLead: read with the rows)
  };
  auto load_window = [&](Window &x) __attribute__((always_inline)) {
    x.n = c < ce ? (ce - c < (uint32_t)kWave ? ce - c : (uint32_t)kWave) : 0u;
    x.c = x.n ? c : 0u;
    const uint32_t p = x.c + (l < x.n ? l : 0u);
    x.x0 = reinterpret_cast<const f32x4 *>(m.box0)[p];
    x.x1 = reinterpret_cast<const f32x4 *>(m.box1)[p];
    if (!kLead) x.nn = v.nn[p];
    c += x.n;
    normalise();
  };
  uint32_t head = 0, cnt = 0;  // ring (wave-uniform)
  auto test_window = [&](const Window &x) __attribute__((always_inline)) {
    float lb = 0.0f;
#pragma unroll
    for (int t = 0; t < kBoxDims; ++t) {
      // y - clamp(y): the gap up to its sign, in three instructions a dimension
      const float y = t < 4 ? x.x0[t & 3] : x.x1[t & 3];
      const float g = y - __builtin_amdgcn_fmed3f(y, blo[t], bhi[t]);
      lb = __builtin_fmaf(g, g, lb);
    }
    const uint64_t valid = x.n < (uint32_t)kWave ? (1ull << x.n) - 1ull : ~0ull;
    uint64_t km = ballot(lb <= m.hi) & valid;
    if (v.skip_below) {
      // candidates of earlier result batches: their pairs were taken there
      const uint64_t early =
          ballot(v.orig_id[x.c + (l < x.n ? l : 0u)] < v.skip_below) & valid;
      n_skip += (uint64_t)__builtin_popcountll(early) * nq;
      km &= ~early;
    }
    if ((km >> l) & 1ull) {
      const uint32_t at = (head + cnt + lanes_below(km)) % kRingW;
      ring[at] = x.c + l;
      if (!kLead) ring_n[at] = x.nn;
    }
    cnt += (uint32_t)__builtin_popcountll(km);
  };
  const V8 *__restrict__ XS = static_cast<const V8 *>(v.XS);
  // The next nb <= 32 survivors on their way to the operands: adjacent lanes
  // load the 16-byte vectors of one row, so a row costs one or two cache
  // accesses, and the wave's LDS turns rows into operands.  The vectors of a row
  // are permuted (by the low bits of the row) against bank conflicts.  The
  // loads are unconditional (ahead of the ring they repeat old entries): under
  // a branch the compiler copies their results at its end, and so waits for
  // them there.
  constexpr int RT = RV / 2;  // vectors per lane
  constexpr uint32_t kSwz = RV < 8 ? RV - 1 : 7;
  struct Rows {
    V8 x[RT];
    float nn;     // kLead: reject value of this column's candidate
    uint32_t at;  // first ring entry
  };
  auto load_rows = [&](Rows &q) __attribute__((always_inline)) {
    q.at = head;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const uint32_t e = (uint32_t)i * kWave + l, row = e / RV;
      const uint32_t pos = ring[(head + row) % kRingW];
      q.x[i] = XS[(uint64_t)pos * RV + ((e % RV) ^ (row & kSwz))];
    }
    if (kLead) q.nn = v.nn[ring[(head + col) % kRingW]];
    head += 32;
    __builtin_amdgcn_sched_barrier(0);  // issued here, ahead of the tiles
  };
  struct Block {
    V8 b[kLead ? 1 : PARTS][KS];
    float an;
    uint32_t cp;
  };
  auto to_block = [&](const Rows &q, Block &b) __attribute__((always_inline)) {
    V8 *t = rows_mem;
#pragma unroll
    for (int i = 0; i < RT; ++i) t[(uint32_t)i * kWave + l] = q.x[i];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < (kLead ? 1 : PARTS); ++i)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        b.b[i][ks] = t[col * RV + (((uint32_t)(i * (K / 8) + 2 * ks) + half) ^ (col & kSwz))];
    const uint32_t at = (q.at + col) % kRingW;
    b.an = kLead ? q.nn : ring_n[at];
    b.cp = ring[at];
    __builtin_amdgcn_wave_barrier();
  };
  // tile j of a block from the leading parts alone
  auto lead = [&](int j, const Block &cur) __attribute__((always_inline)) {
    float16v acc = c0[j];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) acc = Mat<FMT>::mfma(A1[j][ks], cur.b[0][ks], acc);
    return acc;
  };
  // and from all products
  auto product = [&](int j, const Block &cur) __attribute__((always_inline)) {
    float16v acc = kLead ? rows_init(&cinit_mem[j * 32], half) : c0[j];
    // (kLead: the second parts wait in LDS, the block's rows until the next block's)
    auto a2 = [&](int ks) {
      if constexpr (kLead) return a2_mem[(j * KS + ks) * kWave + l];
      else return A2[j][ks];
    };
    auto b2 = [&](int ks) {
      if constexpr (kLead)
        return rows_mem[col * RV + (((uint32_t)(K / 8 + 2 * ks) + half) ^ (col & kSwz))];
      else return cur.b[PARTS - 1][ks];
    };
    if constexpr (PARTS == 1) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = Mat<FMT>::mfma(A1[j][ks], cur.b[0][ks], acc);
    } else if constexpr (kTwo) {
      float16v lo;
#pragma unroll
      for (int e = 0; e < 16; ++e) lo[e] = 0.0f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        lo = Mat<FMT>::mfma(A1[j][ks], b2(ks), lo);
        acc = Mat<FMT>::mfma(A1[j][ks], cur.b[0][ks], acc);
        lo = Mat<FMT>::mfma(a2(ks), cur.b[0][ks], lo);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] += lo[e];
    } else {
      acc = Mat<FMT>::mfma(A1[j][0], b2(0), acc);
      acc = Mat<FMT>::mfma(a2(0), cur.b[0][0], acc);
      acc = Mat<FMT>::mfma(A1[j][0], cur.b[0][0], acc);
    }
    return acc;
  };
  // The tiles of a block: products and minima without a branch, so that they
  // overlap; a tile with a hit is computed again for its masks.  With kLead the
  // first look is at the leading product, whose bound is wider by 2^-10 of the
  // norms, and only tiles that pass take the other two.
  auto first_look = [&](int j, const Block &cur) __attribute__((always_inline)) {
    if constexpr (kLead) return lead(j, cur);
    else return product(j, cur);
  };
  auto tiles = [&](const Block &cur) __attribute__((always_inline)) {
    Min16 mn[QB];
    float least = __builtin_inff();
    const float an1 = kLead ? __builtin_fmaxf(cur.an * v.widen, cur.an) : cur.an;
    float16v acc = first_look(0, cur);
#pragma unroll
    for (int j = 0; j < QB; ++j) {
      float16v next = acc;
      if (j + 1 < QB) next = first_look(j + 1, cur);
      __builtin_amdgcn_sched_barrier(0);  // the next product runs under these minima
      mn[j] = min16(acc);
      least = __builtin_fminf(__builtin_fminf(least, mn[j].a), mn[j].b);
      acc = next;
    }
    if (ballot(least < an1) == 0) return;
    const float nacc =
        PARTS == 1 ? cur.an : (cur.an < 0.0f ? cur.an * v.kacc : -__builtin_inff());
#pragma unroll
    for (int j0 = 0; j0 < QB; j0 += 4) {
      uint64_t hits = 0, within = 0;
#pragma unroll
      for (int j = j0; j < QB && j < j0 + 4; ++j) {
        if (ballot(__builtin_fminf(mn[j].a, mn[j].b) < an1) == 0) continue;
        uint32_t h, a;
        tile_masks<kAccept>(product(j, cur), cur.an, nacc, &delta_mem[j * 32], half, h, a);
        hits |= (uint64_t)h << (16 * (j - j0));
        within |= (uint64_t)a << (16 * (j - j0));
      }
      emit_hits<kAccept>(hits, within, &qpos_mem[j0 * 32], half, cur.cp, PARTS == 1 ? cur.an : 0.0f, kf,
                         st, bs, out, capacity, cursor);
    }
  };

  for (uint32_t i = l; i < kRingW; i += kWave) ring[i] = m.pad_row;
  __builtin_amdgcn_wave_barrier();
  while (cnt || c < ce) {
    {
      // test phase: kWindows windows in flight, all tested before it ends
      if (kLead) {
#pragma unroll
        for (int t = 0; t < kBoxDims; ++t) {
          blo[t] = box_mem[t];
          bhi[t] = box_mem[kBoxDims + t];
        }
      }
      Window x[kWindows];
#pragma unroll
      for (int i = 0; i < kWindows; ++i) load_window(x[i]);
      while (cnt < kBatch && c < ce) {
#pragma unroll
        for (int i = 0; i < kWindows; ++i) {
          test_window(x[i]);
          load_window(x[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < kWindows; ++i) test_window(x[i]);
    }
    if (c >= ce && cnt % 32) {  // the stream is done: fill up the last block
      const uint32_t pad = 32u - cnt % 32;
      if (l < pad) {
        const uint32_t at = (head + cnt + l) % kRingW;
        ring[at] = m.pad_row;
        if (!kLead) ring_n[at] = -__builtin_inff();  // (as the padding row's)
      }
      cnt += pad;
    }
    __builtin_amdgcn_wave_barrier();
    // tile phase: the rows of two blocks in flight behind the current one
    if (cnt >= 32) {
      uint32_t nb = cnt / 32;
      cnt %= 32;
      Rows r0, r1;
      Block blk;
      const uint32_t end = head + 32 * nb;
      load_rows(r0);
      load_rows(r1);
      for (;;) {
        to_block(r0, blk);
        load_rows(r0);
        tiles(blk);
        if (--nb == 0) break;
        to_block(r1, blk);
        load_rows(r1);
        tiles(blk);
        if (--nb == 0) break;
      }
      head = end;
    }
    __builtin_amdgcn_wave_barrier();
  }
  flush(bs.st, bs.buf, bs.cap, bs.cursor);
  if constexpr (kAccept) flush(st, out, capacity, cursor);
  if (l == 0 && n_skip) atomicAdd(v.skipped, (unsigned long long)n_skip);
}

// ---------------------------------------------------------------------------
// Above 24 padded dimensions: one workgroup per work unit of 256 queries.
//
// Group test.  Points are projected on 32 orthonormal directions that span the
// pivots' means (y1 = 2^-4 V x~ in FP16): clusters stay as far apart as they are
// while the scatter inside them falls to its share of 32 dimensions, and the test
// reads 64 bytes per candidate.  The queries form up to 32 groups of consecutive
// ones with the same nearest pivot; c_g is the mean of a group's y1 rounded to
// FP16.  With eta = 2^-11 + 2^-13 (the FP16 rounding, the FP32 sums of up to 128
// terms, sqrt(32) 130 2^-24, the directions' and the centring's rounding), A =
// 2^-4 |a~| and tiny = 2^-20 (FP16 subnormals), |y1(a) - 2^-4 V a~| <= eta A +
// tiny / 2, likewise for a query, and a pair within eps has |V (q~ - a~)| <=
// |q~ - a~| <= R = sqrt(s_hi) (1 + 2^-16).  Hence with r_g the largest
// |y1(q) - c_g| + eta 2^-4 |q~| of a group and x = 2^-4 R + r_g + tiny
//     |y1(a)|^2 + |c_g|^2 - 2 c_g . y1(a) <= (x + eta A)^2
//                                         <= x^2 (1 + eta) + A^2 (eta + eta^2).
// One 32x32 tile tests 32 candidates against all groups: the rows start from
// -T_g, and candidates above pn in every row are dropped.  Margins of 2^-13 on
// both sides cover the FP32 accumulation (gamma_34(2^-23) < 2^-17) and the
// rounding of T_g.
// Against the leading parts of the whole rows, as before, groups of one cluster
// still passed a quarter of the other clusters' points of the 515k x 90 mixture
// (|a - c|^2 about 18 against (R + r)^2 = 16), and the test was bound by reading
// rows of 192 bytes that the caches hold only in part.  The join of that set took
// 50.1 ms then, 37.7 with the projected test and 14.5 with picked pivots (36, 36
// and 7 % of the tests passed); now the tests alone take 7.9 ms, bound by
// instruction issue (two products, 8 minima and 4 LDS reads per 32 candidates).
//
// Survivors' positions enter a ring in LDS; chunks of CH of them are staged,
// split rows and all, into a double-buffered LDS tile that every wave reads.
// ---------------------------------------------------------------------------
constexpr uint32_t kRing = 2048;  // >= 63 pending + one window of up to 1024
constexpr int kTestBlocks = 4;    // blocks of 32 candidates that a wave tests at a time

// Tile shapes by K (dimensions padded to 16): waves per workgroup, query row
// blocks per wave and candidate columns per staged chunk.  Two blocks per wave
// halve the LDS reads per product (uniform 400k x 64 27.5 to 22.9 ms, exponential
// 500k x 45 32.5 to 24.9); above K 64 their registers leave too few waves (515k x
// 90 14.7 to 19.3).
template <int K>
struct Shape {
  static constexpr int NW = K <= 64 ? 4 : 8;
  static constexpr int QB = K <= 64 ? 2 : 1;
  static constexpr int CH = K <= 48 ? 64 : 32;
};

// group lengths tried (the last takes all queries of a pivot)
constexpr int kGroupLens = 6;
__device__ constexpr uint32_t kGroupLen[kGroupLens] = {8, 9, 11, 14, 20, 256};

template <int K>
__global__ __launch_bounds__(Shape<K>::NW * kWave) void k_join_fp32_mxg(
    Mx32View v, const WorkUnit *__restrict__ wus) {
  constexpr int NW = Shape<K>::NW, QB = Shape<K>::QB, CH = Shape<K>::CH;
  constexpr int NT = NW * kWave;    // threads
  constexpr int TQ = NW * QB * 32;  // query rows
  constexpr int KS = K / 16;
  constexpr int RV = 2 * (K / 8);     // 16-byte vectors per split row
  constexpr int RS = RV + 1;          // and per staged row (odd: no bank conflicts)
  constexpr int PER_THREAD = (CH * RV + NT - 1) / NT;
  constexpr uint32_t WIN = NW * 32 * kTestBlocks;  // candidates tested at a time
  constexpr int KT = kMx32Dirs / 16;
  static_assert(TQ == 256, "units hold 256 queries in 32 groups");
  static_assert(RV % 2 == 0, "the padded stride is odd");
  __shared__ uint64_t band_mem[NW][kBandStage];
  __shared__ half8 tile[2][CH * RS];
  __shared__ float tile_n[2][CH];
  __shared__ uint32_t tile_pos[2][CH];
  __shared__ uint32_t ring[kRing];
  __shared__ __align__(16) float cinit[TQ];  // -Thi of each query row
  __shared__ __align__(16) float linit[TQ];  // and that of the leading product
  __shared__ uint32_t qpos_s[TQ];
  __shared__ __align__(16) float ginit[32];  // -T_g
  __shared__ __align__(16) _Float16 gctr[32][kMx32Dirs];
  __shared__ uint32_t wcnt[NW];
  __shared__ uint64_t seg_mask[TQ / kWave];
  __shared__ uint32_t len_cnt[kGroupLens][TQ / kWave];
  __shared__ uint32_t gfirst[33];  // the groups' first queries, then nq
  const MfmaView &m = v.m;
  const WorkUnit wu = wus[blockIdx.x];
  const uint32_t tid = threadIdx.x;
  const uint32_t w = uniform_u32(tid / kWave);
  const uint32_t l = lane_id();
  const uint32_t half = l >> 5, col = l & 31;
  const uint32_t dp = m.dp;
  const uint32_t nq = wu.q1 - wu.q0;  // 1 .. TQ

  // query rows: split operands of -2 q~ and thresholds
  half8 A1[QB][KS], A2[QB][KS];
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const uint32_t idx = (w * QB + (uint32_t)j) * 32 + col;
    const bool live = idx < nq;
    const uint32_t slot = wu.q0 + idx;
    const uint32_t p = live ? (m.qlist ? m.qlist[slot] : slot) : 0u;
    const float *row = m.Xq + (uint64_t)p * dp;
    double n = 0.0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      query_slice(row, v, (uint32_t)ks * 16 + half * 8, live, A1[j][ks], A2[j][ks], n);
    n += __shfl_xor(n, 32);
    if (half == 0) {
      float ci, de;
      query_bounds(v, n, ci, de);
      cinit[idx] = live ? ci : __builtin_inff();
      linit[idx] = live ? lead_bound(v, v.lead_kappa, n) : __builtin_inff();
      qpos_s[idx] = live ? p : 0xffffffffu;
    }
  }
  __syncthreads();
  // groups: runs of up to L queries of one pivot, L the least of kGroupLen for
  // which 32 groups suffice (or eight each, where even 32 pivots do not)
  {
    const uint32_t idx = tid < (uint32_t)TQ ? tid : TQ - 1u;
    const bool live = tid < nq;  // nq <= TQ <= NT
    auto pivot = [&](uint32_t i) { return v.pid ? v.pid[qpos_s[i]] : (uint8_t)0; };
    const bool cut = live && (idx == 0 || pivot(idx) != pivot(idx - 1));
    const uint64_t cuts = ballot(cut);
    if (l == 0 && w < TQ / kWave) seg_mask[w] = cuts;
    __syncthreads();
    uint32_t seg = 0;  // first query of this one's pivot
    if (live) {
      uint32_t i = idx / kWave;
      uint64_t mask = seg_mask[i] & (~0ull >> (63 - idx % kWave));
      while (!mask) mask = seg_mask[--i];  // (query 0 is a cut)
      seg = i * kWave + 63u - (uint32_t)__builtin_clzll(mask);
    }
    uint32_t starts = 0;  // bit j: a group of length kGroupLen[j] starts here
#pragma unroll
    for (int j = 0; j < kGroupLens; ++j) {
      const bool at = live && (idx - seg) % kGroupLen[j] == 0;
      starts |= at ? 1u << j : 0u;
      const uint64_t m64 = ballot(at);
      if (l == 0 && w < TQ / kWave) len_cnt[j][w] = (uint32_t)__builtin_popcountll(m64);
    }
    __syncthreads();
    int pick = -1;
#pragma unroll
    for (int j = kGroupLens - 1; j >= 0; --j) {
      uint32_t total = 0;
#pragma unroll
      for (uint32_t i = 0; i < TQ / kWave; ++i) total += len_cnt[j][i];
      if (total <= 32) pick = j;
    }
    const bool first = live && (pick < 0 ? idx % 8 == 0 : (starts >> pick & 1u) != 0);
    const uint64_t fm = ballot(first);
    if (l == 0 && w < TQ / kWave) wcnt[w] = (uint32_t)__builtin_popcountll(fm);
    if (tid < 33) gfirst[tid] = nq;
    __syncthreads();
    if (first) {
      uint32_t g = lanes_below(fm);
      for (uint32_t i = 0; i < w; ++i) g += wcnt[i];
      gfirst[g] = idx;
    }
    __syncthreads();
  }
  // NT / 32 threads per group: its centre, each over every NT/32-th direction,
  // then its radius, each over every NT/32-th query
  {
    constexpr uint32_t TG = NT / 32;
    const uint32_t g = tid / TG, i0 = tid % TG;
    const uint32_t a = gfirst[g], gn = gfirst[g + 1] - a;
    const _Float16 *__restrict__ yq = static_cast<const _Float16 *>(v.yq);
    double nc = 0.0;
    for (uint32_t t = i0; t < kMx32Dirs; t += TG) {
      float sum = 0.0f;
      for (uint32_t i = 0; i < gn; ++i) sum += (float)yq[(uint64_t)qpos_s[a + i] * kMx32Dirs + t];
      const float cf = (float)(_Float16)(gn ? sum / (float)gn : 0.0f);
      gctr[g][t] = (_Float16)(-2.0f * cf);  // exact
      nc += (double)cf * (double)cf;
    }
    __syncthreads();
    double r = 0.0;
    for (uint32_t i = i0; i < gn; i += TG) {
      const uint32_t p = qpos_s[a + i];
      double d2 = 0.0;
      for (uint32_t t = 0; t < kMx32Dirs; ++t) {
        const double e = (double)(float)yq[(uint64_t)p * kMx32Dirs + t] +
                         0.5 * (double)(float)gctr[g][t];
        d2 += e * e;
      }
      const double x = __builtin_sqrt(d2) * (1.0 + 0x1p-40) + (double)v.ye[p];
      r = x > r ? x : r;
    }
#pragma unroll
    for (uint32_t off = TG / 2; off > 0; off >>= 1) {
      nc += __shfl_xor(nc, off);
      const double o = __shfl_xor(r, off);
      r = o > r ? o : r;
    }
    if (i0 == 0) {
      const double x = __builtin_sqrt(v.s_hi) * (0x1p-4 * (1.0 + 0x1p-16)) + r + 0x1p-20;
      const double T = x * x * (1.0 + kEta) + 0x1p-13 * (x * x + 2.0 * nc) - nc;
      ginit[g] = gn ? -round_up_f32(T) : __builtin_inff();
    }
  }
  __syncthreads();
  half8 G[KT];
#pragma unroll
  for (int ks = 0; ks < KT; ++ks)
    G[ks] = *reinterpret_cast<const half8 *>(&gctr[col][ks * 16 + half * 8]);
  float16v c0[QB];
#pragma unroll
  for (int j = 0; j < QB; ++j)
    c0[j] = rows_init(&(v.lead ? linit : cinit)[(w * QB + (uint32_t)j) * 32], half);

  Stage none{nullptr, 0u, 0u};
  BandSink bs{m.band, m.band_cap, m.band_cursor, Stage{&band_mem[w][0], 0u, kBandStage}};
  uint64_t n_skip = 0;
  const KeyForm kf{m.key_hi, m.pshift, m.symmetric != 0};
  const half8 *__restrict__ XS = static_cast<const half8 *>(v.XS);
  const half8 *__restrict__ YS = static_cast<const half8 *>(v.ys);

  // candidate stream (uniform over the workgroup) and the ring of survivors
  uint32_t r = wu.run_first, c = wu.c_begin;
  uint32_t ce = (r == wu.run_last) ? wu.c_end : scalar_run(m.runs, r).y;
  auto normalise = [&]() {
    while (c >= ce && r < wu.run_last) {
      const uint2 run = scalar_run(m.runs, ++r);
      c = run.x;
      ce = (r == wu.run_last) ? wu.c_end : run.y;
    }
  };
  normalise();
  uint32_t head = 0, tail = 0;  // ring positions (uniform)
  // test windows until at least CH survivors wait or the stream ends
  auto fill = [&]() __attribute__((always_inline)) {
    while (tail - head < (uint32_t)CH && c < ce) {
      const uint32_t wl = ce - c < WIN ? ce - c : WIN;
      const uint32_t first = w * (32u * kTestBlocks) + col;  // (both halves)
      half8 b[kTestBlocks][KT];
      float pnv[kTestBlocks];
#pragma unroll
      for (int i = 0; i < kTestBlocks; ++i) {
        const uint32_t ci = first + 32u * (uint32_t)i, p = c + (ci < wl ? ci : 0u);
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) b[i][ks] = YS[(uint64_t)p * (2 * KT) + 2 * ks + half];
        pnv[i] = v.pn[p];
      }
      uint32_t keep[kTestBlocks], mine = 0;
#pragma unroll
      for (int i = 0; i < kTestBlocks; ++i) {
        const uint32_t ci = first + 32u * (uint32_t)i;
        const bool valid = ci < wl;
        const bool early = v.skip_below && valid && v.orig_id[c + ci] < v.skip_below;
        float16v a = rows_init(ginit, half);
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) a = mfma(G[ks], b[i][ks], a);
        // a column passes when some row of either half does
        const uint64_t pm = ballot(min16(a, __builtin_inff()) <= pnv[i] && valid && !early);
        keep[i] = (uint32_t)pm | (uint32_t)(pm >> 32);
        mine += (uint32_t)__builtin_popcount(keep[i]);
        if (v.skip_below)  // earlier result batches took these pairs (halves agree)
          n_skip += (uint64_t)__builtin_popcount((uint32_t)ballot(early)) * nq;
      }
      if (l == 0) wcnt[w] = mine;
      __syncthreads();
      uint32_t before = 0, total = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const uint32_t k = wcnt[i];
        before += (uint32_t)i < w ? k : 0u;
        total += k;
      }
#pragma unroll
      for (int i = 0; i < kTestBlocks; ++i) {
        if (half == 0 && ((keep[i] >> col) & 1u))
          ring[(tail + before + (uint32_t)__builtin_popcount(keep[i] & ((1u << col) - 1u))) %
               kRing] = c + first + 32u * (uint32_t)i;
        before += (uint32_t)__builtin_popcount(keep[i]);
      }
      __syncthreads();  // the ring is read and wcnt rewritten after this
      tail += total;
      c += wl;
      normalise();
    }
  };
  half8 pre[PER_THREAD];
  uint32_t pre_p = 0;
  float pre_n = 0.0f;
  // rows [head, head + nr) of the ring into registers (padding rows past nr)
  auto gather = [&](uint32_t nr) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const uint32_t e = tid + (uint32_t)i * NT;
      if (e < (uint32_t)(CH * RV)) {
        const uint32_t rr = e / RV;
        const uint32_t pos = rr < nr ? ring[(head + rr) % kRing] : m.pad_row;
        pre[i] = XS[(uint64_t)pos * RV + e % RV];
      }
    }
    if (tid < (uint32_t)CH) {
      pre_p = tid < nr ? ring[(head + tid) % kRing] : m.pad_row;
      pre_n = v.nn[pre_p];
    }
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const uint32_t e = tid + (uint32_t)i * NT;
      if (e < (uint32_t)(CH * RV)) tile[buf][(e / RV) * RS + e % RV] = pre[i];
    }
    if (tid < (uint32_t)CH) {
      tile_pos[buf][tid] = pre_p;
      tile_n[buf][tid] = pre_n;
    }
  };

  fill();
  uint32_t ncur = tail - head < (uint32_t)CH ? tail - head : (uint32_t)CH;
  if (ncur) {
    gather(ncur);
    store(0);
    head += ncur;
    __syncthreads();
  }
  int cur = 0;
  while (ncur) {
    fill();
    const uint32_t nn = tail - head < (uint32_t)CH ? tail - head : (uint32_t)CH;
    if (nn) gather(nn);  // in flight during the tiles below
    if (w * QB * 32 < nq)  // (a wave without queries has no tiles)
#pragma nounroll
    for (int blk = 0; blk < CH / 32; ++blk) {
      if (ncur <= 32u * (uint32_t)blk) break;
      const half8 *brow = &tile[cur][(blk * 32 + col) * RS + half];
      const float an = tile_n[cur][blk * 32 + col];
      float16v acc[QB], lo[QB];
      if (v.lead) {  // the leading product first (see k_join_box)
        const float an1 = __builtin_fmaxf(an * v.widen, an);
        bool pass = false;
#pragma unroll
        for (int j = 0; j < QB; ++j) acc[j] = c0[j];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int j = 0; j < QB; ++j) acc[j] = mfma(A1[j][ks], brow[ks * 2], acc[j]);
#pragma unroll
        for (int j = 0; j < QB; ++j) pass |= min16(acc[j], __builtin_inff()) < an1;
        if (ballot(pass) == 0) continue;
      }
#pragma unroll
      for (int j = 0; j < QB; ++j) {
        acc[j] = v.lead ? rows_init(&cinit[(w * QB + (uint32_t)j) * 32], half) : c0[j];
#pragma unroll
        for (int e = 0; e < 16; ++e) lo[j][e] = 0.0f;
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const half8 b1 = brow[ks * 2], b2 = brow[K / 8 + ks * 2];
#pragma unroll
        for (int j = 0; j < QB; ++j) lo[j] = mfma(A1[j][ks], b2, lo[j]);
#pragma unroll
        for (int j = 0; j < QB; ++j) acc[j] = mfma(A1[j][ks], b1, acc[j]);
#pragma unroll
        for (int j = 0; j < QB; ++j) lo[j] = mfma(A2[j][ks], b1, lo[j]);
      }
#pragma unroll
      for (int j = 0; j < QB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] += lo[j][e];
      bool any = false;
#pragma unroll
      for (int j = 0; j < QB; ++j) any |= min16(acc[j], __builtin_inff()) < an;
      if (ballot(any)) {
        const uint32_t cp = tile_pos[cur][blk * 32 + col];
        uint32_t hits = 0;
#pragma unroll
        for (int j = 0; j < QB; ++j) {
          uint32_t h, a;
          tile_masks<false>(acc[j], an, 0.0f, nullptr, half, h, a);
          hits |= h << (16 * j);
        }
        emit_hits<false>(hits, 0u, &qpos_s[w * QB * 32], half, cp, 0.0f, kf, none, bs, nullptr, 0,
                         nullptr);
      }
    }
    if (!nn) break;
    store(cur ^ 1);
    head += nn;
    __syncthreads();
    cur ^= 1;
    ncur = nn;
  }
  flush(bs.st, bs.buf, bs.cap, bs.cursor);
  if (l == 0 && n_skip) atomicAdd(v.skipped, (unsigned long long)n_skip);
}

// query blocks per wave of k_join_box: FP32 at K = 16 and 32, 16 bits likewise
constexpr int kQbBox16 = 4, kQbBox32 = 2, kQbHalf16 = 8, kQbHalf32 = 4;
constexpr int kQbLead16 = 8, kQbLead32 = 4;  // FP32 with the leading product first: a unit

template <int FMT, int PARTS, int K, int QB, bool kLead = false>
void launch_box(const Mx32View &v, const WorkUnit *wu, uint64_t n_wu, uint32_t parts,
                uint64_t *out, uint64_t capacity, unsigned long long *cursor, hipStream_t s) {
  for_unit_launches(n_wu, parts * kWave, [&](uint64_t u, uint64_t m) {
    hipLaunchKernelGGL((k_join_box<FMT, PARTS, K, QB, kLead>), dim3((uint32_t)(m * parts)),
                       dim3(kWave), 0, s, v, wu + u, parts, out, capacity, cursor);
    SJ_HIP(hipGetLastError());
  });
}

template <int FMT>
void launch_half(const MfmaLaunch &a, const Mx32View &v, uint32_t tq, hipStream_t s) {
  if (a.kp == 16)
    launch_box<FMT, 1, 16, kQbHalf16>(v, a.wu, a.n_wu, tq / (32 * kQbHalf16), a.out, a.capacity,
                                      a.cursor, s);
  else
    launch_box<FMT, 1, 32, kQbHalf32>(v, a.wu, a.n_wu, tq / (32 * kQbHalf32), a.out, a.capacity,
                                      a.cursor, s);
}

template <int K>
void launch_g(const Mx32Launch &a, hipStream_t s) {
  for_unit_launches(a.n_wu, Shape<K>::NW * kWave, [&](uint64_t u, uint64_t m) {
    hipLaunchKernelGGL((k_join_fp32_mxg<K>), dim3((uint32_t)m), dim3(Shape<K>::NW * kWave), 0, s,
                       a.view, a.wu + u);
    SJ_HIP(hipGetLastError());
  });
}

}  // namespace

double mx32_kappa(uint32_t d) {
  const double k = (double)((d + 15) / 16 * 16);
  auto gamma = [](double n, double u) { return n * u / (1.0 - n * u); };
  // sequential adds of the chain that holds the large products: one chain of
  // all 3 K products at K = 16; above it the large products alone, and the
  // small ones (below 2^-10 of them, 2 K adds) in a chain of their own
  const double acc = k <= 16.0 ? gamma(3.0 * k + 2.0, std::ldexp(1.0, -23))
                               : 1.02 * gamma(k + 4.0, std::ldexp(1.0, -23));
  return 1.02 * (acc + 4.2 * std::ldexp(1.0, -24) + 2.0 * std::ldexp(1.0, -21));
}

// + what the leading product leaves out: 2 (|q||a| - q1 a1) <= (2^-10 + 2^-21)
// (|q|^2 + |a|^2)
double mx32_lead_kappa(uint32_t d) { return mx32_kappa(d) + 0x1p-10 * (1.0 + 0x1p-10); }

uint32_t mx32_k(uint32_t dp) { return (dp + 15) / 16 * 16; }

uint32_t mx32_queries(uint32_t dp) {
  return dp <= 16 ? 32u * kQbLead16 : dp <= 24 ? 32u * kQbLead32 : 256u;
}

uint32_t mx32_live_queries(uint32_t dp) {
  return dp <= 16 ? 32u * kQbBox16 : dp <= 24 ? 32u * kQbBox32 : 256u;
}

bool mx32_per_wave(uint32_t dp) { return dp <= 24; }

void launch_mx32_prep(const float *X, uint64_t n, uint64_t n_pad, uint32_t dp, const float *ctr,
                      float sc, double kappa, void *XS, float *nn, hipStream_t s) {
  if (!n_pad) return;
  const uint32_t K = mx32_k(dp);
  const uint64_t vecs = n_pad * (K / 8);
  hipLaunchKernelGGL(k_mx32_split,
                     dim3((uint32_t)std::min<uint64_t>((vecs + kBlock - 1) / kBlock, 1u << 20)),
                     dim3(kBlock), 0, s, X, n, n_pad, dp, K, ctr, sc,
                     static_cast<half8 *>(XS));
  SJ_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_mx32_norms, dim3((uint32_t)((n_pad + kBlock - 1) / kBlock)), dim3(kBlock),
                     0, s, X, n, n_pad, dp, ctr, sc, kappa, nn);
  SJ_HIP(hipGetLastError());
}

void launch_mx32_project(const float *X, uint64_t n, uint64_t n_pad, uint32_t dp,
                         const float *dirs, const float *ctr, float sc, void *ys, float *pn,
                         float *ye, hipStream_t s) {
  if (!n_pad) return;
  hipLaunchKernelGGL(k_mx32_project, dim3((uint32_t)((n_pad + kBlock - 1) / kBlock)), dim3(kBlock),
                     0, s, X, n, n_pad, dp, dirs, ctr, sc, static_cast<half8 *>(ys), pn, ye);
  SJ_HIP(hipGetLastError());
}

void launch_box_rows(const float *X, uint64_t n, uint32_t dp, void *box0, void *box1,
                     hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(k_box_rows,
                     dim3((uint32_t)std::min<uint64_t>((n + kBlock - 1) / kBlock, 1u << 20)),
                     dim3(kBlock), 0, s, X, n, dp, static_cast<f32x4 *>(box0),
                     static_cast<f32x4 *>(box1));
  SJ_HIP(hipGetLastError());
}

void launch_join_mx32(const Mx32Launch &a, hipStream_t s) {
  if (!a.n_wu) return;
  const uint32_t dp = a.view.m.dp;
  auto box = [&](auto launch, int qb) {
    launch(a.view, a.wu, a.n_wu, mx32_queries(dp) / (32u * (uint32_t)qb), a.out, a.capacity,
           a.cursor, s);
  };
  if (dp <= 16)
    return a.view.lead ? box(launch_box<kFmtF16, 2, 16, kQbLead16, true>, kQbLead16)
                       : box(launch_box<kFmtF16, 2, 16, kQbBox16>, kQbBox16);
  if (dp <= 24)
    return a.view.lead ? box(launch_box<kFmtF16, 2, 32, kQbLead32, true>, kQbLead32)
                       : box(launch_box<kFmtF16, 2, 32, kQbBox32>, kQbBox32);
  switch (mx32_k(dp)) {
    case 32: launch_g<32>(a, s); break;
    case 48: launch_g<48>(a, s); break;
    case 64: launch_g<64>(a, s); break;
    case 80: launch_g<80>(a, s); break;
    case 96: launch_g<96>(a, s); break;
    case 112: launch_g<112>(a, s); break;
    case 128: launch_g<128>(a, s); break;
    default: fail(SJ_ERR_INVALID_ARG, "unsupported padded dimension");
  }
}

void launch_join_box16(const MfmaLaunch &a, hipStream_t s) {
  if (!a.n_wu) return;
  const uint32_t tq = mfma_wg_queries(a.kp);
  static_assert(256 % (32 * kQbHalf16) == 0 && 256 % (32 * kQbHalf32) == 0, "whole parts");
  if (tq != 256 || a.kp > 32)
    fail(SJ_ERR_INVALID_ARG, "unsupported box launch");
  Mx32View v{};
  v.m = a.view;
  v.XS = a.view.XA;
  v.nn = a.view.cn;
  if (a.fmt == kFmtF16) launch_half<kFmtF16>(a, v, tq, s);
  else launch_half<kFmtBF16>(a, v, tq, s);
}

}  // namespace sj
