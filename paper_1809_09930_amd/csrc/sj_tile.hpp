// Device helpers shared by the matrix-core filters (sj_mfma.hip, sj_mx32.hip):
// directed rounding, the per-wave result stage and the minimum of a tile's
// accumulators.
#pragma once

#include "sj_internal.hpp"

namespace sj {

constexpr int kStage = 512;  // u64 keys staged per wave

typedef float float16v __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A wave-uniform read of memory that no kernel in flight writes, as a scalar
// load: through an ordinary pointer the compiler must allow for the kernel's
// own stores and takes a vector load and a wait for every load in flight.
__device__ __forceinline__ uint2 scalar_run(const uint2 *runs, uint32_t r) {
  const auto *p = reinterpret_cast<const __attribute__((address_space(4))) uint64_t *>(
      reinterpret_cast<uintptr_t>(runs));
  const uint64_t v = p[uniform_u32(r)];
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}

// next float above a finite f (one ulp step on the bit pattern)
__device__ __forceinline__ float next_up(float f) {
  if (f == 0.0f) return __builtin_bit_cast(float, 1u);
  const uint32_t b = __builtin_bit_cast(uint32_t, f);
  return __builtin_bit_cast(float, f > 0.0f ? b + 1u : b - 1u);
}
__device__ __forceinline__ float round_up_f32(double v) {
  if (v != v || v == __builtin_inf()) return __builtin_inff();
  if (v == -__builtin_inf()) return -__builtin_inff();
  float f = (float)v;
  if ((double)f < v) f = next_up(f);
  return f;
}
__device__ __forceinline__ float round_down_f32(double v) {
  return -round_up_f32(-v);
}

struct Stage {
  uint64_t *buf;
  uint32_t cnt;
  uint32_t size;  // entries of buf, at least 128 (band lists: 64)
};

__device__ __forceinline__ void flush(Stage &st, uint64_t *__restrict__ out, uint64_t capacity,
                                      unsigned long long *__restrict__ cursor) {
  if (st.cnt == 0) return;
  __builtin_amdgcn_wave_barrier();
  unsigned long long base = 0;
  if (lane_id() == 0) base = atomicAdd(cursor, (unsigned long long)st.cnt);
  base = uniform_u64(__shfl(base, 0));
  for (uint32_t i = lane_id(); i < st.cnt; i += kWave) {
    const uint64_t pos = base + i;
    if (pos < capacity) out[pos] = st.buf[i];
  }
  __builtin_amdgcn_wave_barrier();
  st.cnt = 0;
}

// Where the hit path sends band pairs: a per-wave LDS stage flushed to the
// deferred-recheck list.
constexpr int kBandStage = 128;
struct BandSink {
  uint64_t *buf;
  uint64_t cap;
  unsigned long long *cursor;
  Stage st;
};

// Minimum of 16 accumulators as two values, seven three-operand minima: the
// eighth takes both of them together with what the caller compares or collects
// (a two-operand minimum of raw matrix results would first be canonicalised).
struct Min16 {
  float a, b;
};

__device__ __forceinline__ Min16 min16(const float16v &v) {
  auto min3 = [](float x, float y, float z) {
    return __builtin_fminf(__builtin_fminf(x, y), z);
  };
  const float a = min3(v[0], v[1], v[2]), b = min3(v[3], v[4], v[5]);
  const float c = min3(v[6], v[7], v[8]), d = min3(v[9], v[10], v[11]);
  const float e = min3(v[12], v[13], v[14]);
  return {min3(a, b, c), min3(d, e, v[15])};
}

__device__ __forceinline__ float min16(const float16v &v, float with) {
  const Min16 m = min16(v);
  return __builtin_fminf(__builtin_fminf(with, m.a), m.b);
}

// Waits for this wave's outstanding loads.  Placed before a loop that keeps
// loads in flight: what was loaded ahead of it (a unit's queries) would
// otherwise be waited for at its first use inside, in every iteration, and the
// loop's own loads with it.
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
}

// Tiles.  Rows are queries, columns candidates: lane l holds column l & 31, and
// element e of its 16 accumulators is row 8 (e / 4) + 4 (l >> 5) + e % 4.  The
// rows' thresholds are the initial accumulators (kept in registers for the
// whole unit) and a candidate's norm is one value per lane, so a tile reads
// nothing but its operands: with candidates as rows every tile had to reload
// 16 norms per lane from LDS, which bound the 16-dimensional joins.

// Initial accumulators of 32 rows from their 32 values.
__device__ __forceinline__ float16v rows_init(const float *rows32, uint32_t half) {
  float16v c;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = *reinterpret_cast<const f32x4 *>(rows32 + 8 * g + 4 * half);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[4 * g + i] = x[i];
  }
  return c;
}

// One tile's hits (element < nn) as a 16-bit mask per lane, and with kAccept
// the mask of the pairs proven within eps (element + its row's delta < nacc).
// Element e is bit 15 - e: the sign bits of the differences are shifted in one
// by one (v_alignbit).  A candidate with nn = -inf (padding) has none of finite
// elements; the sign of -inf - -inf is open, and emit_hits drops what it leaves.
template <bool kAccept>
__device__ __forceinline__ void tile_masks(const float16v &acc, float nn, float nacc,
                                           const float *delta32, uint32_t half, uint32_t &hit,
                                           uint32_t &within) {
  hit = within = 0u;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 d = {0, 0, 0, 0};
    if constexpr (kAccept) d = *reinterpret_cast<const f32x4 *>(delta32 + 8 * g + 4 * half);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = acc[4 * g + i];
      hit = __builtin_amdgcn_alignbit(hit, __builtin_bit_cast(uint32_t, x - nn), 31);
      if constexpr (kAccept)
        within =
            __builtin_amdgcn_alignbit(within, __builtin_bit_cast(uint32_t, x + d[i] - nacc), 31);
    }
  }
}

// How emitted keys are formed: key_hi | pos_q << pshift | pos_c.
struct KeyForm {
  uint64_t key_hi;
  uint32_t pshift;
  bool sym;  // both orders, of pairs with pos_q <= pos_c only
};

// Emits the hits of up to 64 / 16 tiles of one 32-candidate block: every lane
// with hits left takes its lowest one per round, so the rounds are few (a lane
// rarely has two) and there is one copy of the emission code.  hits / within:
// tile j's masks at bits 16 j; cp: the lane's candidate and nn its reject value
// (-inf: padding, nothing is emitted; 0 where all thresholds are finite, and padding
// has no hits); qpos: the tiles' query positions, 32 per tile.  Pairs proven within
// eps go to the result stage, the others to the recheck list.
template <bool kAccept, class M>
__device__ __forceinline__ void emit_hits(M hits, M within, const uint32_t *qpos, uint32_t half,
                                          uint32_t cp, float nn, const KeyForm &kf, Stage &st,
                                          BandSink &bs, uint64_t *__restrict__ out,
                                          uint64_t capacity,
                                          unsigned long long *__restrict__ cursor) {
  // queries below this take part (0xffffffff: a row without a query)
  const uint32_t end_q = nn == -__builtin_inff() ? 0u : kf.sym ? cp + 1u : 0xffffffffu;
  while (ballot(hits != 0)) {
    const bool live = hits != 0;
    const uint32_t b = live ? (uint32_t)__builtin_ctzll((uint64_t)hits) : 0u;
    const uint32_t e = 15u - (b & 15u);
    const uint32_t qp = qpos[(b & ~15u) * 2 + 8 * (e / 4) + 4 * half + (e & 3u)];
    const bool ok = live && qp < end_q;
    const bool acc_ok = kAccept && ok && ((within >> b) & 1) != 0;
    const bool band = ok && !acc_ok;
    const uint64_t key = kf.key_hi | ((uint64_t)qp << kf.pshift) | cp;
    const uint64_t bm = ballot(band);
    if (bm) {
      const uint32_t nb = (uint32_t)__builtin_popcountll(bm);
      if (bs.st.cnt + nb > bs.st.size) flush(bs.st, bs.buf, bs.cap, bs.cursor);
      if (band) bs.st.buf[bs.st.cnt + lanes_below(bm)] = key;
      bs.st.cnt += nb;
    }
    if constexpr (kAccept) {
      const uint64_t am = ballot(acc_ok);
      if (am) {
        const bool two = acc_ok && kf.sym && qp != cp;
        const uint64_t m2 = ballot(two);
        const uint32_t total = (uint32_t)(__builtin_popcountll(am) + __builtin_popcountll(m2));
        if (st.cnt + total > st.size) flush(st, out, capacity, cursor);
        const uint32_t off = st.cnt + lanes_below(am) + lanes_below(m2);
        if (acc_ok) {
          st.buf[off] = key;
          if (two) st.buf[off + 1] = kf.key_hi | ((uint64_t)cp << kf.pshift) | qp;
        }
        st.cnt += total;
      }
    }
    if (live) hits &= hits - 1;
  }
}

// The smallest float above a reject value, so that "value <= v" is "value < w".
__device__ __forceinline__ float strict(float v) {
  return v == -__builtin_inff() ? v : next_up(v);
}

}  // namespace sj
