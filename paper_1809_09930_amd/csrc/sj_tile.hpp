// Device helpers shared by the matrix-core filters (sj_mfma.hip, sj_mx32.hip):
// directed rounding, the per-wave result stage and the minimum of a tile's
// accumulators.
#pragma once

#include "sj_internal.hpp"

namespace sj {

constexpr int kStage = 512;  // u64 keys staged per wave

typedef float float16v __attribute__((ext_vector_type(16)));

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
// deferred-recheck list, or (buf == null) nowhere: the pair is rechecked in
// place.
constexpr int kBandStage = 128;
struct BandSink {
  uint64_t *buf;
  uint64_t cap;
  unsigned long long *cursor;
  Stage st;
};

__device__ __forceinline__ float min16(const float16v &v) {
  float a = __builtin_fminf(__builtin_fminf(v[0], v[1]), v[2]);
  float b = __builtin_fminf(__builtin_fminf(v[3], v[4]), v[5]);
  float c = __builtin_fminf(__builtin_fminf(v[6], v[7]), v[8]);
  float e = __builtin_fminf(__builtin_fminf(v[9], v[10]), v[11]);
  float f = __builtin_fminf(__builtin_fminf(v[12], v[13]), v[14]);
  a = __builtin_fminf(__builtin_fminf(a, b), c);
  e = __builtin_fminf(__builtin_fminf(e, f), v[15]);
  return __builtin_fminf(a, e);
}

}  // namespace sj
