// FP32 filter on the matrix cores (sj_mx32.hip).
#pragma once

#include "sj_mfma.hpp"

namespace sj {

// What a work unit reads: rows, runs, queries and the band list of `m` (its
// 16-bit operands and thresholds stay unused), the bounds on the exact squared
// distance implied by canonical acceptance / rejection (in units of 1 / sc) and
// the error factor.
struct Mx32View {
  MfmaView m;
  double s_hi, s_lo;
  double kappa;   // mx32_kappa(d)
  double tiny;    // absolute error of FP16 parts below the normal range
  double lead_kappa;  // mx32_lead_kappa(d)
  int lead;       // 1: tiles start with the leading product alone (mx32_lead_kappa)
  float widen;    // factor from a candidate's reject value to that of the leading product
  float kacc;     // 1 + 4 kappa, rounded up; FLT_MAX: no pair is accepted without FP64
  const void *XS;     // [n_pad][2][K] split candidate rows
  const float *nn;    // [n_pad] reject values of the tiles
  // group test above 24 dimensions (see k_join_fp32_mxg): projected candidates
  // and queries, the candidates' reject values and the queries' error radii
  const void *ys, *yq;  // [n_pad][kMx32Dirs] FP16
  const float *pn, *ye;
  float sc;           // scale of the centred coordinates (a power of two)
  const uint8_t *pid; // nearest pivot of each query position (null: none), see k_join_fp32_mxg
  const float *ctr;   // [K] centre, reordered dimensions, zero padded
  uint32_t skip_below;           // candidates with caller index below this are skipped (0: none)
  const uint32_t *orig_id;       // candidate position -> caller index
  unsigned long long *skipped;   // += skipped candidates x queries of the unit
};

struct Mx32Launch {
  Mx32View view;
  const WorkUnit *wu;
  uint64_t n_wu;
  uint64_t *out;  // keys pos_q << 32 | pos_c
  uint64_t capacity;
  unsigned long long *cursor;
};

// K padding, query slots of a work unit and whether a unit is one wave's
// (else a workgroup's), for padded dimension dp.
uint32_t mx32_k(uint32_t dp);
uint32_t mx32_queries(uint32_t dp);
// Query slots over which the share of live ones decides for this form (the least
// that its waves take at a time).
uint32_t mx32_live_queries(uint32_t dp);
bool mx32_per_wave(uint32_t dp);
// Split rows and reject values of the cell-ordered rows X ([n][dp]); rows
// n .. n_pad - 1 become padding.
void launch_mx32_prep(const float *X, uint64_t n, uint64_t n_pad, uint32_t dp, const float *ctr,
                      float sc, double kappa, void *XS, float *nn, hipStream_t s);
// Directions of the group test and the rows projected on them: dirs is
// [dp][kMx32Dirs], orthonormal columns (zero rows past d).
constexpr uint32_t kMx32Dirs = 32;
void launch_mx32_project(const float *X, uint64_t n, uint64_t n_pad, uint32_t dp,
                         const float *dirs, const float *ctr, float sc, void *ys, float *pn,
                         float *ye, hipStream_t s);
// Planes of the rows' dimensions 0 .. 3 and 4 .. 7 (16 bytes per point each).
void launch_box_rows(const float *X, uint64_t n, uint32_t dp, void *box0, void *box1,
                     hipStream_t s);
// Relative error factor of the leading product alone.
double mx32_lead_kappa(uint32_t d);
// Relative error factor of the filter for d dimensions.
double mx32_kappa(uint32_t d);
void launch_join_mx32(const Mx32Launch &a, hipStream_t s);
// The 16-bit filters' workgroup units (256 queries, K <= 32) behind the query
// box (MfmaLaunch::box).
void launch_join_box16(const MfmaLaunch &a, hipStream_t s);

}  // namespace sj
