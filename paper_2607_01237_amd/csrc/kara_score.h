// Declarations shared by the scoring kernels (kara_score.hip: two sweeps and
// single sweep over streamed keys; kara_score_res.hip: keys resident in LDS).
#pragma once

#include "kara_internal.h"

namespace kara {

struct ScoreArgs {
  Geom g;
  const char* q;              // [n_layers][n_trig][W][Hq][d]
  PoolPtrs k;                 // per-layer K pools
  const int32_t* trig;
  const int32_t* bt;
  const int32_t* win_start;
  const int32_t* status;
  float* partials;            // [units][n_splits][N] (unused with one split)
  float* scores;              // [units][N]
  int n_splits;
  int rows_split;             // query rows per split (single-sweep and resident kernels)
  int64_t n_blocks;
};

constexpr int kScoreCUs = 256;
// Workgroups up to which a launch of few units splits their rows further
// than the kernels need; bounds the partial sums such a launch adds to the
// workspace.
constexpr int kSplitMaxWgs = 1024;

// Resident-key kernel: false where g does not fit it.
bool resident_fits(const Geom& g);
// rows per workgroup (a multiple of 32) for n_units units of g
int resident_rows(const Geom& g, int64_t n_units);
hipError_t launch_score_resident(const ScoreArgs& a, hipStream_t stream);

}  // namespace kara
