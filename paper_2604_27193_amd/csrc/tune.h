// tune.h -- launch-shape table of the block-structured integration kernels,
// per precision (FP64 / FP32C) and obstacle kind, filled with defaults,
// a JSON cache, or the autotuner (tune.cpp).
#pragma once

#include <vector>

namespace aeb {

struct TuneCfg {
  int k;               // steps per unchecked block (16, 32, 64; FP64 also 128)
  int block;           // threads per workgroup (64, 128, 256)
  int waves_per_simd;  // 0: one pass, one workgroup per `block` samples; else a persistent
                       // grid of this many wavefronts per SIMD claiming 64-sample chunks
  int spt = 1;         // samples per thread: 1, or 2 (FP64 explicit Euler without a lead
                       // vehicle or controller: each lane integrates two sorted samples)
};

// The built-in shapes, [precision 0 FP64, 1 FP32C][obstacle none, stationary,
// lead], measured on MI355X (1,048,576-sample workloads, launch shapes timed in
// one process, interleaved): FP64 256 threads and 4 persistent wavefronts per
// SIMD, 128-step blocks with an obstacle and 64-step blocks without; FP32C
// 64-step blocks, 256 threads, one pass
constexpr TuneCfg TUNE_BUILTIN[2][3] = {
    {{64, 256, 4, 1}, {128, 256, 4, 1}, {128, 256, 4, 1}},
    {{64, 256, 0, 1}, {64, 256, 0, 1}, {64, 256, 0, 1}},
};

// Whether t is the built-in shape: only that one may start fewer wavefronts
// than it says (shape() of the integration kernels); one that was set, tuned or
// loaded runs as it is.
inline bool tune_is_builtin(int precision, int obstacle, const TuneCfg& t) {
  const TuneCfg& b = TUNE_BUILTIN[precision == 0 ? 0 : 1][obstacle < 0 || obstacle > 2 ? 0 : obstacle];
  return t.k == b.k && t.block == b.block && t.waves_per_simd == b.waves_per_simd && t.spt == b.spt;
}

// One timed candidate of the last autotuner sweep.
struct TuneResult {
  TuneCfg t;
  float ms;
};

// candidates of the last sweep for (precision, obstacle), fastest first
std::vector<TuneResult> tune_results(int precision, int obstacle);

// precision: AEB_FP64 or AEB_FP32C (the fix-up mode uses the FP32C entry)
TuneCfg tune_get(int precision, int obstacle);
bool tune_valid(int precision, const TuneCfg& t, int obstacle);
void tune_set(int precision, int obstacle, const TuneCfg& t);

}  // namespace aeb
