// Autotuner of the H*v launch: times the built-in launch and every admissible (variant,
// grid size, columns per lane) on the caller's buffers with HIP events, times the built-in
// one and the four fastest again with more launches, and keeps the fastest in the handle
// (the built-in one unless another is clearly faster); subsequent ftlm_apply / ftlm_run
// launches with the same precision and column count use it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <string>
#include <utility>
#include <vector>

#include "ftlm_internal.hpp"

using namespace ftlm;

extern "C" {

int ftlm_hamiltonian_set_tuning(ftlm_hamiltonian *h, int32_t precision, int32_t n_cols, int32_t variant,
                                int32_t grid_cap, int32_t kc) {
  if (!h || (precision != FTLM_C128 && precision != FTLM_C64) || n_cols < 1 || n_cols > 64 || variant < 0 ||
      variant > 6 || grid_cap < 0 || kc < 0) {
    set_error("bad tuning arguments");
    return FTLM_EINVAL;
  }
  HvTuning &t = h->dev.tune[precision][n_cols];
  t.variant = variant;
  t.grid_cap = grid_cap;
  t.kc = kc;
  return FTLM_OK;
}

int ftlm_hamiltonian_autotune(ftlm_hamiltonian *h, int32_t precision, int32_t n_cols, const void *v, void *w,
                              void *stream, int32_t *variant, int32_t *grid_cap, int32_t *kc,
                              float *best_ms) {
  if (!h || !v || !w || (precision != FTLM_C128 && precision != FTLM_C64) || n_cols < 1 || n_cols > 64) {
    set_error("bad autotune arguments");
    return FTLM_EINVAL;
  }
  hipStream_t s = (hipStream_t)stream;
  const HamGeom &g = h->dev.geom;
  struct Cand {
    int variant, cap, kc;
  };
  // the built-in launch first, with its own grid
  const int own = hv_builtin_variant(h->dev, precision, n_cols);
  std::vector<Cand> cands{{own, 0, 0}};
  const bool f32 = precision == FTLM_C64;
  const bool sweep = (f32 ? h->dev.sw32 : h->dev.sw64).ok, single = (f32 ? h->dev.sp32 : h->dev.sp64).ok;
  const bool half = hv_half_sweeps(h->dev, precision, n_cols);
  if (own != 1) cands.push_back({1, 0, 0});
  const int caps[5] = {0, 512, 1024, 2048, 4096};  // 0: the launch's own, of those that have one
  for (int cap : caps) {
    // half sweep (its threads are fixed)
    if (half && cap <= 2048 && (cap || own != 5)) cands.push_back({5, cap, 0});
    // tile sweep: chunks of 1, 4, 16 or 64 tiles per XCD; its block follows from the tile
    if (n_cols == 1 && cap <= 2048 && sweep)
      for (int ch : {0, 2, 4, 6})
        if (cap || ch || own != 6) cands.push_back({6, cap, ch << 4});
    if (!cap) continue;
    for (int k : {1, 2, 4, 8})
      if (n_cols % k == 0) cands.push_back({1, cap, k});
    if (n_cols == 1) cands.push_back({2, cap, 0});
    if (n_cols == 1 && g.spin_half && g.n >= kTileBits) cands.push_back({3, cap, 0});
    if (n_cols == 1 && cap <= 2048) cands.push_back({4, cap, 0});
    // stream kernel: 1024 or 256 threads per block, chunks of 1, 4, 16 or 64 tiles per
    // XCD, the mixed pairs' partner tiles read directly or staged in LDS
    if (n_cols == 1 && cap <= 2048 && single && !sweep)
      for (int st : {0, 1})
        for (int nt : {0, 1})
          for (int ch : {0, 2, 4, 6}) cands.push_back({6, cap, nt | (ch << 4) | (st << 8)});
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    set_error("hipEventCreate failed");
    return FTLM_EHIP;
  }
  // (an earlier choice would stand in for a candidate's zeros)
  const HvTuning saved = h->dev.tune[precision][n_cols];
  h->dev.tune[precision][n_cols] = HvTuning{};
  float best = FLT_MAX;
  int bestc = 0;
  int rc = FTLM_OK;
  // mean time of reps launches after one warm-up launch; < 0 if the shape is
  // inadmissible, NaN on a HIP error
  auto time_cand = [&](const Cand &c, int reps) -> float {
    HvLaunch L{};
    L.precision = precision;
    L.K = n_cols;
    L.v = v;
    L.w = w;
    L.variant = c.variant;
    L.grid_cap = c.cap;
    L.kc = c.kc;
    if (launch_hv(h->dev, L, s) != FTLM_OK) return -1.0f;
    if (hipEventRecord(e0, s) != hipSuccess) return NAN;
    for (int r = 0; r < reps; r++) launch_hv(h->dev, L, s);
    if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) return NAN;
    float ms = 0;
    (void)hipEventElapsedTime(&ms, e0, e1);
    return ms / (float)reps;
  };
  // a quick pass over every candidate, then the built-in launch and the four fastest others
  // again with more launches each (neighbouring grid sizes often differ by a few per
  // cent, within the noise of three launches; of grid sizes alone at most two, as those
  // beyond a launch's tiles are one launch)
  std::vector<std::pair<float, int>> timed;
  for (size_t i = 0; i < cands.size() && !rc; i++) {
    const float ms = time_cand(cands[i], 3);
    if (std::isnan(ms)) rc = FTLM_EHIP;
    else if (ms >= 0) timed.push_back({ms, (int)i});
  }
  std::sort(timed.begin(), timed.end());
  std::vector<int> finals{0};
  for (const auto &t : timed) {
    const Cand &c = cands[t.second];
    const int same = (int)std::count_if(finals.begin(), finals.end(),
                                        [&](int i) { return cands[i].variant == c.variant && cands[i].kc == c.kc; });
    if (t.second && same < 2 && finals.size() < 5) finals.push_back(t.second);
  }
  for (int i : finals) {
    if (rc) break;
    const float ms = time_cand(cands[i], 10);
    if (std::isnan(ms)) rc = FTLM_EHIP;
    // (two means of ten launches differ by a few per cent by themselves)
    else if (ms >= 0 && (best == FLT_MAX || ms < best * (bestc == 0 ? 0.97f : 1.0f))) {
      best = ms;
      bestc = i;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) {
    h->dev.tune[precision][n_cols] = saved;
    set_error("autotune timing failed");
    return rc;
  }
  if (best == FLT_MAX) {
    h->dev.tune[precision][n_cols] = saved;
    set_error("no admissible H*v configuration");
    return FTLM_EINVAL;
  }
  HvTuning &t = h->dev.tune[precision][n_cols];
  t.variant = cands[bestc].variant;
  t.grid_cap = cands[bestc].cap;
  t.kc = cands[bestc].kc;
  if (variant) *variant = t.variant;
  if (grid_cap) *grid_cap = t.grid_cap;
  if (kc) *kc = t.kc;
  if (best_ms) *best_ms = best;
  return FTLM_OK;
}

}  // extern "C"
