// Autotuner of the projection kernel's tile shape.
//
// Candidates differ in how samples map to MFMA columns (4 axis slots per
// sample; 2 in 2D so that 8 samples fill the 16 columns; or 8, two samples
// per block, which doubles the block count for small batches), in how many
// 16-step time blocks one wave carries (1 or 2: more independent items per
// lane, fewer waves per block), and in the grid (one block per tile, or a
// persistent grid of resident blocks looping over tiles), or whether one wave
// owns a sample group over the whole horizon (no block barrier per
// iteration; for batches large enough to fill the chip).  All candidates
// compute bit-identical results, so the choice only affects time: each
// candidate runs one warm-up launch of one iteration, then a timed one of
// kShortTrial iterations; those within kAgain of the fastest (the clocks are
// still rising then, which costs the first candidates up to a third) are timed
// twice over kTrial iterations, and the fastest of these is kept (by a 3%
// margin).  All launches take the caller's real arguments but the iteration
// count (outputs redirected by the caller), timed by HIP events on the caller's
// stream.
#include <algorithm>
#include <vector>

#include "priest_internal.h"

namespace priest {

std::vector<TileCfg> tile_candidates(int dims, int K) {
  std::vector<TileCfg> out;
  const int slots[3] = {4, 2, 8};
  const int rts[3] = {1, 2, 0};
  for (int rt : rts)
    for (int s : slots)
      for (int pers = 0; pers <= 1; ++pers)
        if (tiling_valid(dims, s, rt, K)) out.push_back(TileCfg{s, rt, pers});
  return out;
}

void apply_tiling(ProjArgs& a, const TileCfg& t) {
  a.axis_slots = t.axis_slots;
  a.row_tiles = t.row_tiles;
  a.persistent = t.persistent;
  a.S = samples_per_block(a);
  a.blocks_per_problem = (a.N + a.S - 1) / a.S;
}

// kTrial iterations are enough for the searching loop to be typical: with 8 of
// 100, 16 2D problems of 1000 samples got the whole-horizon shape at 27 ms a plan
// instead of the time-split one at 20.  The tiles choose their loop as in a launch
// of kTrialOf iterations.  The pick serves calls of any length, so the trial does
// not depend on the length of the one that happens to come first.  Over 120 random
// calls, their shape picked in a shorter one, it took 0.55% more time than the
// best shape, and the picking call 3.8 ms (two launches of every shape over
// min(n, 24) iterations, then two more of the near ones: 1.0% and 5.1 ms).
constexpr int kTrial = 24, kTrialOf = 100, kShortTrial = 8;
constexpr float kAgain = 1.6f;

ProjArgs trial_args(const ProjArgs& a) {
  ProjArgs t = a;
  t.n_iter = kTrial;
  t.trial_of = kTrialOf;
  t.bf16_iters = a.bf16_iters > 0 ? kTrial : 0;  // (the same kernel instance)
  t.xi_src = nullptr;
  t.resid2 = nullptr;
  t.c12 = nullptr;
  t.xi_out2 = nullptr;
  return t;
}

hipError_t time_tilings(const ProjArgs& trial, int n_problems, size_t lds_limit, hipStream_t s,
                        const std::vector<TileCfg>& cands, std::vector<float>* ms) {
  ms->assign(cands.size(), -1.0f);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t err = hipEventCreate(&e0);
  if (err == hipSuccess) err = hipEventCreate(&e1);
  auto timed = [&](ProjArgs a, int iters, float* t) {
    a.n_iter = std::min(a.n_iter, iters);
    a.bf16_iters = std::min(a.bf16_iters, iters);
    if (err == hipSuccess) err = hipEventRecord(e0, s);
    if (err == hipSuccess) err = launch_project(a, n_problems, s);
    if (err == hipSuccess) err = hipEventRecord(e1, s);
    if (err == hipSuccess) err = hipEventSynchronize(e1);
    if (err == hipSuccess) err = hipEventElapsedTime(t, e0, e1);
  };
  std::vector<float> first(cands.size(), -1.0f);
  float fastest = -1.0f;
  for (size_t i = 0; i < cands.size() && err == hipSuccess; ++i) {
    ProjArgs a = trial;
    apply_tiling(a, cands[i]);
    if (project_lds_bytes(a) > lds_limit) continue;
    float t = 0.0f;
    timed(a, 1, &t);  // warm-up (first use of the instance)
    timed(a, kShortTrial, &first[i]);
    if (err == hipSuccess && (fastest < 0.0f || first[i] < fastest)) fastest = first[i];
  }
  for (int pass = 0; pass < 2 && err == hipSuccess; ++pass)
    for (size_t i = 0; i < cands.size() && err == hipSuccess; ++i) {
      if (first[i] < 0.0f || first[i] > kAgain * fastest) continue;
      ProjArgs a = trial;
      apply_tiling(a, cands[i]);
      float t = 0.0f;
      timed(a, trial.n_iter, &t);
      if (err == hipSuccess && ((*ms)[i] < 0.0f || t < (*ms)[i])) (*ms)[i] = t;
    }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  return err;
}

int pick_tiling(const std::vector<float>& ms) {
  // a candidate replaces the current pick only if it is more than 3% faster,
  // so timing noise between near-equal shapes does not flip the choice
  int best = 0;
  for (size_t i = 1; i < ms.size(); ++i)
    if (ms[i] >= 0.0f && (ms[best] < 0.0f || ms[i] < ms[best] * 0.97f)) best = static_cast<int>(i);
  return best;
}

}  // namespace priest
