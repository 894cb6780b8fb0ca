// Test helper: the gradient's work of a sharing plan (gst::GradWork) unrolled as
// the kernel runs it, next to the plan's own records, for the CPU test.
#include <cstring>

#include "gst_plan.h"

namespace {
std::vector<int64_t> plan_recs, work_recs;  // (gate, adjoint row, state row)
int64_t tiles_seen = 0, tiles_bad = 0, groups = 0;
}

extern "C" int64_t grad_work(const int64_t* off, const uint8_t* gates, int64_t S, int K, int64_t* info) {
  gst::HostPlan P;
  gst::PlanOptions opt;
  opt.max_share_ratio = 10.0;
  if (!gst::build_plan(off, gates, S, K, opt, &P)) return 0;
  const gst::GradWork w(P, K);
  plan_recs.clear();
  work_recs.clear();
  std::vector<char> seen(w.tile_ptr[K], 0);
  tiles_bad = 0;
  auto tile = [&](int64_t t, int k) {
    if (t < w.tile_ptr[k] || t >= w.tile_ptr[k + 1] || seen[t]) ++tiles_bad;
    else seen[t] = 1;
  };
  auto gate_of = [&](int64_t t) {
    int k = 0;
    while (k + 1 < K && t >= w.tile_ptr[k + 1]) ++k;
    return k;
  };
  for (int k = 0; k < K; ++k)
    for (int64_t r = P.rec_gate_ptr[k]; r < P.rec_gate_ptr[k + 1]; ++r) plan_recs.insert(plan_recs.end(), {k, P.rec_b[r], P.rec_f[r]});
  for (size_t c = 0; c < w.chunk_tile.size(); ++c) {
    const int k = gate_of(w.chunk_tile[c]);
    tile(w.chunk_tile[c], k);
    if (w.chunk_end[c] - w.chunk_beg[c] > 128 || w.chunk_end[c] <= w.chunk_beg[c]) ++tiles_bad;
    for (int64_t r = w.chunk_beg[c]; r < w.chunk_end[c]; ++r) work_recs.insert(work_recs.end(), {k, w.rec_b[r], w.rec_f[r]});
  }
  groups = (int64_t)w.jump_meta.size() / 8;
  for (int64_t g = 0; g < groups; ++g) {
    const int32_t* m = &w.jump_meta[8 * g];
    const uint32_t pat = (uint32_t)m[1];
    const int per = (int)(pat & 0xffu);
    if (per < 1 || per > 4 || m[0] % per != 0 || w.jump_first[16 * g] < 0) ++tiles_bad;
    for (int ph = 0; ph < per; ++ph) tile(m[4 + ph], ph < 3 ? (int)((pat >> (8 * (ph + 1))) & 0xffu) : m[2]);
    for (int c = 0; c < 16; ++c) {
      const int64_t first = w.jump_first[16 * g + c], in = w.jump_in[16 * g + c];
      if (first < 0) continue;
      for (int x = 0; x < m[0]; ++x)
        work_recs.insert(work_recs.end(), {gate_of(m[4 + x % per]), first + x, x > 0 ? first + x : in});
    }
  }
  for (char s : seen) tiles_bad += !s;
  info[0] = tiles_bad;
  info[1] = groups;
  info[2] = (int64_t)work_recs.size() / 3;
  return (int64_t)plan_recs.size() / 3;
}

extern "C" void grad_work_copy(int64_t* plan, int64_t* work) {
  std::memcpy(plan, plan_recs.data(), plan_recs.size() * 8);
  std::memcpy(work, work_recs.data(), work_recs.size() * 8);
}
