// What the two history-side kernels (mfma_history.hip, mfma_history_walk.hip) share.
#pragma once

#include "mfma.hpp"

namespace lime {

struct HistArgs {
  const bf16_t* E;
  const int32_t* lens;
  const bf16x8 *WkA, *WvB, *QB;
  int64_t qb_user_frags;  // size of one user's query image in bf16x8 units (0 = shared links)
  float* part_acc;        // [B][chunks][h][m][dh]
  float* part_ml;         // [B][chunks][h][m][2]  (running max, running sum)
  int N, chunk_items, chunks;
  float scale;
};

// mfma_history_walk.hip: the cut into chunks, and the launch (softmax only).
struct WalkPlan {
  int chunk_items, chunks;
  bool coop;  // h-wave workgroups that stage each tile once through LDS
};
WalkPlan walk_plan(int B, int N, int d, int h);
// mfma_history_raw.hip: the kernel that takes its operands as they are; `workgroups` of it and those of `beside`.
bool history_raw_fits(const LinksOverHistory& q, int64_t workgroups, const PackJobs& beside);
hipError_t history_raw(const HistArgs& a, const LinksOverHistory& q, hipStream_t s);
hipError_t walk_history(const HistArgs& a, int d, int h, int m, int users, bool coop, hipStream_t s);

}  // namespace lime
