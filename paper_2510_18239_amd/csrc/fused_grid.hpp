// How the fused stages (fused.hpp) are launched, and how large a launch may be.
#pragma once

#include <algorithm>
#include <cstdint>

namespace lime {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kChunkKeys = 32 * kWaves;  // history items of a workgroup: a tile per wave

// Workgroups of a history, a chunk and a head each: the most there are.
constexpr int64_t history_workgroups(int64_t B, int64_t N, int64_t h) { return B * ((N + kChunkKeys - 1) / kChunkKeys) * h; }

// How the users' last chunks are shared out: `users` of them to a workgroup, `tiles` tiles of 32 items (a wave each) of every user.
// Wave w has tile w - tiles * (w * per_tile >> 16).  Ahead of them come `first` workgroups (a head) of whole chunks.
struct HistoryTails {
  int first, users, tiles, per_tile;
};
// As many users as leave a workgroup for each of the `at_once` that run at a time, if so many fit; 0 = one each.
inline HistoryTails history_tails(int64_t B, int64_t N, int64_t h, int64_t at_once) {
  const int64_t chunks = (N + kChunkKeys - 1) / kChunkKeys, tiles = (N - (chunks - 1) * kChunkKeys + 31) / 32;
  const int64_t wanted = at_once > 0 ? (B * chunks * h + at_once - 1) / at_once : 1;
  const int64_t users = std::max<int64_t>(1, std::min(wanted, kWaves / tiles));
  return {static_cast<int>(B * (chunks - 1)), static_cast<int>(users), static_cast<int>(tiles), static_cast<int>((65536 + tiles - 1) / tiles)};
}
constexpr int64_t tails_workgroups(const HistoryTails& t, int64_t B, int64_t h) { return (t.first + (B + t.users - 1) / t.users) * h; }
// Workgroups are launched in eights, an XCD's share each.
constexpr int64_t launched_workgroups(int64_t total) { return (total + 7) / 8 * 8; }
// HIP takes fewer than 2^32 work items in a dimension of a grid: 2^23 - 1 workgroups.
constexpr bool launch_fits(int64_t total) { return launched_workgroups(total) < (int64_t{1} << 32) / kThreads; }

}  // namespace lime
