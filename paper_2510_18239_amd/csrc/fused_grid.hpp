// How the fused stages (fused.hpp) are launched, and how large a launch may be.
#pragma once

#include <cstdint>

namespace lime {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kChunkKeys = 32 * kWaves;  // history items of a workgroup: a tile per wave

// Workgroups of a history, a chunk and a head each.
constexpr int64_t history_workgroups(int64_t B, int64_t N, int64_t h) { return B * ((N + kChunkKeys - 1) / kChunkKeys) * h; }
// Workgroups are launched in eights, an XCD's share each.
constexpr int64_t launched_workgroups(int64_t total) { return (total + 7) / 8 * 8; }
// HIP takes fewer than 2^32 work items in a dimension of a grid: 2^23 - 1 workgroups.
constexpr bool launch_fits(int64_t total) { return launched_workgroups(total) < (int64_t{1} << 32) / kThreads; }

}  // namespace lime
