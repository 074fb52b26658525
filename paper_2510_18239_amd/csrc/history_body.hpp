// User-side link personalisation on the matrix cores: the m links attend over the N history
// rows, by softmax (Eq. 3) or by the target-to-source half of XORA, O[T] (Eq. 7, phi = SiLU/n_s).
//
// Design: one fused pass over E.  A workgroup owns a chunk of one user's history and HG heads, and walks the chunk in
// steps of TP tiles of 32 items.  A wave owns 32 columns of a head (a head has MB = d/h / 32 such blocks) and one tile of
// every step; its slices of W_K^T and W_V stay in its registers.  Per tile, with X = the 32 history rows:
//   K~^T (32 x 32) = W_K^T . X^T      X is the B operand
//   V~   (32 x 32) = X . W_V          the same X fragments are the A operand
// The MB waves of a head and tile then trade their blocks of K~ and V~ through LDS and share out the links:
//   S^T  (32 x links) = K~ . Q~_a^T   A operand = accumulators of the first product
//   L^P^T(d/h x links) += V~^T . phi(S)^T   both operands are accumulators (of the 2nd and 3rd product)
// Each lane owns one link (column of S^T and of L^P^T): the running maximum, the running sum and the rescaling of the
// accumulator are all lane-local, plus one exchange with lane ^ 32.  Rows at or beyond lens[b] are
// replaced by zeros before they are read and masked out of phi, so their content is never used.
// The rows go from memory straight to LDS, a step ahead; the TP waves of a block combine their tiles' results in LDS
// at the end.
// Every chunk writes an un-normalised partial (maximum, sum, accumulator); a small merge kernel
// combines the chunks of a user in a fixed order (deterministic) and writes L^P.
#pragma once

#include <algorithm>

#include "history.hpp"
#include "pack.hpp"

namespace lime {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

// How a workgroup's waves are laid out: heads x tiles of a step x 32-column blocks of a head.
// RAW: the operands come as they are (RawArgs) and are laid out by the workgroup, whose steps are one: a chunk is a step.
template <int DH, int M, int H, int HG_, int TP_, bool RAW = false>
struct HistShape {
  static constexpr int D = DH * H, HG = HG_, TP = TP_;
  static constexpr int MB = DH / 32, K1 = D / 16, K2 = DH / 16, LB = M / 32;
  static constexpr int LBW = (LB + MB - 1) / MB;  // 32-link blocks per wave
  static constexpr int kWaves = HG * TP * MB, kThreads = 64 * kWaves, kRows = 32 * TP;
  static constexpr int kXBytes = kRows * 2 * D, kExchange = MB > 1 ? kWaves * 4 * 1024 : 0, kQueries = HG * K2 * LB * 1024;
  // Two buffers for the rows and the exchange (one barrier a step) where a compute unit then still holds eight waves,
  // otherwise one (two barriers).
  static constexpr int kLdsPerUnit = 160 * 1024 / (8 / kWaves);
  static constexpr int NX = !RAW && 2 * kXBytes + 2 * kExchange + kQueries <= kLdsPerUnit ? 2 : 1;
  static constexpr int kPerWave = MB * LBW * 4096 + LBW * 512, kCombine = TP > 1 ? TP * HG * MB * kPerWave : 0;
  // RAW: the head's columns of a weight matrix, as tiles of 16 rows x 32 columns; the links' rows, with those of W_Q where the
  // exchange and the queries come to lie once they have been read; W_K and W_V behind them
  static constexpr int kSlice = K1 * MB * 1024, kLinks = M * 2 * D;
  static constexpr int kShared = std::max(kLinks + kSlice, kExchange + kQueries);
  static constexpr int kLds = RAW ? std::max(kXBytes + kShared + 2 * kSlice, kCombine) : std::max(NX * (kXBytes + kExchange) + kQueries, kCombine);
  // What the compiler is held to.  RAW: three where LDS lets a compute unit have three workgroups (of four waves, one a SIMD).
  static constexpr int kWavesPerSimd = RAW && 3 * kLds <= 160 * 1024 ? 3 : 2;
};

// What a launch brings besides HistArgs: RAW, the operands, and jobs for as many workgroups more (blockIdx.z from H on).
struct RawArgs {
  const bf16_t *LC, *Wq, *Wk, *Wv;
  int64_t lc_user_stride;
  int negate;    // the logit scale is negative: its sign is the queries'
  int pack_blocks;
  PackArgs pack;
};
struct PackedArgs {};

// A 16-byte piece c of row r of a staged tile lies at piece c ^ row_swizzle<D>(r) of the row, so that the 16 lanes that an
// LDS read serves at once (16 rows, one column) touch all banks.
template <int D>
__device__ __forceinline__ int row_swizzle(int r) {
  constexpr int CPR = D / 8;  // pieces per row
  return CPR >= 16 ? r & 15 : r / (16 / CPR) & (CPR - 1);
}

// (Both forms from one text, but each a kernel of its own body: as a function that two kernels call, the same text takes up to 31
// registers more (softmax, d/h = 32, 96 or 128 links), spills 46 instead of 17 at h = 8 and m = 128, and is slower by a quarter there:
// 8 prepared users of 8000 items, d=256 h=8, m=128 71.6 | 57.1 us, m=96 48.3 | 45.6.)
template <int DH, int M, int H, int PHI, int HG, int TP, bool RAW>
__global__ __launch_bounds__((HistShape<DH, M, H, HG, TP, RAW>::kThreads), (HistShape<DH, M, H, HG, TP, RAW>::kWavesPerSimd)) void links_over_history_kernel(HistArgs a, std::conditional_t<RAW, RawArgs, PackedArgs> r) {
  using S = HistShape<DH, M, H, HG, TP, RAW>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  if constexpr (RAW) {
    if (blockIdx.z >= H) {  // uniform
      const int i = ((blockIdx.z - H) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
      if (i < r.pack_blocks) pack_block<DH * H, 0, 0>(r.pack, i, lds);
      return;
    }
  }
  constexpr int D = S::D, K1 = S::K1, MB = S::MB, K2 = S::K2, LB = S::LB, LBW = S::LBW, NX = S::NX, kWaves = S::kWaves;
  constexpr int CPR = D / 8, LW = S::kXBytes / (kWaves * 1024);  // 1 KiB loads per wave and step
  unsigned char* const ex_lds = lds + NX * S::kXBytes;
  bf16x8* const q_lds = reinterpret_cast<bf16x8*>(ex_lds + NX * S::kExchange);
  const int lane = threadIdx.x & 63, n = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave % MB, hl = wave / MB % HG, tp = wave / (MB * HG);  // column block, head of the group, tile of a step
  const int head = blockIdx.z * HG + hl;
  const int b = blockIdx.y, chunk = blockIdx.x;
  const int len = __builtin_amdgcn_readfirstlane(a.lens ? min(a.lens[b], a.N) : a.N);
  const int i_begin = chunk * a.chunk_items;
  if (i_begin >= len) return;  // uniform over the workgroup: nothing for this chunk
  const int i_end = min(len, i_begin + a.chunk_items);

  const bf16_t* Eb = a.E + static_cast<int64_t>(b) * a.N * D;
  // This wave's part of a step.  A load's rows are RPL j past its first one's, whose row number has those bits clear: the pieces
  // of the others lie where its own do, but for a constant in the swizzle.
  constexpr int RPL = 64 / CPR;
  static_assert((LW & (LW - 1)) == 0 && LW > 0, "row numbers split into bits");
  auto ask_rows = [&](int i0, int buf) {
    const bf16_t* base = Eb + static_cast<int64_t>(i0) * D;
    const unsigned dst = lds_offset_of(lds) + buf * S::kXBytes + wave * LW * 1024;
    int l = lane;
    asm volatile("" : "+v"(l));  // (what follows from it is formed here, not carried through the loop: registers)
    const int first_row = wave * (LW * RPL) + l / CPR;
    if (i0 + S::kRows <= a.N) {  // uniform
      const int piece = first_row * (2 * D) + (l % CPR ^ row_swizzle<D>(first_row)) * 16;
#pragma unroll
      for (int j = 0; j < LW; ++j) load_to_lds(dst + j * 1024, piece ^ (row_swizzle<D>(RPL * j) * 16), base + RPL * j * D);
      return;
    }
    const int last = a.N - 1 - i0;  // rows past the tensor's end as its last one
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int r = first_row + RPL * j;
      load_to_lds(dst + j * 1024, min(r, last) * (2 * D) + (l % CPR ^ row_swizzle<D>(r)) * 16, base);
    }
  };
  auto clear_tail = [&](int i0, int buf) {  // what this wave asked for past the chunk's end becomes zeros
    if (i0 + S::kRows <= i_end) return;     // uniform
    bf16x8 zero;
#pragma unroll
    for (int t = 0; t < 8; ++t) zero[t] = static_cast<__bf16>(0.f);
    int q0 = wave * LW * 64 + lane;
    asm volatile("" : "+v"(q0));
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int q = q0 + j * 64;
      if (i0 + q / CPR >= i_end) *reinterpret_cast<bf16x8*>(lds + buf * S::kXBytes + q * 16) = zero;
    }
  };

  bf16x8 wk[K1], wv[K1];

  // RAW: everything is asked for at once, the links and W_Q first of the operands; the queries are formed while W_K and W_V
  // arrive.  Sums and roundings are those of the pack kernel's projection.
  constexpr int kSliceLoads = (K1 * MB + kWaves - 1) / kWaves, kLinkLoads = S::kLinks / 1024 / kWaves;
  unsigned char *const links_lds = ex_lds + S::kSlice, *const keys_lds = ex_lds + S::kShared, *const values_lds = keys_lds + S::kSlice;
  static_assert(!RAW || (HG == 1 && S::kLinks % (1024 * kWaves) == 0 && (K1 * MB) % kWaves == 0), "every wave asks for as many lines");
  auto ask_slice = [&](const bf16_t* w, unsigned char* to) {
#pragma unroll
    for (int i = 0; i < kSliceLoads; ++i) {
      const int f = wave * kSliceLoads + i;  // tile (k-step f / MB, block f % MB)
      load_to_lds(lds_offset_of(to) + f * 1024, (lane / 4) * (2 * D) + lane % 4 * 16, w + static_cast<int64_t>(16 * (f / MB)) * D + head * DH + 32 * (f % MB));
    }
  };
  auto ask_raw = [&](const auto& r) {
    const bf16_t* lc = r.LC + b * r.lc_user_stride;
#pragma unroll
    for (int j = 0; j < kLinkLoads; ++j) {
      const int q = (wave * kLinkLoads + j) * 64 + lane, row = q / CPR;
      load_to_lds(lds_offset_of(links_lds) + (wave * kLinkLoads + j) * 1024, row * (2 * D) + (q % CPR ^ row_swizzle<D>(row)) * 16, lc);
    }
    ask_slice(r.Wq, ex_lds);
    ask_slice(r.Wk, keys_lds);
    ask_slice(r.Wv, values_lds);
  };
  auto lay_out_raw = [&](const auto& r) {
    constexpr int kBlocks = LB * MB, kMine = (kBlocks + kWaves - 1) / kWaves;
    wait_lds_loads<2 * kSliceLoads>();
    lds_barrier();
    bf16x8 q[kMine][2];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int block = wave + i * kWaves, lb = block / MB, mb = block % MB;
      if (block >= kBlocks) break;  // uniform
      const int link = 32 * lb + n;
      bf16x8 w[K1], x[K1];
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) {
        w[kk] = column_fragment(ex_lds + (kk * MB + mb) * 1024, 64, lane);
        x[kk] = *reinterpret_cast<const bf16x8*>(links_lds + link * (2 * D) + ((2 * kk + g) ^ row_swizzle<D>(link)) * 16);
      }
      f32x16 block_sum = project_block<K1>(w, x);
      if (r.negate) block_sum = -block_sum;
      q[i][0] = pack_half(block_sum, 0), q[i][1] = pack_half(block_sum, 1);
    }
    wait_lds_loads<0>();
    clear_tail(i_begin, 0);
    lds_barrier();  // (and the links and W_Q have been read: the queries lie where they were)
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int block = wave + i * kWaves, lb = block / MB, mb = block % MB;
      if (block >= kBlocks) break;
#pragma unroll
      for (int f = 0; f < 2; ++f) q_lds[((2 * mb + f) * LB + lb) * 64 + lane] = q[i][f];
    }
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      wk[kk] = column_fragment(keys_lds + (kk * MB + half) * 1024, 64, lane);
      wv[kk] = column_fragment(values_lds + (kk * MB + half) * 1024, 64, lane);
    }
  };

  // The rows come from HBM and are asked for ahead of the operands, which come from L2.
  ask_rows(i_begin, 0);
  if constexpr (RAW) {
    ask_raw(r);
  } else {
    {
      // the heads' query fragments: kept in LDS, read once per tile
      const bf16x8* src = a.QB + b * a.qb_user_frags + static_cast<int64_t>(blockIdx.z) * HG * K2 * LB * 64;
      for (int f = wave; f < HG * K2 * LB; f += kWaves) load_to_lds(lds_offset_of(q_lds) + f * 1024, lane * 16, src + f * 64);
    }
    if (NX == 2 && i_begin + S::kRows < i_end) ask_rows(i_begin + S::kRows, 1);
  #pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      wk[kk] = a.WkA[((head * K1 + kk) * MB + half) * 64 + lane];
      wv[kk] = a.WvB[((head * K1 + kk) * MB + half) * 64 + lane];
    }
  }

  f32x16 acc[MB][LBW];
  float run_max[LBW], run_sum[LBW];
#pragma unroll
  for (int l = 0; l < LBW; ++l) {
    run_max[l] = -INFINITY;
    run_sum[l] = 0.f;
#pragma unroll
    for (int ob = 0; ob < MB; ++ob)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[ob][l][i] = 0.f;
  }
  const float c = a.scale * kLog2e;                    // >= 0: a negative scale is folded into the sign of the packed queries
  const int row = 32 * tp + n, row_base = row * (2 * D) + (g ^ row_swizzle<D>(row)) * 16;

  if constexpr (RAW) {
    lay_out_raw(r);
  } else {
    // (the weights are waited for here: left pending, the loop would wait for them, and with them for the rows, every time)
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) asm volatile("" : "+v"(wk[kk]), "+v"(wv[kk]));
    wait_lds_loads<0>();
    clear_tail(i_begin, 0);
    lds_barrier();
  }

  int s = 0;
  for (int i0 = i_begin; i0 < i_end; i0 += S::kRows, ++s) {
    const int buf = NX == 2 ? s & 1 : 0;
    const int t0 = i0 + 32 * tp;       // this wave's tile
    const bool live = t0 < i_end;      // uniform over the wave
    bf16x8 kf[K2], vf[MB][2];
    unsigned char* const ex = ex_lds + buf * S::kExchange;
    if (live) {
      f32x16 d1, d2;
#pragma unroll
      for (int i = 0; i < 16; ++i) d1[i] = d2[i] = 0.f;
      int base = row_base + buf * S::kXBytes;
      asm volatile("" : "+v"(base));  // (the addresses are formed here, not carried through the loop)
      // (the reads run kAhead k-steps ahead of their use and, fenced, no further: registers)
      constexpr int kAhead = K1 < 3 ? K1 : 3;
      bf16x8 x[K1];
#pragma unroll
      for (int kk = 0; kk < K1 + kAhead; ++kk) {
        if (kk < K1) x[kk] = *reinterpret_cast<const bf16x8*>(lds + ((base ^ (kk % 8 * 32)) + kk / 8 * 256));
        if (kk >= kAhead) {
          d1 = mfma32(wk[kk - kAhead], x[kk - kAhead], d1);
          d2 = mfma32(x[kk - kAhead], wv[kk - kAhead], d2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (MB == 1) {
        kf[0] = pack_half(d1, 0), kf[1] = pack_half(d1, 1);
        vf[0][0] = pack_half(d2, 0), vf[0][1] = pack_half(d2, 1);
      } else {
        bf16x8* dst = reinterpret_cast<bf16x8*>(ex) + (wave * 4) * 64 + lane;
#pragma unroll
        for (int f = 0; f < 2; ++f) dst[f * 64] = pack_half(d1, f), dst[(2 + f) * 64] = pack_half(d2, f);
      }
    }
    const int next = i0 + S::kRows;
    if constexpr (NX == 2) {
      if (next < i_end) {
        wait_lds_loads<0>();
        clear_tail(next, buf ^ 1);
      }
    }
    // publishes the next step's rows (NX == 2) and this step's exchange; everybody has read this step's rows
    if (MB > 1 || RAW || next < i_end) lds_barrier();
    const int after = NX == 2 ? next + S::kRows : next;
    if (after < i_end) ask_rows(after, buf);

    // A wave that projects always has a matrix instruction ready: without priority the other wave of its SIMD would wait
    // for it to finish before each of the few that stand between its vector instructions.
    __builtin_amdgcn_s_setprio(2);
    if (live) {
      if constexpr (MB == 2) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          const bf16x8* src = reinterpret_cast<const bf16x8*>(ex) + ((wave - half + mb) * 4) * 64 + lane;
#pragma unroll
          for (int f = 0; f < 2; ++f) kf[2 * mb + f] = src[f * 64];
        }
      }
      const bool ragged = t0 + 32 > i_end;  // uniform; only a chunk's last tile can be
#pragma unroll
      for (int l = 0; l < LBW; ++l) {
        const int lb = half * LBW + l;
        if (LB % MB != 0 && lb >= LB) break;  // uniform
        f32x16 sc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < K2; ++kk) sc = mfma32(kf[kk], q_lds[((hl * K2 + kk) * LB + lb) * 64 + lane], sc);
        // register 4j + r of this lane is item t0 + 8j + 4g + r
        if (PHI == kPhiSoftmax) {
          auto mask = [&](float to) {
            if (!ragged) return;
            int valid = i_end - t0 - 4 * g;
            asm volatile("" : "+v"(valid));  // (the comparisons stay in here)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (8 * (i >> 2) + (i & 3) >= valid) sc[i] = to;
          };
          mask(-INFINITY);
          float tmax = sc[0];
#pragma unroll
          for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, sc[i]);
          // The weights are relative to the running maximum, so that the largest is one exactly.  (A base that moves only
          // once a logit passes it by eight powers of two saves 1 us of 99 at B=16 N=4096 C=8192 d=256 m=128, but rounds
          // the largest weight like any other: link states up to 1.3 % further from the exact ones.)
          if (__any(tmax > run_max[l])) {  // uniform
            const float new_max = fmaxf(run_max[l], pair_max(tmax));  // finite: the tile holds at least one valid item
            const float alpha = run_max[l] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((run_max[l] - new_max) * c);
            run_sum[l] *= alpha;
            run_max[l] = new_max;
#pragma unroll
            for (int ob = 0; ob < MB; ++ob)
#pragma unroll
              for (int i = 0; i < 16; ++i) acc[ob][l][i] *= alpha;
          }
          const float shift = -run_max[l] * c;  // exp2(raw * c + shift) = exp(scale * raw - running maximum)
          float psum = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) sc[i] = __builtin_amdgcn_exp2f(fmaf(sc[i], c, shift));
          mask(0.f);  // (explicit: also right for scale = 0)
#pragma unroll
          for (int i = 0; i < 16; ++i) psum += sc[i];
          run_sum[l] += psum;
        } else {
          // SiLU(scale * s) = scale * s * sigmoid(scale * s); the factor `scale` is applied by the merge
#pragma unroll
          for (int i = 0; i < 16; ++i) sc[i] = sc[i] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-sc[i] * c));
          // (no mask is needed here: rows past the end of the chunk are zeros, so their projected keys are zero, their
          // logits are zero and SiLU(0) = 0 exactly)
        }
        const bf16x8 p0 = pack_half(sc, 0), p1 = pack_half(sc, 1);
        if constexpr (MB == 2) {
          if (LBW > 1) __builtin_amdgcn_sched_barrier(0);  // (fetched no earlier: registers)
#pragma unroll
          for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int f = 0; f < 2; ++f) vf[mb][f] = reinterpret_cast<const bf16x8*>(ex)[((wave - half + mb) * 4 + 2 + f) * 64 + lane];
        }
#pragma unroll
        for (int ob = 0; ob < MB; ++ob) {
          acc[ob][l] = mfma32(vf[ob][0], p0, acc[ob][l]);
          acc[ob][l] = mfma32(vf[ob][1], p1, acc[ob][l]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if constexpr (NX == 1) {
      if (next < i_end) {
        wait_lds_loads<0>();
        clear_tail(next, 0);
        lds_barrier();
      }
    }
  }

  // The tiles of a step are combined in ascending order, through LDS: the TP waves of a block share out its pieces, a piece
  // being what a lane stores at once: four head columns 32 ob + 8 j + 4 g .. + 3 of its link.  (By the first tile's waves alone
  // this took 1.6 us with eight tiles, and their stores 2.0, at B=32 N=1024 d=128 m=64; 0.5 and 1.1 so.)
  const int64_t slot = (static_cast<int64_t>(b) * a.chunks + chunk) * H + head;
  auto store_piece = [&](int l, int ob, int j, float4 v) {
    const int link = 32 * (half * LBW + l) + n;
    *reinterpret_cast<float4*>(a.part_acc + (slot * M + link) * DH + 4 * g + 32 * ob + 8 * j) = v;
  };
  auto store_sums = [&](int l, float top, float sum) {
    const int link = 32 * (half * LBW + l) + n;
    const float total = pair_sum(sum);
    if (g == 0) *reinterpret_cast<float2*>(a.part_ml + (slot * M + link) * 2) = make_float2(top * a.scale, total);  // (the merge works on scaled logits)
  };
  auto past_links = [&](int l) { return LB % MB != 0 && half * LBW + l >= LB; };  // uniform
  if constexpr (TP > 1) {
    constexpr int kPer = S::kPerWave;
    lds_barrier();  // the rows' and the exchange's last readers are done
    unsigned char* const block = lds + (hl * MB + half) * kPer;  // a tile's part, HG MB kPer apart
    {
      unsigned char* dst = block + tp * HG * MB * kPer;
#pragma unroll
      for (int l = 0; l < LBW; ++l) {
#pragma unroll
        for (int ob = 0; ob < MB; ++ob)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            *reinterpret_cast<float4*>(dst + ((ob * LBW + l) * 4 + j) * 1024 + lane * 16) =
                make_float4(acc[ob][l][4 * j], acc[ob][l][4 * j + 1], acc[ob][l][4 * j + 2], acc[ob][l][4 * j + 3]);
        *reinterpret_cast<float2*>(dst + MB * LBW * 4096 + l * 512 + lane * 8) = make_float2(run_max[l], run_sum[l]);
      }
    }
    lds_barrier();
#pragma unroll
    for (int l = 0; l < LBW; ++l) {
      if (past_links(l)) break;
      float2 ms[TP];
#pragma unroll
      for (int p = 0; p < TP; ++p) ms[p] = *reinterpret_cast<const float2*>(block + p * HG * MB * kPer + MB * LBW * 4096 + l * 512 + lane * 8);
      float top = ms[0].x;
#pragma unroll
      for (int p = 1; p < TP; ++p) top = fmaxf(top, ms[p].x);
      // (a tile without items has maximum -inf and weight zero; the first tile of a chunk has one; phi = SiLU has no maximum)
      float w[TP];
#pragma unroll
      for (int p = 0; p < TP; ++p)
        w[p] = PHI != kPhiSoftmax ? 1.f : ms[p].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ms[p].x - top) * c);
      if (tp == l % TP) {
        float sum = ms[0].y * w[0];
#pragma unroll
        for (int p = 1; p < TP; ++p) sum = fmaf(ms[p].y, w[p], sum);
        store_sums(l, top, sum);
      }
#pragma unroll
      for (int piece = 0; piece < MB * 4; ++piece) {
        const int ob = piece / 4, j = piece % 4;
        if ((l * MB * 4 + piece) % TP != tp) continue;  // uniform
        float4 v[TP];
#pragma unroll
        for (int p = 0; p < TP; ++p) v[p] = *reinterpret_cast<const float4*>(block + p * HG * MB * kPer + ((ob * LBW + l) * 4 + j) * 1024 + lane * 16);
        float4 sum = make_float4(v[0].x * w[0], v[0].y * w[0], v[0].z * w[0], v[0].w * w[0]);
#pragma unroll
        for (int p = 1; p < TP; ++p)
          sum.x = fmaf(v[p].x, w[p], sum.x), sum.y = fmaf(v[p].y, w[p], sum.y), sum.z = fmaf(v[p].z, w[p], sum.z), sum.w = fmaf(v[p].w, w[p], sum.w);
        store_piece(l, ob, j, sum);
      }
    }
  } else {
#pragma unroll
    for (int l = 0; l < LBW; ++l) {
      if (past_links(l)) break;
#pragma unroll
      for (int ob = 0; ob < MB; ++ob)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          store_piece(l, ob, j, make_float4(acc[ob][l][4 * j], acc[ob][l][4 * j + 1], acc[ob][l][4 * j + 2], acc[ob][l][4 * j + 3]));
      store_sums(l, run_max[l], run_sum[l]);
    }
  }
}

// Forms of a workgroup, by the amount of work (plan()):
//   kShort   one head, four waves: one step is all there is.  The most compute units share the first loads.
//   kNarrow  one head, eight waves: a row goes to h workgroups, but a workgroup covers many rows, which leaves few partials.
//   kWide    several heads, eight waves: for long histories, whose rows cost more than their partials.
//   kWalk, kWalkTogether  the kernels of mfma_history_walk.hip, one wave or one per head
enum Form { kShort, kNarrow, kWide, kWalk, kWalkTogether };
constexpr int waves_per_group(int form) { return form == kShort ? 4 : 8; }
constexpr int heads_per_group(int dh, int h, int form) { return form != kWide ? 1 : dh == 64 ? std::min(h, 2) : std::min(h, 4); }
constexpr int tiles_per_step(int dh, int h, int form) { return waves_per_group(form) / (heads_per_group(dh, h, form) * (dh / 32)); }

}  // namespace
}  // namespace lime
