// Baseline on the matrix cores: full target attention (Eq. 1 with the candidates as queries and
// the history as keys and values; the "MHA skyline" of Section 4.1).  Every candidate attends over
// all N history rows, so the work is O(C N d) per user - the cost LIME avoids.
//
// Two kernels.  (1) project_history_kernel computes K~ = E W_K and V~ = E W_V with the weight slices stationary in
// registers and writes both as MFMA fragment images, a head's tiles one after the other.  (2) target_attention_kernel
// projects its own queries, Q~ = T W_Q, keeps them in registers and walks the user's 32-item tiles:
//   S^T (32 items x 32 q) = K~_tile . Q~^T        O^T (d/h x 32 q) += V~_tile^T . P^T
// History rows at or beyond lens[b] are written as zeros by (1) and masked out of the softmax by (2).
#include <algorithm>
#include <type_traits>

#include "mfma.hpp"

namespace lime {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Fragments of one (user, head, tile of 32 items), 64 lanes of 16 bytes each: first the keys, then the values
//   keys   [K2]    : lane (item n, g), slot t = K~[32 tile + n][a dh + 16 kk + chain_k(g, t)]
//   values [2][MB] : lane (col c, g),  slot t = V~[32 tile + 16 f + chain_k(g, t)][a dh + 32 ob + c]
// Both are halves of accumulator blocks as they stand.  Tiles are stored in pairs (a stage of the attention kernel).
template <int DH>
struct TileImage {
  static constexpr int K2 = DH / 16, MB = DH / 32, kFrags = K2 + 2 * MB;
};

struct ProjArgs {
  const bf16_t* X;        // [B][rows][d]
  const int32_t* lens;    // nullable; rows >= lens[b] are treated as zeros
  const bf16x8 *Wk, *Wv;  // weight images
  bf16x8* Y;              // [B][h][tiles rounded up to pairs][frags][64]
  int B, rows, tiles;
};

// 2 H waves: H heads' keys, then H heads' values, so that a row is read from memory once for both; the waves copy a tile
// together through a register ring into LDS.  A user's tiles are filled up to whole pairs with zeros (the attention kernel
// walks pairs).  Tiles past a user's
// length are left out.  Consecutive tile numbers go to consecutive users, shifted by one from round to round, so that
// a workgroup's tiles differ both in user and in position (lengths are ragged).
// Bound by the rows' latency and the image's stores; at B=16 N=4096 d=256 it takes the place of two passes of 24-26 us
// each (one for keys, one for values, both over the rows past the lengths too).
template <int DH, int H>
__global__ __launch_bounds__(128 * H) void project_history_kernel(ProjArgs a) {
  using Img = TileImage<DH>;
  constexpr int D = DH * H, K1 = D / 16, MB = DH / 32, kThreads = 128 * H;
  constexpr int LW = DH / 32, CPR = D / 8;  // 16-byte loads per lane and tile, and per row
  constexpr int PITCH = 2 * D + 16;         // LDS row pitch of a tile, bytes
  __shared__ __attribute__((aligned(16))) unsigned char xs[2][32 * PITCH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, head = wave % H;
  const bool values = wave >= H;
  const int n = lane & 31, g = lane >> 5;
  const int tiles_alloc = (a.tiles + 1) & ~1, total = a.B * tiles_alloc;
  const bf16x8* img = (values ? a.Wv : a.Wk) + static_cast<int64_t>(head) * K1 * MB * 64 + lane;
  bf16x8 w[K1][MB];
#pragma unroll
  for (int kk = 0; kk < K1; ++kk)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) w[kk][mb] = img[(kk * MB + mb) * 64];

  // the next tile at or after number t with a valid row: its user and first row
  struct Tile {
    int t, b, i0, len;
  };
  auto find = [&](int t) {
    Tile r{t, 0, 0, 0};
    for (; r.t < total; r.t += gridDim.x) {
      const int pos = r.t / a.B;
      r.b = (r.t - pos * a.B + pos) % a.B, r.i0 = pos * 32;
      r.len = a.lens ? min(a.lens[r.b], a.rows) : a.rows;
      if (r.i0 < (r.len + 63) / 64 * 64) break;
    }
    return r;
  };
  // this wave's share of a tile; rows past the length as zeros
  auto issue = [&](const Tile& r, bf16x8 (&v)[LW]) {
    const bf16_t* X = a.X + static_cast<int64_t>(r.b) * a.rows * D;
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int q = j * kThreads + threadIdx.x, row = r.i0 + q / CPR;
      v[j] = *reinterpret_cast<const bf16x8*>(X + static_cast<int64_t>(min(row, a.rows - 1)) * D + q % CPR * 8);
      if (r.i0 + 32 > r.len) {  // uniform
#pragma unroll
        for (int t = 0; t < 8; ++t) v[j][t] = row < r.len ? v[j][t] : static_cast<__bf16>(0.f);
      }
    }
  };

  constexpr int P = 2;  // tiles in flight, besides the one in LDS
  Tile tile[P];
  bf16x8 ring[P][LW];
  tile[0] = find(blockIdx.x);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (p > 0) tile[p] = find(tile[p - 1].t + gridDim.x);
    if (tile[p].t < total) issue(tile[p], ring[p]);
  }
  auto step = [&](auto p_tag) {
    constexpr int p = decltype(p_tag)::value;
    const Tile now = tile[p];
    if (now.t >= total) return false;  // uniform
    unsigned char* buf = xs[p];
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int q = j * kThreads + threadIdx.x;
      *reinterpret_cast<bf16x8*>(buf + q / CPR * PITCH + q % CPR * 16) = ring[p][j];
    }
    // a wave arrives here only after it has read the tile before, so nobody still reads this buffer's last tile
    __syncthreads();
    tile[p] = find(tile[(p + P - 1) % P].t + gridDim.x);
    if (tile[p].t < total) issue(tile[p], ring[p]);

    bf16x8* dst = a.Y + ((static_cast<int64_t>(now.b) * H + head) * tiles_alloc + now.i0 / 32) * Img::kFrags * 64 + lane;
    const unsigned char* xrow = buf + n * PITCH + 16 * g;
    f32x16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
    if (values) {
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(xrow + 32 * kk);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = mfma32(x, w[kk][mb], acc[mb]);
        if (H == 8 && kk % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (128 registers a wave: fetch no further ahead)
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int f = 0; f < 2; ++f) dst[(Img::K2 + f * MB + mb) * 64] = pack_half(acc[mb], f);
    } else {
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(xrow + 32 * kk);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = mfma32(w[kk][mb], x, acc[mb]);
        if (H == 8 && kk % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (128 registers a wave: fetch no further ahead)
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int f = 0; f < 2; ++f) dst[(2 * mb + f) * 64] = pack_half(acc[mb], f);
    }
    return true;
  };
  while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
  }
}

struct AttnArgs {
  const bf16_t* T;       // [B][C][d]
  const bf16x8* Wq;      // weight image
  const bf16x8* KV;      // [B][h][tiles rounded up to pairs][frags][64]
  const int32_t* lens;
  bf16_t* O;
  int C, N, tiles, q_groups, pairs;  // q_groups: workgroups per (user, head) pair
  float scale;           // >= 0 (a negative scale is folded into the sign of the packed W_K)
};

// A workgroup is four waves of 64 queries of one (user, head).  The logits come out of the matrix instruction ready for
// the exponential: scale * log2(e) is multiplied into Q~ before its rounding, and the accumulator starts at minus the
// query's running maximum (kept as a block of 16 equal registers), which moves as soon as a logit passes it, so that the
// largest weight is one exactly.  The maximum over a tile costs one three-way instruction per two logits and a compare per
// block.  (Letting the maximum lag, so that it moves less often, rounds the largest weight like any other: at B=16 N=4096
// C=8192 d=256, by up to eight powers of two, 448 instead of 521 us, but outputs 0.1 to 2.5 % further from the exact ones.)
// Half a step is a (tile, 32-query block): its 16 logits per lane are turned into weights between the eight matrix
// instructions of S^T of the same queries' next tile and O^T of the half step before, one instruction and its share of
// the vector work at a time.
// Keys and values go from memory to LDS without registers, stages of two tiles in four buffers, asked for two stages
// ahead; a buffer is asked to be filled after the barrier that follows its last read.
// What bounds it: the vector ALUs, with 12.4 instructions per matrix instruction where the weights themselves need six (16
// exponentials, 16 additions, 8 conversions and 8 maxima for eight); most of the others are moves of the maximum.  The matrix cores are
// busy 41 % of the time (B=16 N<=4096 C=8192 d=256).
template <int DH, int H>
__global__ __launch_bounds__(256, 2) void target_attention_kernel(AttnArgs a) {
  using Img = TileImage<DH>;
  constexpr int D = DH * H, MB = DH / 32, K2 = DH / 16, K1 = D / 16;
  constexpr int QB = 2, kBuffers = 4, kStageFrags = 2 * Img::kFrags, kLoads = kStageFrags / 4;
  __shared__ bf16x8 kv_lds[kBuffers * kStageFrags * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, g = lane >> 5;
  // Consecutive workgroups go to consecutive XCDs.  A pair's workgroups share its keys and values, so an XCD gets whole
  // pairs: every eighth one (users' lengths differ: neighbours are spread), or a contiguous run of workgroups where the
  // pairs do not divide by eight.
  int pair, group;
  {
    const int xcd = blockIdx.x % 8, i = blockIdx.x / 8;
    if (a.pairs % 8 == 0) {
      pair = xcd + 8 * (i / a.q_groups), group = i % a.q_groups;
    } else {
      const int total = a.pairs * a.q_groups, per = (total + 7) / 8, l = xcd * per + i;
      if (l >= total) return;  // uniform over the workgroup
      pair = l / a.q_groups, group = l % a.q_groups;
    }
  }
  const int b = pair / H, head = pair % H;
  const int q0 = (group * 4 + wave) * QB * 32;  // (a wave past the last query works on the last row and stores nothing)
  const int len = __builtin_amdgcn_readfirstlane(a.lens ? min(a.lens[b], a.N) : a.N);
  const int tiles = (len + 31) / 32;

  const bf16x8* kv = a.KV + (static_cast<int64_t>(b) * H + head) * ((a.tiles + 1) & ~1) * Img::kFrags * 64;
  const int last_stage = (tiles - 1) / 2;
  // (a stage past the last is the last one again: the number of outstanding loads is then the same at every wait)
  auto load_stage = [&](int stage, int slot) {
    const bf16x8* src = kv + (static_cast<int64_t>(min(stage, last_stage)) * kStageFrags + wave * kLoads) * 64;
    const unsigned dst = lds_offset_of(kv_lds) + (slot * kStageFrags + wave * kLoads) * 1024;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load_to_lds(dst + j * 1024, lane * 16, src + j * 64);
  };
  auto publish = [&] {  // this wave's part of the stage about to be read has arrived; so has everybody's
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(kLoads) : "memory");  // all but the youngest stage
  };
  if (tiles > 0) {  // uniform
    load_stage(0, 0);
    load_stage(1, 1);
  }

  bf16x8 qf[QB][K2];
  {
    const bf16x8* wimg = a.Wq + static_cast<int64_t>(head) * K1 * MB * 64 + lane;
    f32x16 q[QB][MB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) q[qb][mb][i] = 0.f;
    const bf16_t* row[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) row[qb] = a.T + (static_cast<int64_t>(b) * a.C + min(q0 + 32 * qb + n, a.C - 1)) * D + 8 * g;
    // all rows are asked for at once, the weights (which every workgroup reads) kAhead k-steps ahead of their use
    constexpr int kAhead = K1 < 4 ? K1 : 4;
    bf16x8 x[QB][K1], w[K1][MB];
#pragma unroll
    for (int kk = 0; kk < K1; ++kk)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) x[qb][kk] = *reinterpret_cast<const bf16x8*>(row[qb] + 16 * kk);
#pragma unroll
    for (int kk = 0; kk < K1 + kAhead; ++kk) {
      if (kk < K1) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) w[kk][mb] = wimg[(kk * MB + mb) * 64];
      }
      if (kk >= kAhead) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) q[qb][mb] = mfma32(w[kk - kAhead][mb], x[qb][kk - kAhead], q[qb][mb]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const float c = a.scale * kLog2e;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        q[qb][mb] *= c;
        qf[qb][2 * mb] = pack_half(q[qb][mb], 0);
        qf[qb][2 * mb + 1] = pack_half(q[qb][mb], 1);
      }
  }

  f32x16 acc[QB][MB], base[QB];  // base: minus the running maximum
  float run_sum[QB][2];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    run_sum[qb][0] = run_sum[qb][1] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      base[qb][i] = 0.f;
#pragma unroll
      for (int ob = 0; ob < MB; ++ob) acc[qb][ob][i] = 0.f;
    }
  }

  if (tiles > 0) {  // uniform
    auto mask_tail = [&](f32x16& s, int t) {  // register 4j + r of this lane is item 32t + 8j + 4g + r
      int valid = len - 32 * t - 4 * g;
      asm volatile("" : "+v"(valid));  // (the comparisons stay in here)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float v = s[i];
        if (8 * (i >> 2) + (i & 3) >= valid) v = -INFINITY;
        asm volatile("" : "+v"(v));  // (kept apart from the unmasked maximum, which is one instruction only if nobody shares its halves)
        s[i] = v;
      }
    };
    auto move_base = [&](int qb, f32x16& s, float mx) {
      const float by = pair_max(mx);  // the query's other items are in the other lane of the pair
      // (> 0 except for the first tile, whose logits may be so low that 2^-by is infinite: there is nothing to keep yet)
      const float keep = by > 0.f ? __builtin_amdgcn_exp2f(-by) : 1.f;
      run_sum[qb][0] *= keep, run_sum[qb][1] *= keep;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        base[qb][i] -= by;
        s[i] -= by;
#pragma unroll
        for (int ob = 0; ob < MB; ++ob) acc[qb][ob][i] *= keep;
      }
    };
    // larger of mx >= 0 and two of the 16 logits, compared as integers: one instruction (a float maximum is two more to
    // quiet its operands)
    auto max_step = [&](const f32x16& s, int j, float mx) {
      return __int_as_float(max(max(__float_as_int(s[2 * j]), __float_as_int(s[2 * j + 1])), __float_as_int(mx)));
    };

    bf16x8 kf[K2], vf[2][MB];
    u32x4 pf[QB][2];  // weights in pairs
    f32x16 s[QB];
    float smax[QB];
    auto read_keys = [&](const bf16x8* tile) {
#pragma unroll
      for (int kk = 0; kk < K2; ++kk) kf[kk] = tile[kk * 64 + lane];
    };

    publish();
    load_stage(2, 2);
    read_keys(kv_lds);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      s[qb] = base[qb];
#pragma unroll
      for (int kk = 0; kk < K2; ++kk) s[qb] = mfma32(kf[kk], qf[qb][kk], s[qb]);
      mask_tail(s[qb], 0);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[qb][i]);
      move_base(qb, s[qb], mx);  // finite: the tile holds at least one valid item
      smax[qb] = 0.f;
    }
    read_keys(kv_lds + Img::kFrags * 64);
#pragma unroll
    for (int f = 0; f < 2; ++f) {
#pragma unroll
      for (int t = 0; t < 4; ++t) pf[1][f][t] = 0;  // there is no half step before the first
#pragma unroll
      for (int ob = 0; ob < MB; ++ob)
#pragma unroll
        for (int t = 0; t < 8; ++t) vf[f][ob][t] = static_cast<__bf16>(0.f);
    }

    // Half step (t, QBI): weights of s[QBI] (tile t), whose registers then take the logits of tile t + 1.
    constexpr int kSlots = K2 + 2 * MB;  // matrix instructions of a half step
    // After its last use a key or value fragment is read again for the next tile (half a step before its first use there):
    // the keys of `next_tile` in the second half of a tile, its values in the first.
    auto half_step = [&](auto qb_tag, int t, const bf16x8* next_tile) {
      constexpr int qb = decltype(qb_tag)::value, other = 1 - qb;
      if (32 * t + 32 > len) {  // uniform: the user's last tile; the maximum has to leave out what is masked
        mask_tail(s[qb], t);
        smax[qb] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) smax[qb] = max_step(s[qb], j, smax[qb]);
      }
      if (__any(smax[qb] > 0.f)) move_base(qb, s[qb], smax[qb]);
      f32x16 next = base[qb];
      float mx = 0.f, p0 = 0.f, p1 = 0.f;
      // a pair of weights, one step after its exponentials were asked for
      // (pinned where it stands: the compiler would sink all of it to the weights' use, behind the matrix instructions)
      auto finish = [&](int j) {
        run_sum[qb][0] += p0;
        run_sum[qb][1] += p1;
        bf16x2 pair;
        pair[0] = static_cast<__bf16>(p0), pair[1] = static_cast<__bf16>(p1);
        unsigned bits = __builtin_bit_cast(unsigned, pair);
        asm volatile("" : "+v"(bits), "+v"(run_sum[qb][0]), "+v"(run_sum[qb][1]));
        pf[qb][j / 4][j % 4] = bits;
      };
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kSlots; ++i) {
        // the product whose fragments this half step replaces comes first, so that they are there when it starts again
        const int u = i % (kSlots / 2);
        if ((i < kSlots / 2) == (qb == 1)) next = mfma32(kf[u], qf[qb][u], next);
        else acc[other][u % MB] = mfma32(vf[u / MB][u % MB], __builtin_bit_cast(bf16x8, pf[other][u / MB]), acc[other][u % MB]);
        if (i >= 1 && i <= kSlots / 2) {
          const int r = i - 1;
          if (qb == 1) kf[r] = next_tile[r * 64 + lane];
          else vf[r / MB][r % MB] = next_tile[(K2 + r) * 64 + lane];
        }
#pragma unroll
        for (int j = i * 8 / kSlots; j < (i + 1) * 8 / kSlots; ++j) {
          const float n0 = __builtin_amdgcn_exp2f(s[qb][2 * j]), n1 = __builtin_amdgcn_exp2f(s[qb][2 * j + 1]);
          if (j > 0) mx = max_step(s[other], j - 1, mx);
          if (j > 0) finish(j - 1);
          p0 = n0, p1 = n1;
          asm volatile("" : "+v"(p0), "+v"(p1), "+v"(mx));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      mx = max_step(s[other], 7, mx);
      finish(7);
      smax[other] = mx;
      s[qb] = next;
    };

    int slot = 0;  // buffer of the current stage
    for (int t = 0; t < tiles; t += 2) {
      const bf16x8* cur = kv_lds + slot * kStageFrags * 64;
      slot = (slot + 1) % kBuffers;
      const bf16x8* nxt = kv_lds + slot * kStageFrags * 64;
      half_step(std::integral_constant<int, 0>{}, t, cur);  // reads the values of tile t
      publish();
      load_stage(t / 2 + 3, (slot + 2) % kBuffers);
      half_step(std::integral_constant<int, 1>{}, t, nxt);  // the keys of tile t + 2
      half_step(std::integral_constant<int, 0>{}, t + 1, cur + Img::kFrags * 64);
      half_step(std::integral_constant<int, 1>{}, t + 1, nxt + Img::kFrags * 64);
    }
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int ob = 0; ob < MB; ++ob) acc[1][ob] = mfma32(vf[f][ob], __builtin_bit_cast(bf16x8, pf[1][f]), acc[1][ob]);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");  // nothing may arrive in LDS after the workgroup has gone
  }

  // lane (query n of block qb, g) holds head columns 32 ob + 8 j + 4 g + r in register 4 j + r
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int q = q0 + 32 * qb + n;
    const float total = pair_sum(run_sum[qb][0] + run_sum[qb][1]);
    const float inv = tiles > 0 ? 1.f / total : 0.f;
    if (q >= a.C) continue;
    bf16_t* orow = a.O + (static_cast<int64_t>(b) * a.C + q) * D + head * DH + 4 * g;
#pragma unroll
    for (int ob = 0; ob < MB; ++ob)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = static_cast<__bf16>(acc[qb][ob][4 * j + r] * inv);
        *reinterpret_cast<bf16x4*>(orow + 32 * ob + 8 * j) = v;
      }
  }
}

template <int DH, int H>
hipError_t run(const TargetAttention& q, void* workspace, hipStream_t s) {
  constexpr int D = DH * H;
  const int tiles = (q.N + 31) / 32;
  char* ws = static_cast<char*>(workspace);
  const size_t wimg = align_up(static_cast<size_t>(D) * D * 2);
  void *Wq = ws, *Wk = ws + wimg, *Wv = ws + 2 * wimg;
  bf16x8* KV = reinterpret_cast<bf16x8*>(ws + 3 * wimg);

  // a negative logit scale becomes an exact sign flip of the packed W_K
  PackWeight wjobs[3] = {{q.Wq, Wq, 1.f}, {q.Wk, Wk, q.scale < 0.f ? -1.f : 1.f}, {q.Wv, Wv, 1.f}};
  hipError_t e = pack_operands(wjobs, 3, nullptr, 0, D, H, 32, s);
  if (e != hipSuccess) return e;

  const int64_t total_tiles = static_cast<int64_t>(q.B) * ((tiles + 1) & ~1);
  // one resident workgroup per compute unit, two where the weight slices are small
  const int64_t resident = static_cast<int64_t>(compute_units()) * (D <= 128 && H <= 4 ? 2 : 1);
  ProjArgs p{static_cast<const bf16_t*>(q.E), q.lens, static_cast<const bf16x8*>(Wk), static_cast<const bf16x8*>(Wv), KV, q.B, q.N, tiles};
  launch_timed(kKernelProjection, project_history_kernel<DH, H>, dim3(static_cast<unsigned>(std::min(total_tiles, resident))), dim3(128 * H), 0, s, p);
  e = hipGetLastError();
  if (e != hipSuccess) return e;

  AttnArgs a{static_cast<const bf16_t*>(q.T), static_cast<const bf16x8*>(Wq), KV, q.lens, static_cast<bf16_t*>(q.O),
             q.C, q.N, tiles, (q.C + 255) / 256, q.B * H, fabsf(q.scale)};
  const int64_t groups = (static_cast<int64_t>(a.pairs) * a.q_groups + 7) / 8 * 8;
  if (groups >= (int64_t{1} << 31)) return hipErrorInvalidValue;
  launch_timed(kKernelTargetAttention, target_attention_kernel<DH, H>, dim3(static_cast<unsigned>(groups)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool target_attention_supported(int d, int h) {
  const int dh = d / h;
  return (dh == 32 || dh == 64) && (h == 1 || h == 2 || h == 4 || h == 8) && d <= 256;
}

size_t target_attention_workspace(int B, int C, int N, int d) {
  (void)C;
  const int tiles = (N + 31) / 32;
  return 3 * align_up(static_cast<size_t>(d) * d * 2) + align_up(static_cast<size_t>(B) * ((tiles + 1) & ~1) * 32 * d * 4);
}

hipError_t target_attention(const TargetAttention& q, void* workspace, hipStream_t s) {
  const int dh = q.d / q.h;
  if (dh == 32) {
    switch (q.h) {
      case 1: return run<32, 1>(q, workspace, s);
      case 2: return run<32, 2>(q, workspace, s);
      case 4: return run<32, 4>(q, workspace, s);
      case 8: return run<32, 8>(q, workspace, s);
    }
  } else if (dh == 64) {
    switch (q.h) {
      case 1: return run<64, 1>(q, workspace, s);
      case 2: return run<64, 2>(q, workspace, s);
      case 4: return run<64, 4>(q, workspace, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace lime
