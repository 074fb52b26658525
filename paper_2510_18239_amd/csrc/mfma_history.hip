// User-side link personalisation on the matrix cores: the launches of the kernels of history_body.hpp on packed operands, and
// the merge of their chunks.
#include "history_body.hpp"

namespace lime {
namespace {

struct MergeArgs {
  const float* part_acc;
  const float* part_ml;
  const int32_t* lens;
  bf16_t* LP;
  int N, chunk_items, chunks, h, m, dh;
  float scale;  // |logit scale|: the factor the SiLU partials still lack
};

// The merged link states of a user's chunks, one row LP[b][link] at a time by a workgroup of 2 d threads.  The sum over the
// chunks is one chain in ascending order per column, relative to a maximum that moves once per kMergeSpan chunks: the same in
// every kernel, so that a link state has the same bits whichever of them finishes it.
// The partials were written by other compute units and every read of them is a long-latency miss: thread (quad, group) asks
// for four adjacent columns of every eighth chunk, all reads of a batch of kMergeBatch before any is used, whether or not a
// user has that many chunks (what lies past its last one counts as zero, and need not have been written).  They meet in LDS,
// where thread (head, chunk) has left the chunk's weight, and a thread per column takes the chain.
// (With two batches of 16 chunks one after the other in 128 threads, each reading its columns of every chunk from memory, this
// took 3.5 of a merge_values_kernel's 5.9 us between its first and last instruction, at B=1 N=2048 d=256 m=64.)
constexpr int kMergeBatch = 32, kMergeSpan = 16, kMergeGroups = 8;
template <int PHI, int D>
struct MergeRow {
  static constexpr int kThreads = 2 * D, kQuads = D / 4, kLoads = kMergeBatch / kMergeGroups, kMaxHeads = D / 32;
  static constexpr int kMlPitch = kMergeBatch + 4;
  static_assert(kThreads == kQuads * kMergeGroups && 32 * kMaxHeads <= kThreads, "every chunk and every (head, chunk) has its thread");
  struct alignas(16) Lds {
    float part[kMergeBatch * D];
    float w[PHI == kPhiSoftmax ? kMaxHeads * kMlPitch : 1];  // the chunks' weights and sums, by head
    float sum[PHI == kPhiSoftmax ? kMaxHeads * kMlPitch : 1];
    float keep[PHI == kPhiSoftmax ? kMaxHeads * 2 : 1];      // what a span leaves of the sums before it
  };
  float4 ac[kLoads];
  float2 ml;
  int quad, group, head;
  int64_t first, stride;  // (head, link) slots: of the row in the user's first chunk, per chunk

  // asks for the first batch
  __device__ __forceinline__ void begin(const MergeArgs& a, int b, int link) {
    quad = threadIdx.x % kQuads, group = threadIdx.x / kQuads, head = 4 * quad / a.dh;
    stride = static_cast<int64_t>(a.h) * a.m;
    first = static_cast<int64_t>(b) * a.chunks * stride + link;
    ask(a, 0);
  }
  __device__ __forceinline__ void ask(const MergeArgs& a, int c0) {
    if (PHI == kPhiSoftmax) {
      // thread (head, chunk of the batch); the threads past the last head's repeat it
      const int hd = min(static_cast<int>(threadIdx.x) / kMergeBatch, a.h - 1), c = c0 + threadIdx.x % kMergeBatch;
      ml = *reinterpret_cast<const float2*>(a.part_ml + (first + hd * a.m + min(c, a.chunks - 1) * stride) * 2);
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      ac[i] = *reinterpret_cast<const float4*>(
          a.part_acc + (first + head * a.m + min(c0 + group + kMergeGroups * i, a.chunks - 1) * stride) * a.dh + 4 * quad % a.dh);
  }
  // the finished value of column threadIdx.x, in the first D threads
  __device__ __forceinline__ float finish(const MergeArgs& a, int len, Lds& lds) {
    const int used = (len + a.chunk_items - 1) / a.chunk_items;  // chunks that hold at least one valid item
    const int col = threadIdx.x, col_head = min(col, D - 1) / a.dh;
    float num = 0.f, den = 0.f, top = -INFINITY;
    for (int c0 = 0; c0 < used; c0 += kMergeBatch) {  // uniform
      if (c0 > 0) {
        ask(a, c0);
        lds_barrier();  // the last batch's have been read
      }
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const int c = group + kMergeGroups * i;
        *reinterpret_cast<float4*>(&lds.part[c * D + 4 * quad]) = c0 + c < used ? ac[i] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      if (PHI == kPhiSoftmax) {
        const int hd = threadIdx.x / kMergeBatch, c = threadIdx.x % kMergeBatch;  // (a head's two spans are two 16-lane rows)
        const bool live = c0 + c < used;
        const float x = live ? ml.x : -INFINITY, span = row_max(x);
        const u32x2 rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(span), __float_as_uint(span), false, false);
        const float top0 = fmaxf(top, __uint_as_float(rows[0])), top1 = fmaxf(top0, __uint_as_float(rows[1]));
        const float before = c < kMergeSpan ? top : top0, now = c < kMergeSpan ? top0 : top1;
        if (hd < a.h) {
          lds.w[hd * kMlPitch + c] = live ? __builtin_amdgcn_exp2f((x - now) * kLog2e) : 0.f;
          lds.sum[hd * kMlPitch + c] = live ? ml.y : 0.f;
          if (c % kMergeSpan == 0) lds.keep[hd * 2 + c / kMergeSpan] = __builtin_amdgcn_exp2f((before - now) * kLog2e);  // 0 on the first
        }
        top = top1;
      }
      lds_barrier();
      if (col >= D) continue;
#pragma unroll
      for (int s = 0; s < kMergeBatch; s += kMergeSpan) {
        if (c0 + s >= used) break;  // uniform
        if (PHI == kPhiSoftmax) {
          const float keep = lds.keep[col_head * 2 + s / kMergeSpan];
          num *= keep, den *= keep;
        }
#pragma unroll
        for (int c = s; c < s + kMergeSpan; c += 4) {
          float p[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) p[j] = lds.part[(c + j) * D + col];
          if (PHI == kPhiSoftmax) {
            const float4 w = *reinterpret_cast<const float4*>(&lds.w[col_head * kMlPitch + c]);
            const float4 l = *reinterpret_cast<const float4*>(&lds.sum[col_head * kMlPitch + c]);
            num = fmaf(w.w, p[3], fmaf(w.z, p[2], fmaf(w.y, p[1], fmaf(w.x, p[0], num))));
            den = fmaf(w.w, l.w, fmaf(w.z, l.z, fmaf(w.y, l.y, fmaf(w.x, l.x, den))));
          } else {
            num = (((num + p[0]) + p[1]) + p[2]) + p[3];
          }
        }
      }
    }
    if (used <= 0) return 0.f;
    return PHI == kPhiSoftmax ? num / den : num * (a.scale / static_cast<float>(len));
  }
};

// The same by one thread for its four columns, kMergeGroups chunks at a time: for calls with many rows, whose threads have
// few chunks each.  The maxima and sums of a batch are asked for together and stay in registers, and a group's partials are
// asked for during the group before (lime_request_prepared, 512 candidates, against reading the maxima group by group and
// again: 41.5 -> 39.6 us at B=5 N=13000 d=128 h=2 m=128, 36.7 -> 35.8 at B=3 N=8000 d=256 m=96, 31.9 -> 31.4 at B=4 N=4096
// d=256 m=128).  GROUPS: of a batch; 1 where a history has no more than kMergeGroups chunks, which the registers of the
// general form would slow (15.3 | 15.6 us at B=5 N=300 d=256 m=64, 14.5 | 14.8 at B=16 N=1024 d=128).
template <int PHI, int D, int GROUPS>
struct MergeQuad {
  static constexpr int kBatch = GROUPS * kMergeGroups;
  static_assert(kBatch == kMergeBatch || GROUPS == 1, "batches as in MergeRow, or one group and no other");
  int64_t first, stride;
  int link, quad;
  float2 ml[kMergeGroups];  // of the first group of a batch
  float4 ac[kMergeGroups];
  __device__ __forceinline__ void ask_ml(const MergeArgs& a, int c0, float2* to) {
#pragma unroll
    for (int q = 0; q < kMergeGroups; ++q) to[q] = *reinterpret_cast<const float2*>(a.part_ml + (first + min(c0 + q, a.chunks - 1) * stride) * 2);
  }
  __device__ __forceinline__ void ask(const MergeArgs& a, int c0, float4* to) {
#pragma unroll
    for (int q = 0; q < kMergeGroups; ++q)
      to[q] = *reinterpret_cast<const float4*>(a.part_acc + (first + min(c0 + q, a.chunks - 1) * stride) * a.dh + 4 * quad % a.dh);
  }
  __device__ __forceinline__ void begin(const MergeArgs& a, int b, int link_, int quad_) {
    link = link_, quad = quad_, stride = static_cast<int64_t>(a.h) * a.m;
    first = (static_cast<int64_t>(b) * a.chunks * a.h + 4 * quad / a.dh) * a.m + link;
    if (PHI == kPhiSoftmax) ask_ml(a, 0, ml);
    ask(a, 0, ac);
  }
  __device__ __forceinline__ float4 finish(const MergeArgs& a, int len) {
    const int used = (len + a.chunk_items - 1) / a.chunk_items;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f, top = -INFINITY;
    for (int c0 = 0; c0 < (GROUPS > 1 ? used : min(used, 1)); c0 += kBatch) {  // uniform, as every branch on `used` below
      float2 m[kBatch];
      if (c0 > 0) {
        if (PHI == kPhiSoftmax) ask_ml(a, c0, ml);
        ask(a, c0, ac);
      }
      float4 next[kMergeGroups];
      if (PHI == kPhiSoftmax) {
#pragma unroll
        for (int q = 0; q < kBatch; ++q) m[q] = q < kMergeGroups ? ml[q % kMergeGroups] : make_float2(-INFINITY, 0.f);
#pragma unroll
        for (int c = kMergeGroups; c < kBatch; c += kMergeGroups)
          if (c0 + c < used) ask_ml(a, c0 + c, m + c);
      }
      if (GROUPS > 1 && c0 + kMergeGroups < used) ask(a, c0 + kMergeGroups, next);
#pragma unroll
      for (int c = 0; c < kBatch; c += kMergeGroups) {
        if (c0 + c >= used) break;
        if (c > 0) {
#pragma unroll
          for (int q = 0; q < kMergeGroups; ++q) ac[q] = next[q];
          if (c + kMergeGroups < kBatch && c0 + c + kMergeGroups < used) ask(a, c0 + c + kMergeGroups, next);
        }
        if (PHI == kPhiSoftmax && c % kMergeSpan == 0) {
          float span_top = top;
#pragma unroll
          for (int q = c; q < c + kMergeSpan && q < kBatch; ++q) span_top = fmaxf(span_top, c0 + q < used ? m[q].x : -INFINITY);
          const float keep = __builtin_amdgcn_exp2f((top - span_top) * kLog2e);  // 0 on the first span
          num.x *= keep, num.y *= keep, num.z *= keep, num.w *= keep, den *= keep;
          top = span_top;
        }
#pragma unroll
        for (int q = 0; q < kMergeGroups; ++q) {
          if (c0 + c + q >= used) continue;
          if (PHI == kPhiSoftmax) {
            const float w = __builtin_amdgcn_exp2f((m[c + q].x - top) * kLog2e);
            num.x = fmaf(w, ac[q].x, num.x), num.y = fmaf(w, ac[q].y, num.y);
            num.z = fmaf(w, ac[q].z, num.z), num.w = fmaf(w, ac[q].w, num.w);
            den = fmaf(w, m[c + q].y, den);
          } else {
            num.x += ac[q].x, num.y += ac[q].y, num.z += ac[q].z, num.w += ac[q].w;
          }
        }
      }
    }
    if (used <= 0) return make_float4(0.f, 0.f, 0.f, 0.f);
    if (PHI == kPhiSoftmax) return make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
    const float f = a.scale / static_cast<float>(len);
    return make_float4(num.x * f, num.y * f, num.z * f, num.w * f);
  }
};

// Four rounded link-state values as one 8-byte store.
__device__ __forceinline__ void store_rounded(bf16_t* dst, const float4& v, bf16_t* again = nullptr) {
  alignas(8) bf16_t r[4];
  store_as(&r[0], v.x), store_as(&r[1], v.y), store_as(&r[2], v.z), store_as(&r[3], v.w);
  *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(r);
  if (again != nullptr) *reinterpret_cast<uint2*>(again) = *reinterpret_cast<const uint2*>(r);
}

// A workgroup per link state.
template <int PHI, int D>
__global__ __launch_bounds__(2 * D) void merge_kernel(MergeArgs a) {
  __shared__ typename MergeRow<PHI, D>::Lds lds;
  const int b = blockIdx.y, link = blockIdx.x;
  MergeRow<PHI, D> row;
  row.begin(a, b, link);
  const int len = a.lens ? min(a.lens[b], a.N) : a.N;
  const float v = row.finish(a, len, lds);
  if (threadIdx.x < D) store_as(a.LP + (static_cast<int64_t>(b) * a.m + link) * D + threadIdx.x, v);
}

// A thread per four columns of a link state.
constexpr int kMergeManyThreads = 64;
template <int PHI, int D, int GROUPS>
__global__ __launch_bounds__(kMergeManyThreads) void merge_many_kernel(MergeArgs a) {
  const int b = blockIdx.y, idx = blockIdx.x * kMergeManyThreads + threadIdx.x;  // (m d / 4 is a multiple of 64)
  MergeQuad<PHI, D, GROUPS> task;
  task.begin(a, b, idx / (D / 4), idx % (D / 4));
  const int len = a.lens ? min(a.lens[b], a.N) : a.N;
  store_rounded(a.LP + (static_cast<int64_t>(b) * a.m + task.link) * D + 4 * task.quad, task.finish(a, len));
}

// Layer normalisation of a finished link state by a wavefront, from x(k) to put(k, value): mean, centred second moment, then
// the normalised row rounded to bf16, as a normalisation pass of its own would have stored it.
// (the lane through an opaque copy: what is derived from it - addresses, the scale and the shift - is then computed and
// fetched here, not ahead of the merge, which has no registers to carry it; the fetches are in flight during the two
// reductions)
template <int D, typename X, typename Put>
__device__ __forceinline__ void normalise_state(const bf16_t* gamma, const bf16_t* beta, float eps, X x, Put put) {
  constexpr int kPerLane = (D + 63) / 64;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  bf16_t ga[kPerLane], be[kPerLane];
#pragma unroll
  for (int i = 0; i < kPerLane; ++i) {
    const int k = min(lane + 64 * i, D - 1);
    ga[i] = gamma[k], be[i] = beta[k];
  }
  float v[kPerLane], sum = 0.f, q = 0.f;
#pragma unroll
  for (int i = 0; i < kPerLane; ++i) v[i] = lane + 64 * i < D ? x(lane + 64 * i) : 0.f, sum += v[i];
  const float mean = wave_sum(sum) * (1.f / D);
#pragma unroll
  for (int i = 0; i < kPerLane; ++i) {
    v[i] = lane + 64 * i < D ? v[i] - mean : 0.f;
    q = fmaf(v[i], v[i], q);
  }
  const float inv = 1.f / sqrtf(wave_sum(q) * (1.f / D) + eps);
#pragma unroll
  for (int i = 0; i < kPerLane; ++i)
    if (lane + 64 * i < D) put(lane + 64 * i, static_cast<__bf16>(fmaf(v[i] * inv, to_float(ga[i]), to_float(be[i]))));
}

// Merge and the candidate stage's value projection in one kernel: a workgroup finishes link states of one user, stores them,
// and projects their bf16-rounded values onto Wv: V~ = LP Wv, written as the value image (kPackValues) that the
// candidate-side kernel loads.  (The sums of the projection are in another order than the pack kernel's: V~ of a request and
// of lime_score_candidates on its link states agree to the last bits of fp32, before their rounding to bf16.)
struct MergeValuesArgs {
  MergeArgs m;
  const bf16_t* Wv;  // [d][d], nullable = identity
  bf16_t* VA;        // [B] value images
  // layer normalisation of the finished link states before the projection (ln_on; LP is stored un-normalised)
  const bf16_t *ln_gamma, *ln_beta;
  float ln_eps;
  int ln_on;
};

// A link state per workgroup, for calls whose workgroups then all run at once.  The projection is on the vector ALUs: thread
// (cg, kc) owns 8 adjacent columns and every sixteenth k; the partial sums meet in LDS.
template <int PHI, int D>
__global__ __launch_bounds__(2 * D) void merge_values_kernel(MergeValuesArgs a) {
  constexpr int kThreads = 2 * D, CG = D / 8, nkc = 16, kMaxK = D / nkc;
  static_assert(CG * nkc == kThreads, "one thread per (column group, k-group)");
  __shared__ typename MergeRow<PHI, D>::Lds lds;
  __shared__ __attribute__((aligned(16))) float lp[D];  // bf16-rounded values
  // (a column c sits at c + c / 32: the writers' columns are 8 apart, which would otherwise share four banks)
  constexpr int kRedRow = D + D / 32;
  __shared__ float red[nkc * kRedRow];
  const int tid = threadIdx.x, b = blockIdx.y, link = blockIdx.x;
  const int cg = tid % CG, kc = tid / CG;
  MergeRow<PHI, D> merge;
  merge.begin(a.m, b, link);
  bf16x8 wreg[kMaxK];
  if (a.Wv != nullptr) {  // asked for behind the partials, used after them
#pragma unroll
    for (int it = 0; it < kMaxK; ++it)
      wreg[it] = *reinterpret_cast<const bf16x8*>(a.Wv + static_cast<int64_t>(kc + it * nkc) * D + 8 * cg);
  }
  const int len = a.m.lens ? min(a.m.lens[b], a.m.N) : a.m.N;
  const float v = merge.finish(a.m, len, lds);
  if (tid < D) {
    bf16_t r;
    store_as(&r, v);
    a.m.LP[(static_cast<int64_t>(b) * a.m.m + link) * D + tid] = r;
    lp[tid] = to_float(r);
  }
  __syncthreads();
  if (a.ln_on) {  // uniform
    if (tid < 64) normalise_state<D>(a.ln_gamma, a.ln_beta, a.ln_eps, [&](int k) { return lp[k]; }, [&](int k, __bf16 y) { lp[k] = static_cast<float>(y); });
    __syncthreads();
  }
  float out = 0.f;
  if (a.Wv == nullptr) {
    if (tid < D) out = lp[tid];
  } else {
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll
    for (int it = 0; it < kMaxK; ++it) {
      const float x = lp[kc + it * nkc];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] = fmaf(x, static_cast<float>(wreg[it][j]), acc[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[kc * kRedRow + 8 * cg + j + (cg >> 2)] = acc[j];
    __syncthreads();
    if (tid < D)
#pragma unroll
      for (int c = 0; c < nkc; ++c) out += red[c * kRedRow + tid + tid / 32];
  }
  if (tid < D) store_as(a.VA + values_slot(b, link, tid, D, a.m.dh, a.m.m, true), out);
}

// ROWS (8 or 16) link states per workgroup, for calls with many: the projection is on the matrix cores (a 32-row block repeats
// them), W_V goes straight to LDS and is turned on its way out, a wavefront's 32 columns in its own part.
template <int PHI, int D, int ROWS>
struct MergeTile {
  static constexpr int kRows = ROWS, NK = D / 16, kWaves = D / 32, kPitch = D + 8, kTasks = kRows * (D / 4) / (2 * D);
  static constexpr int kLds = kWaves * NK * 1024 + kRows * kPitch * 2;
};
template <int PHI, int D, int ROWS, int GROUPS>
__global__ __launch_bounds__(2 * D) void merge_values_tile_kernel(MergeValuesArgs a) {
  using T = MergeTile<PHI, D, ROWS>;
  constexpr int NK = T::NK, kTasks = T::kTasks, kQuads = D / 4;
  extern __shared__ unsigned char lds[];
  bf16_t* const rows = reinterpret_cast<bf16_t*>(lds + T::kWaves * NK * 1024);
  const int lane = threadIdx.x & 63, n = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.y, link0 = blockIdx.x * T::kRows, dh = a.m.dh;
  unsigned char* const mine = lds + wave * NK * 1024;
  MergeQuad<PHI, D, GROUPS> task[kTasks];
#pragma unroll
  for (int i = 0; i < kTasks; ++i) {
    const int idx = threadIdx.x + i * 2 * D;
    task[i].begin(a.m, b, link0 + idx / kQuads, idx % kQuads);
  }
  if (a.Wv != nullptr) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
      load_to_lds(lds_offset_of(mine) + kk * 1024, (lane / 4) * (2 * D) + lane % 4 * 16, a.Wv + static_cast<int64_t>(16 * kk) * D + 32 * wave);
  }
  const int len = a.m.lens ? min(a.m.lens[b], a.m.N) : a.m.N;
#pragma unroll
  for (int i = 0; i < kTasks; ++i) {
    const int link = task[i].link, quad = task[i].quad;
    store_rounded(a.m.LP + (static_cast<int64_t>(b) * a.m.m + link) * D + 4 * quad, task[i].finish(a.m, len), rows + (link - link0) * T::kPitch + 4 * quad);
  }
  wait_lds_loads<0>();  // W_V's part of this wave
  __syncthreads();
  if (a.ln_on) {  // uniform
    for (int r = wave; r < T::kRows; r += T::kWaves) {
      bf16_t* x = rows + r * T::kPitch;
      normalise_state<D>(a.ln_gamma, a.ln_beta, a.ln_eps, [&](int k) { return to_float(x[k]); },
                         [&](int k, __bf16 y) { x[k].bits = __builtin_bit_cast(uint16_t, y); });
    }
    __syncthreads();
  }
  bf16x8 values;  // lane (column 32 wave + n, g), slot t = link chain_k(g, t) of sixteen (of eight: the first four slots)
  if (a.Wv == nullptr) {
#pragma unroll
    for (int t = 0; t < 8; ++t) values[t] = __builtin_bit_cast(__bf16, rows[chain_k(g, t) % ROWS * T::kPitch + 32 * wave + n].bits);
  } else {
    bf16x8 x[NK], w[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      x[kk] = *reinterpret_cast<const bf16x8*>(rows + n % ROWS * T::kPitch + 16 * kk + 8 * g);
      w[kk] = column_fragment(mine + kk * 1024, 64, lane);
    }
    values = pack_half(project_block<NK>(x, w), 0);
  }
  const int64_t frag = ((static_cast<int64_t>(b) * a.m.h + 32 * wave / dh) * (a.m.m / 16) + link0 / 16) * (dh / 32) + 32 * wave % dh / 32;
  bf16_t* dst = a.VA + (frag * 64 + out_rho(n) + 32 * g) * 8;
  if constexpr (ROWS == 16)
    *reinterpret_cast<bf16x8*>(dst) = values;
  else  // (links 8 .. 15 of the sixteen are the last four slots)
    *reinterpret_cast<bf16x4*>(dst + link0 % 16 / 2) = __builtin_shufflevector(values, values, 0, 1, 2, 3);
}

template <int DH, int M, int H, int PHI, int FORM>
hipError_t launch_shape(const HistArgs& a, int users, hipStream_t s) {
  constexpr int HG = heads_per_group(DH, H, FORM), TP = tiles_per_step(DH, H, FORM);
  using S = HistShape<DH, M, H, HG, TP>;
  static_assert(S::kLds <= 160 * 1024, "LDS");
  auto kernel = links_over_history_kernel<DH, M, H, PHI, HG, TP, false>;
  if (S::kLds > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), S::kLds); e != hipSuccess) return e;
  }
  launch_timed(kKernelLinksOverHistory, kernel, dim3(a.chunks, users, H / HG), dim3(S::kThreads), S::kLds, s, a, PackedArgs{});
  return hipGetLastError();
}

template <int DH, int M, int H, int PHI>
hipError_t launch_form(const HistArgs& a, int users, int form, hipStream_t s) {
  if constexpr (H > 1) {
    if (form == kWide) return launch_shape<DH, M, H, PHI, kWide>(a, users, s);
  }
  return form == kShort ? launch_shape<DH, M, H, PHI, kShort>(a, users, s) : launch_shape<DH, M, H, PHI, kNarrow>(a, users, s);
}

template <int DH, int M, int H>
hipError_t launch_main(const HistArgs& a, int phi, int users, int form, hipStream_t s) {
  return phi == kPhiSoftmax ? launch_form<DH, M, H, kPhiSoftmax>(a, users, form, s) : launch_form<DH, M, H, kPhiSilu>(a, users, form, s);
}

template <int DH, int H>
hipError_t dispatch_m(const HistArgs& a, int links, int phi, int users, int form, hipStream_t s) {
  switch (links) {
    case 32: return launch_main<DH, 32, H>(a, phi, users, form, s);
    case 64: return launch_main<DH, 64, H>(a, phi, users, form, s);
    case 96: return launch_main<DH, 96, H>(a, phi, users, form, s);
    case 128: return launch_main<DH, 128, H>(a, phi, users, form, s);
  }
  return hipErrorInvalidValue;
}

template <int DH>
hipError_t dispatch_h(const HistArgs& a, int h, int links, int phi, int users, int form, hipStream_t s) {
  switch (h) {
    case 1: return dispatch_m<DH, 1>(a, links, phi, users, form, s);
    case 2: return dispatch_m<DH, 2>(a, links, phi, users, form, s);
    case 4: return dispatch_m<DH, 4>(a, links, phi, users, form, s);
    case 8: if (DH == 32) return dispatch_m<32, 8>(a, links, phi, users, form, s);
  }
  return hipErrorInvalidValue;
}

// One link state per workgroup where all of them run at once with eight waves a compute unit.  What a workgroup takes off is
// the wait for many chunks, so the two sides cross at different numbers of rows.  In us, a workgroup a row | the other form,
// lime_request_prepared with 16 candidates: d=256 m=64 B=4 (256 rows) N=2048 18.4|20.3, N=300 15.6|15.5, B=6 N=300 17.2|16.2; m=128
// B=2 N=2048 23.2|28.0; d=128 m=64 B=4 N=2048 12.8|13.7, B=8 (512 rows) N=500 13.2|12.6, B=12 13.9|12.6.  lime_link_history: d=256 m=64
// B=1 N=2048 12.6|14.7; d=128 m=64 B=8 N=16384 26.7|28.0, N=500 12.1|11.5, B=32 N=1024 17.3|15.5.
bool few_rows(int64_t rows, int d) { return rows <= static_cast<int64_t>(compute_units()) * (256 / d); }

template <int PHI, int D>
hipError_t launch_merge(const MergeArgs& a, int users, hipStream_t s) {
  if (few_rows(static_cast<int64_t>(users) * a.m, D))
    hipLaunchKernelGGL((merge_kernel<PHI, D>), dim3(a.m, users), dim3(2 * D), 0, s, a);
  else if (a.chunks <= kMergeGroups)
    hipLaunchKernelGGL((merge_many_kernel<PHI, D, 1>), dim3(a.m * (D / 4) / kMergeManyThreads, users), dim3(kMergeManyThreads), 0, s, a);
  else
    hipLaunchKernelGGL((merge_many_kernel<PHI, D, kMergeBatch / kMergeGroups>), dim3(a.m * (D / 4) / kMergeManyThreads, users), dim3(kMergeManyThreads), 0, s, a);
  return hipGetLastError();
}

template <int PHI, int D, int ROWS, int GROUPS>
hipError_t launch_merge_values_tile(const MergeValuesArgs& a, int users, hipStream_t s) {
  using T = MergeTile<PHI, D, ROWS>;
  auto kernel = merge_values_tile_kernel<PHI, D, ROWS, GROUPS>;
  if (T::kLds > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), T::kLds); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(a.m.m / ROWS, users), dim3(2 * D), T::kLds, s, a);
  return hipGetLastError();
}
template <int PHI, int D, int ROWS>
hipError_t launch_merge_values_tile(const MergeValuesArgs& a, int users, hipStream_t s) {
  if (a.m.chunks <= kMergeGroups) return launch_merge_values_tile<PHI, D, ROWS, 1>(a, users, s);
  // (sixteen rows a workgroup: users x m d > 2048 compute units, and plan() then makes no more than eight chunks; only the
  // histories of mfma_history_walk.hip, softmax all, come in more)
  if constexpr (ROWS == 16 && PHI == kPhiSilu)
    return hipErrorInvalidValue;
  else
    return launch_merge_values_tile<PHI, D, ROWS, kMergeBatch / kMergeGroups>(a, users, s);
}
template <int PHI, int D>
hipError_t launch_merge_values(const MergeValuesArgs& a, int users, hipStream_t s) {
  const int64_t rows = static_cast<int64_t>(users) * a.m.m;
  if (few_rows(rows, D)) {
    hipLaunchKernelGGL((merge_values_kernel<PHI, D>), dim3(a.m.m, users), dim3(2 * D), 0, s, a);
    return hipGetLastError();
  }
  // Eight rows each as long as the workgroups then all run at once, counted as in few_rows.  lime_request_prepared with 16
  // candidates, N=60, eight | sixteen rows, us: d=256 m=64 1536 rows 15.6|17.4, 2048 16.0|17.5, 2560 19.8|18.1, 4096 21.7|19.2
  // (m=128 20.4|21.9, 21.6|22.2, 25.1|22.5, 26.6|23.8); d=128 m=64 2048 rows 13.0|13.7, 4096 14.8|14.8, 8192 25.6|24.8; d=64 m=64
  // 6144 rows 12.7|13.2, 8192 13.2|13.5, 16384 22.1|21.8.  (Below d = 256 the form for few chunks leaves room for more at once,
  // and the two are within 6 % of each other around the line.)
  return few_rows(rows / 8, D) ? launch_merge_values_tile<PHI, D, 8>(a, users, s) : launch_merge_values_tile<PHI, D, 16>(a, users, s);
}

struct Layout {
  int chunk_items, chunks, form;
  size_t wk, wv, qb, acc, ml, total;
};

Layout plan(int B, int N, int d, int h, int m, bool q_per_user, bool walk) {
  Layout l{};
  auto sized = [&] {
    l.wk = l.wv = align_up(static_cast<size_t>(d) * d * 2);
    l.qb = align_up(static_cast<size_t>(q_per_user ? B : 1) * m * d * 2);
    l.acc = align_up(static_cast<size_t>(B) * l.chunks * m * d * sizeof(float));
    l.ml = align_up(static_cast<size_t>(B) * l.chunks * h * m * 2 * sizeof(float));
    l.total = l.wk + l.wv + l.qb + l.acc + l.ml;
    return l;
  };
  if (walk) {
    const WalkPlan w = walk_plan(B, N, d, h);
    l.chunk_items = w.chunk_items, l.chunks = w.chunks, l.form = w.coop ? kWalkTogether : kWalk;
    return sized();
  }
  // A workgroup per compute unit, and the smallest form that then has one step, or the one for the amount of work.
  // Measured, history + merge kernel in us, for four-wave, narrow and wide groups:
  //   B=1 N=2048 d=256: 11.7, 12.9, 13.1     B=32 N=1024 d=128: 15.0, 15.1, 18.1     B=32 N=2048 d=128: 20.2, 18.8, 20.5
  //   B=8 N=16384 d=128: 31.1, 26.3, 25.5    B=16 N=4096 d=256: 36.4, 34.2, 32.4
  // The line between narrow and wide, at B tiles d = 2048 slots: where they cross depends on the shape.  lime_link_history
  // on prepared operands in us, narrow | wide, at 1434, 1741, 2048, 2458 and 3072 slots (SiLU crosses at the same places):
  //   B=8 d=128 h=4 m=64:  20.2|22.5  22.3|23.6  24.2|24.8  28.1|27.9  32.1|31.1
  //   B=32 d=128 h=4 m=64: 20.5|21.9  22.2|22.6  24.5|24.1  28.0|27.4  32.0|30.4
  //   B=8 d=256 h=4 m=64:  24.7|24.1  27.1|26.5  29.9|28.7  34.1|32.6  39.7|37.7
  //   B=8 d=256 h=4 m=128: 33.7|32.2  37.1|35.6  41.1|39.3  47.1|43.9  54.5|50.8
  // With h = 8 wide is ahead from 1000 slots on (30.3|27.1 at 1741), with h = 2 from 4096, for one user later still
  // (36.6|37.2 at 1741, 33.7|38.8 at 2048, d=256).  One line for all, where four heads of width 32 cross.
  const int64_t slots = compute_units();
  const int tiles = (N + 31) / 32;
  int tp = 1, groups = 1, steps = tiles;
  auto shape = [&](int form) {
    l.form = form;
    tp = tiles_per_step(d / h, h, form), groups = h / heads_per_group(d / h, h, form), steps = (tiles + tp - 1) / tp;
  };
  shape(kShort);
  if (static_cast<int64_t>(B) * steps * groups > slots) shape(h > 1 && static_cast<int64_t>(B) * tiles * d >= 2048 * slots ? kWide : kNarrow);
  int chunk_steps = static_cast<int>((static_cast<int64_t>(B) * steps * groups + slots - 1) / slots);
  if (chunk_steps > steps) chunk_steps = steps;
  l.chunk_items = chunk_steps * tp * 32;
  l.chunks = (steps + chunk_steps - 1) / chunk_steps;
  return sized();
}

}  // namespace

bool links_over_history_takes(const LinksOverHistory& q, const PackJobs& beside) {
  if (q.walk || q.prepared != nullptr || q.images[0] != nullptr || q.packed || q.q_norm.on) return false;
  const Layout l = plan(q.B, q.N, q.d, q.h, q.m, q.lc_user_stride != 0, false);
  return l.form == kShort && history_raw_fits(q, static_cast<int64_t>(q.B) * l.chunks * q.h, beside);
}

bool links_over_history_supported(int d, int h, int m) { return queries_over_links_supported(d, h, m); }

size_t links_over_history_workspace(int B, int N, int d, int h, int m, bool q_per_user) {
  return std::max(plan(B, N, d, h, m, q_per_user, false).total, plan(B, N, d, h, m, q_per_user, true).total);
}

void links_over_history_jobs(const LinksOverHistory& q, void* workspace, PackJobs& jobs) {
  const Layout l = plan(q.B, q.N, q.d, q.h, q.m, q.lc_user_stride != 0, q.walk);
  char* ws = static_cast<char*>(workspace);
  jobs.weights[jobs.n_weights++] = PackWeight{q.Wk, ws};
  jobs.weights[jobs.n_weights++] = PackWeight{q.Wv, ws + l.wk};
  // a negative logit scale is folded into the sign of the packed queries, so the kernels see scale >= 0
  jobs.projections[jobs.n_projections++] = PackProject{q.LC, q.Wq, ws + l.wk + l.wv, q.lc_user_stride,
                                                       q.lc_user_stride != 0 ? q.B : 1, kPackKeys, q.scale < 0.f ? -1.f : 1.f, q.q_norm};
}

hipError_t links_over_history(const LinksOverHistory& q, void* workspace, hipStream_t s) {
  const int d = q.d, h = q.h, m = q.m, dh = d / h;
  const bool per_user = q.lc_user_stride != 0;
  const Layout l = plan(q.B, q.N, d, h, m, per_user, q.walk);
  char* ws = static_cast<char*>(workspace);
  void* WkA = ws;
  void* WvB = ws + l.wk;
  void* QB = ws + l.wk + l.wv;
  float* part_acc = reinterpret_cast<float*>(ws + l.wk + l.wv + l.qb);
  float* part_ml = reinterpret_cast<float*>(ws + l.wk + l.wv + l.qb + l.acc);

  hipError_t e = hipSuccess;
  if (q.prepared != nullptr) {  // nothing to pack
    const PreparedLayout pl = prepared_layout(d, m);
    char* base = const_cast<char*>(static_cast<const char*>(q.prepared));
    WkA = base + pl.wk, WvB = base + pl.wv, QB = base + pl.qb;
  } else if (q.images[0] != nullptr) {
    WkA = const_cast<void*>(q.images[0]), WvB = const_cast<void*>(q.images[1]), QB = const_cast<void*>(q.images[2]);
  } else if (!q.packed && q.beside == nullptr) {
    PackJobs jobs;
    links_over_history_jobs(q, workspace, jobs);
    e = pack_operands(jobs, d, h, m, s);
    if (e != hipSuccess) return e;
  }

  HistArgs a{};
  a.E = static_cast<const bf16_t*>(q.E), a.lens = q.lens;
  a.WkA = static_cast<const bf16x8*>(WkA), a.WvB = static_cast<const bf16x8*>(WvB);
  a.QB = static_cast<const bf16x8*>(QB);
  a.qb_user_frags = per_user ? static_cast<int64_t>(m) * d / 8 : 0;
  a.part_acc = part_acc, a.part_ml = part_ml;
  a.N = q.N, a.chunk_items = l.chunk_items, a.chunks = l.chunks, a.scale = fabsf(q.scale);
  if (q.beside != nullptr)
    e = history_raw(a, q, s);
  else if (q.walk)
    e = walk_history(a, d, h, m, q.B, l.form == kWalkTogether, s);
  else
    e = dh == 32 ? dispatch_h<32>(a, h, m, q.phi, q.B, l.form, s) : dispatch_h<64>(a, h, m, q.phi, q.B, l.form, s);
  if (e != hipSuccess) return e;

  MergeArgs g{part_acc, part_ml, q.lens, static_cast<bf16_t*>(q.LP), q.N, l.chunk_items, l.chunks, h, m, dh, fabsf(q.scale)};
  const bool softmax = q.phi == kPhiSoftmax;
  if (q.values_image != nullptr) {
    MergeValuesArgs mv{g, static_cast<const bf16_t*>(q.Wv_values), static_cast<bf16_t*>(q.values_image),
                       static_cast<const bf16_t*>(q.values_norm.gamma), static_cast<const bf16_t*>(q.values_norm.beta),
                       q.values_norm.eps, q.values_norm.on ? 1 : 0};
    switch (d) {  // every d the matrix-core kernels take
      case 32: return softmax ? launch_merge_values<kPhiSoftmax, 32>(mv, q.B, s) : launch_merge_values<kPhiSilu, 32>(mv, q.B, s);
      case 64: return softmax ? launch_merge_values<kPhiSoftmax, 64>(mv, q.B, s) : launch_merge_values<kPhiSilu, 64>(mv, q.B, s);
      case 128: return softmax ? launch_merge_values<kPhiSoftmax, 128>(mv, q.B, s) : launch_merge_values<kPhiSilu, 128>(mv, q.B, s);
      case 256: return softmax ? launch_merge_values<kPhiSoftmax, 256>(mv, q.B, s) : launch_merge_values<kPhiSilu, 256>(mv, q.B, s);
    }
    return hipErrorInvalidValue;
  }
  switch (d) {
    case 32: return softmax ? launch_merge<kPhiSoftmax, 32>(g, q.B, s) : launch_merge<kPhiSilu, 32>(g, q.B, s);
    case 64: return softmax ? launch_merge<kPhiSoftmax, 64>(g, q.B, s) : launch_merge<kPhiSilu, 64>(g, q.B, s);
    case 128: return softmax ? launch_merge<kPhiSoftmax, 128>(g, q.B, s) : launch_merge<kPhiSilu, 128>(g, q.B, s);
    case 256: return softmax ? launch_merge<kPhiSoftmax, 256>(g, q.B, s) : launch_merge<kPhiSilu, 256>(g, q.B, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lime
