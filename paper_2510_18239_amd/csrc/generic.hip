// General kernels: fp32 arithmetic, any shape with d/h <= 256.
// They serve the fp32 storage type and every bf16 shape the bf16 matrix-core kernels do
// not cover.  Each step is the plain definition (Eq. 1): a projection X~ = X W and an
// attention (phi(scale * Q~ K~^T) restricted to the valid keys) V~.
//
// Both run on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums, twice the rate of
// the vector ALUs' unpacked multiply-add), whose fragments are one float per lane:
//   A (32 x 2): lane (n, g) = A[row n][k = g];  B (2 x 32): lane (n, g) = B[k = g][col n];
//   D (32 x 32): lane (n, g), register 4j + r = D[row 8j + 4g + r][col n]          (lane = 32 g + n)
// A sum does not care about the order of its terms, so the two k of an instruction need not be neighbours: with
// k = 8j + i and 8j + 4 + i, i = 0..3, a lane's operands of four instructions are four consecutive floats, one 16-byte
// load; and a D block is, register by register, the B operand of a product that sums over its rows.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "mfma.hpp"

namespace lime {
namespace {

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// ----------------------------------------------------------------------------- projections
// Up to kMaxProjections products Y[rows][d] (fp32) = X[rows][d] W[d][d] in one launch: what a call has to project
// before its attention is independent, and at a few hundred rows each a launch costs more than the product.
// A workgroup computes a TM x TN tile (TM TN = 4096, a 32 x 32 block per wave; 128 x 32 for d <= 32), k in steps of 32
// through two LDS buffers, the next step's loads in flight during the current one's products.  A lane's A operands of
// four instructions are one 16-byte LDS read (row pitch 36 floats: eight rows cover all banks), its B operands four
// 4-byte reads of a row of W (pitch TN + 8: the lane halves, four rows apart, fall on different banks).
// What bounds it: at 16016 x 128 fp32 rows the matrix instruction (64 cycles per 32 x 32 x 2); at a few rows the launch.
constexpr int kProjK = 32;
struct ProjectJob {
  const void* X;
  const void* W;  // nullable = identity: X is copied
  float* Y;
  const int32_t* lens;  // nullable; rows of a user at or past its length need not be computed
  int64_t rows;
  int64_t rows_per_user;
};
struct ProjectArgs {
  int first_tile[kMaxProjections];  // of each job; past the last job the largest int
  int d;
  ProjectJob job[kMaxProjections];  // (a workgroup reads the first tiles and then its job: two scalar loads, one after the other)
};

template <typename T>
struct Vec8 {  // eight consecutive elements as one or two 16-byte loads
  float v[8];
  __device__ __forceinline__ void load(const T* p) {
    if constexpr (sizeof(T) == 4) {
      const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
      v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    } else {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = static_cast<float>(a[t]);
    }
  }
};

// VEC: d is a multiple of 8 and every X and W is 16-byte aligned.
template <typename T, int TN, bool VEC>
__global__ __launch_bounds__(256) void project_kernel(ProjectArgs a) {
  constexpr int TM = 4096 / TN, XP = kProjK + 4, WP = TN + 8;
  constexpr int XL = TM * kProjK / 8 / 256;  // 8-element pieces of the X tile per thread (1 or 2)
  constexpr int WL = kProjK * TN / 8;        // 8-element pieces of the W tile (256, or 128: the first half of the threads)
  __shared__ __attribute__((aligned(16))) float xs[2][TM * XP];
  __shared__ __attribute__((aligned(16))) float ws[2][kProjK * WP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, g = lane >> 5, d = a.d;
  int job = 0;
#pragma unroll
  for (int i = 1; i < kMaxProjections; ++i) job += static_cast<int>(blockIdx.x) >= a.first_tile[i];
  const ProjectJob j = a.job[job];
  const int tile = blockIdx.x - a.first_tile[job], col_tiles = (d + TN - 1) / TN;
  const int64_t r0 = static_cast<int64_t>(tile / col_tiles) * TM, rows = j.rows;
  const int c0 = (tile % col_tiles) * TN;
  if (j.lens != nullptr) {  // a tile that holds one user's padding only is skipped: nothing reads it
    // (32-bit divisions where they do: a 64-bit one is a hundred instructions)
    const int64_t b = rows <= 0x7fffffff ? static_cast<int64_t>(static_cast<int>(r0) / static_cast<int>(j.rows_per_user)) : r0 / j.rows_per_user;
    const int first = static_cast<int>(r0 - b * j.rows_per_user);
    if (first >= j.lens[b] && first + TM <= j.rows_per_user) return;
  }
  const T* X = static_cast<const T*>(j.X);
  const T* W = static_cast<const T*>(j.W);
  float* Y = j.Y;
  if (W == nullptr) {
    for (int i = tid; i < TM * TN; i += 256) {
      const int64_t row = r0 + i / TN;
      const int c = c0 + i % TN;
      if (row < rows && c < d) Y[row * d + c] = to_float(X[row * d + c]);
    }
    return;
  }
  Vec8<T> px[XL], pw;
  auto fetch = [&](int k0) {
#pragma unroll
    for (int l = 0; l < XL; ++l) {
      const int i = tid + 256 * l;
      const int64_t row = r0 + i / (kProjK / 8);
      const int k = k0 + 8 * (i % (kProjK / 8));
      if constexpr (VEC) {
        // (rows past the end are read from the last one and not stored; columns past the end count as zeros)
        if (k < d) px[l].load(X + (row < rows ? row : rows - 1) * d + k);
        else
#pragma unroll
          for (int t = 0; t < 8; ++t) px[l].v[t] = 0.f;
      } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) px[l].v[t] = (row < rows && k + t < d) ? to_float(X[row * d + k + t]) : 0.f;
      }
    }
    if (WL == 256 || tid < WL) {
      const int k = k0 + tid / (TN / 8), c = c0 + 8 * (tid % (TN / 8));
      if constexpr (VEC) {
        if (k < d && c < d) pw.load(W + static_cast<int64_t>(k) * d + c);
        else
#pragma unroll
          for (int t = 0; t < 8; ++t) pw.v[t] = 0.f;
      } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) pw.v[t] = (k < d && c + t < d) ? to_float(W[static_cast<int64_t>(k) * d + c + t]) : 0.f;
      }
    }
  };
  auto park = [&](int buf) {
#pragma unroll
    for (int l = 0; l < XL; ++l) {
      const int i = tid + 256 * l;
      float* dst = xs[buf] + (i / (kProjK / 8)) * XP + 8 * (i % (kProjK / 8));
      *reinterpret_cast<float4*>(dst) = make_float4(px[l].v[0], px[l].v[1], px[l].v[2], px[l].v[3]);
      *reinterpret_cast<float4*>(dst + 4) = make_float4(px[l].v[4], px[l].v[5], px[l].v[6], px[l].v[7]);
    }
    if (WL == 256 || tid < WL) {
      float* dst = ws[buf] + (tid / (TN / 8)) * WP + 8 * (tid % (TN / 8));
      *reinterpret_cast<float4*>(dst) = make_float4(pw.v[0], pw.v[1], pw.v[2], pw.v[3]);
      *reinterpret_cast<float4*>(dst + 4) = make_float4(pw.v[4], pw.v[5], pw.v[6], pw.v[7]);
    }
  };
  constexpr int WC = TN / 32;  // waves across the tile's columns
  const int wr = wave / WC, wc = wave % WC;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  const int steps = (d + kProjK - 1) / kProjK;
  fetch(0);
  for (int s = 0; s < steps; ++s) {
    park(s & 1);
    __syncthreads();  // (the other buffer was last read before this barrier's predecessor)
    if (s + 1 < steps) fetch((s + 1) * kProjK);
    const float* xrow = xs[s & 1] + (32 * wr + n) * XP + 4 * g;
    const float* wcol = ws[s & 1] + 4 * g * WP + 32 * wc + n;
#pragma unroll
    for (int j = 0; j < kProjK / 8; ++j) {
      const float4 x = *reinterpret_cast<const float4*>(xrow + 8 * j);
      const float w0 = wcol[(8 * j) * WP], w1 = wcol[(8 * j + 1) * WP], w2 = wcol[(8 * j + 2) * WP], w3 = wcol[(8 * j + 3) * WP];
      acc = mfma_f32(x.x, w0, acc), acc = mfma_f32(x.y, w1, acc), acc = mfma_f32(x.z, w2, acc), acc = mfma_f32(x.w, w3, acc);
    }
  }
  const int c = c0 + 32 * wc + n;
  if (c >= d) return;
  // (written through as it is produced, see store_through: 28.1 -> 27.4 us a pass of the small-model request, 56.5 -> 54.3 of
  // the fp32 batch's)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(Y + r0 * d, 0, TM * d * 4, 0x00020000);
  const int left = static_cast<int>(min(rows - r0, static_cast<int64_t>(TM)));
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = 32 * wr + 8 * (i >> 2) + 4 * g + (i & 3);
    if (row < left) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i]), rsrc, (row * d + c) * 4, 0, 16 /* sc1 */);
  }
}

template <typename T>
hipError_t launch_project(const ProjectArgs& a, int tiles, bool vec, hipStream_t s) {
  if (a.d <= 32) {
    if (vec) hipLaunchKernelGGL((project_kernel<T, 32, true>), dim3(tiles), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((project_kernel<T, 32, false>), dim3(tiles), dim3(256), 0, s, a);
  } else {
    if (vec) hipLaunchKernelGGL((project_kernel<T, 64, true>), dim3(tiles), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((project_kernel<T, 64, false>), dim3(tiles), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- attention
// A wave takes 32 query rows of one (user, head) and walks the keys 32 at a time; everything but the operands stays in
// registers.  S^T = K Q^T (A = key rows, B = query rows, the head's columns summed), so a lane owns a query (column) and
// 16 of the 32 keys, the other 16 in lane ^ 32: the online softmax is lane-local plus one exchange.  Then
// O^T += V^T P^T: register i of S^T is the B operand whose two k are the keys that register stands for in the two lane
// halves, and the A operand is one float of each of those two rows of V: coalesced row reads, no LDS.
// The order of the sums over the keys is the same however the work is cut, so that a user's result has the same bits in
// every batch and with every workspace: the keys are taken in chunks of kChunkTiles tiles; of a chunk, tiles 0, 4, 8, ..,
// then 1, 5, .., up to 3, 7, .. each give a state (running maximum, running sum, sums), which are folded in this order, and
// the chunks' states in ascending order.
// SPLIT: the four waves of a workgroup share 32 query rows, a state of every chunk each, folded through LDS.  Chosen where
// the queries alone would leave the compute units idle (the m links over a history); with few workgroups besides, each
// chunk has a workgroup of its own and attention_merge_kernel folds the chunks' states.  Without SPLIT a wave forms all
// four states in turn (one chunk only: the third state that more would need has no registers).  What bounds it: two key
// tiles per wave are two dependent round trips to the cache, the matrix instruction (64 cycles each, d/h / 2 + 16 per tile
// at d/h <= 32) from a few thousand tiles up.
constexpr int kChunkTiles = 32;

struct AttnDev {
  const float *Q, *K, *V;
  int64_t qs, ks, vs;
  void* O;
  const int32_t *q_lens, *k_lens;
  int q_rows, n_keys, d, dh, q_tiles, h, chunks;  // chunks > 1: a workgroup takes one chunk
  float scale;
  float *part_acc, *part_ml;  // chunks > 1: [B][chunks][q_rows][d], [B][chunks][q_rows][h][2] (running max, running sum)
  int chunk_keys = 32 * kChunkTiles;
};

// The weights of two states that are folded into one: their maxima relative to the common one, which `mx` becomes.  (A
// maximum is -inf where every logit of the state was.)
struct FoldWeights {
  float into, from;
};
template <int PHI>
__device__ __forceinline__ FoldWeights fold_weights(float& mx, float from) {
  if (PHI != kPhiSoftmax) return {1.f, 1.f};
  const float top = fmaxf(mx, from);
  const FoldWeights w{mx == -INFINITY ? 0.f : expf(mx - top), from == -INFINITY ? 0.f : expf(from - top)};
  mx = top;
  return w;
}
__device__ __forceinline__ float folded(float into, float from, FoldWeights w) { return fmaf(w.from, from, into * w.into); }

// How a head's row is read: kWhole d/h = 8 KJ, kQuads d/h is a multiple of 4 (both from 16-byte aligned rows), kSingly.
enum Rows { kWhole, kQuads, kSingly };

// KJ: groups of eight head columns (d/h <= 8 KJ; the columns past d/h are zeros in Q and K).  Loads carry no condition: a
// test per load costs a branch and the copies of a join (12.9 -> 6 us for the 16 links of a one-user request at d/h = 64).
// Waves per SIMD: as many as the operands' registers leave room for (at d/h = 8 and a wave per query tile the allocator by
// itself takes 144 registers, three waves instead of four: 29.8 instead of 29.0 us for B=64 N=256 C=501 d=32).
template <typename OutT, int PHI, int KJ, bool SPLIT, Rows ROWS>
__global__ __launch_bounds__(256, KJ == 1 ? 4 : KJ == 2 ? 3 : KJ == 4 ? 2 : 1) void attention_kernel(AttnDev a) {
  constexpr bool VEC = ROWS != kSingly;
  constexpr int DB = (KJ + 3) / 4;     // 32-column blocks of the head's output
  constexpr int VB = DB < 4 ? DB : 4, KB = KJ < 16 ? KJ : 16;  // blocks of V and column groups of K in registers at a time
  constexpr bool kPrefetch = KJ <= 8;  // the next tile's K and V in flight during the current one (registers permitting)
  __shared__ float red[SPLIT ? 4 * (DB * 16 + 2) * 64 : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 31, g = lane >> 5;
  const int b = blockIdx.z, d = a.d, dh = a.dh;
  const int unit = SPLIT ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * 4 + wave;  // (query tile, head), heads innermost
  const int head = unit % a.h, q0 = unit / a.h * 32;
  if (!SPLIT && q0 >= a.q_rows) return;
  const int qlen = a.q_lens ? min(a.q_lens[b], a.q_rows) : a.q_rows;
  const int klen = a.k_lens ? min(a.k_lens[b], a.n_keys) : a.n_keys;
  const int tiles = (klen + 31) / 32;
  const int chunk = SPLIT && a.chunks > 1 ? blockIdx.y : 0;
  if (chunk > 0 && chunk * kChunkTiles >= tiles) return;  // uniform: no key in this chunk
  const bool dead = q0 >= qlen;                           // only rows that are written as zeros
  const int tile_last = dead ? 0 : SPLIT && a.chunks > 1 ? min(tiles, (chunk + 1) * kChunkTiles) : tiles;

  // head columns 8j + 4g .. + 3 of a row, j = j0 ..; past the head's width its last columns (zero_past clears them)
  // (the lane half through an opaque copy: what follows from it is formed here, not carried through the loop)
  auto load_row = [&](const float* row, int j0, float4 (&x)[KB]) {
    int g_ = g;
    if constexpr (KJ > KB) asm volatile("" : "+v"(g_));
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const int k = 8 * (j0 + j) + 4 * g_;
      if constexpr (VEC) {
        x[j] = *reinterpret_cast<const float4*>(row + (ROWS == kWhole ? k : min(k, dh - 4)));
      } else {
        x[j] = make_float4(row[min(k, dh - 1)], row[min(k + 1, dh - 1)], row[min(k + 2, dh - 1)], row[min(k + 3, dh - 1)]);
      }
    }
  };
  auto zero_past = [&](int j0, float4 (&x)[KB]) {
    if constexpr (ROWS == kWhole) return;
    int left = dh - 8 * j0 - 4 * g;
    asm volatile("" : "+v"(left));
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      x[j].x = left > 8 * j ? x[j].x : 0.f;
      x[j].y = left > 8 * j + (VEC ? 0 : 1) ? x[j].y : 0.f;  // (VEC: all four or none)
      x[j].z = left > 8 * j + (VEC ? 0 : 2) ? x[j].z : 0.f;
      x[j].w = left > 8 * j + (VEC ? 0 : 3) ? x[j].w : 0.f;
    }
  };
  float4 q[KJ / KB][KB];
#pragma unroll
  for (int p = 0; p < KJ / KB; ++p)
    load_row(a.Q + b * a.qs + static_cast<int64_t>(min(q0 + n, a.q_rows - 1)) * d + head * dh, p * KB, q[p]);
  const float* Kb = a.K + b * a.ks + head * dh;
  const float* Vb = a.V + b * a.vs + head * dh;
  // rows past the last valid key are read from it instead: their weights are zero
  auto load_k = [&](int k0, int j0, float4 (&k)[KB]) { load_row(Kb + static_cast<int64_t>(min(k0 + n, klen - 1)) * d, j0, k); };
  int vcol[DB];
#pragma unroll
  for (int ob = 0; ob < DB; ++ob) vcol[ob] = min(32 * ob + n, dh - 1);
  auto load_v = [&](int k0, int ob0, float (&v)[VB][16]) {
    if (k0 + 32 <= klen) {  // uniform: a scalar row base plus a lane offset that never changes
      const float* base = Vb + static_cast<int64_t>(k0) * d;
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int ob = 0; ob < VB; ++ob) v[ob][i] = (base + static_cast<int64_t>(8 * (i >> 2) + (i & 3)) * d)[4 * g * d + vcol[ob0 + ob]];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float* vrow = Vb + static_cast<int64_t>(min(k0 + 8 * (i >> 2) + 4 * g + (i & 3), klen - 1)) * d;
#pragma unroll
        for (int ob = 0; ob < VB; ++ob) v[ob][i] = vrow[vcol[ob0 + ob]];
      }
    }
  };
  float4 kn[KB];
  float vn[VB][16];
  auto prefetch = [&](int t) {
    if constexpr (kPrefetch) load_k(t * 32, 0, kn), load_v(t * 32, 0, vn);
  };
  int t = chunk * kChunkTiles + (SPLIT ? wave : 0);
  if (kPrefetch && t < tile_last) prefetch(t);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < KJ / KB; ++p) {
    zero_past(p * KB, q[p]);
#pragma unroll
    for (int j = 0; j < KB; ++j) q[p][j].x *= a.scale, q[p][j].y *= a.scale, q[p][j].z *= a.scale, q[p][j].w *= a.scale;
  }

  f32x16 acc[DB];  // the state that is being formed
  float run_max, run_sum;
  auto begin_state = [&] {
#pragma unroll
    for (int ob = 0; ob < DB; ++ob)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[ob][i] = 0.f;
    run_max = -INFINITY, run_sum = 0.f;
  };
  begin_state();
  auto take_tile = [&](int t, int next) {  // next: the tile after it, or one past tile_last
    const int k0 = t * 32;
    float4 k[KB];
    float v[VB][16];
    if constexpr (kPrefetch) {
#pragma unroll
      for (int j = 0; j < KB; ++j) k[j] = kn[j];
#pragma unroll
      for (int ob = 0; ob < VB; ++ob)
#pragma unroll
        for (int i = 0; i < 16; ++i) v[ob][i] = vn[ob][i];
      if (next < tile_last) prefetch(next);
    } else {
      load_k(k0, 0, k);
    }
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int p = 0; p < KJ / KB; ++p) {
      if (p > 0) {
        __builtin_amdgcn_sched_barrier(0);  // (fetched no earlier: registers)
        load_k(k0, p * KB, k);
      }
      zero_past(p * KB, k);
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        s = mfma_f32(k[j].x, q[p][j].x, s), s = mfma_f32(k[j].y, q[p][j].y, s);
        s = mfma_f32(k[j].z, q[p][j].z, s), s = mfma_f32(k[j].w, q[p][j].w, s);
      }
    }
    if constexpr (!kPrefetch) load_v(k0, 0, v);
    // register i of this lane is key k0 + 8 (i / 4) + 4g + i % 4
    const bool ragged = k0 + 32 > klen;  // uniform
    auto past = [&](int i) { return 8 * (i >> 2) + (i & 3) >= klen - k0 - 4 * g; };
    if (ragged) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (past(i)) s[i] = PHI == kPhiSoftmax ? -INFINITY : 0.f;  // (SiLU(0) = 0)
    }
    if (PHI == kPhiSoftmax) {
      float tmax = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
      const float new_max = fmaxf(run_max, pair_max(tmax));
      const float base = new_max == -INFINITY ? 0.f : new_max;  // (every logit so far is -inf: weights of zero)
      const float alpha = expf(run_max - base);                 // run_max = -inf on the first tile -> 0
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = expf(s[i] - base), psum += s[i];  // masked logits are -inf -> 0
      run_sum = fmaf(run_sum, alpha, psum);
      run_max = new_max;
#pragma unroll
      for (int ob = 0; ob < DB; ++ob)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[ob][i] *= alpha;
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = s[i] / (1.f + expf(-s[i]));
    }
#pragma unroll
    for (int ob0 = 0; ob0 < DB; ob0 += VB) {
      if (ob0 > 0) {
        __builtin_amdgcn_sched_barrier(0);  // (fetched no earlier: registers)
        load_v(k0, ob0, v);
      }
      if (ragged) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int ob = 0; ob < VB; ++ob) v[ob][i] = past(i) ? 0.f : v[ob][i];  // (what was read in its place may be infinite)
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int ob = 0; ob < VB; ++ob) acc[ob0 + ob] = mfma_f32(v[ob][i], s[i], acc[ob0 + ob]);
    }
  };

  // the result: acc, run_max and run_sum (the lane pair's), for SPLIT in the first wave
  if constexpr (!SPLIT) {
    f32x16 out[DB];  // the states folded so far
    float out_max = -INFINITY, out_sum = 0.f;
#pragma unroll
    for (int ob = 0; ob < DB; ++ob)
#pragma unroll
      for (int i = 0; i < 16; ++i) out[ob][i] = 0.f;
    while (t < tile_last) {  // tiles 0, 4, 8, .., 1, 5, .. (t & 3: the state)
      const bool ends = t + 4 >= tile_last;
      const int next = !ends ? t + 4 : (t & 3) < 3 ? (t & 3) + 1 : tile_last;
      take_tile(t, next);
      if (ends) {  // uniform
        run_sum = pair_sum(run_sum);
        if ((t & 3) == 0) {
          out_max = run_max, out_sum = run_sum;
#pragma unroll
          for (int ob = 0; ob < DB; ++ob) out[ob] = acc[ob];
        } else {
          const FoldWeights w = fold_weights<PHI>(out_max, run_max);
          out_sum = folded(out_sum, run_sum, w);
#pragma unroll
          for (int ob = 0; ob < DB; ++ob)
#pragma unroll
            for (int i = 0; i < 16; ++i) out[ob][i] = folded(out[ob][i], acc[ob][i], w);
        }
        begin_state();
      }
      t = next;
    }
    run_max = out_max, run_sum = out_sum;
#pragma unroll
    for (int ob = 0; ob < DB; ++ob) acc[ob] = out[ob];
  } else {
    constexpr int kState = (DB * 16 + 2) * 64;
    float* const kept = red + 3 * kState + lane;  // the first wave's: the chunks folded so far
    for (int c = chunk; c * kChunkTiles < tile_last; ++c) {  // uniform over the workgroup
      const int end = min(tile_last, (c + 1) * kChunkTiles), states = min(4, end - c * kChunkTiles);
      if (c > chunk) {
        __syncthreads();  // the last chunk's states have been read
        begin_state();
      }
      for (t = c * kChunkTiles + wave; t < end; t += 4) take_tile(t, t + 4);  // (a chunk is a multiple of four tiles)
      run_sum = pair_sum(run_sum);
      if (wave > 0) {
        float* mine = red + (wave - 1) * kState + lane;
        mine[0] = run_max, mine[64] = run_sum;
#pragma unroll
        for (int ob = 0; ob < DB; ++ob)
#pragma unroll
          for (int i = 0; i < 16; ++i) mine[(2 + ob * 16 + i) * 64] = acc[ob][i];
      }
      __syncthreads();
      if (wave > 0) continue;
#pragma unroll
      for (int o = 0; o < 3; ++o) {
        if (o + 1 >= states) break;  // uniform
        const float* theirs = red + o * kState + lane;
        const FoldWeights w = fold_weights<PHI>(run_max, theirs[0]);
        run_sum = folded(run_sum, theirs[64], w);
#pragma unroll
        for (int ob = 0; ob < DB; ++ob)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[ob][i] = folded(acc[ob][i], theirs[(2 + ob * 16 + i) * 64], w);
      }
      if (c > chunk) {
        float top = kept[0];
        const FoldWeights w = fold_weights<PHI>(top, run_max);
        run_max = top, run_sum = folded(kept[64], run_sum, w);
#pragma unroll
        for (int ob = 0; ob < DB; ++ob)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[ob][i] = folded(kept[(2 + ob * 16 + i) * 64], acc[ob][i], w);
      }
      if (end < tile_last) {
        kept[0] = run_max, kept[64] = run_sum;
#pragma unroll
        for (int ob = 0; ob < DB; ++ob)
#pragma unroll
          for (int i = 0; i < 16; ++i) kept[(2 + ob * 16 + i) * 64] = acc[ob][i];
      }
    }
    if (wave > 0) return;
  }

  // lane (query n, g) holds head columns 32 ob + 8 j + 4 g + r in register 4 j + r
  auto store4 = [&](auto* dst, int t, const f32x16& x, int j, float f) {
    using D = std::remove_reference_t<decltype(*dst)>;
    if constexpr (VEC) {
      if (t >= dh) return;
      if constexpr (sizeof(D) == 4) {
        *reinterpret_cast<float4*>(dst + t) = make_float4(x[4 * j] * f, x[4 * j + 1] * f, x[4 * j + 2] * f, x[4 * j + 3] * f);
      } else {
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = static_cast<__bf16>(x[4 * j + r] * f);
        *reinterpret_cast<bf16x4*>(dst + t) = v;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (t + r < dh) store_as(dst + t + r, x[4 * j + r] * f);
    }
  };
  const int row = q0 + n;
  if (row >= a.q_rows) return;
  if (SPLIT && a.chunks > 1) {
    const int64_t slot = (static_cast<int64_t>(b) * a.chunks + chunk) * a.q_rows + row;
    float* dst = a.part_acc + slot * d + head * dh;
#pragma unroll
    for (int ob = 0; ob < DB; ++ob)
#pragma unroll
      for (int j = 0; j < 4; ++j) store4(dst, 32 * ob + 8 * j + 4 * g, acc[ob], j, 1.f);
    if (g == 0) {
      float* ml = a.part_ml + (slot * a.h + head) * 2;
      ml[0] = run_max, ml[1] = run_sum;
    }
    return;
  }
  const bool live = row < qlen && klen > 0;
  const float inv = live ? 1.f / (PHI == kPhiSoftmax ? run_sum : static_cast<float>(klen)) : 0.f;
  OutT* orow = static_cast<OutT*>(a.O) + (static_cast<int64_t>(b) * a.q_rows + row) * d + head * dh;
#pragma unroll
  for (int ob = 0; ob < DB; ++ob)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!live)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[ob][4 * j + r] = 0.f;
      store4(orow, 32 * ob + 8 * j + 4 * g, acc[ob], j, inv);
    }
}

// The chunks' states folded in ascending order, one thread per output element.
template <typename OutT, int PHI>
__global__ __launch_bounds__(256) void attention_merge_kernel(AttnDev a) {
  const int b = blockIdx.y;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(a.q_rows) * a.d) return;
  const int row = static_cast<int>(idx / a.d), col = static_cast<int>(idx % a.d), head = col / a.dh;
  const int qlen = a.q_lens ? min(a.q_lens[b], a.q_rows) : a.q_rows;
  const int klen = a.k_lens ? min(a.k_lens[b], a.n_keys) : a.n_keys;
  const int used = (klen + a.chunk_keys - 1) / a.chunk_keys;
  float out = 0.f;
  if (used > 0 && row < qlen) {
    const int64_t slot0 = static_cast<int64_t>(b) * a.chunks * a.q_rows + row;
    const float* ml = a.part_ml + (slot0 * a.h + head) * 2;
    const float* acc = a.part_acc + slot0 * a.d + col;
    float mx = ml[0], den = ml[1], num = acc[0];
#pragma unroll 4
    for (int c = 1; c < used; ++c) {
      const int64_t row_c = static_cast<int64_t>(c) * a.q_rows;
      const FoldWeights w = fold_weights<PHI>(mx, ml[row_c * a.h * 2]);
      num = folded(num, acc[row_c * a.d], w), den = folded(den, ml[row_c * a.h * 2 + 1], w);
    }
    out = num * (1.f / (PHI == kPhiSoftmax ? den : static_cast<float>(klen)));
  }
  store_as(static_cast<OutT*>(a.O) + static_cast<int64_t>(b) * a.q_rows * a.d + idx, out);
}

template <typename OutT, int PHI>
hipError_t launch_merge(const AttnDev& dev, int B, hipStream_t s) {
  const int64_t total = static_cast<int64_t>(dev.q_rows) * dev.d;
  hipLaunchKernelGGL((attention_merge_kernel<OutT, PHI>), dim3(static_cast<unsigned>((total + 255) / 256), B), dim3(256), 0, s, dev);
  return hipGetLastError();
}

// (a workgroup's waves share the keys, chunks with workgroups of their own) of an attention: what fills the compute units.
struct AttnSplit {
  bool split;
  int chunks;
};
AttnSplit attention_split(int64_t B, int64_t q_rows, int64_t n_keys, int64_t h) {
  const int64_t units = B * h * ((q_rows + 31) / 32);  // (user, head, query tile)
  const int cus = compute_units();
  const int chunks = static_cast<int>((n_keys + 32 * kChunkTiles - 1) / (32 * kChunkTiles));
  if (units >= 4 * static_cast<int64_t>(cus) && chunks <= 1) return {false, 1};  // a wave per SIMD without splitting
  if (units >= cus) return {true, 1};                                           // a workgroup per compute unit
  return {true, chunks};
}

template <typename OutT, int PHI, int KJ, Rows ROWS>
hipError_t launch_attention(const AttnDev& dev, int B, bool split, hipStream_t s) {
  const int units = dev.q_tiles * dev.h;
  if (split)
    hipLaunchKernelGGL((attention_kernel<OutT, PHI, KJ, true, ROWS>), dim3(units, dev.chunks, B), dim3(256), 0, s, dev);
  else
    hipLaunchKernelGGL((attention_kernel<OutT, PHI, KJ, false, ROWS>), dim3((units + 3) / 4, 1, B), dim3(256), 0, s, dev);
  if (dev.chunks > 1) return launch_merge<OutT, PHI>(dev, B, s);
  return hipGetLastError();
}

template <typename OutT, int PHI>
hipError_t dispatch_attention(const AttnDev& dev, int B, bool split, hipStream_t s) {
  const bool vec = dev.dh % 4 == 0 &&
                   ((reinterpret_cast<uintptr_t>(dev.Q) | reinterpret_cast<uintptr_t>(dev.K) | reinterpret_cast<uintptr_t>(dev.O)) & 15u) == 0;
#define LIME_ATTN_CASE(KJ)                                                                              \
  if (vec && dev.dh == 8 * KJ) return launch_attention<OutT, PHI, KJ, kWhole>(dev, B, split, s); \
  if (vec && dev.dh < 8 * KJ) return launch_attention<OutT, PHI, KJ, kQuads>(dev, B, split, s);
  LIME_ATTN_CASE(1) LIME_ATTN_CASE(2) LIME_ATTN_CASE(4) LIME_ATTN_CASE(8) LIME_ATTN_CASE(16) LIME_ATTN_CASE(32)
  if (dev.dh <= 32) return launch_attention<OutT, PHI, 4, kSingly>(dev, B, split, s);
  if (dev.dh <= 256) return launch_attention<OutT, PHI, 32, kSingly>(dev, B, split, s);
#undef LIME_ATTN_CASE
  return hipErrorInvalidValue;
}

// ----------------------------------------------------------------------------- QK cache (Section 3.3)
// One wave per (user, candidate, head): weights = softmax over the m links of the scaled logits.
template <typename OutT>
__global__ __launch_bounds__(256) void qk_weights_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                                                         OutT* __restrict__ W, int64_t rows, int d, int h, int m,
                                                         float scale) {
  const int lane = threadIdx.x & 63;
  const int64_t item = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);  // (row, head)
  if (item >= rows * h) return;
  const int64_t row = item / h;
  const int head = static_cast<int>(item % h), dh = d / h;
  const float* q = Q + row * d + head * dh;
  float mx = -INFINITY;
  for (int i = lane; i < m; i += 64) {
    const float* k = K + static_cast<int64_t>(i) * d + head * dh;
    float s = 0.f;
    for (int t = 0; t < dh; ++t) s = fmaf(q[t], k[t], s);
    mx = fmaxf(mx, s * scale);
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  float sum = 0.f;
  for (int i = lane; i < m; i += 64) {
    const float* k = K + static_cast<int64_t>(i) * d + head * dh;
    float s = 0.f;
    for (int t = 0; t < dh; ++t) s = fmaf(q[t], k[t], s);
    sum += expf(s * scale - mx);
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  for (int i = lane; i < m; i += 64) {
    const float* k = K + static_cast<int64_t>(i) * d + head * dh;
    float s = 0.f;
    for (int t = 0; t < dh; ++t) s = fmaf(q[t], k[t], s);
    store_as(W + (row * h + head) * m + i, expf(s * scale - mx) / sum);
  }
}

// One thread per output element: O[b][c][col] = sum_i W[b][c][head(col)][i] * V[b][i][col]; with ids, the
// weight row is row ids[b][c] of a table of n_items rows, and an id outside the table gives zero.
template <typename T>
__global__ __launch_bounds__(256) void cached_sum_kernel(const T* __restrict__ W, const int32_t* __restrict__ ids,
                                                         int n_items, const float* __restrict__ V, T* __restrict__ O,
                                                         int64_t total, int C, int d, int h, int m) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= total) return;
  const int col = static_cast<int>(idx % d);
  const int64_t row = idx / d, b = row / C;
  const int head = col / (d / h);
  int64_t wrow = row;
  if (ids != nullptr) {
    const int id = ids[row];
    if (static_cast<unsigned>(id) >= static_cast<unsigned>(n_items)) {
      store_as(O + idx, 0.f);
      return;
    }
    wrow = id;
  }
  const T* w = W + (wrow * h + head) * m;
  const float* v = V + b * m * d + col;
  float acc = 0.f;
  for (int i = 0; i < m; ++i) acc = fmaf(to_float(w[i]), v[static_cast<int64_t>(i) * d], acc);
  store_as(O + idx, acc);
}

}  // namespace

hipError_t generic_qk_weights(const float* Q, const float* K, void* W, int64_t rows, int d, int h, int m, float scale,
                              int dtype, hipStream_t s) {
  const int64_t items = rows * h;
  dim3 grid(static_cast<unsigned>((items + 3) / 4));
  if (dtype == 0)
    hipLaunchKernelGGL(qk_weights_kernel<float>, grid, dim3(256), 0, s, Q, K, static_cast<float*>(W), rows, d, h, m, scale);
  else
    hipLaunchKernelGGL(qk_weights_kernel<bf16_t>, grid, dim3(256), 0, s, Q, K, static_cast<bf16_t*>(W), rows, d, h, m, scale);
  return hipGetLastError();
}

hipError_t generic_cached_sum(const void* W, const int32_t* ids, int n_items, const float* V, void* O, int B, int C,
                              int d, int h, int m, int dtype, hipStream_t s) {
  const int64_t total = static_cast<int64_t>(B) * C * d;
  dim3 grid(static_cast<unsigned>((total + 255) / 256));
  if (dtype == 0)
    hipLaunchKernelGGL(cached_sum_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(W), ids, n_items, V,
                       static_cast<float*>(O), total, C, d, h, m);
  else
    hipLaunchKernelGGL(cached_sum_kernel<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t*>(W), ids, n_items, V,
                       static_cast<bf16_t*>(O), total, C, d, h, m);
  return hipGetLastError();
}

hipError_t generic_project(const Projection* jobs, int n, int d, int dtype, hipStream_t s) {
  if (n > kMaxProjections) return hipErrorInvalidValue;
  ProjectArgs a{};
  a.d = d;
  const int tn = d <= 32 ? 32 : 64, tm = 4096 / tn;
  bool vec = d % 8 == 0;
  int64_t tiles = 0;
  int used = 0;
  for (int i = 0; i < kMaxProjections; ++i) a.first_tile[i] = 0x7fffffff;
  for (int i = 0; i < n; ++i) {
    const Projection& j = jobs[i];
    if (j.rows <= 0) continue;
    a.first_tile[used] = static_cast<int>(tiles);
    a.job[used++] = ProjectJob{j.X, j.W, j.Y, j.lens, j.rows, j.rows_per_user > 0 ? j.rows_per_user : 1};
    vec = vec && ((reinterpret_cast<uintptr_t>(j.X) | reinterpret_cast<uintptr_t>(j.W)) & 15u) == 0;
    tiles += (j.rows + tm - 1) / tm * ((d + tn - 1) / tn);
    if (tiles >= 0x7fffffff) return hipErrorInvalidValue;
  }
  if (tiles == 0) return hipSuccess;
  return dtype == 0 ? launch_project<float>(a, static_cast<int>(tiles), vec, s) : launch_project<bf16_t>(a, static_cast<int>(tiles), vec, s);
}

namespace {

// Z = A * SiLU(P), P = X Wu in fp32 (one block of rows for all users when p_user_stride == 0)
template <typename T>
__global__ __launch_bounds__(256) void gate_kernel(const float* __restrict__ P, int64_t p_user_stride, const T* __restrict__ A,
                                                   const int32_t* __restrict__ lens, T* __restrict__ Z, int rows, int d,
                                                   int64_t total) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t per_user = static_cast<int64_t>(rows) * d;
  const int b = static_cast<int>(i / per_user);
  const int64_t rem = i - b * per_user;
  const int row = static_cast<int>(rem / d);
  const bool valid = row < (lens ? min(lens[b], rows) : rows);
  const float p = P[b * p_user_stride + rem];
  store_as(Z + i, valid ? to_float(A[i]) * p / (1.f + expf(-p)) : 0.f);
}

// Y = X + P, P = Z Wo in fp32; the running sum of P over the layers
template <typename T>
__global__ __launch_bounds__(256) void residual_kernel(const float* __restrict__ P, const T* __restrict__ X, int64_t x_user_stride,
                                                       const int32_t* __restrict__ lens, T* __restrict__ Y,
                                                       const float* __restrict__ sum_in, float* __restrict__ sum_out,
                                                       T* __restrict__ sum_rounded, int rows, int d, int64_t total) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t per_user = static_cast<int64_t>(rows) * d;
  const int b = static_cast<int>(i / per_user);
  const int64_t rem = i - b * per_user;
  const int row = static_cast<int>(rem / d);
  const bool valid = row < (lens ? min(lens[b], rows) : rows);
  const float p = P[i];
  if (Y != nullptr) store_as(Y + i, valid ? to_float(X[b * x_user_stride + rem]) + p : 0.f);
  if (sum_out != nullptr || sum_rounded != nullptr) {
    const float t = (sum_in != nullptr ? sum_in[i] : 0.f) + p;
    if (sum_out != nullptr) sum_out[i] = t;
    if (sum_rounded != nullptr) store_as(sum_rounded + i, t);
  }
}

template <typename T>
hipError_t gated_block_typed(const GenericGatedBlock& g, hipStream_t s) {
  const int64_t total = static_cast<int64_t>(g.B) * g.rows * g.d;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256));
  const bool shared = g.x_user_stride == 0;
  const Projection gate{g.X, g.Wu, g.P, shared ? g.rows : static_cast<int64_t>(g.B) * g.rows};
  hipError_t e = generic_project(&gate, 1, g.d, g.dtype, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gate_kernel<T>, grid, dim3(256), 0, s, g.P, shared ? int64_t{0} : static_cast<int64_t>(g.rows) * g.d,
                     static_cast<const T*>(g.A), g.lens, static_cast<T*>(g.Z), g.rows, g.d, total);
  const Projection out{g.Z, g.Wo, g.P, static_cast<int64_t>(g.B) * g.rows};
  e = generic_project(&out, 1, g.d, g.dtype, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(residual_kernel<T>, grid, dim3(256), 0, s, g.P, static_cast<const T*>(g.X), g.x_user_stride, g.lens,
                     static_cast<T*>(g.Y), g.sum_in, g.sum_out, static_cast<T*>(g.sum_rounded), g.rows, g.d, total);
  return hipGetLastError();
}

}  // namespace

hipError_t generic_gated_block(const GenericGatedBlock& g, hipStream_t s) {
  if (g.B <= 0 || g.rows <= 0) return hipSuccess;
  return g.dtype == 0 ? gated_block_typed<float>(g, s) : gated_block_typed<bf16_t>(g, s);
}

hipError_t generic_merge_chunks(const float* acc, const float* ml, const int32_t* lens, void* O, int B, int m, int N, int chunk_keys,
                                int d, int h, int phi, int dtype, hipStream_t s) {
  AttnDev dev{};
  dev.O = O, dev.k_lens = lens, dev.q_rows = m, dev.n_keys = N, dev.d = d, dev.dh = d / h, dev.h = h;
  dev.chunks = (N + chunk_keys - 1) / chunk_keys, dev.chunk_keys = chunk_keys;
  dev.part_acc = const_cast<float*>(acc), dev.part_ml = const_cast<float*>(ml);
  if (dtype == 0) return phi == kPhiSoftmax ? launch_merge<float, kPhiSoftmax>(dev, B, s) : launch_merge<float, kPhiSilu>(dev, B, s);
  return phi == kPhiSoftmax ? launch_merge<bf16_t, kPhiSoftmax>(dev, B, s) : launch_merge<bf16_t, kPhiSilu>(dev, B, s);
}

size_t generic_attention_scratch(int64_t B, int64_t q_rows, int64_t n_keys, int64_t d, int64_t h) {
  const AttnSplit sp = attention_split(B, q_rows, n_keys, h);
  if (sp.chunks <= 1) return 0;
  return align_up(static_cast<size_t>(B) * sp.chunks * q_rows * d * sizeof(float)) +
         align_up(static_cast<size_t>(B) * sp.chunks * q_rows * h * 2 * sizeof(float));
}

hipError_t generic_attention(const GenericAttention& a, hipStream_t s) {
  if (a.B <= 0 || a.q_rows <= 0) return hipSuccess;
  AttnSplit sp = attention_split(a.B, a.q_rows, a.n_keys, a.h);
  if (a.scratch == nullptr) sp.chunks = 1;
  AttnDev dev{a.Q, a.K, a.V, a.q_user_stride, a.k_user_stride, a.v_user_stride, a.O, a.q_lens, a.k_lens,
              a.q_rows, a.n_keys, a.d, a.d / a.h, (a.q_rows + 31) / 32, a.h, sp.chunks, a.scale, nullptr, nullptr};
  if (sp.chunks > 1) {
    dev.part_acc = static_cast<float*>(a.scratch);
    dev.part_ml = reinterpret_cast<float*>(static_cast<char*>(a.scratch) +
                                           align_up(static_cast<size_t>(a.B) * sp.chunks * a.q_rows * a.d * sizeof(float)));
  }
  if (a.dtype == 0)
    return a.phi == kPhiSoftmax ? dispatch_attention<float, kPhiSoftmax>(dev, a.B, sp.split, s)
                                : dispatch_attention<float, kPhiSilu>(dev, a.B, sp.split, s);
  return a.phi == kPhiSoftmax ? dispatch_attention<bf16_t, kPhiSoftmax>(dev, a.B, sp.split, s)
                              : dispatch_attention<bf16_t, kPhiSilu>(dev, a.B, sp.split, s);
}

}  // namespace lime
