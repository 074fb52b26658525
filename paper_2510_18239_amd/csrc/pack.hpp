// Operand packing for the matrix-core kernels, a workgroup of four wavefronts at a time: in a launch of its own
// (mfma_pack.hip), or beside the history kernel of a call (mfma_history_raw.hip).
#pragma once

#include "mfma.hpp"

namespace lime {
namespace {

constexpr int kMaxJobs = kMaxPackProjections, kMaxWeights = kMaxPackWeights;

struct WeightJob {
  const bf16_t* src;
  bf16x8* img;
  float sign;
  int pad;
};
struct ProjectJob {
  const bf16_t *x, *w, *gamma, *beta;  // gamma, beta: of the layer normalisation of a job's rows (norm set)
  bf16_t* img;
  int64_t stride;
  int layout, norm;
  float sign, eps;
};
// (a workgroup reads the numbers and then its job: two scalar loads, one after the other)
struct PackArgs {
  int n_weights, blocks_per_weight;
  int d, dh, m;
  int first_unit[kMaxJobs + 1];     // ranges of the projection jobs' units, after the weight jobs
  int units_per_block;              // of the projection jobs: 1 or 4
  const bf16_t *s_wq, *s_k, *s_wk;  // the score job (at most one), after the projection jobs
  bf16_t* s_img;
  float s_sign;
  WeightJob weight[kMaxWeights];
  ProjectJob job[kMaxJobs];
};

// One wavefront of a score job: the 32 x 32 block (links 32lb.., rows j = 32jb..) of head a's
//   G_a^T[l][j] = sum_c K~[l][a dh + c] Wq[j][a dh + c],   K~ = Ksrc Wk,
// computed on the matrix cores as Ksrc (Wk_a Wq_a^T): in that order both products read their operands row-major
// with the summed index contiguous, so no transposed copy of a weight is needed.  For each block of 32 rows k of
// Wk the wave forms M = Wk_a[k-block] Wq_a[j-block]^T (summed over the head's columns) and feeds it straight back
// as the B operand of Ksrc[l-block][k-block] . M (chained order, see mfma.hpp).
template <int DH, int M, int NKB>
__device__ void score_wave(const PackArgs& p, int combo) {
  constexpr int D = 32 * NKB, H = D / DH, LB = M / 32, KC = DH / 16, K1 = D / 16;
  const int lane = threadIdx.x & 63, n = lane & 31, g = lane >> 5;
  const int lb = combo % LB, jb = (combo / LB) % NKB, a = combo / (LB * NKB);
  if (a >= H) return;  // uniform over the wave
  // a null weight stands for the identity
  auto rows_of = [&](const bf16_t* W, int row, int kc) {
    const int c0 = a * DH + 16 * kc + 8 * g;
    if (W != nullptr) return *reinterpret_cast<const bf16x8*>(W + static_cast<int64_t>(row) * D + c0);
    bf16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(row == c0 + t ? 1.f : 0.f);
    return v;
  };
  bf16x8 wq[KC], wk[NKB][KC], lf[NKB][2];
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) wq[kc] = rows_of(p.s_wq, 32 * jb + n, kc);
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) wk[kb][kc] = rows_of(p.s_wk, 32 * kb + n, kc);
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      // slot t stands for k = 32kb + 16f + chain_k(g, t): columns 4g..4g+3 and 8+4g..8+4g+3 of the 16
      const bf16_t* src = p.s_k + static_cast<int64_t>(32 * lb + n) * D + 32 * kb + 16 * f + 4 * g;
      const bf16x4 lo = *reinterpret_cast<const bf16x4*>(src), hi = *reinterpret_cast<const bf16x4*>(src + 8);
#pragma unroll
      for (int t = 0; t < 4; ++t) lf[kb][f][t] = lo[t], lf[kb][f][4 + t] = hi[t];
    }
  }
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    f32x16 mk;
#pragma unroll
    for (int i = 0; i < 16; ++i) mk[i] = 0.f;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) mk = mfma32(wk[kb][kc], wq[kc], mk);
#pragma unroll
    for (int f = 0; f < 2; ++f) acc = mfma32(lf[kb][f], pack_half(mk, f), acc);
  }
  // register 4jj + r is link 32lb + 8jj + 4g + r, the lane's column is row j = 32jb + n of G_a
  const int j = 32 * jb + n;
  const int64_t frag = (static_cast<int64_t>(a) * K1 + j / 16) * LB + lb + a * kQueryImageHeadPad;
  bf16_t* dst = p.s_img + (frag * 64 + 32 * ((j % 16) / 8)) * 8 + j % 8;
#pragma unroll
  for (int i = 0; i < 16; ++i) store_as(dst + (8 * (i / 4) + 4 * g + i % 4) * 8, acc[i] * p.s_sign);
}

// 32 rows taken by a workgroup of four wavefronts into LDS, from where every wavefront reads its fragments: eight lanes per
// row, D / 64 pieces of eight columns per lane.  With a normalisation a row's statistics are a lane's own sums and three
// exchanges; mean first, then the centred second moment, in fp32, the rows rounded to bf16 where a normalisation pass of its
// own would have stored them.  `take` asks for what is needed, `finish` leaves the rows in LDS.
template <int D>
struct GroupRows {
  static constexpr int J = D / 64, kPitch = D + 8;  // (16 rows of a fragment read then cover all banks)
  bf16x8 x[J], gamma[J], beta[J];
  __device__ __forceinline__ void take(const bf16_t* rows, bool norm, const bf16_t* ga, const bf16_t* be) {
    const int r = threadIdx.x / 8, c = 8 * (threadIdx.x % 8);
#pragma unroll
    for (int j = 0; j < J; ++j) x[j] = *reinterpret_cast<const bf16x8*>(rows + static_cast<int64_t>(r) * D + 64 * j + c);
    if (!norm) return;  // uniform
#pragma unroll
    for (int j = 0; j < J; ++j) {
      gamma[j] = *reinterpret_cast<const bf16x8*>(ga + 64 * j + c);
      beta[j] = *reinterpret_cast<const bf16x8*>(be + 64 * j + c);
    }
  }
  __device__ __forceinline__ void finish(bf16_t* lds, bool norm, float eps) {
    bf16_t* dst = lds + threadIdx.x / 8 * kPitch + 8 * (threadIdx.x % 8);
    if (norm) {  // uniform
      float v[J][8], sum = 0.f, q = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int t = 0; t < 8; ++t) v[j][t] = static_cast<float>(x[j][t]), sum += v[j][t];
      const float mean = group_sum<8>(sum) * (1.f / D);
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int t = 0; t < 8; ++t) v[j][t] -= mean, q = fmaf(v[j][t], v[j][t], q);
      const float inv = 1.f / sqrtf(group_sum<8>(q) * (1.f / D) + eps);
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int t = 0; t < 8; ++t)
          x[j][t] = static_cast<__bf16>(fmaf(v[j][t] * inv, static_cast<float>(gamma[j][t]), static_cast<float>(beta[j][t])));
    }
#pragma unroll
    for (int j = 0; j < J; ++j) *reinterpret_cast<bf16x8*>(dst + 64 * j) = x[j];
  }
};

// A projection job's unit: 32 rows x 32 columns of X_u W on the matrix cores (project_block), written as two fragments of
// the job's image.  The unit's columns of W are read along its rows, 16 rows of 64 bytes per load, and turned in LDS.
//
// Up to d = 64 a wavefront does a unit by itself.  From d = 128 on (a multiple of four column blocks: a workgroup's units
// then belong to one job and to the same rows) the workgroup takes the rows together, and normalises them where that is
// asked for; with few units (one per workgroup) its wavefronts also share the loads of W, and the first does the product.
// What counts is the bytes a compute unit asks for, 64 a cycle: with four units a workgroup, each wavefront fetching its
// rows as fragments (32 lines a load), the loads of the request's 32 units at d = 256 took 2.1 us to be issued.
template <int D>
struct PackLds {
  static constexpr int NK = D / 16, kTurn = NK < 8 ? NK : 8;  // k-steps of W that a wavefront has in LDS at a time
  static constexpr bool kTogether = D / 32 % 4 == 0;
  static constexpr int kRows = kTogether ? 32 * (D + 8) * 2 : 0, kBytes = kRows + 4 * kTurn * 1024;
};
template <int D>
__device__ __forceinline__ void project_unit(const PackArgs& p, const ProjectJob& job, int unit, unsigned char* lds) {
  constexpr int NK = D / 16, CB = D / 32;
  constexpr bool kTogether = PackLds<D>::kTogether;
  constexpr int kTurn = PackLds<D>::kTurn;
  bf16_t* const rows_lds = reinterpret_cast<bf16_t*>(lds);
  unsigned char* const turned = lds + PackLds<D>::kRows;
  static_assert(!kTogether || NK <= 4 * kTurn, "a unit's columns of W fit the workgroup's part of LDS");
  const int lane = threadIdx.x & 63, n = lane & 31, g = lane >> 5, dh = p.dh, m = p.m;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lbs = m / 32, u = unit / (lbs * CB);
  const int lb = kTogether ? unit / CB % lbs : unit % lbs, cb = kTogether ? unit % CB : unit / lbs % CB;
  const bf16_t* Xu = job.x + u * job.stride;
  const bf16_t* W = job.w;
  const bool alone = kTogether && p.units_per_block == 1;  // uniform
  const int a = 32 * cb / dh, hc = 32 * cb % dh / 32;  // head, and 32-column block of the head
  const bool keys = job.layout == kPackKeys;
  bf16x8* img = reinterpret_cast<bf16x8*>(job.img);
  bf16x8 lo, hi;  // the block's accumulators, or what they would be
  if (W == nullptr) {
    // the identity: the rows as they are (normalised rows always come with a weight)
    if (alone && wave > 0) return;
    auto element = [&](int k) { return keys ? Xu[static_cast<int64_t>(32 * lb + n) * D + 32 * cb + k] : Xu[static_cast<int64_t>(32 * lb + k) * D + 32 * cb + n]; };
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      lo[t] = __builtin_bit_cast(__bf16, element(chain_k(g, t)).bits);
      hi[t] = __builtin_bit_cast(__bf16, element(16 + chain_k(g, t)).bits);
    }
    if (job.sign < 0.f) lo = -lo, hi = -hi;
  } else {
    const bf16_t* wrow = W + static_cast<int64_t>(lane / 4) * D + 32 * cb + 8 * (lane % 4);
    bf16x8 x[NK], w[NK], raw[NK];
    auto take_weights = [&] {
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) raw[kk] = *reinterpret_cast<const bf16x8*>(wrow + 16 * kk * D);
    };
    auto turn_weights = [&] {  // (a wavefront's LDS accesses are served in order, so its part needs no barrier)
      unsigned char* mine = turned + wave * kTurn * 1024;
#pragma unroll
      for (int k0 = 0; k0 < NK; k0 += kTurn) {
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < kTurn; ++k) *reinterpret_cast<bf16x8*>(mine + k * 1024 + lane * 16) = raw[k0 + k];
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < kTurn; ++k) w[k0 + k] = column_fragment(mine + k * 1024, 64, lane);
      }
    };
    if constexpr (kTogether) {
      const bool norm = job.norm;
      GroupRows<D> group;
      group.take(Xu + static_cast<int64_t>(32 * lb) * D, norm, job.gamma, job.beta);
      if (alone) {
        bf16x8 part[NK / 4];
#pragma unroll
        for (int k = 0; k < NK / 4; ++k) part[k] = *reinterpret_cast<const bf16x8*>(wrow + 16 * (NK / 4 * wave + k) * D);
        group.finish(rows_lds, norm, job.eps);
#pragma unroll
        for (int k = 0; k < NK / 4; ++k) *reinterpret_cast<bf16x8*>(turned + (NK / 4 * wave + k) * 1024 + lane * 16) = part[k];
        lds_barrier();
        if (wave > 0) return;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) w[kk] = column_fragment(turned + kk * 1024, 64, lane);
      } else {
        take_weights();
        group.finish(rows_lds, norm, job.eps);
        lds_barrier();
        turn_weights();
      }
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) x[kk] = *reinterpret_cast<const bf16x8*>(rows_lds + n * GroupRows<D>::kPitch + 16 * kk + 8 * g);
    } else {
      const bf16_t* X = Xu + static_cast<int64_t>(32 * lb + n) * D + 8 * g;  // row 32 lb + n
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) x[kk] = *reinterpret_cast<const bf16x8*>(X + 16 * kk);
      bf16x8 gamma[NK], beta[NK];
      if (job.norm) {  // asked for with everything else
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          gamma[kk] = *reinterpret_cast<const bf16x8*>(job.gamma + 16 * kk + 8 * g);
          beta[kk] = *reinterpret_cast<const bf16x8*>(job.beta + 16 * kk + 8 * g);
        }
      }
      take_weights();
      if (job.norm) normalise_rows<D>(x, gamma, beta, job.eps);
      turn_weights();
    }
    f32x16 acc = keys ? project_block<NK>(w, x) : project_block<NK>(x, w);
    if (job.sign < 0.f) acc = -acc;
    lo = pack_half(acc, 0), hi = pack_half(acc, 1);
  }
  if (keys) {
    // lane (row 32 lb + n, g), registers = the block's columns in chained order: k-steps 2 hc and 2 hc + 1 of the head
    const int64_t frag = ((static_cast<int64_t>(u) * (D / dh) + a) * (dh / 16) + 2 * hc) * lbs + lb;
    img[frag * 64 + lane] = lo;
    img[(frag + lbs) * 64 + lane] = hi;
  } else {
    // lane (column 32 cb + n, g), registers = the block's rows in chained order: k-steps 2 lb and 2 lb + 1
    const int64_t frag = ((static_cast<int64_t>(u) * (D / dh) + a) * (m / 16) + 2 * lb) * (dh / 32) + hc;
    const int slot = out_rho(n) + 32 * g;
    const bool natural = job.layout == kPackValuesNatural;
    img[frag * 64 + slot] = natural ? natural_from_chained(lo) : lo;
    img[(frag + dh / 32) * 64 + slot] = natural ? natural_from_chained(hi) : hi;
  }
}

// D: embedding width.  SDH, SM: shape of the score job (d/h, m) this instance can run after its other jobs; 0 = none.
// A block is four wavefronts: 256 slots of a weight image, or one or four units of the projection jobs, or four of the
// score job.  What bounds it is latency (a few KiB per compute unit): every load of a unit is independent of every other.
template <int D, int SDH, int SM>
__device__ __forceinline__ void pack_block(const PackArgs& p, int blk, unsigned char* lds) {
  constexpr int d = D;
  const int dh = p.dh, tid = threadIdx.x;
  if (blk < p.n_weights * p.blocks_per_weight) {
    // one thread per (8 consecutive k, column): a 16-byte slot of the weight image
    const int job = blk / p.blocks_per_weight;
    const int idx = (blk % p.blocks_per_weight) * 256 + tid;
    if (idx >= d * d / 8) return;
    const WeightJob w = p.weight[job];
    const bf16_t* W = w.src;
    const int col = idx % d, k0 = (idx / d) * 8;
    // (one uniform branch around all eight loads: a test per element would make each load wait for the one before)
    float x[8];
    if (W != nullptr) {
      bf16_t raw[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) raw[t] = W[static_cast<int64_t>(k0 + t) * d + col];
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = to_float(raw[t]);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = k0 + t == col ? 1.f : 0.f;
    }
    bf16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(x[t] * w.sign);
    const int a = col / dh, c = col % dh, mb = c / 32, n = c % 32;
    const int kk = k0 / 16, g = (k0 % 16) / 8;
    const int64_t frag = (static_cast<int64_t>(a) * (d / 16) + kk) * (dh / 32) + mb;
    // (768 KiB of a request's images at d = 256: written through, 19.6 -> 19.4 us a pass with 16 candidates)
    store_through(w.img, d * d * 2 + (d / dh) * w.pad * 1024, static_cast<int>(((frag + a * w.pad) * 64 + 32 * g + n) * 16), v);
    return;
  }
  blk -= p.n_weights * p.blocks_per_weight;
  const int projection_blocks = (p.first_unit[kMaxJobs] + p.units_per_block - 1) / p.units_per_block;
  if constexpr (SDH != 0) {
    if (blk >= projection_blocks) {  // uniform
      score_wave<SDH, SM, D / 32>(p, (blk - projection_blocks) * 4 + tid / 64);
      return;
    }
  }
  int unit = p.units_per_block == 1 ? blk : __builtin_amdgcn_readfirstlane(blk * 4 + tid / 64);
  if (unit >= p.first_unit[kMaxJobs]) return;
  int job = 0;
#pragma unroll
  for (int i = 1; i < kMaxJobs; ++i) job += unit >= p.first_unit[i];
  const ProjectJob j = p.job[job];
  project_unit<D>(p, j, unit - p.first_unit[job], lds);
}

// The weight and projection jobs as an argument, and how many workgroups they take.
inline int pack_args(PackArgs& p, const PackWeight* weights, int n_weights, const PackProject* projections, int n_projections, int d, int h, int m) {
  p = PackArgs{};
  p.d = d, p.dh = d / h, p.m = m;
  p.n_weights = n_weights;
  p.blocks_per_weight = (d * d / 8 + 255) / 256;
  for (int i = 0; i < n_weights; ++i) {
    p.weight[i] = WeightJob{static_cast<const bf16_t*>(weights[i].W), static_cast<bf16x8*>(weights[i].image), weights[i].sign, weights[i].head_pad};
  }
  int units = 0;
  for (int i = 0; i < kMaxJobs; ++i) {
    p.first_unit[i] = units;
    if (i < n_projections) {
      const PackProject& q = projections[i];
      p.job[i] = ProjectJob{static_cast<const bf16_t*>(q.X), static_cast<const bf16_t*>(q.W), static_cast<const bf16_t*>(q.norm.gamma),
                            static_cast<const bf16_t*>(q.norm.beta), static_cast<bf16_t*>(q.image), q.user_stride, q.layout, q.norm.on ? 1 : 0,
                            q.sign, q.norm.eps};
      units += q.users * (m / 32) * (d / 32);
    }
  }
  p.first_unit[kMaxJobs] = units;
  // A unit per workgroup as long as every workgroup then has a compute unit to itself; project_unit takes four from there on.
  p.units_per_block = d >= 128 && units <= compute_units() ? 1 : 4;
  return n_weights * p.blocks_per_weight + (units + p.units_per_block - 1) / p.units_per_block;
}

}  // namespace
}  // namespace lime
