// The m links over a history with its projections inside, see fused.hpp.
#include "fused.hpp"

namespace lime {
namespace {

// ----------------------------------------------------------------------------- the m links over a history
struct HistoryDev {
  const void *E, *L, *Wq, *Wk, *Wv;
  const int32_t* lens;
  int64_t l_user_stride;
  void* LP;
  float *part_acc, *part_ml;  // more than one chunk: [B][chunks][m][d], [B][chunks][m][h][2]
  int B, N, h, m, chunks, total;
  HistoryTails tails;
  float scale;
};

template <typename T, int D, int DH, int MT>
struct HistoryLds {
  using H = Head<DH>;
  using W = Weights<T, D, DH>;
  static constexpr int kQueries = MT * H::KF * 3 * 1024, kParts = kWaves * 4096;
  static constexpr int kState = MT * (DH / 2 + 2) * 256;  // a wave's state
  static constexpr int kBytes = std::max(W::kBytes + kQueries + kParts, kWaves * kState);
};

// A workgroup: one chunk of a user's history, one head, 32 MT links; a wave: a tile of 32 items.  What bounds it: at the sizes
// of these calls the chain of latencies of one tile (rows and weights from memory, projections, logits, weights), which is why
// a tile has a wave of its own and the small operands are computed by all waves, a part of the sum each.  With more workgroups than
// run at once it is the weights' way to planes in LDS: where the users' last (or only) chunks are short, several of them share a
// workgroup (HistoryTails; a tile's and a user's sums are the same in every place).
// SHARED: with such workgroups (which cost the others 0.25 us).
template <typename T, int D, int DH, int MT, int PHI, bool SHARED>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(fused_waves(D, DH), fused_waves(D, DH)))) void fused_history_kernel(HistoryDev a) {
  using H = Head<DH>;
  using Lds = HistoryLds<T, D, DH, MT>;
  constexpr bool kAlternate = sizeof(T) == 4;  // every other item negated
  constexpr int K1 = D / 16, DB = H::DB, NP = kPlanes<T>, kBlocks = MT * DB, kSplits = std::min(kWaves / kBlocks, K1);
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  using W = typename Lds::W;
  unsigned char* const weights = lds;
  bf16x8* const queries = reinterpret_cast<bf16x8*>(lds + W::kBytes);
  float* const parts = reinterpret_cast<float*>(queries + Lds::kQueries / 16);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, g = lane >> 5;
  int id = block_on_xcd(a.total);
  if (id >= a.total) return;
  const int head = id % a.h;
  const int c0 = n % DH;  // this lane's column of the head's (first) block
  id /= a.h;
  int chunk, b0, users = 1, tiles = kWaves, slot = 0;  // this wave's user is b0 + slot
  if constexpr (!SHARED) {
    chunk = id % a.chunks, b0 = id / a.chunks;
  } else if (id < a.tails.first) {
    chunk = id % (a.chunks - 1), b0 = id / (a.chunks - 1);
  } else {
    chunk = a.chunks - 1, b0 = (id - a.tails.first) * a.tails.users, users = min(a.tails.users, a.B - b0), tiles = a.tails.tiles;
    slot = wave * a.tails.per_tile >> 16;
  }
  const int tile = wave - slot * tiles, b = b0 + min(slot, users - 1);
  auto link_row = [&](int lt, int i) {
    return static_cast<const T*>(a.L) + b * a.l_user_stride + static_cast<int64_t>(min(32 * lt + i, a.m - 1)) * D;
  };
  const int block = wave % kBlocks, part = wave / kBlocks;  // queries: block (link tile, 32 columns), a part of its sum
  const T *const wq = static_cast<const T*>(a.Wq) + head * DH, *const wk = static_cast<const T*>(a.Wk) + head * DH, *const wv = static_cast<const T*>(a.Wv) + head * DH;
  unsigned char* const own = reinterpret_cast<unsigned char*>(parts) + wave * 4096;

  // everything the workgroup reads is asked for here, in the order of its use
  W share;
  RowTile<T, D / kSplits> links;
  RowTile<T, D> items;
  share.load(wq, wk, wv, threadIdx.x);
  if (part < kSplits) links.load([&](int i) { return link_row(block / DB, i) + part * (D / kSplits); }, lane);
  __builtin_amdgcn_sched_barrier(0);  // (ahead of the wait for the length)
  const int klen = a.lens ? min(a.lens[b], a.N) : a.N;
  if (users == 1 && chunk > 0 && chunk * kChunkKeys >= klen) return;  // uniform: nothing in this chunk
  const int k0 = chunk * kChunkKeys + 32 * tile;
  const bool live = slot < users && k0 < klen;  // uniform over the wave
  const int last = max(klen, 1) - 1;
  auto item_row = [&](int i) { return static_cast<const T*>(a.E) + (static_cast<int64_t>(b) * a.N + min(k0 + i, last)) * D; };
  if (live) items.load(item_row, lane);
  __builtin_amdgcn_sched_barrier(0);
  share.park(weights, threadIdx.x);
  lds_barrier();
  f32x16 q_part = zeros(), kv[2 * DB];  // keys (lane = item), values (lane = column)
  if (part < kSplits) q_part = partial_block<W>(links, weights, 0, block % DB, part, own, true, lane);
  if (live) {
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) kv[i] = zeros();
    Planes<NP> w[2][2 * DB];
    items.each(own, lane, kAlternate && n % 2 ? -kUp<T> : kUp<T>, [&](int kk) {
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) w[kk & 1][i] = W::fragment(weights, 1 + i / DB, i % DB, kk, lane);
    }, [&](int kk, const Planes<NP>& x) {
      Planes<NP> l[2 * DB], r[2 * DB];
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) l[ob] = w[kk & 1][ob], r[ob] = x, l[DB + ob] = x, r[DB + ob] = w[kk & 1][DB + ob];
      products(l, r, kv);
    });
  }
  if (part < kSplits) park_block(reinterpret_cast<float*>(own), q_part, lane);
  lds_barrier();
  if (wave < 2 * kBlocks) {  // half a block's sum each: registers 8f .. of block (link tile, 32 columns)
    const int lt = wave / 2 / DB, ob = wave / 2 % DB, f = wave % 2;
    const float* src = parts + (wave / 2) * 1024 + 512 * f + lane;
    float q[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      q[t] = src[t * 64];
#pragma unroll
      for (int p = 1; p < kSplits; ++p) q[t] += src[p * kBlocks * 1024 + t * 64];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) q[t] *= kSum<T>;
    if (__any(any_not_finite(q, 8))) {
      const f32x16 x = exact_block<T, D, true>(link_row(lt, n), wq + c0 + 32 * ob, g);
#pragma unroll
      for (int t = 0; t < 8; ++t) q[t] = !not_finite(q[t]) ? q[t] : f ? x[8 + t] : x[t];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) q[t] = q[t] * a.scale * kUp<T>;
    // (a narrow head's columns are in the first registers)
    if (DH >= 32 || f == 0) park(queries + (lt * H::KF + (DH >= 32 ? 2 * ob + f : 0)) * 3 * 64, column_planes<DH, false>(q), lane);
  }
  lds_barrier();

  float mx[MT], sum[MT], res[MT][DH / 2];
  const int left = klen - k0 - 4 * g;
  const bool ragged = k0 + 32 > klen;  // uniform over the wave
  auto past = [&](int i) { return 8 * (i >> 2) + (i & 3) >= left; };
  // logits of a tile (kUnit) to weights (`up` times as large) in place, those of odd items negated before and after, all as they are
  // the exact way: register i of this lane is item k0 + 8 (i / 4) + 4g + i % 4
  auto sign = [](int i) { return kAlternate && i % 2 ? -1.f : 1.f; };
  const float tile_sign = kAlternate && tile % 2 ? -1.f : 1.f, up = tile_sign * kUp<T>;  // uniform
  auto to_weights = [&](f32x16& s, float& top, float& total, auto exact_tag) {
    constexpr bool kExact = decltype(exact_tag)::value;
    if (ragged) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (past(i)) s[i] = PHI != kPhiSoftmax ? 0.f : kExact ? -INFINITY : sign(i) * kMaskedLogit;  // (SiLU(0) = 0)
    }
    top = -INFINITY, total = 0.f;
    if (PHI == kPhiSoftmax) {
#pragma unroll
      for (int i = 0; i < 16; ++i) top = fmaxf(top, kExact ? s[i] : sign(i) * s[i]);
      top = pair_max(top);
      const float base = kExact && top == -INFINITY ? 0.f : top;  // (every logit is -inf: weights of zero)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = kExact ? expf(s[i] - base) : exp_finite(sign(i) * s[i] - base, kUnit<T>, sign(i) * up);
        total += kExact ? s[i] : sign(i) * s[i];
      }
      total = pair_sum(total);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = kExact ? silu(s[i]) : silu_finite(sign(i) * s[i], kUnit<T>, sign(i) * up);
    }
  };
  // items past the last: what was read in their place may be infinite
  auto clear_past = [&](f32x16& v) {
    if (!ragged) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = past(i) ? 0.f : v[i];
  };
  if (live) {
    Planes<3> kf[H::KF];
    Planes<H::VP> vf[2][DB];
#pragma unroll
    for (int f = 0; f < H::KF; ++f) kf[f] = column_planes<DH, true>(half_of(kv[f / 2], f % 2).x);
#pragma unroll
    for (int ob = 0; ob < DB; ++ob) {
      clear_past(kv[DB + ob]);
#pragma unroll
      for (int f = 0; f < 2; ++f) vf[f][ob] = value_planes<DH>(split_half(kv[DB + ob], f), n);
    }
    bool bad[MT];  // (both lanes of a link)
    f32x16 s[MT], acc[MT][DB];
    Planes<3> q[MT][H::KF];
#pragma unroll
    for (int lt = 0; lt < MT; ++lt) {
      s[lt] = zeros();
#pragma unroll
      for (int f = 0; f < H::KF; ++f) q[lt][f] = parked<3>(queries + (lt * H::KF + f) * 3 * 64, lane);
    }
#pragma unroll
    for (int t = 0; t < kColumnTerms<DH>; ++t)
#pragma unroll
      for (int f = 0; f < H::KF; ++f)
#pragma unroll
        for (int lt = 0; lt < MT; ++lt) s[lt] = column_term<DH>(t, kf[f], q[lt][f], s[lt]);
#pragma unroll
    for (int lt = 0; lt < MT; ++lt) {
      to_weights(s[lt], mx[lt], sum[lt], std::false_type{});
      const Planes<3> w[2] = {split_half(s[lt], 0), split_half(s[lt], 1)};
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) acc[lt][ob] = zeros();
#pragma unroll
      for (int t = 0; t < kValueTerms<DH>; ++t)
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int ob = 0; ob < DB; ++ob) acc[lt][ob] = value_term<DH>(t, vf[f][ob], w[f], acc[lt][ob]);
    }
#pragma unroll
    for (int lt = 0; lt < MT; ++lt) {
      head_result<DH>(acc[lt], res[lt]);
      bad[lt] = either_lane(any_not_finite(res[lt], DH / 2) || sum[lt] != sum[lt] || (PHI == kPhiSoftmax && mx[lt] < kLowLogit));
      mx[lt] *= kUnit<T>, sum[lt] *= tile_sign * kDown<T>;
#pragma unroll
      for (int i = 0; i < DH / 2; ++i) res[lt][i] *= tile_sign * kUnit<T>;
    }
    bool any = bad[0];
#pragma unroll
    for (int lt = 1; lt < MT; ++lt) any = any || bad[lt];
    if (__any(any)) {
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) {
        kv[ob] = exact_block<T, D, true>(item_row(n), wk + c0 + 32 * ob, g);
        kv[DB + ob] = exact_block<T, D, false>(item_row(n), wv + c0 + 32 * ob, g);
        clear_past(kv[DB + ob]);
      }
#pragma unroll
      for (int lt = 0; lt < MT; ++lt) {
        f32x16 s = zeros();
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          const f32x16 q = exact_block<T, D, true>(link_row(lt, n), wq + c0 + 32 * ob, g);
#pragma unroll
          for (int i = 0; i < std::min(DH / 2, 16); ++i) s = mfma_f32(kv[ob][i], q[i] * a.scale, s);
        }
        float top, total;
        to_weights(s, top, total, std::true_type{});
        mx[lt] = bad[lt] ? top : mx[lt], sum[lt] = bad[lt] ? total : sum[lt];
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          f32x16 x = zeros();
#pragma unroll
          for (int i = 0; i < 16; ++i) x = mfma_f32(kv[DB + ob][i], s[i], x);
#pragma unroll
          for (int i = 0; i < std::min(DH / 2, 16); ++i) res[lt][16 * ob + i] = bad[lt] ? x[i] : res[lt][16 * ob + i];
        }
      }
    }
  }

  // A user's tiles' states, folded in ascending order: a quad of a link tile's result by one wave.
  lds_barrier();  // weights and queries have been read
  float* const states = reinterpret_cast<float*>(lds);
  constexpr int kState = Lds::kState / 4, kTile = (4 * H::QUADS + 2) * 64;
  if (live) {
#pragma unroll
    for (int lt = 0; lt < MT; ++lt) {
      float* st = states + wave * kState + lt * kTile + lane;
      st[0] = mx[lt], st[64] = sum[lt];
#pragma unroll
      for (int i = 0; i < DH / 2; ++i) st[(2 + i) * 64] = res[lt][i];
    }
  }
  lds_barrier();
  auto fold = [&](int s, int lt, int q) {  // user b0 + s
    const int link = 32 * lt + n, b = b0 + s;
    const int len = !SHARED || !a.lens ? klen : min(a.lens[b], a.N);
    const int used = min(tiles, (len - chunk * kChunkKeys + 31) / 32);  // (none for a user without history)
    if (SHARED && chunk > 0 && used <= 0) return;  // uniform over the wave
    const float* st = states + s * tiles * kState + lt * kTile + lane;
    float m[kWaves], top = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      m[w] = w < used ? st[w * kState] : -INFINITY;
      top = fmaxf(top, m[w]);
    }
    float x[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w >= used) break;  // uniform
      // (-200: maxima of tiles taken the exact way may lie further apart than exp_finite, which is NaN from -2.36e38 on, takes; a NaN
      // among the operands is in the sums)
      const float f = PHI != kPhiSoftmax ? 1.f : exp_finite(fmaxf(m[w] - top, -200.f), 1.f, 1.f);
      den = fmaf(f, st[w * kState + 64], den);
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = fmaf(f, st[w * kState + (2 + 4 * q + r) * 64], x[r]);
    }
    if (link >= a.m) return;
    const int col = head * DH + 8 * q + 4 * g;
    if (a.chunks > 1) {
      const int64_t slot = (static_cast<int64_t>(b) * a.chunks + chunk) * a.m + link;
      store_quad(a.part_acc + slot * D + col, x);
      if (q == 0 && g == 0) {
        float* ml = a.part_ml + (slot * a.h + head) * 2;
        ml[0] = top, ml[1] = den;
      }
    } else {
      const float inv = len > 0 ? 1.f / (PHI == kPhiSoftmax ? den : static_cast<float>(len)) : 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] *= inv;
      store_quad(static_cast<T*>(a.LP) + (static_cast<int64_t>(b) * a.m + link) * D + col, x);
    }
  };
  constexpr int kUnits = MT * H::QUADS;
  if constexpr (SHARED) {
#pragma unroll 1
    for (int u = wave; u < users * kUnits; u += kWaves) fold(u / kUnits, u / H::QUADS % MT, u % H::QUADS);
  } else {
#pragma unroll
    for (int u = wave; u < kUnits; u += kWaves) fold(0, u / H::QUADS, u % H::QUADS);
  }
}

template <typename T, int D, int DH, int MT, int PHI, bool SHARED>
hipError_t launch_form(const HistoryDev& a, hipStream_t s) {
  constexpr int kBytes = HistoryLds<T, D, DH, MT>::kBytes;
  static_assert(kBytes <= 160 * 1024);
  auto kernel = fused_history_kernel<T, D, DH, MT, PHI, SHARED>;
  if constexpr (kBytes > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), kBytes); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(launched_workgroups(a.total)), dim3(kThreads), kBytes, s, a);
  return hipGetLastError();
}

template <typename T, int D, int DH, int MT, int PHI>
hipError_t launch_history(const HistoryDev& a, hipStream_t s) {
  return a.tails.users > 1 ? launch_form<T, D, DH, MT, PHI, true>(a, s) : launch_form<T, D, DH, MT, PHI, false>(a, s);
}

// Whether a head of dh columns is one that this kernel is for, see fused_history_supported.
constexpr bool narrow_pays(int d, int dh, bool fp32) { return dh >= 32 || (fp32 ? d == 32 : d != 64 || dh > 8); }

template <typename T, int D, int DH>
hipError_t dispatch_history(const HistoryDev& a, int phi, hipStream_t s) {
  if constexpr (DH >= 32)
    if (a.m > 32) return phi == kPhiSoftmax ? launch_history<T, D, DH, 2, kPhiSoftmax>(a, s) : launch_history<T, D, DH, 2, kPhiSilu>(a, s);
  return phi == kPhiSoftmax ? launch_history<T, D, DH, 1, kPhiSoftmax>(a, s) : launch_history<T, D, DH, 1, kPhiSilu>(a, s);
}

template <typename T>
hipError_t dispatch_history_shape(const HistoryDev& a, int d, int phi, hipStream_t s) {
#define LIME_CASE(D, DH) \
  if constexpr (narrow_pays(D, DH, sizeof(T) == 4)) \
    if (d == D && d / a.h == DH) return dispatch_history<T, D, DH>(a, phi, s);
  LIME_FUSED_SHAPES(LIME_CASE)
#undef LIME_CASE
  return hipErrorInvalidValue;
}

int history_chunks(int64_t N) { return static_cast<int>((N + kChunkKeys - 1) / kChunkKeys); }

}  // namespace

// As many links as one workgroup takes, since a second one would project the history once more (64 links of 8 heads of 16
// columns, 128 users of 512 items in fp32: 186 us, the general kernels 110); and narrow heads, each of whose workgroups projects
// 32 columns whatever it uses, where that is cheap: in bf16 but for the narrowest of eight (57 us for the 65 536 items and 16
// candidates, the general kernels 56), in fp32 at d = 32.  In fp32 at d = 64 four heads take 39 and 43 us, but 123 and 112 at four
// times the items, eight heads 77 and 53.  lime_link_history, general kernels | this one, us, at one user's 100 items, one user's 16 384
// and 64 users' 4096: fp32 d=32 h=4 m=16 9.0|5.6 25.0|18.8 79.5|64.8, d=32 h=2 m=32 9.1|5.4 26.2|18.4 55.5|40.3, d=64 h=1 m=16 12.2|8.4
// 46.7|24.5 94.7|57.4, d=128 h=4 m=64 11.7|9.5 43.9|26.9 301|251; bf16 d=32 h=4 m=16 9.0|4.8 25.3|17.3 80.5|50.0, d=64 h=4 m=16 9.6|5.1
// 29.8|18.4 117|60.2, d=128 h=8 m=16 11.7|5.7 40.8|25.9 291|209.
// The states of a history's chunks fit where separate kernels keep its keys and values (2 N d numbers of a user; m (d + 2h) of
// each 256 items or part of them), with room to align them.
bool fused_history_supported(int64_t B, int64_t N, int d, int h, int m, int dtype) {
  if (!fused_shape(d, h) || m > (d / h >= 32 ? 64 : 32)) return false;
  return narrow_pays(d, d / h, dtype == 0) && launch_fits(history_workgroups(B, N, h));
}

hipError_t fused_history(const FusedHistory& q, hipStream_t s) {
  HistoryDev a{q.E, q.L, q.Wq, q.Wk, q.Wv, q.lens, q.l_user_stride, q.LP, nullptr, nullptr, q.B, q.N, q.h, q.m, history_chunks(q.N), 0, {}, q.scale};
  // (links of a user's own are projected by a workgroup of the user's own)
  const int64_t at_once = static_cast<int64_t>(compute_units()) * fused_waves(q.d, q.d / q.h) / 2;
  a.tails = history_tails(q.B, q.N, q.h, q.l_user_stride != 0 ? 0 : at_once);
  a.total = static_cast<int>(tails_workgroups(a.tails, q.B, q.h));
  if (a.chunks > 1) {
    char* scratch = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(q.scratch) + 15) & ~uintptr_t{15});
    a.part_acc = reinterpret_cast<float*>(scratch);
    a.part_ml = a.part_acc + static_cast<int64_t>(q.B) * a.chunks * q.m * q.d;
  }
  hipError_t e = q.dtype == 0 ? dispatch_history_shape<float>(a, q.d, q.phi, s) : dispatch_history_shape<bf16_t>(a, q.d, q.phi, s);
  if (e != hipSuccess || a.chunks == 1) return e;
  return generic_merge_chunks(a.part_acc, a.part_ml, q.lens, q.LP, q.B, q.m, q.N, kChunkKeys, q.d, q.h, q.phi, q.dtype, s);
}

}  // namespace lime
