// Rows over the m links with its projections inside, see fused.hpp.
#include "fused.hpp"

namespace lime {
namespace {

// ----------------------------------------------------------------------------- rows over the m links
struct RowsDev {
  const void *X, *Ksrc, *Vsrc, *Wq, *Wk, *Wv;
  const int32_t* row_lens;
  int64_t k_user_stride, v_user_stride;
  void* O;
  int B, rows, h, m, parts, total;  // workgroups per (user, head); by wave: per head
  float scale;
};

template <typename T, int D, int DH, int MH>
struct RowsLds {
  using H = Head<DH>;
  static constexpr int MT = (MH + 1) / 2;
  using W = Weights<T, D, DH>;
  static constexpr int kKeys = MT * H::KF * 3 * 1024, kValues = MH * H::DB * H::VP * 1024, kParts = kWaves * 4096;
  static constexpr int kBytes = W::kBytes + kKeys + kValues + kParts;
};

// (by wave: the values of a user's links lie in registers)
constexpr int rows_waves(int D, int DH, bool by_wave) { return by_wave ? 2 : fused_waves(D, DH); }

// A workgroup: a part of a user's rows, one head, all m <= 16 MH links; a wave takes every eighth tile of 32 rows.  Keys and
// values of the links are computed by all waves first.  What bounds it: as above at few rows; from a few thousand tiles on the
// vector ALUs (exponentials, and the planes of queries and weights).
// BY_WAVE: a user to a wave, one after the other, with the same sums in the same order; the workgroup shares the weights and the keys
// (which all users have in common) and no barrier stands between users.  For many users of few rows, where a workgroup each would
// bring the weights into LDS for a tile or two: lime_score_candidates, general kernels | a workgroup a user | so, in us, 2000 users' 16
// candidates: fp32 d=128 h=4 m=64 92.5|261|84.4, d=64 h=2 m=32 34.0|75.9|16.6, d=32 h=4 m=16 20.8|54.6|16.7; bf16 d=128 h=8 m=16 56.4|212|27.
// (fp32 at d=128 stays behind with fewer: 256 users' 19.1|31.8|22.4, 75 users', a workgroup each, 13.5|16.9; 512 users' 30.6|64.8|27.)
template <typename T, int D, int DH, int MH, int PHI, bool BY_WAVE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(rows_waves(D, DH, BY_WAVE), rows_waves(D, DH, BY_WAVE)))) void fused_rows_kernel(RowsDev a) {
  using H = Head<DH>;
  using Lds = RowsLds<T, D, DH, MH>;
  constexpr int K1 = D / 16, DB = H::DB, NP = kPlanes<T>, MT = Lds::MT, kBlocks = MT * DB, kSplits = std::max(1, std::min(kWaves / (2 * kBlocks), K1));
  constexpr int kRegs = MH == 1 ? 8 : 16;  // registers of a tile of links that count
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  using W = typename Lds::W;
  unsigned char* const weights = lds;
  bf16x8* const keys = reinterpret_cast<bf16x8*>(lds + W::kBytes);
  bf16x8* const values = keys + Lds::kKeys / 16;
  float* const parts = reinterpret_cast<float*>(values + Lds::kValues / 16);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, g = lane >> 5;
  int id = block_on_xcd(a.total);
  if (id >= a.total) return;
  const int head = id % a.h;
  id /= a.h;
  const int share = id % a.parts;
  int b = BY_WAVE ? share * kWaves + wave : id / a.parts;
  const int tiles = (a.rows + 31) / 32, step = BY_WAVE ? 1 : a.parts * kWaves;
  // keys and values of the links: blocks (side, link tile, 32 columns), each by kSplits waves
  const int c0 = n % DH;  // this lane's column of the head's (first) block
  const T* const keys_from = static_cast<const T*>(a.Ksrc) + (BY_WAVE ? 0 : b) * a.k_user_stride;
  const T* values_from = static_cast<const T*>(a.Vsrc) + b * a.v_user_stride;
  const T *const wk = static_cast<const T*>(a.Wk) + head * DH, *const wv = static_cast<const T*>(a.Wv) + head * DH, *const wq = static_cast<const T*>(a.Wq) + head * DH;
  auto link_row = [&](const T* from, int lt, int i) { return from + static_cast<int64_t>(min(32 * lt + i, a.m - 1)) * D; };
  const int block = wave % (2 * kBlocks), part = wave / (2 * kBlocks);
  const bool of_values = block >= kBlocks;  // uniform over the wave
  const bool has_part = part < kSplits && !(BY_WAVE && of_values);
  unsigned char* const own = reinterpret_cast<unsigned char*>(parts) + wave * 4096;

  // everything the workgroup reads at first is asked for here, in the order of its use
  W columns;
  RowTile<T, D / kSplits> links;
  RowTile<T, D> items;
  columns.load(wk, wv, wq, threadIdx.x);
  if (has_part)
    links.load([&](int i) { return link_row(of_values ? values_from : keys_from, block / DB % MT, i) + part * (D / kSplits); }, lane);
  __builtin_amdgcn_sched_barrier(0);  // (ahead of the wait for the length)
  int rlen = 0;
  auto take_length = [&] { rlen = a.row_lens ? min(a.row_lens[b], a.rows) : a.rows; };
  if (!BY_WAVE) take_length();
  auto row_of = [&](int t, int i) { return static_cast<const T*>(a.X) + (static_cast<int64_t>(b) * a.rows + min(32 * t + i, max(rlen, 1) - 1)) * D; };
  auto wanted = [&](int t) { return t < tiles && 32 * t < rlen; };  // uniform over the wave
  auto fetch = [&](int t) {
    if (wanted(t)) items.load([&](int i) { return row_of(t, i); }, lane);
  };
  f32x16 q[DB];  // queries of a tile (lane = row)
  auto project = [&] {
    Planes<NP> w[2][DB];
#pragma unroll
    for (int ob = 0; ob < DB; ++ob) q[ob] = zeros();
    items.each(own, lane, kUp<T>, [&](int kk) {
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) w[kk & 1][ob] = W::fragment(weights, 2, ob, kk, lane);
    }, [&](int kk, const Planes<NP>& x) {
      Planes<NP> r[DB];
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) r[ob] = x;
      products(w[kk & 1], r, q);
    });
  };
  int t = BY_WAVE ? 0 : share * kWaves + wave;
  if (!BY_WAVE) fetch(t);
  __builtin_amdgcn_sched_barrier(0);
  columns.park(weights, threadIdx.x);
  lds_barrier();
  f32x16 links_part = zeros();
  if (has_part) links_part = partial_block<W>(links, weights, of_values, block % DB, part, own, !of_values, lane);
  if (!BY_WAVE && wanted(t)) project();
  if (has_part) park_block(reinterpret_cast<float*>(own), links_part, lane);
  if (!BY_WAVE) fetch(t + step);
  lds_barrier();
  // half a block of the links' values (registers 8f ..) to fragments; links past the last have weight zero, but what was read in
  // their place may be infinite
  auto finish_values = [&](float (&x)[8], int lt, int f, int ob) {
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] *= kSum<T>;
    if (__any(any_not_finite(x, 8))) {
      const f32x16 y = exact_block<T, D, false>(link_row(values_from, lt, n), wv + c0 + 32 * ob, g);
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = !not_finite(x[t]) ? x[t] : f ? y[8 + t] : y[t];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = 32 * lt + 16 * f + 8 * (t >> 2) + 4 * g + (t & 3) < a.m ? x[t] * kUp<T> : 0.f;
    return value_planes<DH>(split(x), n);
  };
#pragma unroll
  for (int u = wave; u < 4 * kBlocks; u += kWaves) {  // half a block's sum each: registers 8f .. of block (side, link tile, 32 columns)
    const int f = u % 2, ob = u / 2 % DB, lt = u / 2 / DB % MT;
    const bool is_value = u >= 2 * kBlocks;
    if (BY_WAVE && is_value) continue;
    const float* src = parts + (u / 2) * 1024 + 512 * f + lane;
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      x[t] = src[t * 64];
#pragma unroll
      for (int p = 1; p < kSplits; ++p) x[t] += src[p * 2 * kBlocks * 1024 + t * 64];
    }
    if (is_value) {
      if (2 * lt + f < MH) park(values + ((2 * lt + f) * DB + ob) * H::VP * 64, finish_values(x, lt, f, ob), lane);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] *= kSum<T>;
      if (__any(any_not_finite(x, 8))) {
        const f32x16 y = exact_block<T, D, true>(link_row(keys_from, lt, n), wk + c0 + 32 * ob, g);
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = !not_finite(x[t]) ? x[t] : f ? y[8 + t] : y[t];
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = x[t] * a.scale * kUp<T>;
      // (a narrow head's columns are in the first registers)
      if (DH >= 32 || f == 0) park(keys + (lt * H::KF + (DH >= 32 ? 2 * ob + f : 0)) * 3 * 64, column_planes<DH, true>(x), lane);
    }
  }
  lds_barrier();

  // logits of all links (kUnit) to weights (kUp times as large) in place, all as they are the exact way; the factor of the result
  auto to_weights = [&](f32x16 (&s)[MT], float& top, auto exact_tag) {
    constexpr bool kExact = decltype(exact_tag)::value;
    if (a.m < 16 * MH) {  // uniform
#pragma unroll
      for (int lt = 0; lt < MT; ++lt)
#pragma unroll
        for (int i = 0; i < kRegs; ++i)
          if (32 * lt + 8 * (i >> 2) + 4 * g + (i & 3) >= a.m) s[lt][i] = PHI != kPhiSoftmax ? 0.f : kExact ? -INFINITY : kMaskedLogit;
    }
    if (PHI != kPhiSoftmax) {
#pragma unroll
      for (int lt = 0; lt < MT; ++lt)
#pragma unroll
        for (int i = 0; i < kRegs; ++i) s[lt][i] = kExact ? silu(s[lt][i]) : silu_finite(s[lt][i], kUnit<T>, kUp<T>);
      return (kExact ? 1.f : kSum<T>) / static_cast<float>(a.m);
    }
    float total = 0.f;
    top = s[0][0];
#pragma unroll
    for (int lt = 0; lt < MT; ++lt)
#pragma unroll
      for (int i = 0; i < kRegs; ++i) top = fmaxf(top, s[lt][i]);
    top = pair_max(top);
    const float base = kExact && top == -INFINITY ? 0.f : top;
#pragma unroll
    for (int lt = 0; lt < MT; ++lt)
#pragma unroll
      for (int i = 0; i < kRegs; ++i)
        s[lt][i] = kExact ? expf(s[lt][i] - base) : exp_finite(s[lt][i] - base, kUnit<T>, kUp<T>), total += s[lt][i];
    return (kExact ? 1.f : kDown<T>) / pair_sum(total);
  };

  Planes<H::VP> own_values[BY_WAVE ? MH : 1][DB];  // BY_WAVE: the user's
  auto compute_values = [&] {
    constexpr int kPart = K1 / kSplits;
#pragma unroll
    for (int lt = 0; lt < MT; ++lt) {
      RowTile<T, D> rows;
      rows.load([&](int i) { return link_row(values_from, lt, i); }, lane);
      f32x16 acc[DB], total[DB];
      Planes<NP> w[2][DB];
      rows.each(own, lane, kUp<T>, [&](int kk) {
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) w[kk & 1][ob] = W::fragment(weights, 1, ob, kk, lane);
      }, [&](int kk, const Planes<NP>& x) {
        Planes<NP> l[DB];
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          l[ob] = x;
          if (kk % kPart == 0) acc[ob] = zeros();
        }
        products(l, w[kk & 1], acc);
        if (kk % kPart == kPart - 1) {
#pragma unroll
          for (int ob = 0; ob < DB; ++ob) total[ob] = kk < kPart ? acc[ob] : total[ob] + acc[ob];
        }
      });
#pragma unroll
      for (int f = 0; f < 2 && 2 * lt + f < MH; ++f)
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          Half x = half_of(total[ob], f);
          own_values[BY_WAVE ? 2 * lt + f : 0][ob] = finish_values(x.x, lt, f, ob);
        }
    }
  };
  // (BY_WAVE: no barrier in here)
  for (; b < a.B; b += BY_WAVE ? a.parts * kWaves : a.B) {
  if constexpr (BY_WAVE) {
    take_length();
    values_from = static_cast<const T*>(a.Vsrc) + b * a.v_user_stride;
    t = 0;
    compute_values();
    fetch(0);  // (not ahead of it: registers)
    if (wanted(0)) project();
    fetch(1);
  }
  for (bool first = true; t < tiles; t += step, first = false) {
    float res[DH / 2], inv = 0.f;
    if (32 * t < rlen) {  // uniform over the wave
      if (!first) {
        project();
        fetch(t + step);
      }
      f32x16 s[MT];
      {
        Planes<3> x[H::KF], k[MT][H::KF];
#pragma unroll
        for (int f = 0; f < H::KF; ++f) {
          x[f] = column_planes<DH, false>(half_of(q[f / 2], f % 2).x);
#pragma unroll
          for (int lt = 0; lt < MT; ++lt) k[lt][f] = parked<3>(keys + (lt * H::KF + f) * 3 * 64, lane);
        }
#pragma unroll
        for (int lt = 0; lt < MT; ++lt) s[lt] = zeros();
#pragma unroll
        for (int t = 0; t < kColumnTerms<DH>; ++t)
#pragma unroll
          for (int f = 0; f < H::KF; ++f)
#pragma unroll
            for (int lt = 0; lt < MT; ++lt) s[lt] = column_term<DH>(t, k[lt][f], x[f], s[lt]);
      }
      float top = 0.f;
      inv = to_weights(s, top, std::false_type{});
      f32x16 acc[DB];
      Planes<3> p[MH];
#pragma unroll
      for (int ob = 0; ob < DB; ++ob) acc[ob] = zeros();
#pragma unroll
      for (int f = 0; f < MH; ++f) p[f] = split_half(s[f / 2], f % 2);
      // (the last term apart: with two blocks the values' planes are read again rather than kept)
      auto terms = [&](int from, int to) {
        Planes<H::VP> v[MH][DB];
#pragma unroll
        for (int f = 0; f < MH; ++f)
#pragma unroll
          for (int ob = 0; ob < DB; ++ob)
            if constexpr (BY_WAVE) v[f][ob] = own_values[f][ob];
            else v[f][ob] = parked<H::VP>(values + (f * DB + ob) * H::VP * 64, lane);
        auto term = [&](int t, int f) {
#pragma unroll
          for (int ob = 0; ob < DB; ++ob) acc[ob] = value_term<DH>(t, v[f][ob], p[f], acc[ob]);
        };
        if constexpr (DB == 1) {
#pragma unroll
          for (int t = from; t < to; ++t)
#pragma unroll
            for (int f = 0; f < MH; ++f) term(t, f);
        } else {
#pragma unroll
          for (int f = 0; f < MH; ++f)
#pragma unroll
            for (int t = from; t < to; ++t) term(t, f);
        }
      };
      if constexpr (DB == 1) {
        terms(0, kValueTerms<DH>);
      } else {
        terms(0, kValueTerms<DH> - 1);
        wave_lds_fence();
        terms(kValueTerms<DH> - 1, kValueTerms<DH>);
      }
      head_result<DH>(acc, res);
      const bool bad = either_lane(any_not_finite(res, DH / 2) || inv != inv || top < kLowLogit);  // (both lanes of a row)
      if (__any(bad)) {
#pragma unroll
        for (int lt = 0; lt < MT; ++lt) s[lt] = zeros();
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          const f32x16 x = exact_block<T, D, true>(row_of(t, n), wq + c0 + 32 * ob, g);
#pragma unroll
          for (int lt = 0; lt < MT; ++lt) {
            const f32x16 k = exact_block<T, D, true>(link_row(keys_from, lt, n), wk + c0 + 32 * ob, g);
#pragma unroll
            for (int i = 0; i < std::min(DH / 2, 16); ++i) s[lt] = mfma_f32(k[i] * a.scale, x[i], s[lt]);
          }
        }
        const float exact_inv = to_weights(s, top, std::true_type{});
        inv = bad ? exact_inv : inv;
#pragma unroll
        for (int ob = 0; ob < DB; ++ob) {
          f32x16 x = zeros();
#pragma unroll
          for (int lt = 0; lt < MT; ++lt) {
            const f32x16 v = exact_block<T, D, false>(link_row(values_from, lt, n), wv + c0 + 32 * ob, g);
#pragma unroll
            for (int i = 0; i < kRegs; ++i) x = mfma_f32(32 * lt + 8 * (i >> 2) + 4 * g + (i & 3) < a.m ? v[i] : 0.f, s[lt][i], x);
          }
#pragma unroll
          for (int i = 0; i < std::min(DH / 2, 16); ++i) res[16 * ob + i] = bad ? x[i] : res[16 * ob + i];
        }
      }
    }
    const int r = 32 * t + n;
    if (r >= a.rows) continue;
    T* orow = static_cast<T*>(a.O) + (static_cast<int64_t>(b) * a.rows + r) * D + head * DH + 4 * g;
#pragma unroll
    for (int q = 0; q < H::QUADS; ++q) {
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = r < rlen ? res[4 * q + i] * inv : 0.f;
      store_quad(orow + 8 * q, x);
    }
  }
  if (!BY_WAVE) break;
  }
}

template <typename T, int D, int DH, int MH, int PHI, bool BY_WAVE>
hipError_t launch_form(const RowsDev& a, hipStream_t s) {
  constexpr int kBytes = RowsLds<T, D, DH, MH>::kBytes;
  static_assert(kBytes <= 160 * 1024);
  auto kernel = fused_rows_kernel<T, D, DH, MH, PHI, BY_WAVE>;
  if constexpr (kBytes > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), kBytes); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(launched_workgroups(a.total)), dim3(kThreads), kBytes, s, a);
  return hipGetLastError();
}

template <typename T, int D, int DH, int MH, int PHI>
hipError_t launch_rows(const RowsDev& a, bool by_wave, hipStream_t s) {
  if constexpr (DH < 64)
    if (by_wave) return launch_form<T, D, DH, MH, PHI, true>(a, s);
  return launch_form<T, D, DH, MH, PHI, false>(a, s);
}

template <typename T, int D, int DH, int PHI>
hipError_t dispatch_rows(const RowsDev& a, bool by_wave, hipStream_t s) {
  if (a.m <= 16) return launch_rows<T, D, DH, 1, PHI>(a, by_wave, s);
  if (a.m <= 32) return launch_rows<T, D, DH, 2, PHI>(a, by_wave, s);
  if constexpr (DH >= 32) return launch_rows<T, D, DH, 4, PHI>(a, by_wave, s);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t dispatch_rows_shape(const RowsDev& a, int d, int phi, bool by_wave, hipStream_t s) {
#define LIME_CASE(D, DH) \
  if (d == D && d / a.h == DH) return phi == kPhiSoftmax ? dispatch_rows<T, D, DH, kPhiSoftmax>(a, by_wave, s) : dispatch_rows<T, D, DH, kPhiSilu>(a, by_wave, s);
  LIME_FUSED_SHAPES(LIME_CASE)
#undef LIME_CASE
  return hipErrorInvalidValue;
}

}  // namespace

// All links' logits of a row lie in registers: 64 of them, 32 where the head is narrow.  Narrow heads of any width, though each of
// their workgroups reads whole rows and projects 32 columns: lime_score_candidates, general kernels | this one, us, at one user's 300
// candidates, 64 users' 501 and 32 users' 4000: fp32 d=32 h=4 m=16 8.1|5.2 13.7|7.4 39.1|18.8, d=64 h=8 m=16 8.6|7.1 23.5|16.8
// 62.0|50.5, d=64 h=4 m=32 8.6|7.9 19.9|12.8 44.0|35.0, d=128 h=8 m=31 10.2|9.7 34.6|30.8 106|92.5; bf16 d=32 h=4 m=16 8.5|4.8 13.7|5.6
// 38.4|12.9, d=64 h=8 m=16 8.8|4.9 23.0|8.7 67.3|25.2, d=128 h=8 m=31 11.0|6.7 37.7|18.2 108|44.1.
bool fused_rows_supported(int64_t B, int64_t rows, int d, int h, int m) {
  if (!fused_shape(d, h) || m > (d / h >= 32 ? 64 : 32)) return false;
  return launch_fits(B * h + compute_units()) && rows < (int64_t{1} << 31) - 64 * kWaves * compute_units();
}

hipError_t fused_rows(const FusedRows& q, hipStream_t s) {
  // a workgroup per compute unit where the rows are many, a tile per wave where they are few
  const int64_t pairs = static_cast<int64_t>(q.B) * q.h, tiles = (static_cast<int64_t>(q.rows) + 31) / 32;
  const int parts = static_cast<int>(std::min((compute_units() + pairs - 1) / pairs, (tiles + kWaves - 1) / kWaves));
  RowsDev a{q.X, q.Ksrc, q.Vsrc, q.Wq, q.Wk, q.Wv, q.row_lens, q.k_user_stride, q.v_user_stride, q.O,
            q.B, q.rows, q.h, q.m, parts, static_cast<int>(pairs * parts), q.scale};
  // By wave: in turns of a user each, a workgroup of eight per compute unit.  Such a turn takes as long as three workgroups of one user of
  // few rows, and half a one more for each tile (in us, a workgroup | a wave a user, pairs a multiple of the compute units: fp32 d=128 h=4 m=64 16
  // candidates 4 times 31.8|22.4, 8 times 62.0|28, 300 candidates 8 times 132|112, 4 times 60.0|88; d=32 h=4 m=16 16 candidates 2 times
  // 5.1|6.4, 4 times 8.2|6.4; bf16 d=128 h=8 m=16 15.0|6.4, 300 candidates 24.8|22.5).
  const int64_t units = compute_units(), turns = (pairs + kWaves * units - 1) / (kWaves * units);
  const bool by_wave = q.d / q.h < 64 && q.k_user_stride == 0 && turns * (5 + tiles) <= 2 * ((pairs + units - 1) / units);
  if (by_wave) {
    a.parts = static_cast<int>(std::min((units + q.h - 1) / q.h, (static_cast<int64_t>(q.B) + kWaves - 1) / kWaves));
    a.total = a.parts * q.h;
  }
  return q.dtype == 0 ? dispatch_rows_shape<float>(a, q.d, q.phi, by_wave, s) : dispatch_rows_shape<bf16_t>(a, q.d, q.phi, by_wave, s);
}

}  // namespace lime
