// The history-side softmax with a chunk walked by one wave per head (mfma_history.hip is the faster form).
//
// Every lime_scores call runs on this one.  Behind the link states its pipeline has two layer normalisations and the
// interaction network, and a score may come out near zero, where the bf16 rounding of the softmax weights shows.  A weight
// is rounded relative to the running maximum of its chunk; the other kernel's chunks and tiles are others, and with them
// the roundings.  Both are equally far from the exact scores (2-norm, relative: 0.0025 and 0.0025 at N=2048 C=32768 d=256,
// 0.024 and 0.024 at N=16384 C=512, 0.037 and 0.039 at N=50 C=16), but apart from each other they are as far: 0.0025,
// 0.021, 0.023: a program that holds scores against recorded ones, or splits its users over two builds, would see the
// larger of these.  What keeping them costs, whole calls on this kernel and on the other: 77.4 and 75.0 us, 96.9 and 77.4 us,
// 60.0 and 57.9 us.
//
// A wave owns one head of a chunk of one user's history, keeps the head's slices of W_K^T and W_V and the projected link
// queries in fragment form (W_K^T in LDS when d = 256, otherwise in registers) and walks its chunk in tiles of 32 items,
// requesting the next tile's rows before it computes the current one.
#include "history.hpp"

namespace lime {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

// COOP = false: a workgroup is one wave (one head of one chunk; grid.z = heads) that reads its rows
// straight from memory, one tile ahead.  COOP = true (long histories, d <= 128): a workgroup is h waves
// (all heads of one chunk) that copy each tile once, cooperatively and several tiles ahead, through a
// register ring into LDS, as the candidate-side kernel does.
template <int DH, int M, int H, bool WK_LDS, bool COOP>
__global__ __launch_bounds__(COOP ? 64 * H : 64) void walk_history_kernel(HistArgs a) {
  constexpr int D = DH * H;
  constexpr int K1 = D / 16, MB = DH / 32;  // projections: k-steps over d, blocks over d/h
  constexpr int K2 = DH / 16, LB = M / 32;  // scores: k-steps over d/h, blocks over links
  constexpr int P = WK_LDS ? (M >= 128 ? 1 : 2) : 4;  // COOP: tiles in flight per workgroup (registers permitting)
  constexpr int NXS = COOP ? (WK_LDS ? 1 : 2) : 1;  // COOP: LDS tile buffers (one when W_K^T fills the LDS)
  constexpr int LW = DH / 16;               // COOP: 1 KiB loads per wave and tile
  constexpr int CPR = D / 8, PITCH = 2 * D + 16;
  extern __shared__ bf16x8 lds_wk_all[];
  __shared__ __attribute__((aligned(16))) unsigned char xs[NXS][COOP ? 32 * PITCH : 16];
  const int lane = threadIdx.x & 63, head = COOP ? threadIdx.x >> 6 : blockIdx.z;
  const int n = lane & 31, g = lane >> 5;
  const int b = blockIdx.y, chunk = blockIdx.x;
  const int len = a.lens ? min(a.lens[b], a.N) : a.N;
  const int i_begin = chunk * a.chunk_items;
  if (i_begin >= len) return;  // uniform over the workgroup: nothing for this chunk
  const int i_end = min(len, i_begin + a.chunk_items);

  const bf16_t* Eb = a.E + static_cast<int64_t>(b) * a.N * D;
  // rows at or beyond the end of the chunk are replaced by zeros (their content is never used)
  auto load_tile = [&](int i0, bf16x8 (&x)[K1]) {
    const int item = i0 + n;
    const bf16_t* xrow = Eb + static_cast<int64_t>(min(item, a.N - 1)) * D + 8 * g;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      bf16x8 v;
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(0.f);
      if (item < i_end) v = *reinterpret_cast<const bf16x8*>(xrow + 16 * kk);
      x[kk] = v;
    }
  };
  // The first tile's rows come from HBM and are asked for ahead of the operands, which come from L2: behind them, as
  // the loop's own order has it, their latency would begin only once the operands had arrived (the W_K^T slice is
  // waited for on its way into LDS).
  bf16x8 xnext[COOP ? 1 : K1];
  if constexpr (!COOP) load_tile(i_begin, xnext);

  bf16x8* lds_wk = lds_wk_all + (COOP ? head * K1 * MB * 64 : 0);  // this wave's slice
  bf16x8 wk[WK_LDS ? 1 : K1][WK_LDS ? 1 : MB];
  if (WK_LDS) {
    // this head's W_K^T image: the lane moves exactly the K1*MB fragments it will read back itself
    bf16x8 tmp[K1 * MB];
#pragma unroll
    for (int it = 0; it < K1 * MB; ++it) tmp[it] = a.WkA[(head * K1 * MB + it) * 64 + lane];
#pragma unroll
    for (int it = 0; it < K1 * MB; ++it) lds_wk[it * 64 + lane] = tmp[it];
  } else {
#pragma unroll
    for (int kk = 0; kk < K1; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) wk[kk][mb] = a.WkA[((head * K1 + kk) * MB + mb) * 64 + lane];
  }
  bf16x8 wv[K1][MB];
#pragma unroll
  for (int kk = 0; kk < K1; ++kk)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) wv[kk][mb] = a.WvB[((head * K1 + kk) * MB + mb) * 64 + lane];
  bf16x8 qb[K2][LB];
  {
    const bf16x8* src = a.QB + b * a.qb_user_frags + static_cast<int64_t>(head) * K2 * LB * 64;
#pragma unroll
    for (int kk = 0; kk < K2; ++kk)
#pragma unroll
      for (int lb = 0; lb < LB; ++lb) qb[kk][lb] = src[(kk * LB + lb) * 64 + lane];
  }

  if constexpr ((!COOP && M < 128) || (COOP && WK_LDS)) {  // (not where the accumulators of 128 links need the room)
    // W_V only ever feeds the matrix cores, which read AGPRs as readily as VGPRs: pinned there, it leaves the
    // VGPRs to the values the vector ALUs touch and needs no copies.
#pragma unroll
    for (int kk = 0; kk < K1; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+a"(wv[kk][mb]));
  }
  f32x16 acc[MB][LB];
  float run_max[LB], run_sum[LB];
#pragma unroll
  for (int lb = 0; lb < LB; ++lb) {
    run_max[lb] = -INFINITY;
    run_sum[lb] = 0.f;
#pragma unroll
    for (int ob = 0; ob < MB; ++ob)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[ob][lb][i] = 0.f;
  }

  // COOP: this wave's share of a tile (32 rows = 64 D contiguous bytes), 16 bytes per lane and load
  auto issue = [&](int i0, bf16x8 (&r)[LW]) {
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int q = (head * LW + j) * 64 + lane;
      const int item = i0 + q / CPR;
      bf16x8 v;
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(0.f);
      if (item < i_end) v = *reinterpret_cast<const bf16x8*>(Eb + static_cast<int64_t>(item) * D + (q % CPR) * 8);
      r[j] = v;
    }
  };

  auto process_tile = [&](int i0, const bf16x8 (&x)[K1]) {
    // The LDS copy of W_K^T must be re-read for every tile (that is the point of keeping it in LDS
    // rather than in registers); an opaque base index stops the compiler from hoisting the reads.
    int wk_base = lane;
    asm volatile("" : "+v"(wk_base));

    f32x16 d1[MB], d2[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) d1[mb][i] = d2[mb][i] = 0.f;
    // the LDS reads run kAhead k-steps ahead of the MFMAs that use them (one wave per SIMD: nobody else
    // covers the LDS latency)
    constexpr int kAhead = 3;
    bf16x8 wkf[WK_LDS ? K1 : 1][MB];
    auto fetch = [&](int kk) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) wkf[WK_LDS ? kk : 0][mb] = lds_wk[wk_base + (kk * MB + mb) * 64];
    };
    if (WK_LDS) {
#pragma unroll
      for (int kk = 0; kk < kAhead && kk < K1; ++kk) fetch(kk);
    }
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      if (WK_LDS && kk + kAhead < K1) fetch(kk + kAhead);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const bf16x8 w = WK_LDS ? wkf[WK_LDS ? kk : 0][mb] : wk[WK_LDS ? 0 : kk][WK_LDS ? 0 : mb];
        d1[mb] = mfma32(w, x[kk], d1[mb]);
        d2[mb] = mfma32(x[kk], wv[kk][mb], d2[mb]);
      }
    }
    bf16x8 kf[K2], vf[MB][2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      kf[2 * mb] = pack_half(d1[mb], 0);
      kf[2 * mb + 1] = pack_half(d1[mb], 1);
      vf[mb][0] = pack_half(d2[mb], 0);
      vf[mb][1] = pack_half(d2[mb], 1);
    }

#pragma unroll
    for (int lb = 0; lb < LB; ++lb) {
      f32x16 sc;
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < K2; ++kk) sc = mfma32(kf[kk], qb[kk][lb], sc);
      // register 4j + r of this lane is item i0 + 8j + 4g + r; only a chunk's last tile can be ragged
      const float c = a.scale * kLog2e;  // >= 0: a negative scale is folded into the sign of the packed queries
      const bool ragged = i0 + 32 > i_end;  // uniform
      if (ragged) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (i0 + 8 * (i >> 2) + 4 * g + (i & 3) >= i_end) sc[i] = -INFINITY;
      }
      float tmax = sc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, sc[i]);
      tmax = pair_max(tmax);
      const float new_max = fmaxf(run_max[lb], tmax);  // finite: the tile holds at least one valid item
      if (__any(new_max > run_max[lb])) {  // uniform; after the first tiles the maximum rarely moves
        const float alpha = run_max[lb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((run_max[lb] - new_max) * c);
        run_sum[lb] *= alpha;
        run_max[lb] = new_max;
#pragma unroll
        for (int ob = 0; ob < MB; ++ob)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[ob][lb][i] *= alpha;
      }
      const float shift = -new_max * c;  // exp2(raw * c + shift) = exp(scale * raw - running maximum)
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float raw = sc[i];
        sc[i] = __builtin_amdgcn_exp2f(fmaf(raw, c, shift));
        if (ragged && raw == -INFINITY) sc[i] = 0.f;  // (explicit: also right for scale = 0)
        psum += sc[i];
      }
      run_sum[lb] += psum;
      const bf16x8 p0 = pack_half(sc, 0), p1 = pack_half(sc, 1);
#pragma unroll
      for (int ob = 0; ob < MB; ++ob) {
        acc[ob][lb] = mfma32(vf[ob][0], p0, acc[ob][lb]);
        acc[ob][lb] = mfma32(vf[ob][1], p1, acc[ob][lb]);
      }
    }
  };

  if constexpr (COOP) {
    bf16x8 ring[P][LW];
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (i_begin + 32 * p < i_end) issue(i_begin + 32 * p, ring[p]);
    for (int base = i_begin; base < i_end; base += 32 * P) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int i0 = base + 32 * p;
        if (i0 >= i_end) break;  // uniform over the workgroup
        unsigned char* buf = xs[NXS == 2 ? p & 1 : 0];
#pragma unroll
        for (int j = 0; j < LW; ++j) {
          const int q = (head * LW + j) * 64 + lane;
          *reinterpret_cast<bf16x8*>(buf + (q / CPR) * PITCH + (q % CPR) * 16) = ring[p][j];
        }
        // with two buffers a wave arrives here only after it has finished reading the tile before the
        // previous one, which is the one this buffer held; with one, a second barrier follows the reads
        __syncthreads();
        if (i0 + 32 * P < i_end) issue(i0 + 32 * P, ring[p]);
        bf16x8 x[K1];
#pragma unroll
        for (int kk = 0; kk < K1; ++kk) x[kk] = *reinterpret_cast<const bf16x8*>(buf + n * PITCH + 32 * kk + 16 * g);
        if (NXS == 1) __syncthreads();
        process_tile(i0, x);
      }
    }
  } else {
    for (int i0 = i_begin; i0 < i_end; i0 += 32) {
      bf16x8 x[K1];
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) x[kk] = xnext[kk];
      if (i0 + 32 < i_end) load_tile(i0 + 32, xnext);
      process_tile(i0, x);
    }
  }

  // partials: lane (link n of block lb) holds head columns 32ob + 8j + 4g + r in register 4j + r
  const int64_t slot = (static_cast<int64_t>(b) * a.chunks + chunk) * H + head;
#pragma unroll
  for (int lb = 0; lb < LB; ++lb) {
    const int link = 32 * lb + n;
    float* dst = a.part_acc + (slot * M + link) * DH + 4 * g;
#pragma unroll
    for (int ob = 0; ob < MB; ++ob)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float4 v = make_float4(acc[ob][lb][4 * j], acc[ob][lb][4 * j + 1], acc[ob][lb][4 * j + 2], acc[ob][lb][4 * j + 3]);
        *reinterpret_cast<float4*>(dst + 32 * ob + 8 * j) = v;
      }
    const float total = pair_sum(run_sum[lb]);
    if (g == 0) {
      float* ml = a.part_ml + (slot * M + link) * 2;
      ml[0] = run_max[lb] * a.scale;  // the merge works on scaled logits
      ml[1] = total;
    }
  }
}

template <int DH, int M, int H>
hipError_t launch_main(const HistArgs& a, int users, bool coop, hipStream_t s) {
  constexpr bool kWkLds = DH * H >= 256;
  constexpr size_t slice = kWkLds ? static_cast<size_t>(DH) * H * DH * 2 : 0;  // one head's slice of W_K^T
  if constexpr (H > 1 && !(kWkLds && H > 4)) {  // (eight waves of d = 256 would not fit the register file)
    if (coop) {
      constexpr size_t lds = slice * H;
      auto kernel = walk_history_kernel<DH, M, H, kWkLds, true>;
      if (lds > 64 * 1024) {
        static PerDevice granted;
        if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), static_cast<int>(lds)); e != hipSuccess) return e;
      }
      launch_timed(kKernelLinksOverHistory, kernel, dim3(a.chunks, users), dim3(64 * H), lds, s, a);
      return hipGetLastError();
    }
  }
  auto kernel = walk_history_kernel<DH, M, H, kWkLds, false>;
  if (slice > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), static_cast<int>(slice)); e != hipSuccess) return e;
  }
  launch_timed(kKernelLinksOverHistory, kernel, dim3(a.chunks, users, H), dim3(64), slice, s, a);
  return hipGetLastError();
}

template <int DH, int H>
hipError_t dispatch_m(const HistArgs& a, int links, int users, bool coop, hipStream_t s) {
  switch (links) {
    case 32: return launch_main<DH, 32, H>(a, users, coop, s);
    case 64: return launch_main<DH, 64, H>(a, users, coop, s);
    case 96: return launch_main<DH, 96, H>(a, users, coop, s);
    case 128: return launch_main<DH, 128, H>(a, users, coop, s);
  }
  return hipErrorInvalidValue;
}

template <int DH>
hipError_t dispatch_h(const HistArgs& a, int h, int links, int users, bool coop, hipStream_t s) {
  switch (h) {
    case 1: return dispatch_m<DH, 1>(a, links, users, coop, s);
    case 2: return dispatch_m<DH, 2>(a, links, users, coop, s);
    case 4: return dispatch_m<DH, 4>(a, links, users, coop, s);
    case 8: if (DH == 32) return dispatch_m<32, 8>(a, links, users, coop, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

WalkPlan walk_plan(int B, int N, int d, int h) {
  WalkPlan l{};
  const int tiles = (N + 31) / 32;
  // Short histories: every (chunk, head) pair is a one-wave workgroup and a compute unit runs four of
  // them at once (eight when d/h = 32); aim at one round of workgroups.  Long histories with d <= 128
  // (at least four tiles per compute unit): h-wave workgroups, two per compute unit.  At least two
  // tiles per chunk so that the stationary operands are fetched for more than one tile and the merge
  // stays small.
  l.coop = h > 1 && !(d >= 256 && h > 4) && static_cast<int64_t>(B) * tiles >= 4 * static_cast<int64_t>(compute_units());
  // (at d = 256 the cooperative workgroup keeps all of W_K^T in LDS and is alone on its compute unit)
  const int64_t slots = static_cast<int64_t>(l.coop ? (d >= 256 ? 1 : 2) : (d / h == 32 ? 8 : 4)) * compute_units();
  int chunk_tiles = static_cast<int>((static_cast<int64_t>(B) * tiles * (l.coop ? 1 : h) + slots - 1) / slots);
  if (chunk_tiles < 2) chunk_tiles = 2;
  if (chunk_tiles > tiles) chunk_tiles = tiles;
  l.chunk_items = chunk_tiles * 32;
  l.chunks = (tiles + chunk_tiles - 1) / chunk_tiles;
  return l;
}

hipError_t walk_history(const HistArgs& a, int d, int h, int m, int users, bool coop, hipStream_t s) {
  return d / h == 32 ? dispatch_h<32>(a, h, m, users, coop, s) : dispatch_h<64>(a, h, m, users, coop, s);
}

}  // namespace lime
