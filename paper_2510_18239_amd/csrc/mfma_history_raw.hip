// The links over a history of few rows on operands as the caller has them: each workgroup lays its head's out itself, and the
// operands that another kernel of the call needs are packed by workgroups of the same launch.  It takes the place of a pack
// launch ahead of the history kernel, with the same sums and roundings.
#include "history_body.hpp"

namespace lime {
namespace {

constexpr int kUnitLds = 160 * 1024;

template <int DH, int M, int H>
struct RawShape {
  static constexpr int HG = heads_per_group(DH, H, kShort), TP = tiles_per_step(DH, H, kShort), D = DH * H;
  using S = HistShape<DH, M, H, HG, TP, true>;
  static_assert(HG == 1 && S::kThreads == 256, "a workgroup of the pack jobs is as large");
  static constexpr int kLds = std::max(S::kLds, PackLds<D>::kBytes);
  static constexpr int kPerUnit = std::min(kUnitLds / kLds, S::kWavesPerSimd);  // workgroups of a compute unit, by LDS and by registers
};

// What bounds this form is the wait for its operands, 64 to 160 KiB a workgroup, all asked for at once; the queries (16 products a wave
// at d = 256) are formed while the last of them arrive.  A pass of the request, with a pack launch | so, in us: d=256 h=4 m=64
// N=2048 with 16 candidates 19.4 | 16.6, with 32 768 26.3 | 23.9 (15.2 instead of 16.5 with four requests in flight).
template <int DH, int M, int H, int PHI>
hipError_t launch(const HistArgs& a, const RawArgs& r, int users, hipStream_t s) {
  using R = RawShape<DH, M, H>;
  auto kernel = links_over_history_kernel<DH, M, H, PHI, R::HG, R::TP, true>;
  if (R::kLds > 64 * 1024) {
    static PerDevice granted;
    if (hipError_t e = allow_lds(granted, reinterpret_cast<const void*>(kernel), R::kLds); e != hipSuccess) return e;
  }
  const int plane = a.chunks * users;
  launch_timed(kKernelLinksOverHistory, kernel, dim3(a.chunks, users, H + (r.pack_blocks + plane - 1) / plane), dim3(256), R::kLds, s, a, r);
  return hipGetLastError();
}

// Calls f(shape) with the RawShape of (d/h, m, h), if there is a kernel of it: embeddings from 64 on whose operands fit.
template <int DH, int M, int H, typename F>
bool with_shape(F f) {
  if constexpr (DH * H >= 64 && RawShape<DH, M, H>::kLds <= kUnitLds) return f(RawShape<DH, M, H>{}, std::integral_constant<int, M>{}), true;
  return false;
}
template <int DH, int H, typename F>
bool for_links(int m, F f) {
  switch (m) {
    case 32: return with_shape<DH, 32, H>(f);
    case 64: return with_shape<DH, 64, H>(f);
    case 96: return with_shape<DH, 96, H>(f);
    case 128: return with_shape<DH, 128, H>(f);
  }
  return false;
}
template <typename F>
bool for_shape(int dh, int h, int m, F f) {
  if (dh == 64) return h == 1 ? for_links<64, 1>(m, f) : h == 2 ? for_links<64, 2>(m, f) : h == 4 && for_links<64, 4>(m, f);
  if (dh == 32) return h == 2 ? for_links<32, 2>(m, f) : h == 4 ? for_links<32, 4>(m, f) : h == 8 && for_links<32, 8>(m, f);
  return false;
}

int pack_jobs(PackArgs& p, const PackJobs& jobs, int d, int h, int m) {
  return pack_args(p, jobs.weights, jobs.n_weights, jobs.projections, jobs.n_projections, d, h, m);
}

}  // namespace

bool history_raw_fits(const LinksOverHistory& q, int64_t workgroups, const PackJobs& beside) {
  if (beside.has_score) return false;
  PackArgs p;
  const int64_t all = workgroups + pack_jobs(p, beside, q.d, q.h, q.m);
  bool fits = false;
  for_shape(q.d / q.h, q.h, q.m, [&](auto shape, auto) { fits = all <= static_cast<int64_t>(compute_units()) * decltype(shape)::kPerUnit; });
  return fits;
}

hipError_t history_raw(const HistArgs& a, const LinksOverHistory& q, hipStream_t s) {
  RawArgs r{static_cast<const bf16_t*>(q.LC), static_cast<const bf16_t*>(q.Wq), static_cast<const bf16_t*>(q.Wk),
            static_cast<const bf16_t*>(q.Wv), q.lc_user_stride, q.scale < 0.f, 0, {}};
  r.pack_blocks = pack_jobs(r.pack, *q.beside, q.d, q.h, q.m);
  hipError_t e = hipErrorInvalidValue;
  for_shape(q.d / q.h, q.h, q.m, [&](auto shape, auto links) {
    using R = decltype(shape);
    constexpr int M = decltype(links)::value, H = R::D / (32 * R::S::MB);
    e = q.phi == kPhiSoftmax ? launch<32 * R::S::MB, M, H, kPhiSoftmax>(a, r, q.B, s) : launch<32 * R::S::MB, M, H, kPhiSilu>(a, r, q.B, s);
  });
  return e;
}

}  // namespace lime
