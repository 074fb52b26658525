// Operand packing for the matrix-core kernels: weight matrices and the small projected link
// matrices (m rows) are written once per call in MFMA fragment order.
#include "pack.hpp"

namespace lime {
namespace {

template <int D, int SDH, int SM>
__global__ __launch_bounds__(256) void pack_kernel(PackArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[PackLds<D>::kBytes];
  pack_block<D, SDH, SM>(p, blockIdx.x, lds);
}

}  // namespace

hipError_t pack_operands(const PackWeight* weights, int n_weights, const PackProject* projections, int n_projections,
                         int d, int h, int m, hipStream_t s, const PackScore* score) {
  if (n_weights > kMaxWeights || n_projections > kMaxJobs) return hipErrorInvalidValue;
  PackArgs p;
  int grid = pack_args(p, weights, n_weights, projections, n_projections, d, h, m);
  const int dh = d / h, nkb = d / 32;
  if (score == nullptr) {
    if (grid == 0) return hipSuccess;
    switch (d) {  // every d the matrix-core kernels take
      case 32: hipLaunchKernelGGL((pack_kernel<32, 0, 0>), dim3(grid), dim3(256), 0, s, p); break;
      case 64: hipLaunchKernelGGL((pack_kernel<64, 0, 0>), dim3(grid), dim3(256), 0, s, p); break;
      case 128: hipLaunchKernelGGL((pack_kernel<128, 0, 0>), dim3(grid), dim3(256), 0, s, p); break;
      case 256: hipLaunchKernelGGL((pack_kernel<256, 0, 0>), dim3(grid), dim3(256), 0, s, p); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  p.s_wq = static_cast<const bf16_t*>(score->Wq), p.s_k = static_cast<const bf16_t*>(score->Ksrc);
  p.s_wk = static_cast<const bf16_t*>(score->Wk), p.s_img = static_cast<bf16_t*>(score->image);
  p.s_sign = score->sign;
  grid += (h * nkb * (m / 32) + 3) / 4;  // four wavefronts per block, one 32 x 32 block of the image each
#define LIME_SCORE_CASE(DH_, M_, NKB_)                                                              \
  if (dh == DH_ && m == M_ && nkb == NKB_) {                                                        \
    hipLaunchKernelGGL((pack_kernel<32 * NKB_, DH_, M_>), dim3(grid), dim3(256), 0, s, p);          \
    return hipGetLastError();                                                                       \
  }
  LIME_SCORE_CASE(64, 64, 8) LIME_SCORE_CASE(64, 64, 4) LIME_SCORE_CASE(64, 64, 2)
  LIME_SCORE_CASE(64, 32, 8) LIME_SCORE_CASE(64, 32, 4) LIME_SCORE_CASE(64, 32, 2)
  LIME_SCORE_CASE(32, 32, 8) LIME_SCORE_CASE(32, 32, 4) LIME_SCORE_CASE(32, 32, 2) LIME_SCORE_CASE(32, 32, 1)
#undef LIME_SCORE_CASE
  return hipErrorInvalidValue;
}

hipError_t pack_operands(const PackJobs& jobs, int d, int h, int m, hipStream_t s) {
  return pack_operands(jobs.weights, jobs.n_weights, jobs.projections, jobs.n_projections, d, h, m, s,
                       jobs.has_score ? &jobs.score : nullptr);
}

PreparedLayout prepared_layout(int d, int m) {
  PreparedLayout l{};
  const size_t w = align_up(static_cast<size_t>(d) * d * 2 + kQueryImagePadBytes), links = align_up(static_cast<size_t>(m) * d * 2);
  l.wk = 0, l.wv = w, l.qb = 2 * w, l.wq = 2 * w + links, l.ka = 3 * w + links, l.total = 3 * w + 2 * links;
  return l;
}

hipError_t prepare_operands(const PrepareOperands& p, void* prepared, hipStream_t s) {
  const PreparedLayout l = prepared_layout(p.d, p.m);
  char* base = static_cast<char*>(prepared);
  const float sign_cand = p.scale_cand < 0.f ? -1.f : 1.f;
  PackWeight wjobs[3] = {{p.Wk_hist, base + l.wk}, {p.Wv_hist, base + l.wv}, {p.Wq_cand, base + l.wq, 1.f, kQueryImageHeadPad}};
  PackProject pjobs[2] = {{p.LC, p.Wq_hist, base + l.qb, 0, 1, kPackKeys, p.scale_hist < 0.f ? -1.f : 1.f},
                          {p.L, p.Wk_cand, base + l.ka, 0, 1, kPackKeys, sign_cand}};
  if (fused_scores(p.d, p.h, p.m, false)) {
    // the candidate stage then wants G = W_Q (L W_K)^T per head in place of W_Q^T and K~
    PackScore sjob{p.Wq_cand, p.L, p.Wk_cand, base + l.wq, sign_cand};
    return pack_operands(wjobs, 2, pjobs, 1, p.d, p.h, p.m, s, &sjob);
  }
  return pack_operands(wjobs, 3, pjobs, 2, p.d, p.h, p.m, s);
}

}  // namespace lime
