"""The small kernels around the two attention stages, at the edges of their dispatch: the pack kernel's projections (one or
four 32 x 32 blocks per workgroup)."""

import pytest
import torch

from paper_2510_18239_amd import binding

pytestmark = pytest.mark.gpu


def _tensors(seed, *shapes):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [(torch.randn(s, generator=g, device="cuda") * (s[-1] ** -0.5 if len(s) == 2 and s[0] == s[1] else 1.0)).bfloat16() for s in shapes]


# 256 units of the value projection fill the compute units one each; from there on a workgroup takes four
@pytest.mark.parametrize("B,d,h,m", [(64, 128, 4, 32), (65, 128, 4, 32), (8, 256, 4, 128), (9, 256, 8, 128), (257, 64, 2, 32), (3, 32, 1, 32)])
def test_projected_links_do_not_depend_on_the_batch(B, d, h, m):
    C = 33
    LP, Wv, logits = _tensors(d + B, (B, m, d), (d, d), (B, C, h, m))
    W = torch.softmax(logits.float(), -1).bfloat16()
    O = binding.lime_score_candidates_cached(W, LP, Wv)
    for b in {0, B // 2, B - 1}:
        assert torch.equal(binding.lime_score_candidates_cached(W[b:b + 1], LP[b:b + 1], Wv)[0], O[b]), b
    b = B - 1
    V = (LP[b].double() @ Wv.double()).reshape(m, h, d // h).transpose(0, 1)
    ref = (W[b].double().transpose(0, 1) @ V).transpose(0, 1).reshape(C, d)
    # V~ and the output are rounded to bf16 (2^-9 each), fp32 sums of m and d terms besides
    assert ((O[b].double() - ref).abs() <= 2 ** -7 * ref.abs().max()).all()
