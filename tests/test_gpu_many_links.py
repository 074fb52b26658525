"""Rows over 96 or 128 links at d = 256, four heads (128: the candidate-side kernel with its operands pinned in AGPRs), against plain
64-bit arithmetic: one row, remainders of a 32-row tile, and workgroups that pass from one user to the next."""

import pytest
import torch

from paper_2510_18239_amd import binding

pytestmark = pytest.mark.gpu

D, H = 256, 4
# bf16: projected rows, keys, values and weights are rounded to 2^-9 once each, and so is the result
TOLERANCE = 1e-2


def _heads(x):
    return x.reshape(*x.shape[:-1], H, D // H).transpose(-2, -3)


def _rows_over_links(q, k, v, scale, silu):
    s = _heads(q) @ _heads(k).transpose(-1, -2) * scale
    w = s * torch.sigmoid(s) / k.shape[-2] if silu else torch.softmax(s, dim=-1)
    return (w @ _heads(v)).transpose(-2, -3).reshape(q.shape)


@pytest.mark.parametrize("m", [96, 128])
@pytest.mark.parametrize("B,rows", [(1, 1), (2, 33), (1, 8200), (9, 1000)])
@pytest.mark.parametrize("silu", [False, True])
def test_against_64_bits(m, B, rows, silu):
    g = torch.Generator(device="cuda").manual_seed(m + B + rows)
    rn = lambda shape, std=1.0: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)  # noqa: E731
    X, L, LP, W = rn((B, rows, D)), rn((B, m, D)), rn((B, m, D)), [rn((D, D), D ** -0.5) for _ in range(3)]
    scale, D64 = (D // H) ** -0.5, lambda x: x.double()
    if silu:  # O[S] of an XOR layer: links of each user, keys and values both
        got = binding.lime_xor_history(X, None, L, *W, H, scale, want_os=True)[1]
        keys, values = D64(L) @ D64(W[1]), D64(L) @ D64(W[2])
    else:
        got = binding.lime_score_candidates(X, L[0], LP, *W, H, scale)
        keys, values = (D64(L[0]) @ D64(W[1])).expand(B, m, D), D64(LP) @ D64(W[2])
    ref = _rows_over_links(D64(X) @ D64(W[0]), keys, values, scale, silu)
    assert float((got.double() - ref).norm() / ref.norm()) <= TOLERANCE
