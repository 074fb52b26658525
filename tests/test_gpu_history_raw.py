"""The history kernel that lays its operands out itself (mfma_history_raw.hip, calls of few rows) against the one that reads
images packed ahead of it, which calls on prepared operands take: the same sums and roundings, so the same bits."""

import pytest
import torch

from paper_2510_18239_amd import binding

pytestmark = pytest.mark.gpu


# every width, number of heads and of links; one row, the edges of a wave's tile (32 rows) and of a step (64 or 128), several chunks
@pytest.mark.parametrize("d,h", [(64, 1), (64, 2), (128, 2), (128, 4), (256, 4), (256, 8)])
@pytest.mark.parametrize("m", [32, 64, 96, 128])
@pytest.mark.parametrize("B,N,scale", [(1, 1, 0.3), (2, 33, -0.3), (1, 64, 0.3), (3, 129, 0.3), (1, 700, -0.3)])
def test_same_bits_as_packed(d, h, m, B, N, scale):
    g = torch.Generator(device="cuda").manual_seed(d + 10 * h + 100 * m + N)
    rn = lambda shape, std=1.0: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)  # noqa: E731
    E, L, T = rn((B, N, d)), rn((m, d)), rn((B, 40, d))
    W = [rn((d, d), d ** -0.5) for _ in range(6)]
    lens = torch.randint(0, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = N
    E[torch.arange(N, device="cuda")[None, :] >= lens[:, None]] = torch.nan  # padding is never read
    prepared = binding.lime_prepare(L, L, *W[:3], *W[3:5], h, scale, scale)
    for xor in (False, True):
        expected = binding.lime_link_history_prepared(E, lens, prepared, h, m, scale, xor_attention=xor)
        if xor:
            alone = binding.lime_xor_history(E, lens, L, *W[:3], h, scale)[0]
            per_user, _ = binding.lime_xor_history(E, lens, L.expand(B, m, d).contiguous(), *W[:3], h, scale)
        else:
            alone = binding.lime_link_history(E, lens, L, *W[:3], h, scale)
            per_user = binding.lime_link_history(E, lens, L.expand(B, m, d).contiguous(), *W[:3], h, scale)
        LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, scale, scale, xor_attention=xor)
        for x in (alone, per_user, LP):
            assert torch.equal(x, expected)
        # the operands packed beside it; the value projection sums in another order (bf16: 2^-9 in each of three roundings)
        ref = binding.lime_score_candidates(T, L, LP, *W[3:], h, scale)
        assert float((O.double() - ref.double()).norm()) <= 6e-3 * float(ref.double().norm())
