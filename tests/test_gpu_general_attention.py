"""The general kernels' attention: the order of its sums over the keys is the same however the work is cut (a wave, the
four waves of a workgroup, a workgroup per chunk of 1024 keys), so that a user's result has the same bits alone and in any
batch, and with every workspace."""

import re

import pytest
import torch

from paper_2510_18239_amd import binding

pytestmark = pytest.mark.gpu


def _users(B, N, d, m, seed, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda shape, std=1.0: (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)  # noqa: E731
    lens = torch.randint(0, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[:3] = torch.tensor([N, (N + 1) // 2, 1], device="cuda")[: min(B, 3)]
    W = [rn((d, d), d ** -0.5) for _ in range(3)]
    return rn((B, N, d)), lens, rn((m, d)), W


@pytest.mark.parametrize("d,h,m,N,B", [
    # B users: a wave each (a thousand or more tiles of queries), a quarter of them: a workgroup each; one: chunks
    (32, 4, 8, 33, 256), (64, 4, 16, 128, 256), (64, 4, 16, 333, 257), (128, 4, 40, 1024, 130), (96, 4, 16, 97, 256),
    (64, 1, 16, 161, 1024), (128, 1, 16, 200, 1024), (192, 1, 16, 75, 1024), (50, 2, 16, 150, 512),
    # more than one chunk: never a wave each
    (64, 4, 16, 2500, 256), (256, 1, 16, 1030, 300),
])
@pytest.mark.parametrize("xor", [False, True])
def test_bits_do_not_depend_on_the_batch(d, h, m, N, B, xor):
    E, lens, L, W = _users(B, N, d, m, seed=d + N)
    call = binding.lime_xor_history if xor else binding.lime_link_history
    run = lambda part: (call(E[part], lens[part], L, *W, h, 0.5) if not xor else call(E[part], lens[part], L, *W, h, 0.5)[0])  # noqa: E731
    whole = run(slice(0, B))
    assert torch.isfinite(whole).all()
    quarter = run(slice(0, (B + 3) // 4))
    assert torch.equal(quarter, whole[: (B + 3) // 4])
    for b in (0, 1, 2, B - 1):
        assert torch.equal(run(slice(b, b + 1))[0], whole[b]), b


def test_request_bits_do_not_depend_on_the_batch():
    B, N, C, d, h, m = 16, 777, 1001, 128, 4, 64
    E, lens, L, W = _users(B, N, d, m, seed=5)
    T = torch.randn((B, C, d), device="cuda")
    run = lambda part: binding.lime_request(E[part], lens[part], L, *W, T[part], L, *W, h, 0.2, 0.2)  # noqa: E731
    LP, O = run(slice(0, B))
    for b in (0, 7):
        LP1, O1 = run(slice(b, b + 1))
        assert torch.equal(LP1[0], LP[b]) and torch.equal(O1[0], O[b]), b


def test_bits_do_not_depend_on_the_workspace():
    """The least workspace that a call accepts has no room for the chunks' states."""
    B, N, C, d, h, m = 2, 2500, 20, 64, 2, 16
    E, lens, L, W = _users(B, N, d, m, seed=9)
    T = torch.randn((B, C, d), device="cuda")
    calls = [lambda **kw: binding.lime_link_history(E, lens, L, *W, h, 0.3, **kw),
             lambda **kw: binding.lime_xor_history(E, lens, L, *W, h, 0.3, **kw)[0],
             lambda **kw: binding.mha_target_attention(T, E, lens, *W, h, 0.3, **kw)]
    for call in calls:
        with pytest.raises(binding.LimeError) as e:
            call(workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
        least = int(re.search(r"workspace of (\d+) bytes needed", str(e.value)).group(1))
        small = call(workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
        assert torch.equal(small, call())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,h,m", [(48, 2, 20), (50, 2, 45), (40, 1, 7), (96, 1, 150), (300, 2, 33), (32, 2, 16), (64, 1, 70)])
def test_infinite_links(d, h, m, dtype):
    """An infinite key entry makes its logit infinite and nothing else (weight zero where it is -inf, also where that are all
    logits of 32 keys in a row); an infinite value stays infinite in its own column.  Keys and values are the links as they
    are, odd counts and head widths among them."""
    dh, C = d // h, 37
    g = torch.Generator(device="cuda").manual_seed(d)
    rand = lambda *shape: (torch.rand(shape, generator=g, device="cuda") + 0.25).to(dtype)  # noqa: E731
    T, L, LP = rand(1, C, d), rand(m, d), rand(1, m, d)
    L[0, dh - 1] = -torch.inf   # the first head's last column
    if m > 64:
        L[:32, d - dh] = -torch.inf  # a whole tile of the last head's logits
    LP[0, m - 1, d - dh] = torch.inf  # the last key's value, in the last head's first column
    O = binding.lime_score_candidates(T, L, LP, None, None, None, h, 0.1).double().cpu()
    q, k, v = (x.double().cpu().reshape(-1, h, dh).transpose(0, 1) for x in (T[0], L, LP[0]))
    ref = (torch.softmax(q @ k.transpose(1, 2) * 0.1, dim=-1) @ v).transpose(0, 1).reshape(1, C, d)
    finite = torch.isfinite(ref)
    assert (~finite).sum() == C and torch.equal(O[~finite], ref[~finite])
    assert (O - ref)[finite].abs().max() <= (1e-4 if dtype == torch.float32 else 2e-2)
