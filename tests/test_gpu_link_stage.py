"""The small kernels around the two attention stages, at the edges of their dispatch: the pack kernel's projections (one or
four 32 x 32 blocks per workgroup) and the merge of a history's chunks, with and without the value projection."""

import re

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


# rows of link states up to and past what runs at once with a workgroup each, and with one per eight of them; up to 8, 32 and
# more chunks of a history
@pytest.mark.parametrize("B,N,d,h,m", [
    (4, 300, 256, 4, 64), (5, 300, 256, 4, 64), (8, 129, 128, 4, 64), (9, 129, 128, 4, 64), (33, 70, 64, 2, 32), (65, 70, 32, 1, 32),
    (17, 200, 256, 4, 128), (129, 33, 32, 1, 128), (33, 400, 128, 4, 128),
    (3, 12000, 256, 4, 128), (5, 26240, 128, 2, 128), (1, 16384, 64, 1, 32), (1, 2048, 256, 8, 96)])
@pytest.mark.parametrize("xor", [False, True])
def test_merged_link_states(B, N, d, h, m, xor):
    C = 40
    E, T, L, Wq, Wk, Wv, Wv2 = _tensors(N + m, (B, N, d), (B, C, d), (m, d), (d, d), (d, d), (d, d), (d, d))
    lens = torch.randint(1, N + 1, (B,), device="cuda", dtype=torch.int32, generator=torch.Generator(device="cuda").manual_seed(B))
    lens[0] = N
    if B > 1:
        lens[1] = 0
    s = (d // h) ** -0.5
    LP, O = binding.lime_request(E, lens, L, Wq, Wk, Wv, T, L, Wq, Wk, Wv2, h, s, s, xor_attention=xor)
    alone = binding.lime_xor_history(E, lens, L, Wq, Wk, Wv, h, s)[0] if xor else binding.lime_link_history(E, lens, L, Wq, Wk, Wv, h, s)
    assert torch.equal(LP, alone)  # the merge kernel's sums, whichever kernel merges
    O2 = binding.lime_score_candidates(T, L, LP, Wq, Wk, Wv2, h, s)
    # V~ summed in another order: at most a bf16 step apart, weighted by probabilities, and the output's rounding
    assert ((O.float() - O2.float()).abs() <= 2 ** -7 * (O2.float().abs().amax(dim=(1, 2), keepdim=True) + 1e-30)).all()
    heads = lambda x: x.float().reshape(-1, h, d // h).transpose(0, 1).contiguous()  # noqa: E731
    for b in sorted({0, 1, B - 1} & set(range(B))):
        n = int(lens[b])
        if n == 0:
            assert not LP[b].any()
            continue
        Eb, q = E[b, :n].float(), heads(L.float() @ Wq.float())
        k, v = heads(Eb @ Wk.float()), heads(Eb @ Wv.float())
        logits = (q @ k.transpose(1, 2).contiguous()) * s
        w = torch.nn.functional.silu(logits) / n if xor else torch.softmax(logits, -1)
        ref = (w @ v).transpose(0, 1).reshape(m, d)
        err = (LP[b].float() - ref).abs().max()
        assert err <= 2e-2 and err <= 2e-2 * ref.abs().max(), (b, float(err))


@pytest.mark.parametrize("d,h,m", [(128, 4, 64), (128, 2, 32), (32, 1, 96)])
def test_xor_layers_with_a_negative_scale(d, h, m):
    """SiLU(-s x) with the sign folded into Q~ and K~: negating W_Q as well gives the same logits, bit for bit."""
    E, L, Wq, Wk, Wv = _tensors(d, (3, 75, d), (m, d), (d, d), (d, d), (d, d))
    Wu, Wo = (torch.stack(_tensors(d + i, (d, d), (d, d), (d, d))) for i in (1, 2))
    lens = torch.tensor([75, 0, 33], dtype=torch.int32, device="cuda")
    a = binding.lime_xor_layers(E, lens, L, Wq, Wk, Wv, Wu, Wo, h, 0.4)
    assert torch.isfinite(a).all() and a[0].any() and not a[1].any()
    assert torch.equal(a, binding.lime_xor_layers(E, lens, L, -Wq, Wk, Wv, Wu, Wo, h, -0.4))


# one user's history in 10, 12, 20, 26 and 41 chunks, its link states by a workgroup each (MergeRow) or by thread (MergeQuad)
@pytest.mark.parametrize("B,N,d,h,m", [
    (2, 640, 256, 4, 128), (1, 768, 256, 4, 32), (2, 1280, 256, 4, 128), (2, 1664, 256, 4, 128), (1, 2624, 256, 4, 64),
    (3, 640, 256, 4, 128), (3, 1280, 256, 4, 128), (9, 1664, 64, 1, 128), (1, 5248, 128, 2, 64)])
@pytest.mark.parametrize("xor", [False, True])
def test_chunks_are_merged_in_one_ascending_chain(B, N, d, h, m, xor):
    """Every logit is the same, and the values of a user's first and last rows are 2^60 and -2^60, those between one: in
    ascending order the first absorbs the ones (2^60 has steps of 2^37), and the last leaves zero, exactly.  (Several sums of
    chunks, added at the end, would keep the ones of those without the first row.)"""
    E = torch.zeros(B, N, d)
    E[:, :, :2] = 1.0
    E[:, 0, 1], E[:, -1, 1] = 2.0 ** 60, -2.0 ** 60
    L, Wq, Wv = torch.zeros(m, d), torch.zeros(d, d), torch.zeros(d, d)
    L[:, 0] = 1.0
    Wq[0, ::d // h] = 1.0  # (also W_K)
    Wv[1] = 1.0
    T = torch.zeros(B, 3, d)
    E, L, Wq, Wv, T = (x.bfloat16().cuda() for x in (E, L, Wq, Wv, T))
    LP = binding.lime_xor_history(E, None, L, Wq, Wq, Wv, h, 1.0)[0] if xor else binding.lime_link_history(E, None, L, Wq, Wq, Wv, h, 1.0)
    assert (LP == 0).all()
    LP, O = binding.lime_request(E, None, L, Wq, Wq, Wv, T, L, Wq, Wq, Wv, h, 1.0, 1.0, xor_attention=xor)
    assert (LP == 0).all() and (O == 0).all()


# batches on either side of the line between a workgroup and a thread per link state, with histories in the same chunks
@pytest.mark.parametrize("B,N,d,h,m", [(2, 1300, 256, 4, 128), (2, 500, 256, 4, 128), (4, 1500, 128, 4, 128), (8, 129, 128, 4, 64)])
@pytest.mark.parametrize("xor", [False, True])
def test_a_link_state_has_the_same_bits_in_either_merge(B, N, d, h, m, xor):
    E, T, L, Wq, Wk, Wv = _tensors(N + m, (B + 1, N, d), (B + 1, 5, d), (m, d), (d, d), (d, d), (d, d))
    lens = torch.randint(1, N + 1, (B + 1,), device="cuda", dtype=torch.int32, generator=torch.Generator(device="cuda").manual_seed(B))
    lens[0], lens[1] = N, 0
    s = (d // h) ** -0.5

    def states(n):
        LP, _ = binding.lime_request(E[:n], lens[:n], L, Wq, Wk, Wv, T[:n], L, Wq, Wk, Wv, h, s, s, xor_attention=xor)
        alone = binding.lime_xor_history(E[:n], lens[:n], L, Wq, Wk, Wv, h, s)[0] if xor else binding.lime_link_history(E[:n], lens[:n], L, Wq, Wk, Wv, h, s)
        return LP, alone

    few, many = states(B), states(B + 1)
    for a, b in zip(few, many):
        assert torch.equal(a, few[0]) and torch.equal(b[:B], a)


@pytest.mark.parametrize("B,N,d,h,m,layers", [(1, 31, 128, 4, 96, 3), (3, 31, 128, 2, 32, 2), (1, 1, 128, 4, 64, 3), (1, 31, 64, 2, 64, 3), (1, 1, 32, 1, 32, 2)])
@pytest.mark.parametrize("scale", [0.4, -0.4])
def test_xor_layers_in_the_least_workspace(B, N, d, h, m, layers, scale):
    """Histories no longer than the links: the kernels that hold a layer's operands in registers ask for more workspace than a
    call needs.  With what it needs it runs on the others, to the same bits."""
    E, L, Wq, Wk, Wv = _tensors(d + N, (B, N, d), (B, m, d), (d, d), (d, d), (d, d))
    Wu, Wo = (torch.stack(_tensors(d + i, *[(d, d)] * layers)) for i in (1, 2))
    lens = torch.tensor([N, 0, N // 2][:B], dtype=torch.int32, device="cuda")

    def call(bytes_):
        ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        return binding.lime_xor_layers(E, lens, L, Wq, Wk, Wv, Wu, Wo, h, scale, workspace=ws)

    with pytest.raises(RuntimeError, match="bytes needed") as e:
        call(256)
    needed, full = int(re.search(r"(\d+) bytes needed", str(e.value))[1]), binding.workspace_bytes(binding.OP_XOR_LAYERS, B=B, N=N, d=d, h=h, m=m)
    assert needed < full
    a, b = call(needed), call(full)
    assert a.any() and torch.equal(a, b)


@pytest.mark.parametrize("d,h,m", [(128, 4, 64), (64, 2, 96), (128, 4, 128)])
def test_xor_layers_keep_a_users_infinities(d, h, m):
    """A user with an infinite and a NaN entry in its history leaves the others' link states as they are."""
    B, N = 5, 90
    E, L, Wq, Wk, Wv = _tensors(d + m, (B, N, d), (m, d), (d, d), (d, d), (d, d))
    Wu, Wo = (torch.stack(_tensors(d + i, (d, d), (d, d), (d, d))) for i in (3, 4))
    lens = torch.tensor([90, 33, 64, 0, 90], dtype=torch.int32, device="cuda")
    clean = binding.lime_xor_layers(E, lens, L, Wq, Wk, Wv, Wu, Wo, h, 0.4)
    E[1, 5, 3], E[4, 89, 0] = float("inf"), float("nan")
    E[2, 64:] = float("nan")  # padding
    LP = binding.lime_xor_layers(E, lens, L, Wq, Wk, Wv, Wu, Wo, h, 0.4)
    for b in (0, 2, 3):
        assert torch.equal(LP[b], clean[b]), b
    assert not torch.isfinite(LP[1]).all() and not torch.isfinite(LP[4]).all()


@pytest.mark.parametrize("B,N,d,h,m", [(3, 640, 256, 4, 32), (9, 129, 128, 4, 64), (17, 200, 256, 4, 128)])
@pytest.mark.parametrize("xor", [False, True])
def test_merges_keep_a_users_infinities(B, N, d, h, m, xor):
    E, T, L, Wq, Wk, Wv = _tensors(B, (B, N, d), (B, 5, d), (m, d), (d, d), (d, d), (d, d))
    lens = torch.full((B,), N, device="cuda", dtype=torch.int32)
    lens[0], lens[2] = N - 31, 1
    s = (d // h) ** -0.5

    def request():
        return binding.lime_request(E, lens, L, Wq, Wk, Wv, T, L, Wq, Wk, Wv, h, s, s, xor_attention=xor)

    clean = request()
    E[1, N // 2, 3] = float("inf")
    for b in range(B):
        E[b, int(lens[b]):] = float("nan")  # padding
    for x, y in zip(request(), clean):
        others = [b for b in range(B) if b != 1]
        assert torch.equal(x[others], y[others]) and not torch.isfinite(x[1]).all()
