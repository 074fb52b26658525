"""GPU parity of the scoring pipeline around the attention stages - layer normalisation (Appendix C), link
contextualisation (Eq. 2), the interaction network (Section 3.3) and the whole request from embeddings to scores
(lime_scores) - against the CPU oracle on the same seeded inputs, element by element, through the C ABI."""

import numpy as np
import pytest
import torch

from oracle import lime_oracle as orc
from paper_2510_18239_amd import binding, synth
from parity_util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def _rnd(x, dtype):
    return synth.round_to(np.asarray(x, dtype=np.float32), dtype)


@pytest.mark.parametrize("dtype,rows,d", [("bf16", 1000, 256), ("bf16", 333, 128), ("bf16", 70, 32), ("bf16", 65, 64),
                                          ("bf16", 130, 512), ("bf16", 77, 96), ("bf16", 50, 24), ("fp32", 200, 256),
                                          ("fp32", 33, 40), ("bf16", 1, 256)])
def test_layer_norm(dtype, rows, d):
    r = np.random.default_rng(700 + rows + d)
    X = _rnd(r.standard_normal((rows, d)) * 3.0 + 1.5, dtype)
    g, b = _rnd(1.0 + 0.3 * r.standard_normal(d), dtype), _rnd(0.3 * r.standard_normal(d), dtype)
    Y = binding.lime_layer_norm(dev(X, dtype), dev(g, dtype), dev(b, dtype), 1e-5)
    assert_close(host(Y), orc.layer_norm(X, g, b, 1e-5), dtype, f"layer norm d={d}")
    # without scale and shift, and in place
    Xd = dev(X, dtype)
    binding.lime_layer_norm(Xd, None, None, 1e-3, Y=Xd)
    assert_close(host(Xd), orc.layer_norm(X, None, None, 1e-3), dtype, f"plain layer norm in place d={d}")


@pytest.mark.parametrize("dtype,B,m,d,dc,dhid", [("bf16", 3, 64, 128, 24, 96), ("bf16", 1, 64, 256, 64, 256), ("fp32", 2, 16, 64, 5, 33),
                                                 ("bf16", 5, 20, 40, 7, 50)])
def test_contextualize_links(dtype, B, m, d, dc, dhid):
    w = synth.make_workload(710 + d, B=B, N=8, C=8, d=d, h=1, m=m, dtype=dtype)
    p = synth.scoring_params(710 + d, B, m, d, dc, dhid, [1], dtype)
    LC = binding.lime_contextualize_links(dev(w.L, dtype), dev(p["EC"], dtype), *[dev(x, dtype) for x in p["ctx"]])
    assert LC.shape == (B, m, d)
    assert_close(host(LC), orc.contextualize_links(w.L, p["EC"], *p["ctx"]), dtype, "L^C of Eq. 2")


@pytest.mark.parametrize("dtype,rows,d,widths", [
    ("bf16", 1000, 256, [512, 128, 64, 1]),   # matrix cores; a ragged last block of rows
    ("bf16", 4096, 256, [96, 1]),
    ("bf16", 300, 256, [512, 256, 128, 1]),
    ("bf16", 129, 128, [512, 128, 64, 1]),
    ("bf16", 257, 128, [96, 1]),
    ("bf16", 64, 32, [512, 256, 128, 1]),
    ("bf16", 1, 64, [96, 1]),                 # one chunk and no next one to read ahead
    ("bf16", 31, 32, [96, 1]),
    ("bf16", 200, 64, [40, 8, 1]),            # widths the matrix-core kernel is not built for: fp32 arithmetic
    ("bf16", 100, 256, [1]),                  # no hidden layer: a dot product
    ("fp32", 150, 256, [96, 1]),
    ("fp32", 90, 24, [50, 20, 10, 1]),
])
def test_interaction_mlp(dtype, rows, d, widths):
    r = np.random.default_rng(720 + rows)
    O = _rnd(r.standard_normal((rows, d)) * 0.5, dtype)
    p = synth.scoring_params(720 + d + len(widths), 1, 8, d, 4, 8, widths, dtype)
    Ws, bs = p["mlp"]
    scores = binding.lime_interaction_mlp(dev(O, dtype), [dev(x, dtype) for x in Ws], [dev(x, dtype) for x in bs])
    assert scores.dtype == torch.float32 and scores.shape == (rows,)
    assert_close(scores.double().cpu().numpy(), orc.interaction_mlp(O, Ws, bs), dtype, f"scores d={d} widths={widths}")
    # biases absent
    scores = binding.lime_interaction_mlp(dev(O, dtype), [dev(x, dtype) for x in Ws], [None] * len(Ws))
    assert_close(scores.double().cpu().numpy(), orc.interaction_mlp(O, Ws, [np.zeros_like(b) for b in bs]), dtype, "scores without biases")


@pytest.mark.parametrize("d,widths", [(256, [512, 128, 64, 1]), (128, [512, 256, 128, 1]), (32, [512, 256, 128, 1]), (256, [96, 1]), (64, [96, 1])])
def test_interaction_mlp_sums_a_unit_in_one_chain(d, widths):
    """A hidden unit's sum takes its k-steps of 16 in ascending order into one accumulator: 2^24, which absorbs the ones of the
    steps between, minus 2^24 is zero.  (In two accumulators the ones of every other step would be left over.)  Every product and
    every sum is exact in fp32 but the absorbed ones, so the score is the last bias, exactly."""
    dims = [d] + widths
    for layer in range(len(widths) - 1):
        K = dims[layer]
        x, w = torch.zeros(K), torch.zeros(K)
        x[::16] = w[::16] = 1.0
        x[0] = x[K - 16] = w[0] = 4096.0
        w[K - 16] = -4096.0
        Ws = []
        for i in range(len(widths)):
            W = torch.zeros(dims[i], dims[i + 1])
            if i + 1 == layer:
                W[0] = x         # the first unit, which is one, on to the inputs of the layer in question
            elif i == layer:
                W[:] = w[:, None]
            elif i > layer:
                W[:] = 1.0
            else:
                W[0, 0] = 1.0
            Ws.append(W.bfloat16().cuda())
        O = torch.zeros(130, d)
        if layer == 0:
            O[:] = x
        else:
            O[:, 0] = 1.0
        bias = [None] * (len(widths) - 1) + [torch.tensor([3.0], device="cuda").bfloat16()]
        scores = binding.lime_interaction_mlp(O.bfloat16().cuda(), Ws, bias)
        assert (scores == 3.0).all(), (layer, scores.unique())


def _request(idx, B, N, C, d, h, m, dc, dhid, widths, dtype, len_range, plain_norm=None, lens=None):
    w = synth.make_workload(idx, B=B, N=N, C=C, d=d, h=h, m=m, dtype=dtype, gain=4.0, len_range=len_range,
                            pad_value=np.nan if len_range else None)
    if lens is not None:  # of the first users
        w.lens[:len(lens)] = lens
        for b, n in enumerate(lens):
            w.E[b, n:] = np.nan
            w.E[b, :n] = np.nan_to_num(w.E[b, :n], nan=0.0)  # rows that became valid after the length change
    p = synth.scoring_params(idx, B, m, d, dc, dhid, widths, dtype)
    if plain_norm is not None:  # this normalisation without scale and shift
        p[plain_norm] = (None, None)
    g = lambda x: None if x is None else dev(x, dtype)  # noqa: E731
    pair = lambda t: tuple(g(x) for x in t)  # noqa: E731
    keep = dict(L=g(w.L), ctx=pair(p["ctx"]), hist=pair(p["hist"]), cand=pair(p["cand"]),
                mlp=([g(x) for x in p["mlp"][0]], [g(x) for x in p["mlp"][1]]),
                **{k: pair(p[k]) for k in ("ln_hist_q", "ln_hist_kv", "ln_cand_q", "ln_cand_k", "ln_cand_v")})
    s = w.softmax_scale
    model = binding.scoring_model(keep["L"], keep["ctx"], keep["hist"], keep["cand"], keep["ln_hist_q"], keep["ln_hist_kv"],
                                  keep["ln_cand_q"], keep["ln_cand_k"], keep["ln_cand_v"], keep["mlp"], h, s, s)
    lens = None if w.lens is None else torch.from_numpy(w.lens).cuda()
    scores, LC, LP, O = binding.lime_scores(model, g(w.E), lens, g(p["EC"]), g(w.T), want_intermediates=True)
    torch.cuda.synchronize()
    ref = orc.lime_scores(w.E, w.lens, w.L, p["EC"], w.T, p, h, s, s, return_all=True)
    # every stage against the oracle on what the GPU handed that stage (the tensors travel in the storage type) ...
    ln = orc.layer_norm
    assert_close(host(LC), ref[1], dtype, "lime_scores L^C")
    LP_ref = orc.lime_link_history(ln(w.E, *p["ln_hist_kv"]), w.lens, ln(host(LC), *p["ln_hist_q"]), *p["hist"], h, s)
    assert_close(host(LP), LP_ref, dtype, "lime_scores L^P on the GPU's L^C")
    O_ref = orc.lime_score_candidates(ln(w.T, *p["ln_cand_q"]), ln(w.L, *p["ln_cand_k"]), ln(host(LP), *p["ln_cand_v"]), *p["cand"], h, s)
    assert_close(host(O), O_ref, dtype, "lime_scores O on the GPU's L^P")
    assert_close(scores.double().cpu().numpy(), orc.interaction_mlp(host(O), *p["mlp"]), dtype, "lime_scores scores on the GPU's O")
    # ... and the whole chain against the oracle's own chain
    for name, got, want in zip(("L^P", "O"), (LP, O), ref[2:]):
        assert_close(got.double().cpu().numpy(), want, dtype, f"lime_scores {name}, whole chain")
    # The logit at the end of the chain: seven tensors have been stored in the storage type on the way (normalised E, L^C,
    # T, L, L^P; L^P; O) and an MLP logit is a sum with cancellation, so its error is a larger part of the largest logit
    # than any single stage's (up to 2.1 % measured for bf16): the stated absolute bar is asserted, the ratio printed.
    assert_close(scores.double().cpu().numpy(), ref[0], dtype, "lime_scores scores, whole chain", relative=dtype == "fp32")
    # and without the intermediate outputs: the same scores
    again = binding.lime_scores(model, g(w.E), lens, g(p["EC"]), g(w.T))
    assert torch.equal(again, scores)
    del keep
    return scores


@pytest.mark.parametrize("B,N,C,d,h,m,dc,dhid,widths,dtype", [
    (3, 333, 517, 128, 4, 64, 24, 96, [512, 128, 64, 1], "bf16"),
    (2, 257, 130, 256, 4, 32, 16, 128, [96, 1], "bf16"),
    (3, 9000, 40, 256, 4, 32, 16, 64, [96, 1], "bf16"),   # history rows enough for a normalisation launch of their own
    (2, 100, 70, 48, 2, 20, 5, 30, [24, 1], "bf16"),      # everything on the general kernels
    (2, 150, 90, 64, 2, 16, 8, 40, [32, 16, 1], "fp32"),
])
def test_lime_scores_small(B, N, C, d, h, m, dc, dhid, widths, dtype):
    _request(730 + d, B, N, C, d, h, m, dc, dhid, widths, dtype, (max(1, N // 3), N))


def test_lime_scores_with_a_normalisation_without_parameters():
    """Without scale and shift for one of the normalisations the request takes the separate normalisation passes (the
    kernels that normalise on the way in fetch both unconditionally): same shape as the first case above."""
    _request(731, 3, 333, 517, 128, 4, 64, 24, 96, [512, 128, 64, 1], "bf16", (111, 333), plain_norm="ln_cand_q")


def test_lime_scores_config2_full_size():
    """32 users, ragged histories of 512..1024 items, d = 128, 1024 candidates each; Appendix C's [512, 128, 64] network."""
    c = synth.CONFIGS[2]
    _request(2, c["B"], c["N"], c["C"], c["d"], c["h"], c["m"], 32, 128, [512, 128, 64, 1], "bf16", c["len_range"])


@pytest.mark.parametrize("widths", [[96, 1], [512, 128, 64, 1]])
def test_lime_scores_config3_full_size(widths):
    """The headline request (one user, N = 2048, 32 768 candidates, d = 256, 4 heads, 64 links) from embeddings to scores,
    with the industrial interaction network [96] and the largest public one."""
    c = synth.CONFIGS[3]
    _request(3, c["B"], c["N"], c["C"], c["d"], c["h"], c["m"], 64, 256, widths, "bf16", None)


@pytest.mark.parametrize("B,d,h,m", [
    (2, 64, 2, 32),    # two column blocks: each wavefront normalises its rows by itself
    (3, 128, 2, 96),   # four: one workgroup per 32 rows, an odd number of row blocks
    (2, 256, 8, 128),  # eight: two workgroups per 32 rows
])
def test_lime_scores_normalised_link_rows(B, d, h, m):
    """The link rows' normalisation inside the pack launch, in both of its forms."""
    _request(780 + d, B, 70, 45, d, h, m, 8, 40, [96, 1], "bf16", (20, 70))


@pytest.mark.parametrize("B,N,d,h,m", [(17, 2048, 256, 4, 128), (33, 1024, 128, 4, 128)])
def test_lime_scores_many_link_states_of_long_histories(B, N, d, h, m):
    """13 and 11 chunks a history and more link states than run at once with eight a workgroup: sixteen a workgroup in the
    merge's form for many chunks."""
    _request(800 + d, B, N, 9, d, h, m, 8, 40, [96, 1], "bf16", (N // 3, N), lens=[0, 1, N, 161, 160])


@pytest.mark.parametrize("B,m,d,dhid,widths", [(33, 64, 128, 40, [512, 128, 64, 1]), (2, 32, 256, 30, [96, 1])])
def test_lime_scores_without_the_shared_first_launch(B, m, d, dhid, widths):
    """Rows or a width of the hidden layer that the first launch does not take, with the interaction network on the matrix cores
    all the same: its weight images are then packed by its own launch."""
    _request(810 + d, B, 90, 70, d, 4, m, 8, dhid, widths, "bf16", (30, 90))


@pytest.mark.parametrize("d,h,m,B,N", [(256, 4, 64, 40, 1024), (256, 4, 32, 36, 1000), (256, 2, 128, 36, 1000), (128, 2, 64, 70, 600),
                                       (128, 4, 96, 70, 600), (64, 2, 32, 70, 600)])
def test_lime_scores_cooperative_history_walk_on_edge_lengths(d, h, m, B, N):
    """Enough users x tiles (four per compute unit) for the scoring call's cooperative history kernels (at d = 256 the variant
    with all W_K slices in LDS and one tile buffer), with the lengths that stress them: empty users, one item, one short of /
    exactly / one past a tile, a chunk boundary, the full history; padding rows hold NaN."""
    _request(790 + d + m, B, N, 5, d, h, m, 8, 40, [16, 1], "bf16", (1, N), lens=[0, 1, 31, 32, 33, 255, 256, 257, N - 1, N, 0, N])


@pytest.mark.parametrize("d,h,m,B,N", [(256, 4, 64, 3, 777), (128, 4, 64, 70, 600)])
def test_lime_scores_runs_one_history_kernel(d, h, m, B, N):
    """Without scale and shift for the candidates' normalisation the scoring call takes the separate passes, but the same
    history kernel, so that the link states differ only in rows with a normalised element that the other pass rounds the other
    way (its sums run in another order): a few in ten thousand.  Another kernel rounds its softmax weights relative to other
    maxima, which changed 4 and 9 % of all elements."""
    g = torch.Generator(device="cuda").manual_seed(d)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    W = lambda: [(rn(d, d).float() * d ** -0.5).to(torch.bfloat16) for _ in range(3)]  # noqa: E731
    hist, cand = W(), W()
    norms = [((rn(d).float() * 0.2 + 1).to(torch.bfloat16), rn(d)) for _ in range(5)]
    L, E, T, EC, ctx, mlp = rn(m, d), rn(B, N, d), rn(B, 16, d), rn(B, 8), (rn(d + 8, 40), rn(40), rn(40, d), rn(d)), ([rn(d, 1)], [rn(1)])
    s = (d // h) ** -0.5
    LP = []
    for cand_q in (norms[2], (None, None)):
        model = binding.scoring_model(L, ctx, hist, cand, *norms[:2], cand_q, *norms[3:], mlp, h, s, s)
        LP.append(binding.lime_scores(model, E, None, EC, T, want_intermediates=True)[2])
    share = float((LP[0] != LP[1]).float().mean())
    print(f"d={d}: {share:.2e} of the link states' elements differ", flush=True)
    assert share <= 0.01


@pytest.mark.parametrize("d,h", [(64, 2), (32, 1), (128, 4), (256, 8)])
def test_link_rows_are_normalised_as_by_the_separate_pass(d, h):
    """On rows whose sums are exact in fp32 (entries 0 .. 3: mean, centred squares and their sum have at most 24 bits) the
    order of the sums does not matter: the pack launch's normalisation gives the separate pass's bits, and with it the whole
    scoring call those of the call that takes the separate passes.  (Without scale and shift for the candidates'
    normalisation, that is; the link states do not depend on it.)"""
    B, m, N, dc = 512 * 64 // d, 128, 8, 8
    g = torch.Generator(device="cuda").manual_seed(d)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    ints = lambda hi, *s: torch.randint(0, hi + 1, s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    W = lambda: [(rn(d, d).float() * d ** -0.5).to(torch.bfloat16) for _ in range(3)]  # noqa: E731
    hist, cand = W(), W()
    norms = [((rn(d).float() * 0.2 + 1).to(torch.bfloat16), rn(d)) for _ in range(5)]
    zero = torch.zeros(d, dtype=torch.bfloat16, device="cuda")
    eye = torch.eye(d, device="cuda", dtype=torch.bfloat16)
    spread = torch.nn.functional.one_hot(torch.arange(d, device="cuda") % dc, dc).t().to(torch.bfloat16)  # [dc, d]: L^C = L + E^C spread
    L, E, T, EC = ints(2, m, d), rn(B, N, d), rn(B, 1, d), ints(1, B, dc)
    ctx = (torch.cat([eye, spread]).contiguous(), zero, eye, zero)
    s = 3.0 * (d // h) ** -0.5
    LP = []
    for cand_q in (norms[2], (None, None)):
        model = binding.scoring_model(L, ctx, hist, cand, *norms[:2], cand_q, *norms[3:], ([rn(d, 1)], [rn(1)]), h, s, s)
        LP.append(binding.lime_scores(model, E, None, EC, T, want_intermediates=True)[2])
    assert torch.equal(LP[0], LP[1]), f"{int((LP[0] != LP[1]).sum())} of {LP[0].numel()} elements differ"
