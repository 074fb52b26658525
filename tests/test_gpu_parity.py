"""GPU parity: the HIP library, called through the C ABI, against the CPU oracle on the
same seeded inputs, element by element.  Bars: max-abs 1e-4 (fp32) / 2e-2 (bf16) as stated,
unscaled, and the same number relative to the largest reference entry; masks, zero padding
and determinism bit-exact."""

import numpy as np
import pytest
import torch

from oracle import lime_oracle as orc
from paper_2510_18239_amd import binding, synth
from parity_util import DeviceWorkload, assert_close, dev, host, run_all_paths

pytestmark = pytest.mark.gpu


def _sharp(d, h, dtype, value_gain=synth.SHARP_VALUE_GAIN, **kw):
    """Workload whose softmax logits have a standard deviation of about 2 (far from uniform); W_V sized so that
    the outputs stay below one, where the stated absolute bar applies."""
    g = synth.sharp_gain(d, h, (d // h) ** -0.5, 2.0)
    return synth.make_workload(d=d, h=h, dtype=dtype, gain=g, value_gain=value_gain, **kw)


# XORA divides by the history length: over one or two rows O[T] is SiLU(logit) x value, several times a value
# (a softmax weight never exceeds one), so the tests with such users take smaller values still.
TINY_HISTORY_VALUE_GAIN = 0.03


def _xor_scale(w):
    # keeps the XORA logits O(1) on sharp inputs; on benchmark inputs the paper's scale of 1 is used
    return w.softmax_scale if w.meta["gain"] > 1 else 1.0


def _check_all(w, **kw):
    print(f"case B={w.B} N={w.N} C={w.C} d={w.d} h={w.h} m={w.m} {w.dtype} gain={w.meta['gain']:.2f}", flush=True)
    for name, (got, ref) in run_all_paths(w, xor_scale=_xor_scale(w), **kw).items():
        assert_close(got, ref, w.dtype, name)


# ----------------------------------------------------------------------------- configuration 1 (fp32)

@pytest.mark.parametrize("gain", ["bench", "sharp"])
def test_config1_fp32(gain):
    c = dict(synth.CONFIGS[1])
    w = synth.make_workload(1, **c) if gain == "bench" else _sharp(workload=1, **c)
    _check_all(w)


# ----------------------------------------------------------------------------- several tiles and a ragged tail

SHAPES = [
    # B, N, C, d, h, m, dtype
    (3, 333, 517, 128, 4, 64, "bf16"),
    (2, 700, 300, 256, 4, 64, "bf16"),
    (2, 257, 130, 256, 4, 128, "bf16"),
    (2, 190, 77, 64, 2, 32, "bf16"),
    (1, 100, 65, 256, 8, 96, "bf16"),
    (2, 70, 45, 256, 8, 128, "bf16"),  # eight heads, most links: three quarters of W_Q^T go through LDS
    (2, 150, 90, 96, 3, 20, "bf16"),   # m not a multiple of 32: general kernels
    (2, 75, 33, 40, 5, 7, "bf16"),     # d/h = 8: general kernels
    (2, 333, 200, 128, 4, 64, "fp32"),
    (1, 65, 40, 24, 1, 5, "fp32"),
    (1, 50, 20, 512, 2, 16, "fp32"),   # d/h = 256, the largest head the library takes
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}N{}C{}d{}h{}m{}{}".format(*s))
@pytest.mark.parametrize("gain", ["bench", "sharp"])
def test_ragged_shapes(shape, gain):
    B, N, C, d, h, m, dtype = shape
    kw = dict(workload=10 + SHAPES.index(shape), B=B, N=N, C=C, d=d, h=h, m=m, dtype=dtype,
              len_range=(max(1, N // 3), N), pad_value=np.nan)
    w = synth.make_workload(**kw) if gain == "bench" else _sharp(**kw)
    _check_all(w)


# ----------------------------------------------------------------------------- edge cases

@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("fp32", 32, 2, 8), ("bf16", 256, 4, 128)])
def test_empty_and_tiny_histories(dtype, d, h, m):
    w = _sharp(workload=30, B=5, N=70, C=9, d=d, h=h, m=m, dtype=dtype, value_gain=TINY_HISTORY_VALUE_GAIN)
    w.lens = np.array([0, 1, 2, 70, 33], dtype=np.int32)
    for b in range(5):
        w.E[b, w.lens[b]:] = np.nan
    res = run_all_paths(w, xor_scale=w.softmax_scale)
    for name, (got, ref) in res.items():
        assert_close(got, ref, dtype, name)
    assert not res["lime_link_history"][0][0].any()  # empty history -> exact zeros
    assert not res["lime_xor_history.OT"][0][0].any()
    assert not res["mha_target_attention"][0][0].any()
    OS = res["lime_xor_history.OS"][0]
    for b in range(5):
        assert not OS[b, w.lens[b]:].any(), "O[S] rows beyond the history must be exact zeros"


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("fp32", 64, 1, 16), ("bf16", 256, 4, 64)])
def test_single_row_problems(dtype, d, h, m):
    w = _sharp(workload=31, B=1, N=1, C=1, d=d, h=h, m=m, dtype=dtype, value_gain=TINY_HISTORY_VALUE_GAIN)
    _check_all(w)


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("bf16", 256, 4, 64), ("fp32", 64, 2, 16),
                                         ("bf16", 96, 3, 20)])
def test_padding_content_is_never_read(dtype, d, h, m):
    """Results must be bit-identical whatever the rows beyond lens[b] hold."""
    base = dict(workload=32, B=3, N=200, C=50, d=d, h=h, m=m, dtype=dtype, len_range=(20, 200))
    outs = []
    for pad in (0.0, np.nan, np.inf, -3.0e38):
        w = _sharp(pad_value=pad, **base)
        g = DeviceWorkload(w)
        s = w.softmax_scale
        LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)
        OT, OS = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s, want_os=True)
        A = binding.mha_target_attention(g.T, g.E, g.lens, g.Wq, g.Wk, g.Wv, h, s)
        outs.append([t.clone() for t in (LP, OT, OS, A)])
    for o in outs[1:]:
        for x, y in zip(o, outs[0]):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("bf16", 256, 4, 64), ("fp32", 64, 2, 16)])
def test_truncation_equals_masking(dtype, d, h, m):
    """A user with lens = n must get the bits of a call on the tensor cut to n rows."""
    w = _sharp(workload=33, B=1, N=300, C=10, d=d, h=h, m=m, dtype=dtype)
    n = 173
    g = DeviceWorkload(w)
    s = w.softmax_scale
    lens = torch.tensor([n], dtype=torch.int32, device="cuda")
    Ecut = g.E[:, :n].contiguous()
    assert torch.equal(binding.lime_link_history(g.E, lens, g.L, g.Wq, g.Wk, g.Wv, h, s),
                       binding.lime_link_history(Ecut, None, g.L, g.Wq, g.Wk, g.Wv, h, s))
    a = binding.lime_xor_history(g.E, lens, g.L, g.Wq, g.Wk, g.Wv, h, s, want_os=True)
    b = binding.lime_xor_history(Ecut, None, g.L, g.Wq, g.Wk, g.Wv, h, s, want_os=True)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1][:, :n], b[1]) and not a[1][:, n:].any()
    assert torch.equal(binding.mha_target_attention(g.T, g.E, lens, g.Wq, g.Wk, g.Wv, h, s),
                       binding.mha_target_attention(g.T, Ecut, None, g.Wq, g.Wk, g.Wv, h, s))


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("fp32", 64, 2, 16)])
def test_per_user_links(dtype, d, h, m):
    w = _sharp(workload=34, B=3, N=120, C=8, d=d, h=h, m=m, dtype=dtype, len_range=(40, 120), pad_value=np.nan)
    g = DeviceWorkload(w)
    LCu = synth.per_user_links(34, 3, m, d, dtype, gain=w.meta["gain"])
    s = w.softmax_scale
    LP = binding.lime_link_history(g.E, g.lens, dev(LCu, dtype), g.Wq, g.Wk, g.Wv, h, s)
    assert_close(host(LP), orc.lime_link_history(w.E, w.lens, LCu, w.Wq, w.Wk, w.Wv, h, s), dtype, "per-user LP")
    OT, OS = binding.lime_xor_history(g.E, g.lens, dev(LCu, dtype), g.Wq, g.Wk, g.Wv, h, s, want_os=True)
    rt, rs = orc.lime_xor_history(w.E, w.lens, LCu, w.Wq, w.Wk, w.Wv, h, s)
    assert_close(host(OT), rt, dtype, "per-user O[T]")
    assert_close(host(OS), rs, dtype, "per-user O[S]")


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 128, 4, 64), ("bf16", 256, 4, 64), ("fp32", 64, 2, 16)])
def test_identity_projections_in_candidate_stage(dtype, d, h, m):
    """NULL weights give the literal phi(T L^t) L^P of Eq. 4; any subset may be NULL."""
    w = _sharp(workload=35, B=2, N=8, C=150, d=d, h=h, m=m, dtype=dtype)
    g = DeviceWorkload(w)
    LPv = synth.per_user_links(35, 2, m, d, dtype, gain=w.meta["gain"] * synth.SHARP_VALUE_GAIN)  # values: outputs below one
    LP = dev(LPv, dtype)
    s = w.softmax_scale / w.meta["gain"]  # raw embeddings are larger than projected ones
    for mask in [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0)]:
        gw = [x if k else None for x, k in zip((g.Wq, g.Wk, g.Wv), mask)]
        hw = [x if k else None for x, k in zip((w.Wq, w.Wk, w.Wv), mask)]
        O = binding.lime_score_candidates(g.T, g.L, LP, *gw, h, s)
        assert_close(host(O), orc.lime_score_candidates(w.T, w.L, LPv, *hw, h, s), dtype, f"identity mask {mask}")


@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 256, 4, 64), ("bf16", 128, 4, 64), ("fp32", 64, 1, 16)])
def test_determinism_and_row_independence(dtype, d, h, m):
    w = _sharp(workload=36, B=2, N=500, C=700, d=d, h=h, m=m, dtype=dtype, len_range=(100, 500), pad_value=0.0)
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LP1 = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s).clone()
    LP2 = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)
    assert torch.equal(LP1, LP2), "same input twice must give the same bits"
    O1 = binding.lime_score_candidates(g.T, g.L, LP1, g.Wq, g.Wk, g.Wv, h, s).clone()
    perm = torch.randperm(700, generator=torch.Generator().manual_seed(0)).cuda()
    O2 = binding.lime_score_candidates(g.T[:, perm].contiguous(), g.L, LP1, g.Wq, g.Wk, g.Wv, h, s)
    assert torch.equal(O2, O1[:, perm]), "a candidate's result must not depend on its position in the batch"
    X1 = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)[0].clone()
    X2 = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)[0]
    assert torch.equal(X1, X2)


def test_reduces_to_target_attention_when_links_are_the_history():
    """Eq. 4 with L := E_b, L^P := E_b equals Eq. 1 with K = V = E_b (m = N = 64)."""
    w = _sharp(workload=37, B=1, N=64, C=200, d=128, h=4, m=64, dtype="bf16")
    g = DeviceWorkload(w)
    s = w.softmax_scale
    O = binding.lime_score_candidates(g.T, g.E[0].contiguous(), g.E, g.Wq, g.Wk, g.Wv, 4, s)
    A = binding.mha_target_attention(g.T, g.E, None, g.Wq, g.Wk, g.Wv, 4, s)
    ref = orc.mha_target_attention(w.T, w.E, None, w.Wq, w.Wk, w.Wv, 4, s)
    assert_close(host(O), ref, "bf16", "decoupled attention with links = history")
    assert_close(host(A), ref, "bf16", "target attention")


def test_status_codes_on_device_arguments():
    w = synth.make_workload(38, B=1, N=16, C=16, d=64, h=2, m=32, dtype="bf16")
    g = DeviceWorkload(w)
    tiny = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.LimeError) as e:
        binding.lime_score_candidates(g.T, g.L, g.E[:, :32].contiguous(), g.Wq, g.Wk, g.Wv, 2, 1.0, workspace=tiny)
    assert e.value.status == 3
    with pytest.raises(binding.LimeError) as e:
        binding.lime_link_history(g.E, None, g.L, g.Wq, g.Wk, g.Wv, 3, 1.0)
    assert e.value.status == 1


def test_hip_graph_replay_matches_eager():
    """The whole request captured in a HIP graph: every replay, with eager work in between, must give
    the bits of the eager run (the library enqueues kernels only: no memsets, no allocations)."""
    w = _sharp(workload=39, B=2, N=300, C=400, d=256, h=4, m=64, dtype="bf16", len_range=(50, 300), pad_value=0.0)
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LP = torch.empty((2, 64, 256), dtype=torch.bfloat16, device="cuda")
    O = torch.empty_like(g.T)
    XT = torch.empty_like(LP)
    XL = torch.empty_like(LP)
    LP1, O1, LP3, O3 = torch.empty_like(LP), torch.empty_like(O), torch.empty_like(LP), torch.empty_like(O)
    Wu, Wo = (dev(x, "bf16") for x in _layer_weights(5, 2, 256))
    prepared = binding.lime_prepare(g.L, g.L, g.Wq, g.Wk, g.Wv, g.Wq, g.Wk, 4, s, s)
    ws = torch.empty(max(binding.workspace_bytes(binding.OP_XOR_HISTORY, B=2, N=300, d=256, h=4, m=64),
                         binding.workspace_bytes(binding.OP_SCORE_CANDIDATES, B=2, C=400, d=256, h=4, m=64),
                         binding.workspace_bytes(binding.OP_XOR_LAYERS, B=2, N=300, d=256, h=4, m=64),
                         binding.workspace_bytes(binding.OP_REQUEST, B=2, N=300, C=400, d=256, h=4, m=64),
                         binding.workspace_bytes(binding.OP_REQUEST_PREPARED, B=2, N=300, C=400, d=256, h=4, m=64)),
                     dtype=torch.uint8, device="cuda")

    def request():
        binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, s, LP=LP, workspace=ws)
        binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, 4, s, O=O, workspace=ws)
        binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, s, LP=XT, workspace=ws)
        binding.lime_xor_layers(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, Wu, Wo, 4, s, LP=XL, workspace=ws)
        binding.lime_request(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, g.T, g.L, g.Wq, g.Wk, g.Wv, 4, s, s, LP=LP1, O=O1,
                             workspace=ws)
        binding.lime_request_prepared(g.E, g.lens, g.T, g.Wv, prepared, 4, 64, s, s, LP=LP3, O=O3, workspace=ws)

    outs = (LP, O, XT, XL, LP1, O1, LP3, O3)
    request()
    torch.cuda.synchronize()
    want = [t.clone() for t in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        request()
    for _ in range(4):
        for t in outs:
            t.fill_(7.0)
        ws.random_(0, 255)  # the workspace carries nothing from one call to the next
        (torch.randn(1000, device="cuda") * 2).sum().item()  # unrelated eager work and a synchronisation
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip(outs, want):
            assert torch.equal(got, ref)


def test_concurrent_requests_on_separate_streams():
    """Requests of different users in flight at once, each on its own stream with its own link states and
    workspace (how the benchmark's serving loop runs them): the library keeps no state between calls, so
    every request must give the bits it gives when it runs alone."""
    n = 4
    ws_list, inputs, want = [], [], []
    for k in range(n):
        w = _sharp(workload=60 + k, B=1, N=700 + 64 * k, C=3000 + 100 * k, d=256, h=4, m=64, dtype="bf16")
        g = DeviceWorkload(w)
        LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale)
        O = binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale)
        LP1, O1 = binding.lime_request(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, g.T, g.L, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale,
                                       w.softmax_scale)
        torch.cuda.synchronize()
        assert torch.equal(LP1, LP)
        want.append((LP.clone(), O.clone(), O1.clone()))
        inputs.append((w, g))
        ws_list.append(torch.empty(binding.workspace_bytes(binding.OP_REQUEST, B=1, N=w.N, C=w.C, d=256, h=4, m=64),
                                   dtype=torch.uint8, device="cuda"))
    streams = [torch.cuda.Stream() for _ in range(n)]
    got = [(torch.empty_like(lp), torch.empty_like(o)) for lp, o, _ in want]
    reps = 3
    torch.cuda.synchronize()
    for rep in range(reps):
        for k in range(n):
            w, g = inputs[k]
            LP, O = got[k]
            if (k + rep) % 2:  # the request as one call (how bench.py issues it): the same link states, and its own
                # output bits (the value projection sums in another order)
                binding.lime_request(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, g.T, g.L, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale,
                                     w.softmax_scale, LP=LP, O=O, workspace=ws_list[k], stream=streams[k])
                continue
            binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale, LP=LP,
                                      workspace=ws_list[k], stream=streams[k])
            binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, 4, w.softmax_scale, O=O,
                                          workspace=ws_list[k], stream=streams[k])
    torch.cuda.synchronize()
    for k in range(n):
        assert torch.equal(got[k][0], want[k][0]), f"link states of request {k}"
        assert torch.equal(got[k][1], want[k][2 if (k + reps - 1) % 2 else 1]), f"candidate outputs of request {k}"


@pytest.mark.parametrize("scale", [-0.2, 0.0])
@pytest.mark.parametrize("dtype,d,h,m", [("bf16", 256, 4, 64), ("bf16", 128, 4, 64), ("fp32", 64, 2, 16)])
def test_negative_and_zero_logit_scale(scale, dtype, d, h, m):
    """The scale is an arbitrary float: a negative one prefers the smallest raw logits, zero gives
    uniform attention (and SiLU(0) = 0)."""
    w = _sharp(workload=40, B=2, N=150, C=90, d=d, h=h, m=m, dtype=dtype, len_range=(40, 150), pad_value=np.nan)
    g = DeviceWorkload(w)
    LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, scale)
    assert_close(host(LP), orc.lime_link_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, scale), dtype, "LP")
    O = binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, h, scale)
    assert_close(host(O), orc.lime_score_candidates(w.T, w.L, host(LP), w.Wq, w.Wk, w.Wv, h, scale), dtype, "O")
    OT, OS = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, scale, want_os=True)
    rt, rs = orc.lime_xor_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, scale)
    assert_close(host(OT), rt, dtype, "O[T]")
    assert_close(host(OS), rs, dtype, "O[S]")
    A = binding.mha_target_attention(g.T, g.E, g.lens, g.Wq, g.Wk, g.Wv, h, scale)
    assert_close(host(A), orc.mha_target_attention(w.T, w.E, w.lens, w.Wq, w.Wk, w.Wv, h, scale), dtype, "MHA")


def test_unaligned_pointers_take_the_general_kernels():
    """bf16 tensors that are not 16-byte aligned are served (by the general kernels) with the same results."""
    w = _sharp(workload=41, B=2, N=100, C=70, d=128, h=4, m=64, dtype="bf16", len_range=(30, 100), pad_value=0.0)
    g = DeviceWorkload(w)
    s = w.softmax_scale

    def shifted(t):
        buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
        v = buf[1:1 + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 != 0
        return v

    E2, T2 = shifted(g.E), shifted(g.T)
    LP_a = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, s)
    LP_b = binding.lime_link_history(E2, g.lens, g.L, g.Wq, g.Wk, g.Wv, 4, s)
    ref = orc.lime_link_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, 4, s)
    assert_close(host(LP_a), ref, "bf16", "aligned LP")
    assert_close(host(LP_b), ref, "bf16", "unaligned LP")
    O_b = binding.lime_score_candidates(T2, g.L, LP_a, g.Wq, g.Wk, g.Wv, 4, s)
    assert_close(host(O_b), orc.lime_score_candidates(w.T, w.L, host(LP_a), w.Wq, w.Wk, w.Wv, 4, s), "bf16", "unaligned O")
    A_b = binding.mha_target_attention(T2, E2, g.lens, g.Wq, g.Wk, g.Wv, 4, s)
    assert_close(host(A_b), orc.mha_target_attention(w.T, w.E, w.lens, w.Wq, w.Wk, w.Wv, 4, s), "bf16", "unaligned MHA")


@pytest.mark.parametrize("dtype,d,h,m,C", [("bf16", 256, 4, 64, 1000), ("bf16", 128, 4, 64, 333), ("bf16", 256, 4, 128, 200),
                                           ("fp32", 64, 2, 16, 77), ("bf16", 96, 3, 20, 50)])
def test_qk_cache_path(dtype, d, h, m, C):
    """Section 3.3: the cached attention weights and the online weighted sum, against the oracle, and
    chained against the direct candidate call."""
    w = _sharp(workload=42, B=2, N=8, C=C, d=d, h=h, m=m, dtype=dtype)
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LPv = synth.per_user_links(42, 2, m, d, dtype, gain=w.meta["gain"] * synth.SHARP_VALUE_GAIN)
    LP = dev(LPv, dtype)
    W = binding.lime_build_qk_cache(g.T, g.L, g.Wq, g.Wk, h, s)
    assert W.shape == (2, C, h, m)
    W_ref = orc.qk_cache(w.T, w.L, w.Wq, w.Wk, h, s)
    assert_close(host(W), W_ref, dtype, "cached weights")
    sums = host(W).sum(axis=-1)
    assert np.abs(sums - 1.0).max() <= (2e-2 if dtype == "bf16" else 1e-4)
    # the online half is checked on the weights the GPU stored (they travel in the storage type)
    O = binding.lime_score_candidates_cached(W, LP, g.Wv)
    assert_close(host(O), orc.lime_score_candidates_cached(host(W), LPv, w.Wv, h), dtype, "cached O")
    # and the chain against Eq. 4 evaluated directly
    assert_close(host(O), orc.lime_score_candidates(w.T, w.L, LPv, w.Wq, w.Wk, w.Wv, h, s), dtype, "cached chain")
    direct = binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, h, s)
    assert_close(host(O), host(direct).astype(np.float64), dtype, "cached vs direct on the GPU")


@pytest.mark.parametrize("dtype,d,h,m,n_items,C", [("bf16", 256, 4, 64, 5000, 1000), ("bf16", 128, 4, 64, 700, 333),
                                                   ("bf16", 256, 4, 128, 300, 95), ("fp32", 64, 2, 16, 90, 77),
                                                   ("bf16", 96, 3, 20, 60, 50)])
def test_gathered_qk_cache(dtype, d, h, m, n_items, C):
    """Section 3.3 with one cache table for the item corpus and candidates named by id (repeats, a ragged
    last tile, ids outside the table): against the oracle on the table the GPU stored, and against Eq. 4
    evaluated on the gathered embeddings."""
    B = 3
    w = _sharp(workload=44, B=1, N=8, C=n_items, d=d, h=h, m=m, dtype=dtype)  # T[0] is the corpus
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LPv = synth.per_user_links(44, B, m, d, dtype, gain=w.meta["gain"] * synth.SHARP_VALUE_GAIN)
    LP = dev(LPv, dtype)
    table = binding.lime_build_qk_cache(g.T, g.L, g.Wq, g.Wk, h, s)[0]
    rng = np.random.default_rng(4400 + n_items)
    ids = rng.integers(0, n_items, size=(B, C)).astype(np.int32)
    ids[0, :4] = ids[0, 4]           # repeats
    ids[1, 1], ids[2, C - 1], ids[2, 0] = -1, n_items, np.iinfo(np.int32).max  # outside the table
    O = binding.lime_score_candidates_gathered(table, torch.from_numpy(ids).cuda(), LP, g.Wv)
    assert O.shape == (B, C, d)
    ref = orc.lime_score_candidates_gathered(host(table), ids, LPv, w.Wv, h)
    assert_close(host(O), ref, dtype, "gathered O")
    got = host(O)
    assert not got[1, 1].any() and not got[2, C - 1].any() and not got[2, 0].any()
    assert np.array_equal(got[0, 0], got[0, 4])
    valid = (ids >= 0) & (ids < n_items)
    chain = orc.lime_score_candidates(w.T[0][np.where(valid, ids, 0)], w.L, LPv, w.Wq, w.Wk, w.Wv, h, s)
    assert_close(got[valid], chain[valid], dtype, "gathered chain")


@pytest.mark.parametrize("B,N,C,d,h,m,ragged", [(1, 2048, 4096, 256, 4, 64, False), (3, 777, 500, 256, 4, 64, True),
                                                (5, 300, 333, 128, 4, 64, True), (2, 4100, 100, 256, 4, 128, True),
                                                (40, 1024, 64, 128, 4, 32, True)])
def test_prepared_operands_give_the_same_bits(B, N, C, d, h, m, ragged):
    """The stages on operands packed once by lime_prepare (Section 3.3: what does not depend on the user is
    computed ahead of time) run the same kernels on the same images as the per-call entry points: equal bits,
    for softmax and XORA link states and for the candidate stage, with a negative scale for one of them.
    With no more links than head columns the prepared candidate stage folds W_Q and the projected link keys into
    one operand, which rounds differently: there the two agree within the bf16 tolerance."""
    w = _sharp(workload=70 + B, B=B, N=N, C=C, d=d, h=h, m=m, dtype="bf16", len_range=(N // 3, N) if ragged else None,
               pad_value=float("nan") if ragged else 0.0)
    g = DeviceWorkload(w)
    s_h, s_c = w.softmax_scale, -0.5 * w.softmax_scale
    prepared = binding.lime_prepare(g.L, g.L, g.Wq, g.Wk, g.Wv, g.Wq, g.Wk, h, s_h, s_c)
    LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s_h)
    LP_p = binding.lime_link_history_prepared(g.E, g.lens, prepared, h, m, s_h)
    assert torch.equal(LP, LP_p)
    XT, _ = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s_h)
    XT_p = binding.lime_link_history_prepared(g.E, g.lens, prepared, h, m, s_h, xor_attention=True)
    assert torch.equal(XT, XT_p)
    O = binding.lime_score_candidates(g.T, g.L, LP, g.Wq, g.Wk, g.Wv, h, s_c)
    O_p = binding.lime_score_candidates_prepared(g.T, LP, g.Wv, prepared, h, s_c)
    if m <= d // h:
        assert_close(host(O_p), host(O).astype(np.float64), "bf16", "prepared O against the per-call O")
    else:
        assert torch.equal(O, O_p)
    # and against the oracle, so that the equality is not one of two wrong results
    assert_close(host(O_p), orc.lime_score_candidates(w.T, w.L, host(LP), w.Wq, w.Wk, w.Wv, h, s_c), "bf16", "prepared O")


@pytest.mark.parametrize("B,N,C,d,h,m,xor", [(1, 2048, 4096, 256, 4, 64, False), (3, 777, 500, 256, 4, 128, False),
                                             (5, 300, 333, 128, 4, 64, True), (40, 1024, 64, 128, 4, 32, False),
                                             (2, 100, 70, 64, 2, 32, False), (2, 90, 33, 32, 1, 32, False)])
def test_request_on_prepared_operands_in_one_call(B, N, C, d, h, m, xor):
    """lime_request_prepared (three kernels: the merge step also writes the candidate stage's value image) against
    the two prepared calls - the link states bit for bit, the outputs within the bf16 bar - and against the oracle;
    ragged lengths with an empty user, NaN padding, a negative candidate scale, and once without Wv (identity)."""
    w = _sharp(workload=170 + B + m, B=B, N=N, C=C, d=d, h=h, m=m, dtype="bf16", len_range=(1, N), pad_value=np.nan)
    if B > 1:
        w.lens[B - 1] = 0
        w.E[B - 1] = np.nan
    g = DeviceWorkload(w)
    s_h, s_c = (_xor_scale(w) if xor else w.softmax_scale), -0.7 * w.softmax_scale
    Wv_d, Wv_h = (None, None) if m == 128 else (g.Wv, w.Wv)
    prepared = binding.lime_prepare(g.L, g.L, g.Wq, g.Wk, g.Wv, g.Wq, g.Wk, h, s_h, s_c)
    LP2 = binding.lime_link_history_prepared(g.E, g.lens, prepared, h, m, s_h, xor_attention=xor)
    O2 = binding.lime_score_candidates_prepared(g.T, LP2, Wv_d, prepared, h, s_c)
    LP1, O1 = binding.lime_request_prepared(g.E, g.lens, g.T, Wv_d, prepared, h, m, s_h, s_c, xor_attention=xor)
    assert torch.equal(LP1, LP2)
    assert_close(host(O1), host(O2), "bf16", "one call against two calls")
    assert_close(host(O1), orc.lime_score_candidates(w.T, w.L, host(LP1), w.Wq, w.Wk, Wv_h, h, s_c), "bf16", "O against the oracle")
    if B > 1:
        assert not host(LP1)[B - 1].any()


@pytest.mark.parametrize("B,N,C,d,h,m,dtype,xor,per_user", [
    (1, 2048, 4096, 256, 4, 64, "bf16", False, False), (3, 777, 500, 256, 4, 128, "bf16", False, True),
    (5, 300, 333, 128, 4, 64, "bf16", True, False), (40, 1024, 64, 128, 4, 32, "bf16", False, False),
    (2, 90, 33, 32, 1, 32, "bf16", False, True), (2, 333, 200, 128, 4, 64, "fp32", False, False),
    (2, 100, 70, 48, 2, 5, "bf16", True, True), (1, 65, 40, 24, 1, 5, "fp32", True, False)])
def test_request_in_one_call(B, N, C, d, h, m, dtype, xor, per_user):
    """lime_request (per-call packing; on the matrix-core shapes four kernels, elsewhere the two stages in turn) against
    lime_link_history / lime_xor_history followed by lime_score_candidates - the link states bit for bit, the outputs
    within the bar - and against the oracle; ragged lengths with an empty user, NaN padding, shared and per-user
    links, different weights and scales for the two stages, once with the candidate side's weights absent."""
    w = _sharp(workload=190 + B + m, B=B, N=N, C=C, d=d, h=h, m=m, dtype=dtype, len_range=(1, N), pad_value=np.nan)
    if B > 1:
        w.lens[B - 1] = 0
        w.E[B - 1] = np.nan
    g = DeviceWorkload(w)
    s_h, s_c = (_xor_scale(w) if xor else w.softmax_scale), -0.7 * w.softmax_scale
    if per_user:
        rng = np.random.default_rng(7)
        LC_h = np.stack([w.L[rng.permutation(m)] for _ in range(B)])
        LC_d = dev(LC_h, w.dtype)
    else:
        LC_h, LC_d = w.L, g.L
    # the candidate stage gets the history stage's weights in another role, or none at all
    cand_d, cand_h = ((None, None, None), (None, None, None)) if m == 128 else ((g.Wk, g.Wv, g.Wq), (w.Wk, w.Wv, w.Wq))
    if xor:
        LP2 = binding.lime_xor_history(g.E, g.lens, LC_d, g.Wq, g.Wk, g.Wv, h, s_h)[0]
    else:
        LP2 = binding.lime_link_history(g.E, g.lens, LC_d, g.Wq, g.Wk, g.Wv, h, s_h)
    O2 = binding.lime_score_candidates(g.T, g.L, LP2, *cand_d, h, s_c)
    LP1, O1 = binding.lime_request(g.E, g.lens, LC_d, g.Wq, g.Wk, g.Wv, g.T, g.L, *cand_d, h, s_h, s_c, xor_attention=xor)
    assert torch.equal(LP1, LP2)
    assert_close(host(O1), host(O2), dtype, "one call against two calls")
    if xor:
        ref_LP = orc.lime_xor_history(w.E, w.lens, LC_h, w.Wq, w.Wk, w.Wv, h, s_h)[0]
    else:
        ref_LP = orc.lime_link_history(w.E, w.lens, LC_h, w.Wq, w.Wk, w.Wv, h, s_h)
    assert_close(host(LP1), ref_LP, dtype, "LP against the oracle")
    assert_close(host(O1), orc.lime_score_candidates(w.T, w.L, host(LP1), *cand_h, h, s_c), dtype, "O against the oracle")
    if B > 1:
        assert not host(LP1)[B - 1].any()


FOLDED = [(256, 4, 64), (256, 4, 32), (128, 2, 64), (128, 2, 32), (64, 1, 64), (64, 1, 32), (256, 8, 32), (128, 4, 32),
          (64, 2, 32), (32, 1, 32)]


@pytest.mark.parametrize("d,h,m,identity", [s + ("none",) for s in FOLDED] +
                         [s + (i,) for s in [(256, 4, 64), (128, 4, 32), (64, 1, 32)] for i in ("Wq", "Wk")])
def test_prepared_candidate_stage_with_folded_scores(d, h, m, identity):
    """Every shape for which lime_prepare folds the candidate-side query weights and link keys into one operand
    (m <= d/h), and three of them with either weight absent (identity): the prepared candidate stage against the
    oracle, on several users with a candidate count that does not fill the last tile."""
    B, C = 3, 205
    w = _sharp(workload=300 + d + m, B=B, N=64, C=C, d=d, h=h, m=m, dtype="bf16")
    g = DeviceWorkload(w)
    s_c = -w.softmax_scale if d == 128 else w.softmax_scale
    Wq_d, Wq_h = (None, None) if identity == "Wq" else (g.Wq, w.Wq)
    Wk_d, Wk_h = (None, None) if identity == "Wk" else (g.Wk, w.Wk)
    prepared = binding.lime_prepare(g.L, g.L, g.Wq, g.Wk, g.Wv, Wq_d, Wk_d, h, w.softmax_scale, s_c)
    LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, w.softmax_scale)
    O_p = binding.lime_score_candidates_prepared(g.T, LP, g.Wv, prepared, h, s_c)
    assert_close(host(O_p), orc.lime_score_candidates(w.T, w.L, host(LP), Wq_h, Wk_h, w.Wv, h, s_c), "bf16", "prepared O")


@pytest.mark.parametrize("d,h,m,B,N", [(256, 4, 64, 40, 1024), (256, 4, 128, 36, 1000), (128, 4, 64, 70, 600)])
def test_history_kernel_on_edge_lengths(d, h, m, B, N):
    """Enough users x tiles for workgroups of eight waves and several steps, with the lengths that stress them: empty users,
    one item, one short of / exactly / one past a tile, a step's and a chunk's boundary, the full history; padding rows hold
    NaN."""
    w = _sharp(workload=90 + m, B=B, N=N, C=8, d=d, h=h, m=m, dtype="bf16", len_range=(1, N), pad_value=np.nan,
               value_gain=TINY_HISTORY_VALUE_GAIN)
    special = [0, 1, 31, 32, 33, 255, 256, 257, N - 1, N, 0, N]
    w.lens[:len(special)] = special
    for b, n in enumerate(special):
        w.E[b, n:] = np.nan
        w.E[b, :n] = np.nan_to_num(w.E[b, :n], nan=0.0)  # rows that became valid after the length change
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LP = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)
    assert_close(host(LP), orc.lime_link_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, s), "bf16", "LP")
    assert not host(LP)[0].any() and not host(LP)[10].any()
    OT, _ = binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)
    OT_ref, _ = orc.lime_xor_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, s, want_os=False)
    assert_close(host(OT), OT_ref, "bf16", "O[T]")


# ----------------------------------------------------------------------------- stacked XOR layers (Eq. 8)

def _layer_weights(seed, n, d, gain=1.0):
    """eta_j = (Wu[j], Wo[j]) ~ N(0, 1/d) like every other weight, rounded to bf16; `gain` sharpens the gate."""
    r = np.random.default_rng(seed)
    Wu = (r.standard_normal((n, d, d)) * d ** -0.5 * gain).astype(np.float32)
    Wo = (r.standard_normal((n, d, d)) * d ** -0.5).astype(np.float32)
    rnd = lambda x: torch.from_numpy(x).to(torch.bfloat16).float().numpy()  # noqa: E731
    return rnd(Wu), rnd(Wo)


@pytest.mark.parametrize("dtype,B,N,d,h,m,n_layers,per_user", [
    ("fp32", 2, 150, 64, 2, 24, 3, False),   # fp32 storage: the 1e-4 bar
    ("fp32", 3, 70, 128, 4, 64, 2, True),
    ("bf16", 2, 90, 96, 3, 20, 3, False),    # bf16 outside the matrix-core set: general kernels
])
def test_xor_layers_on_general_kernels(dtype, B, N, d, h, m, n_layers, per_user):
    w = _sharp(workload=450 + d + m, B=B, N=N, C=8, d=d, h=h, m=m, dtype=dtype, len_range=(1, N), pad_value=np.nan)
    w.lens[B - 1] = 0
    w.E[B - 1] = np.nan
    Wu, Wo = _layer_weights(99 + d, n_layers, d, gain=1.0)
    if dtype == "fp32":  # fp32 storage takes the weights unrounded as well
        r = np.random.default_rng(99 + d)
        Wu = (r.standard_normal((n_layers, d, d)) * d ** -0.5).astype(np.float32)
        Wo = (r.standard_normal((n_layers, d, d)) * d ** -0.5 * 0.5).astype(np.float32)
    LC = np.stack([np.roll(w.L, b + 1, axis=0) for b in range(B)]) if per_user else w.L
    g = DeviceWorkload(w)
    xs = _xor_scale(w)
    LP = binding.lime_xor_layers(g.E, g.lens, dev(LC, dtype), g.Wq, g.Wk, g.Wv, dev(Wu, dtype), dev(Wo, dtype), h, xs)
    ref = orc.lime_xor_layers(w.E, w.lens, LC, w.Wq, w.Wk, w.Wv, Wu, Wo, h, xs)
    err = assert_close(host(LP), ref, dtype, "LP of stacked XOR layers")
    print(f"{dtype}: max|ref| = {np.abs(ref).max():.3e}, max-abs error {err:.3e}", flush=True)
    assert not host(LP)[B - 1].any()


@pytest.mark.parametrize("B,N,d,h,m,n_layers,per_user", [
    (3, 333, 128, 4, 64, 3, False),      # configuration-4 shape, several tiles and a ragged tail
    (2, 257, 256, 4, 128, 3, False),
    (2, 190, 64, 2, 32, 2, True),        # per-user contextualised links from the start
    (1, 100, 256, 8, 96, 1, False),      # one layer: the gated block on top of lime_xor_history
    (40, 1024, 128, 4, 64, 3, False),    # several steps per workgroup of the history kernel
    # layers whose operands stay in registers: every head count and width, an odd number of link blocks, less than a tile of
    # rows, and 128 links at d = 128, where they do not fit.  (Not one row: the sharp inputs' states are then of size 20, of
    # which bf16 keeps 2^-9, twice the absolute bar.)
    (3, 131, 128, 2, 96, 3, False), (2, 65, 64, 1, 32, 2, False), (5, 33, 32, 1, 64, 3, True), (2, 31, 64, 2, 32, 2, False),
    (2, 97, 128, 4, 128, 2, False),
])
def test_xor_layers(B, N, d, h, m, n_layers, per_user):
    """lime_xor_layers against the oracle's Eq. 8 on sharp inputs (gate pre-activations and XORA logits of order
    one, so that SiLU is far from linear), ragged lengths with an empty user, NaN in the padding rows.  The
    intermediate tensors are bf16; the bar is the single-call one all the same."""
    w = _sharp(workload=400 + d + m + n_layers, B=B, N=N, C=8, d=d, h=h, m=m, dtype="bf16",
               len_range=(max(1, N // 3), N), pad_value=np.nan)
    w.lens[B - 1] = 0 if B > 1 else w.lens[0]
    w.E[B - 1, w.lens[B - 1]:] = np.nan
    Wu, Wo = _layer_weights(77 + d, n_layers, d, gain=2.0)
    LC = w.L
    if per_user:
        LC = np.stack([np.roll(w.L, b + 1, axis=0) for b in range(B)])
    g = DeviceWorkload(w)
    xs = _xor_scale(w)
    LP = binding.lime_xor_layers(g.E, g.lens, dev(LC, "bf16"), g.Wq, g.Wk, g.Wv, dev(Wu, "bf16"), dev(Wo, "bf16"), h, xs)
    ref = orc.lime_xor_layers(w.E, w.lens, LC, w.Wq, w.Wk, w.Wv, Wu, Wo, h, xs)
    err = assert_close(host(LP), ref, "bf16", "LP of stacked XOR layers")
    print(f"max|ref| = {np.abs(ref).max():.3e}, max-abs error {err:.3e}", flush=True)
    if B > 1:
        assert not host(LP)[B - 1].any()
    if n_layers == 1:
        # one layer is the gated block applied to the link states of lime_xor_history
        OT, _ = binding.lime_xor_history(g.E, g.lens, dev(LC, "bf16"), g.Wq, g.Wk, g.Wv, h, xs)
        Lb = LC if LC.ndim == 3 else np.broadcast_to(LC, (B,) + LC.shape)
        want = np.stack([orc.gated_mlp(host(OT)[b], Lb[b], Wu[0], Wo[0]) for b in range(B)])
        assert_close(host(LP), want, "bf16", "one layer on the GPU's own O[T]")


def test_random_shapes_all_paths():
    """Thirty seeded random shapes through every forward entry point (both storage types; d/h = 32 / 64 on the matrix
    cores and 8 .. 48 on the general kernels; 1 .. 129 links; histories and candidate lists of up to 1500 rows; full or
    ragged with NaN padding), half of them from the benchmark distribution, half with sharp logits."""
    rng = np.random.default_rng(777)
    for case in range(30):
        dtype = "bf16" if rng.integers(0, 4) > 0 else "fp32"
        dh = int(rng.choice([32, 64])) if dtype == "bf16" and rng.integers(0, 5) > 0 else int(rng.choice([8, 16, 24, 48]))
        h = int(rng.choice([1, 2, 4]))
        m = int(rng.choice([32, 64, 96, 128])) if rng.integers(0, 3) > 0 else int(rng.integers(1, 130))
        N, C, B = int(rng.integers(8, 1500)), int(rng.integers(1, 1500)), int(rng.integers(1, 4))
        kw = dict(len_range=(8, N), pad_value=np.nan) if rng.integers(0, 3) > 0 else {}
        if case % 2:
            w = _sharp(workload=5000 + case, B=B, N=N, C=C, d=dh * h, h=h, m=m, dtype=dtype, **kw)
        else:
            w = synth.make_workload(5000 + case, B=B, N=N, C=C, d=dh * h, h=h, m=m, dtype=dtype, value_gain=0.25, **kw)
        print(f"case {case}: {dtype} B={B} N={N} C={C} d={dh * h} h={h} m={m} gain={w.meta['gain']:.2f} "
              f"lens={None if w.lens is None else w.lens.tolist()}", flush=True)
        for name, (got, ref) in run_all_paths(w, xor_scale=w.softmax_scale if case % 2 else 1.0).items():
            assert_close(got, ref, dtype, f"case {case} {name}")


@pytest.mark.parametrize("B,N,C,d,h,m,dtype", [
    (1, 2500, 70, 36, 1, 9, "fp32"),    # keys cut into chunks (the last one short); a head width that is no multiple of 8
    (1, 1025, 1, 10, 2, 33, "fp32"),    # one key in the second chunk, one query; heads of width 5 (no 16-byte reads)
    (40, 40, 900, 64, 8, 31, "bf16"),   # candidates without the split over waves, one key short of a tile
    (9, 1030, 300, 96, 1, 70, "fp32"),  # three blocks of head columns
    (3, 31, 129, 32, 4, 16, "bf16"),    # tiles of 128 rows and 32 columns in the projections, one row past a tile
])
def test_general_kernels_at_their_edges(B, N, C, d, h, m, dtype):
    w = _sharp(workload=70 + m, B=B, N=N, C=C, d=d, h=h, m=m, dtype=dtype, len_range=(max(1, N // 3), N), pad_value=np.nan)
    _check_all(w)
    g = DeviceWorkload(w)
    s = w.softmax_scale
    LP, O = binding.lime_request(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, g.T, g.L, g.Wq, g.Wk, g.Wv, h, s, s)
    LP2 = binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, s)
    assert torch.equal(LP, LP2) and torch.equal(O, binding.lime_score_candidates(g.T, g.L, LP2, g.Wq, g.Wk, g.Wv, h, s))


@pytest.mark.parametrize("B,N,C,d,h,m", [
    (1, 1, 1, 256, 4, 64),       # one item, one query
    (2, 65, 257, 256, 4, 96),    # a step of the history kernel and one item; three link blocks over two waves
    (3, 129, 31, 128, 2, 32),    # one link block over two waves; one query short of a block
    (5, 1057, 64, 128, 4, 128),  # four waves and one step per workgroup, the last workgroup's of two tiles, one item in the second
    (2, 2049, 33, 256, 8, 64),   # eight waves, one head and one step per workgroup, the last one's of one item
    (16, 1281, 40, 128, 4, 128), # the same with two steps, the last one item long (two buffers for the rows)
    (6, 2049, 33, 256, 8, 64),   # and without a second buffer: the refill between two barriers
    (33, 2017, 40, 256, 4, 32),  # several heads per workgroup, the last step one tile and one item
    (65, 2080, 20, 128, 4, 64),  # the same with heads of width 32
])
def test_history_and_target_attention_at_their_edges(B, N, C, d, h, m):
    w = _sharp(workload=170 + m, B=B, N=N, C=C, d=d, h=h, m=m, dtype="bf16", len_range=(max(1, N // 3), N), pad_value=np.nan)
    g = DeviceWorkload(w)
    for name, got, ref in [
        ("LP", binding.lime_link_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, w.softmax_scale),
         orc.lime_link_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, w.softmax_scale)),
        ("O[T]", binding.lime_xor_history(g.E, g.lens, g.L, g.Wq, g.Wk, g.Wv, h, 0.1 * w.softmax_scale, want_os=False)[0],
         orc.lime_xor_history(w.E, w.lens, w.L, w.Wq, w.Wk, w.Wv, h, 0.1 * w.softmax_scale, want_os=False)[0]),
        ("target attention", binding.mha_target_attention(g.T, g.E, g.lens, g.Wq, g.Wk, g.Wv, h, w.softmax_scale),
         orc.mha_target_attention(w.T, w.E, w.lens, w.Wq, w.Wk, w.Wv, h, w.softmax_scale)),
    ]:
        assert_close(host(got), ref, "bf16", name)


@pytest.mark.parametrize("d,h", [(128, 4), (256, 4)])
@pytest.mark.parametrize("scale", [0.1, -0.1, 1e-38])
def test_logits_far_from_zero_and_scales_near_it(d, h, scale):
    """All of a head's logits near -64 d/h scale (about -200 and -400, or +200 and +400): the softmax's first base lies
    below the exponent range; a scale so small that eight powers of two divided by it are infinite: uniform weights."""
    rng = np.random.default_rng(5)
    bf = lambda x: torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).float().numpy()  # noqa: E731
    E = bf(-8 + 0.5 * rng.standard_normal((2, 100, d)))
    X = np.full((2, 70, d), 8, np.float32)
    L = np.full((64, d), 8, np.float32)
    I, V = np.eye(d, dtype=np.float32), np.eye(d, dtype=np.float32) / 16  # outputs near -1/2
    lens = np.array([100, 37], np.int32)
    t = lambda x: dev(x, "bf16")  # noqa: E731
    lens_d = torch.from_numpy(lens).cuda()
    A = binding.mha_target_attention(t(X), t(E), lens_d, t(I), t(I), t(V), h, scale)
    assert_close(host(A), orc.mha_target_attention(X, E, lens, I, I, V, h, scale), "bf16", "target attention")
    LP = binding.lime_link_history(t(E), lens_d, t(L), t(I), t(I), t(V), h, scale)
    assert_close(host(LP), orc.lime_link_history(E, lens, L, I, I, V, h, scale), "bf16", "LP")


@pytest.mark.parametrize("d,h,B,N", [
    (128, 4, 33, 2017),  # several steps per workgroup of the history kernel, several heads together
    (256, 4, 3, 1057),   # heads of width 64
    (256, 8, 6, 2049),   # one head per workgroup, two steps
])
def test_largest_softmax_weight_is_not_rounded(d, h, B, N):
    """One item per user has a logit of its own and is the only one with a value; every other logit is zero.  The weights
    are kept in bf16 relative to the running maximum, so that this item's is one exactly, and with logits that are exact
    the output is off by its own rounding only: half a bf16 ulp, at most 2^-8 of the value (beside fp32 sums and the hardware
    exponential, 2^-20 each at most).  A weight that is rounded like any other would add up to 2^-8 of its own.  Head a
    takes its keys from column 2a of E and its values from column 2a + 1, spread over the head by W_V."""
    dh = d // h
    rng = np.random.default_rng(17)
    top = rng.integers(N // 2, N, B)  # past the first tiles, whose logits are all zero
    E = np.zeros((B, N, d), np.float32)
    Wq, Wk, Wv = (np.zeros((d, d), np.float32) for _ in range(3))
    for a in range(h):
        E[np.arange(B), top, 2 * a], E[np.arange(B), top, 2 * a + 1] = 1, 1
        Wq[a * dh, a * dh] = Wk[2 * a, a * dh] = 1
        Wv[2 * a + 1, a * dh:(a + 1) * dh] = 1 + np.arange(dh) / 128  # representable
    m = 64
    X = np.zeros((m, d), np.float32)
    X[:, ::dh] = 1 + np.arange(m)[:, None] / 64  # logits of 4 to 8 powers of two
    scale = float(np.float32(4 * np.log(2)))
    X, E, Wq, Wk, Wv = (torch.from_numpy(x).to(torch.bfloat16).float().numpy() for x in (X, E, Wq, Wk, Wv))
    t = lambda x: dev(x, "bf16")  # noqa: E731
    T = np.broadcast_to(X, (B, m, d)).copy()
    for name, got, ref in [
        ("target attention", binding.mha_target_attention(t(T), t(E), None, t(Wq), t(Wk), t(Wv), h, scale),
         orc.mha_target_attention(T, E, None, Wq, Wk, Wv, h, scale)),
        ("link states", binding.lime_link_history(t(E), None, t(X), t(Wq), t(Wk), t(Wv), h, scale),
         orc.lime_link_history(E, None, X, Wq, Wk, Wv, h, scale)),
    ]:
        worst = float((np.abs(host(got) - ref) / ref).max())
        print(f"{name} d={d} h={h}: largest relative error {worst * 256:.4f} x 2^-8", flush=True)
        assert worst <= 2.0 ** -8 + 2.0 ** -18, name


def test_a_missing_weight_is_refused_by_the_library():
    """None for a weight that a call needs, or for the prepared operands, is the library's error (LIME_INVALID_ARG), as it is
    through the C symbols."""
    bf = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    E, L, W, T = bf(2, 40, 64), bf(32, 64), bf(64, 64), bf(2, 5, 64)
    Wu = bf(1, 64, 64)
    for call in [
        lambda: binding.lime_link_history(E, None, L, W, None, W, 2, 1.0),
        lambda: binding.lime_xor_history(E, None, L, None, W, W, 2, 1.0),
        lambda: binding.lime_xor_layers(E, None, L, W, W, None, Wu, Wu, 2, 1.0),
        lambda: binding.mha_target_attention(T, E, None, W, W, None, 2, 1.0),
        lambda: binding.lime_request(E, None, L, W, W, None, T, L, W, W, W, 2, 1.0, 1.0),
        lambda: binding.lime_request_static(E, None, L, None, W, W, T, L, W, W, W, 2, 1.0, 1.0),
        lambda: binding.lime_link_history_prepared(E, None, None, 2, 32, 1.0),
        lambda: binding.lime_score_candidates_prepared(T, bf(2, 32, 64), W, None, 2, 1.0),
        lambda: binding.lime_request_prepared(E, None, T, W, None, 2, 32, 1.0, 1.0),
    ]:
        with pytest.raises(binding.LimeError, match="NULL") as e:
            call()
        assert e.value.status == 1
