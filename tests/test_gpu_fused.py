"""The stages that project by themselves (fused_history.hip, fused_rows.hip) against plain 64-bit arithmetic, at the edges of
their tiles (32 items, 16 links), chunks (256 items) and forms (one per head width and number of links)."""

import pytest
import torch

from paper_2510_18239_amd import binding

pytestmark = pytest.mark.gpu

# fp32: a result is behind three sums in a row (projection, logits, weighted sum) of at most 48 roundings of 2^-24 each, and an
# error of a logit is one of its weight: 3 * 48 * 2^-24 = 8.6e-6.  bf16: operands and results rounded to 2^-9 once each.
TOLERANCE = {torch.float32: 1e-5, torch.bfloat16: 1e-2}


def _attention(q, k, v, h, scale, lens, silu):
    (B, R, d), n = q.shape, k.shape[1]
    q, k, v = (x.reshape(B, -1, h, d // h).transpose(1, 2) for x in (q, k, v))
    s = q @ k.transpose(2, 3) * scale
    live = torch.ones((B, 1, 1, n), dtype=torch.bool, device=q.device)
    count = torch.full((B, 1, 1, 1), n, device=q.device)
    if lens is not None:
        live = (torch.arange(n, device=q.device)[None, :] < lens[:, None])[:, None, None]
        count = lens[:, None, None, None]
    p = torch.where(live, s * torch.sigmoid(s), 0.0) / count if silu else torch.softmax(torch.where(live, s, -torch.inf), dim=-1)
    return (p @ v).transpose(1, 2).reshape(B, R, d)


def _request(E, lens, L, W, T, LP, h, scale, silu):
    """Both stages in 64 bits; the second from the link states as they were stored."""
    D = lambda x: x.double()  # noqa: E731
    B = E.shape[0]
    rows = lambda w: (D(L) @ D(w))[None].expand(B, -1, -1)  # noqa: E731
    E = torch.where((torch.arange(E.shape[1], device=E.device)[None, :] < lens[:, None])[:, :, None], D(E), 0.0)
    return (_attention(rows(W[0]), E @ D(W[1]), E @ D(W[2]), h, scale, lens, silu),
            _attention(D(T) @ D(W[3]), rows(W[4]), D(LP) @ D(W[5]), h, scale, None, False))


def _inputs(B, N, C, d, m, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda shape, std=1.0: (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)  # noqa: E731
    lens = torch.randint(1, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = N
    E = rn((B, N, d))
    E[torch.arange(N, device="cuda")[None, :] >= lens[:, None]] = torch.nan  # padding is never read
    return E, lens, rn((m, d)), rn((B, C, d)), [rn((d, d), d ** -0.5) for _ in range(6)]


def _error(x, ref):
    return float((x.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,N,C,d,h,m", [
    (2, 1, 1, 32, 4, 1), (3, 31, 33, 32, 4, 8), (2, 32, 31, 32, 2, 16), (1, 33, 300, 32, 1, 17), (2, 255, 257, 64, 8, 16),
    (2, 256, 32, 64, 4, 32), (3, 257, 65, 64, 2, 33), (1, 513, 96, 64, 1, 64), (2, 100, 40, 128, 8, 31), (5, 777, 129, 128, 4, 64),
    (1, 300, 20, 128, 4, 128), (2, 70, 64, 64, 1, 15), (40, 64, 600, 32, 4, 16),
    # a workgroup for every compute unit, and more rows than its waves take at once: several tiles a wave, prefetched, in both row
    # stages (O[S]: lengths that end within, between and before a wave's later tiles)
    (64, 600, 600, 128, 4, 64), (256, 300, 530, 64, 1, 40), (130, 290, 300, 64, 2, 64),
])
@pytest.mark.parametrize("silu", [False, True])
def test_against_64_bits(B, N, C, d, h, m, dtype, silu):
    if dtype == torch.bfloat16 and d // h >= 32 and m % 32 == 0:
        m -= 4  # (the bf16 matrix-core kernels' otherwise)
    E, lens, L, T, W = _inputs(B, N, C, d, m, dtype, seed=N + C)
    scale = (d // h) ** -0.5
    LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, scale, scale, xor_attention=silu)
    refs = _request(E, lens, L, W, T, LP, h, scale, silu)
    assert _error(LP, refs[0]) <= TOLERANCE[dtype] and _error(O, refs[1]) <= TOLERANCE[dtype]
    # the stages by themselves, and O[S] (rows over links with SiLU, per-user links)
    call = binding.lime_xor_history if silu else binding.lime_link_history
    alone = call(E, lens, L, *W[:3], h, scale)
    assert torch.equal(alone[0] if silu else alone, LP)
    assert torch.equal(binding.lime_score_candidates(T, L, LP, *W[3:], h, scale), O)
    if silu:
        links = torch.stack([L.roll(b, 0) for b in range(B)])
        OT, OS = binding.lime_xor_history(E, lens, links, *W[:3], h, scale, want_os=True)
        x = E.double()
        p = [links.double() @ w.double() for w in W[:3]]
        live = torch.arange(N, device="cuda")[None, :] < lens[:, None]
        assert _error(OT[0], _request(E[:1], lens[:1], links[0], W, T[:1], LP[:1], h, scale, True)[0][0]) <= TOLERANCE[dtype]
        ref = _attention(torch.nan_to_num(x) @ W[0].double(), p[1], p[2], h, scale, None, True) * live[:, :, None]
        assert _error(OS, ref) <= TOLERANCE[dtype] and torch.equal(OS[~live], torch.zeros_like(OS[~live]))


@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
@pytest.mark.parametrize("silu", [False, True])
def test_numbers_without_planes(d, h, m, silu):
    """fp32 numbers that round to an infinite bf16 number, and infinities and NaN: each stays with its row."""
    B, N, C = 3, 90, 70
    E, lens, L, T, W = _inputs(B, N, C, d, m, torch.float32, seed=d + m)
    lens[:] = torch.tensor([N, 33, 40])
    E = torch.where((torch.arange(N, device="cuda")[None, :] < lens[:, None])[:, :, None], torch.nan_to_num(E), torch.nan)
    scale = (d // h) ** -0.5
    run = lambda: binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, scale, scale, xor_attention=silu)  # noqa: E731
    plain = run()
    # the same request with the second user's items, and some candidates, at the upper end of the range and the weights at the lower
    big, Wb = 3.4e38, [w.clone() for w in W]
    E2, T2, Wb[1], Wb[2], Wb[3] = E.sign() * big, T.sign() * big, W[1] / big, W[2] / big, W[3] / big
    LP, O = binding.lime_request(E2, lens, L, *Wb[:3], T2, L, *Wb[3:], h, scale, scale, xor_attention=silu)
    refs = _request(E2, lens, L, Wb, T2, LP, h, scale, silu)
    # (W / 3.4e38 is about 2^-131: 18 bits of it are left, and the products' sums are of that precision)
    assert _error(LP, refs[0]) <= 2 ** -14 and _error(O, refs[1]) <= 2 ** -14
    E[1, 5, 3], T[0, 40, 0], T[2, 69, 1] = torch.inf, -torch.inf, torch.nan
    LP, O = run()
    assert torch.equal(LP[::2], plain[0][::2]) and not torch.isfinite(LP[1]).any()
    clean = torch.ones((B, C), dtype=torch.bool, device="cuda")
    clean[1], clean[0, 40], clean[2, 69] = False, False, False
    assert torch.equal(O[clean], plain[1][clean]) and not torch.isfinite(O[~clean]).any()


def _first_column(d, h):
    """Weights under which each head's logit is the product of the two rows' first columns, which the values do not hear of."""
    g = torch.Generator(device="cuda").manual_seed(d)
    Wq, Wk = torch.zeros((d, d), device="cuda"), torch.zeros((d, d), device="cuda")
    Wq[0, :: d // h] = Wk[0, :: d // h] = 1.0
    Wv = torch.randn((d, d), generator=g, device="cuda") * d ** -0.5
    Wv[0] = 0.0
    return Wq, Wk, Wv


@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
def test_tiles_of_a_chunk_at_the_ends_of_the_range(d, h, m):
    """Finite logits of one chunk's tiles so far apart that their difference times log2 e, or the difference itself, is not finite."""
    Wq, Wk, Wv = _first_column(d, h)
    g = torch.Generator(device="cuda").manual_seed(m)
    rn = lambda shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    B, N = 3, 160
    E, L, T = rn((B, N, d)), torch.zeros((m, d), device="cuda"), rn((B, 40, d))
    L[:, 0] = 1.0
    for b, (high, low) in enumerate([(1.2e38, -1.2e38), (3e38, -3e38), (1.0, -1.2e38)]):
        E[b, :, 0] = low
        E[b, 32 * b : 32 * b + 32, 0] = high
    W = [Wq, Wk, Wv] + [rn((d, d)) * d ** -0.5 for _ in range(3)]
    lens = torch.full((B,), N, dtype=torch.int32, device="cuda")
    LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, 1.0, 0.2)
    ref = _attention((L.double() @ Wq.double())[None].expand(B, -1, -1), E.double() @ Wk.double(), E.double() @ Wv.double(), h, 1.0, lens, False)
    for b in range(B):
        assert _error(LP[b], ref[b]) <= TOLERANCE[torch.float32], b
    assert torch.isfinite(O).all()


# Numbers at the lower end of the range (2^-126), whose remainders are below any bf16 number: which operand they come to.
# Powers of two, so that what follows from them is scaled and no digit is lost in the inputs themselves.
@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
@pytest.mark.parametrize("silu", [False, True])
@pytest.mark.parametrize("small", ["rows", "key weights", "value weights", "links"])
def test_small_numbers(d, h, m, silu, small):
    B, N, C = 2, 90, 70
    E, lens, L, T, W = _inputs(B, N, C, d, m, torch.float32, seed=d + m)
    E = torch.where(torch.arange(N, device="cuda")[None, :, None] < lens[:, None, None], E, 0.0)
    down, up = 2.0 ** -118, 2.0 ** 59
    if small == "rows":  # queries and keys that make ordinary logits of them
        E, T, W[0], W[1], W[2], W[3], W[4] = E * down, T * down, W[0] * up, W[1] * up, W[2] * up, W[3] * up, W[4] * up
    elif small == "key weights":  # (SiLU: tiny logits, and weights)
        W[1], W[4] = W[1] * down, W[4] * down
    elif small == "value weights":
        W[2], W[5] = W[2] * down, W[5] * up
    else:
        L, W[0], W[1], W[3], W[4] = L * down, W[0] * up, W[1] * up, W[3] * up, W[4] * up
    scale = (d // h) ** -0.5
    LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, scale, scale, xor_attention=silu)
    refs = _request(E, lens, L, W, T, LP, h, scale, silu)
    assert float(refs[0].abs().max()) < 2.0 ** 100 and float(refs[1].abs().max()) > 2.0 ** -126
    assert _error(LP, refs[0]) <= TOLERANCE[torch.float32] and _error(O, refs[1]) <= TOLERANCE[torch.float32]


# Keys and values of 2^50 to 2^110: sums, products of them with weights, and the numbers themselves pass what the planes hold.
@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
@pytest.mark.parametrize("silu", [False, True])
@pytest.mark.parametrize("power", [50, 60, 85, 110])
def test_large_numbers(d, h, m, silu, power):
    B, N, C = 2, 90, 70
    E, lens, L, T, W = _inputs(B, N, C, d, m, torch.float32, seed=d + m)
    E = torch.where(torch.arange(N, device="cuda")[None, :, None] < lens[:, None, None], E, 0.0)
    W[1], W[2], W[3], W[5] = W[1] * 2.0 ** power, W[2] * 2.0 ** power, W[3] * 2.0 ** power, W[5] * 2.0 ** -power
    scale = (d // h) ** -0.5 * 2.0 ** -power
    LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, scale, scale, xor_attention=silu)
    refs = _request(E, lens, L, W, T, LP, h, scale, silu)
    assert _error(LP, refs[0]) <= TOLERANCE[torch.float32] and _error(O, refs[1]) <= TOLERANCE[torch.float32]


@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
def test_small_attention_weights(d, h, m):
    """A result that comes from the small weights alone: the item (link) with the large one has the value zero."""
    Wq, Wk, Wv = _first_column(d, h)
    B, N, C = 2, 70, 40
    g = torch.Generator(device="cuda").manual_seed(m)
    rows = lambda shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    E, T, L = rows((B, N, d)), rows((B, C, d)), rows((m, d))
    E[:, :, 0] = -86.0 - torch.rand((B, N), generator=g, device="cuda").mul(8).round() / 8
    E[:, 3], L[:, 0] = 0.0, 1.0
    lens = torch.full((B,), N, dtype=torch.int32, device="cuda")
    LP, _ = binding.lime_request(E, lens, L, Wq, Wk, Wv, T, L, Wq, Wk, Wv, h, 1.0, 1.0)
    D = lambda x: x.double()  # noqa: E731
    q = (D(L) @ D(Wq))[None].expand(B, -1, -1)
    assert _error(LP, _attention(q, D(E) @ D(Wk), D(E) @ D(Wv), h, 1.0, lens, False)) <= TOLERANCE[torch.float32]
    # candidates over links: the links' first columns decide, the values are those of given link states
    K, V = L.clone(), rows((B, m, d))
    K[:, 0] = -86.0 - torch.rand((m,), generator=g, device="cuda").mul(8).round() / 8
    K[2], V[:, 2], T[:, :, 0] = 0.0, 0.0, 1.0
    O = binding.lime_score_candidates(T, K, V, Wq, Wk, Wv, h, 1.0)
    k = (D(K) @ D(Wk))[None].expand(B, -1, -1)
    assert _error(O, _attention(D(T) @ D(Wq), k, D(V) @ D(Wv), h, 1.0, None, False)) <= TOLERANCE[torch.float32]


@pytest.mark.parametrize("d,h,m", [(32, 4, 16), (64, 2, 32), (64, 1, 40), (128, 4, 64)])
@pytest.mark.parametrize("silu", [False, True])
def test_long_histories_have_no_error_common_to_all_items(d, h, m, silu):
    """The mean of N items' values (weights all alike) is sqrt(N) times smaller than they are, and so are errors of either sign; an
    error that all items share stays as it is."""
    B, N = 4, 8192
    g = torch.Generator(device="cuda").manual_seed(d + m)
    rn = lambda shape, std=1.0: torch.randn(shape, generator=g, device="cuda") * std  # noqa: E731
    E, L, W = rn((B, N, d)), rn((m, d)), [rn((d, d), d ** -0.5) for _ in range(3)]
    if silu:  # logits of one: every weight is SiLU(1)
        W[0], W[1] = torch.zeros((d, d), device="cuda"), torch.zeros((d, d), device="cuda")
        E[:, :, 0] = L[:, 0] = 1.0
        W[0][0, :: d // h] = W[1][0, :: d // h] = 1.0
        W[2][0] = 0.0
    call = (lambda *a: binding.lime_xor_history(*a)[0]) if silu else binding.lime_link_history
    LP = call(E, None, L, *W, h, 1.0 if silu else 0.0)[:, 0].double()
    ref = (E.double() @ W[2].double()).mean(dim=1) * (torch.sigmoid(torch.ones((), dtype=torch.float64)).item() if silu else 1.0)
    # a value is d products and roundings of 2^-24 at most, in the root mean square a third of that each, and a tile's and the tiles'
    # sums are as good: 2^-24 * sqrt(3 * 128) / 3 = 3.9e-7 (it was 6e-7 to 1e-6 with the shared error)
    assert _error(LP, ref) <= 4e-7


# Histories of one to five tiles, and of a chunk and one, of more users than workgroups run at once.  The workgroups' shares: 8, 5 (the
# last short), 4, 2 and 1 users.
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,N,d,h,m", [(1030, 20, 32, 4, 16), (643, 50, 64, 2, 36), (900, 90, 128, 4, 60), (700, 270, 64, 1, 20), (600, 150, 64, 4, 16)])
@pytest.mark.parametrize("silu", [False, True])
def test_many_users_with_few_rows(B, N, d, h, m, dtype, silu):
    C = 36
    E, lens, L, T, W = _inputs(B, N, C, d, m, dtype, seed=B)
    lens[5], lens[6] = 0, 1
    E[5] = E[6, 1:] = torch.nan
    scale = (d // h) ** -0.5
    run = lambda part: binding.lime_request(E[part], lens[part], L, *W[:3], T[part], L, *W[3:], h, scale, scale, xor_attention=silu)  # noqa: E731
    LP, O = run(slice(0, B))
    for b in (0, 4, 5, 6, B // 2, B - 1):  # (alone: a workgroup each)
        LP1, O1 = run(slice(b, b + 1))
        assert torch.equal(LP1[0], LP[b]) and torch.equal(O1[0], O[b]), b
    assert not LP[5].any()
    live = lens > 0
    refs = _request(E[live], lens[live], L, W, T[live], LP[live], h, scale, silu)
    assert _error(LP[live], refs[0]) <= TOLERANCE[dtype] and _error(O[live], refs[1]) <= TOLERANCE[dtype]
    links = torch.stack([L.roll(b, 0) for b in range(B)])  # links of each user's own
    call = (lambda *a: binding.lime_xor_history(*a)[0]) if silu else binding.lime_link_history
    own = call(E, lens, links, *W[:3], h, scale)
    for b in (0, 5, m, B - 1):
        assert torch.equal(own[b], LP[b].roll(b, 0)), b
    if silu:  # O[S], rows of every length
        rows = lambda part: binding.lime_xor_history(E[part], lens[part], L, *W[:3], h, scale, want_os=True)[1]  # noqa: E731
        OS = rows(slice(0, B))
        for b in (0, 4, 5, 6, B - 1):
            assert torch.equal(rows(slice(b, b + 1))[0], OS[b]), b
        valid = torch.arange(N, device="cuda")[None, :] < lens[:, None]
        p = [(L.double() @ w.double())[None].expand(B, -1, -1) for w in W[1:3]]
        ref = _attention(torch.where(valid[:, :, None], E.double(), 0.0) @ W[0].double(), *p, h, scale, None, True) * valid[:, :, None]
        assert _error(OS, ref) <= TOLERANCE[dtype] and not OS[~valid].any()
    # what is not finite stays with its user, and its row
    lens[7] = N
    E[7], T[9, 3, 1] = torch.nan_to_num(E[7]), torch.nan
    clean = run(slice(0, B))
    E[7, 0, 3] = torch.inf
    LP, O = run(slice(0, B))
    others = torch.arange(B, device="cuda") != 7
    assert torch.equal(LP[others], clean[0][others]) and not torch.isfinite(LP[7]).any() and not torch.isfinite(O[7]).any()
    assert torch.equal(torch.nan_to_num(O[others]), torch.nan_to_num(clean[1][others])) and not torch.isfinite(O[9, 3]).any()
    assert torch.isfinite(O[9, :3]).all() and torch.isfinite(O[10:]).all()


def test_unaligned_rows_take_the_general_kernels():
    B, N, C, d, h, m = 2, 300, 50, 64, 2, 32
    E, lens, L, T, W = _inputs(B, N, C, d, m, torch.float32, seed=3)
    off = lambda x: torch.cat([x.new_zeros(1), x.reshape(-1)])[1:].view(x.shape)  # noqa: E731
    LP, O = binding.lime_request(E, lens, L, *W[:3], T, L, *W[3:], h, 0.2, 0.2)
    LP1, O1 = binding.lime_request(off(E), lens, L, *W[:3], off(T), L, *W[3:], h, 0.2, 0.2)
    assert _error(LP1, LP.double()) <= 1e-5 and _error(O1, O.double()) <= 1e-5
