"""The work that users of this library have it do, as cases to be timed: requests of every size through the public entry
points of `paper_2510_18239_amd.binding`, the XOR layers, their backward pass, the scoring pipeline, the QK-cache path and
the full target attention it is compared with.

Shapes are those of `synth.CONFIGS` (the five benchmark configurations), of the hyper-parameters the paper trains with
(four heads; embeddings of width 32 with 16 or 8 links, width 256 with 32 links; histories of 50 to 1024 items) and of its
latency study (16 to 32768 candidates, histories of up to 16384 items), with odd sizes between them.

Values: embeddings, links and weights are Gaussian with the projections scaled so that a head's logits have a standard
deviation near one (a trained model's regime; the softmaxes are neither uniform nor one-hot), rows past a user's length
are zero padding, ids are uniform over the table.
"""

import math

import torch

from paper_2510_18239_amd import binding

TORCH_DTYPE = {"bf16": torch.bfloat16, "fp32": torch.float32}
BYTES = {"bf16": 2, "fp32": 4}


def listed():
    return [
        # one user of a small fp32 model (configuration 1): the smallest call, all latency and launches
        dict(name="request fp32 smallest", op="request", B=1, N=128, C=64, d=64, h=1, m=16, dtype="fp32", ragged=False, xor=False),
        # one user, a handful of candidates (re-ranking a short list): the low end of the latency study
        dict(name="request few candidates", op="request", B=1, N=2048, C=16, d=256, h=4, m=64, dtype="bf16", ragged=False, xor=False),
        # one user against the largest candidate set of the latency study (configuration 3): the headline request
        dict(name="request headline", op="request", B=1, N=2048, C=32768, d=256, h=4, m=64, dtype="bf16", ragged=False, xor=False),
        # a batch of users with ragged histories (configuration 2)
        dict(name="request batch ragged", op="request", B=32, N=1024, C=1024, d=128, h=4, m=64, dtype="bf16", ragged=True, xor=False),
        # a batch of users of the paper's small public-data model: heads of width 8, 16 links, odd candidate count
        dict(name="request small model", op="request", B=64, N=256, C=501, d=32, h=4, m=16, dtype="bf16", ragged=True, xor=False),
        # a batch in fp32 storage (reference-precision scoring), odd sizes
        dict(name="request fp32 batch", op="request", B=16, N=777, C=1001, d=128, h=4, m=64, dtype="fp32", ragged=True, xor=False),
        # the server with fixed weights (operands prepared once), the largest batch (configuration 5)
        dict(name="prepared request large", op="prepared", B=16, N=4096, C=8192, d=256, h=4, m=128, dtype="bf16", ragged=True, xor=False),
        # embeddings to scores at the headline shape with the larger interaction network
        dict(name="scores headline", op="scores", B=1, N=2048, C=32768, d=256, h=4, m=64, dtype="bf16", ragged=False, net="512,128,64"),
        # the user side of LIME-XOR, three stacked layers, at the longest history (configuration 4)
        dict(name="xor layers long", op="xor_layers", B=8, N=16384, d=128, h=4, m=64, dtype="bf16", ragged=False, layers=3),
        # training: backward of one XOR layer at the same shape
        dict(name="xor backward long", op="xor_backward", B=8, N=16384, d=128, h=4, m=64, dtype="bf16", ragged=False),
        # the comparison every evaluation of the method runs: full target attention (configuration 5)
        dict(name="target attention large", op="target", B=16, N=4096, C=8192, d=256, h=4, dtype="bf16", ragged=True),
        # three-stage inference: candidates named by id, attention weights from a corpus table
        dict(name="gathered qk cache", op="gathered", B=1, C=32768, items=131072, d=256, h=4, m=64, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    """A size spread evenly over the logarithm of [lo, hi], odd as often as even."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["request"] * 5 + ["prepared"] * 2 + ["scores"] * 2 + ["xor_layers", "xor_backward", "target", "gathered"])
    d, h = rng.choice([(64, 2), (128, 2), (128, 4), (256, 4), (256, 8)])
    m = rng.choice([32, 64, 64, 96, 128])
    B = _log(rng, 1, 32)
    N = _log(rng, 50, min(16384, 65536 // B))
    C = _log(rng, 16, min(32768, 131072 // B))
    ragged, xor = rng.random() < 0.5, rng.random() < 0.3
    if op == "request":
        kind = rng.random()
        if kind < 0.25:  # fp32 storage, reference-precision scoring
            d, h, m = rng.choice([(32, 4, 16), (64, 1, 16), (64, 2, 32), (128, 4, 64)])
            B = _log(rng, 1, 16)
            N, C = _log(rng, 50, min(4096, 12432 // B)), _log(rng, 16, min(8192, 16016 // B))
            return dict(op=op, B=B, N=N, C=C, d=d, h=h, m=m, dtype="fp32", ragged=ragged, xor=xor)
        if kind < 0.5:  # the small public-data models
            d, h, m = rng.choice([(32, 4, 16), (32, 4, 8), (64, 4, 16)])
            B = _log(rng, 1, 64)
            N, C = _log(rng, 50, min(1024, 16384 // B)), _log(rng, 16, min(8192, 32064 // B))
        return dict(op=op, B=B, N=N, C=C, d=d, h=h, m=m, dtype="bf16", ragged=ragged, xor=xor)
    if op == "prepared":
        return dict(op=op, B=B, N=N, C=C, d=d, h=h, m=m, dtype="bf16", ragged=ragged, xor=xor)
    if op == "scores":
        d, h = rng.choice([(128, 4), (256, 4)])
        C = _log(rng, 16, min(32768, 32768 // B))
        return dict(op=op, B=B, N=N, C=C, d=d, h=h, m=rng.choice([32, 64]), dtype="bf16", ragged=ragged,
                    net=rng.choice(["96", "512,128,64", "512,256,128"]))
    if op == "xor_layers":
        return dict(op=op, B=min(B, 8), N=_log(rng, 50, 16384), d=128, h=4, m=rng.choice([32, 64]), dtype="bf16", ragged=ragged,
                    layers=rng.choice([1, 2, 3]))
    if op == "xor_backward":
        if rng.random() < 0.25:
            return dict(op=op, B=min(B, 8), N=_log(rng, 50, 2048), d=64, h=2, m=32, dtype="fp32", ragged=ragged)
        return dict(op=op, B=min(B, 8), N=_log(rng, 50, 16384), d=128, h=4, m=rng.choice([32, 64]), dtype="bf16", ragged=ragged)
    if op == "target":
        B = min(B, 16)
        return dict(op=op, B=B, N=_log(rng, 50, 4096), C=_log(rng, 16, 8192), d=d, h=h, dtype="bf16", ragged=ragged)
    return dict(op=op, B=B, C=_log(rng, 16, 32768 // B), items=_log(rng, 4096, 131072), d=d, h=h, m=rng.choice([32, 64]), dtype="bf16")


class _Maker:
    """Seeded tensors on the GPU, rounded to the case's storage type."""

    def __init__(self, case, seed):
        self.dev = torch.device("cuda", torch.cuda.current_device())
        self.dtype = TORCH_DTYPE[case["dtype"]]
        self.g = torch.Generator(device=self.dev).manual_seed(seed)

    def normal(self, shape, std, mean=0.0):
        return (torch.randn(shape, generator=self.g, device=self.dev) * std + mean).to(self.dtype)

    def integers(self, lo, hi, shape):  # uniform on [lo, hi]
        return torch.randint(lo, hi + 1, shape, generator=self.g, device=self.dev, dtype=torch.int32)

    def lens(self, case):
        return self.integers((case["N"] + 1) // 2, case["N"], (case["B"],)) if case["ragged"] else None

    def history(self, rows, lens):
        """Zero padding past each user's length."""
        if lens is None:
            return rows
        live = torch.arange(rows.shape[1], device=self.dev)[None, :] < lens[:, None]
        return (rows * live[:, :, None]).to(self.dtype)


def prepare(case, seed):
    k = _Maker(case, seed)
    op, B, d, h, m = case["op"], case["B"], case["d"], case["h"], case.get("m")
    dh = d // h
    s = dict(op=op, h=h, m=m)
    if op == "gathered":
        logits = torch.randn((case["items"], h, m), generator=k.g, device=k.dev)
        s.update(table=torch.softmax(logits, dim=-1).to(k.dtype), ids=k.integers(0, case["items"] - 1, (B, case["C"])),
                 LP=k.normal((B, m, d), 1.0), Wv=k.normal((d, d), d ** -0.5))
        return s
    s["lens"] = lens = k.lens(case)
    if op == "xor_backward":  # projected tensors; logits of a head with standard deviation one
        qk = dh ** -0.25
        for name, rows, std in (("QS", case["N"], qk), ("KS", case["N"], qk), ("VS", case["N"], 1.0), ("dOS", case["N"], 1.0),
                                ("QT", m, qk), ("KT", m, qk), ("VT", m, 1.0), ("dOT", m, 1.0)):
            x = k.normal((B, rows, d), std)
            s[name] = k.history(x, lens) if rows == case["N"] and name[-1] == "S" else x
        s["scale"] = 1.0
        return s
    s["scale"] = dh ** -0.5
    s["E"] = k.history(k.normal((B, case["N"], d), 1.0), lens)
    weights = lambda: [k.normal((d, d), d ** -0.5) for _ in range(3)]  # noqa: E731
    s["hist"] = weights()
    if op != "target":
        s["L"] = k.normal((m, d), 1.0)
    if "C" in case:
        s["T"] = k.normal((B, case["C"], d), 1.0)
        s["cand"] = weights()
    if op in ("request", "prepared"):
        s["xor"] = case["xor"]
    if op == "prepared":
        s["prepared"] = binding.lime_prepare(s["L"], s["L"], *s["hist"], *s["cand"][:2], h, s["scale"], s["scale"])
    if op == "xor_layers":
        s["Wu"], s["Wo"] = k.normal((case["layers"], d, d), d ** -0.5), k.normal((case["layers"], d, d), d ** -0.5)
    if op == "scores":
        dc, dhid = 64, 256  # widths of the context vector and of Eq. 2's hidden layer
        widths = [int(x) for x in case["net"].split(",")] + [1]
        dims = [d] + widths
        norm = lambda: (k.normal((d,), 0.2, 1.0), k.normal((d,), 0.2))  # noqa: E731
        ctx = (k.normal((d + dc, dhid), (2.0 / (d + dc)) ** 0.5), k.normal((dhid,), 0.1), k.normal((dhid, d), dhid ** -0.5), k.normal((d,), 0.1))
        mlp = ([k.normal((dims[i], dims[i + 1]), (2.0 / dims[i]) ** 0.5) for i in range(len(widths))],
               [k.normal((dims[i + 1],), 0.1) for i in range(len(widths))])
        norms = [norm() for _ in range(5)]
        s["EC"] = k.normal((B, dc), 1.0)
        s["model"] = binding.scoring_model(s["L"], ctx, s["hist"], s["cand"], *norms, mlp, h, s["scale"], s["scale"])
        s["keep"] = (ctx, mlp, norms)  # the struct holds device pointers
    return s


def run(s):
    op, h, scale = s["op"], s["h"], s.get("scale")
    if op == "request":
        return binding.lime_request(s["E"], s["lens"], s["L"], *s["hist"], s["T"], s["L"], *s["cand"], h, scale, scale, xor_attention=s["xor"])
    if op == "prepared":
        return binding.lime_request_prepared(s["E"], s["lens"], s["T"], s["cand"][2], s["prepared"], h, s["m"], scale, scale,
                                             xor_attention=s["xor"])
    if op == "scores":
        return binding.lime_scores(s["model"], s["E"], s["lens"], s["EC"], s["T"])
    if op == "xor_layers":
        return binding.lime_xor_layers(s["E"], s["lens"], s["L"], *s["hist"], s["Wu"], s["Wo"], h, scale)
    if op == "xor_backward":
        return binding.lime_xor_backward(s["QS"], s["KS"], s["VS"], s["QT"], s["KT"], s["VT"], s["dOT"], s["dOS"], s["lens"], h, scale)
    if op == "target":
        return binding.mha_target_attention(s["T"], s["E"], s["lens"], *s["hist"], h, scale)
    return binding.lime_score_candidates_gathered(s["table"], s["ids"], s["LP"], s["Wv"])


def work(case):
    """Each input read once, each output written once; the cheaper of the two orders of the products (projecting the rows,
    or folding the projection into the links' side)."""
    op, B, d, h, m, e = case["op"], case["B"], case["d"], case["h"], case.get("m", 0), BYTES[case["dtype"]]
    N, C = case.get("N", 0), case.get("C", 0)
    valid = B * (0.75 * N if case.get("ragged") else N)  # history rows that count (the expectation of ragged lengths)
    history_pass = valid * min(4 * d * d + 4 * m * d, 4 * h * m * d)           # logits and weighted sum of m links over the rows
    candidate_pass = B * C * (min(2 * d * d + 2 * m * d, 2 * h * m * d) + 2 * m * d)  # logits over the links, weighted sum
    links = 2 * m * d * d                                                      # one projection of one set of links
    if op in ("request", "prepared"):
        weights = 6 * d * d if op == "request" else 3 * d * d + d * d
        return {"bytes": e * (valid * d + 2 * B * C * d + weights + 2 * m * d + B * m * d), "flops": history_pass + candidate_pass + (2 + B) * links}
    if op == "scores":
        dims = [d] + [int(x) for x in case["net"].split(",")] + [1]
        net = sum(dims[i] * dims[i + 1] for i in range(len(dims) - 1))
        return {"bytes": e * (valid * d + B * C * d + 6 * d * d + net + m * d) + 4 * B * C,
                "flops": history_pass + candidate_pass + B * C * 2 * net + (2 + 2 * B) * links + B * m * 2 * (d + 64 + d) * 256}
    if op == "xor_layers":
        last = history_pass + B * links
        full = valid * (min(4 * d * d + 4 * m * d, 4 * h * m * d) + 2 * d * d + 4 * m * d + 4 * d * d) + B * links * 5
        return {"bytes": e * (valid * d + (3 + 2 * case["layers"]) * d * d + m * d + B * m * d), "flops": last + (case["layers"] - 1) * full}
    if op == "xor_backward":
        return {"bytes": e * ((4 * valid + 3 * B * N) * d + 7 * B * m * d), "flops": 20 * valid * m * d}
    if op == "target":
        return {"bytes": e * (valid * d + 2 * B * C * d + 3 * d * d), "flops": 4 * C * valid * d + 4 * valid * d * d + 2 * B * C * d * d}
    return {"bytes": e * (B * C * (h * m + d) + B * m * d + d * d) + 4 * B * C, "flops": 2 * B * C * m * d + B * links}


def tolerance(case):
    """fp32 storage: fp32 sums in another order.  bf16: operands, intermediate operands of chained products and outputs are
    rounded to bf16 (2^-9 each); the interaction network and the stacked layers chain several such stages."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 2e-2 if case["op"] in ("scores", "xor_layers") else 1e-2}
