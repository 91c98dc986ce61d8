"""Performance cases: the calls that a program serving 4-bit decoder models makes of this library, over the sizes it makes
them at.  Five kinds:

  linear  one `wq_gemv` call: a layer's linear or the final projection run alone, for one token, a small batch of
          sequences, or a prompt (M rows of x).
  step    one `wq_decode_linears` call over every linear of a decoder's layers (and, with a vocabulary, the final
          projection): a decoding step of M concurrent sequences, or a prompt of M tokens.
  attn    one `paged_attention` call: a decoding step's attention of `seqs` sequences of mixed length over their paged
          keys and values.
  chain   one `wq_fused_linears` call: the dependent layer chain of one token, with its norms, gated products, residuals
          and the choice of the next token.
  pack    one `wq_pack` call: quantizing a weight matrix at load time.

Shapes are those of the 3B- and 8B-class decoders that the tests and the benchmark use, their tensor-parallel shards, and
generic ones.  `draw` spreads sizes, ragged ones among them, over the same ranges.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2412_15803_amd import wq

HEAD = 128
EPS = 1e-5
MODEL_3B = dict(hidden=3072, q_heads=24, kv_heads=8, inter=8192)
MODEL_8B = dict(hidden=4096, q_heads=32, kv_heads=8, inter=14336)


def listed():
    return [
        # The smallest call: a 512 x 512 linear for one token, where the launch and the host path are all there is.
        dict(name="linear_512_m1", kind="linear", n=512, k=512, m=1),
        # The final projection (a 128256-word vocabulary) for five concurrent sequences.
        dict(name="linear_head_m5", kind="linear", n=128256, k=3072, m=5),
        # One GPU's share of the 8B-class gate/up projection at eight-way tensor parallelism, on a short prompt.
        dict(name="linear_tp8_m100", kind="linear", n=3584, k=4096, m=100),
        # The 3B-class gate/up projection over a 2048-token prompt.
        dict(name="linear_gate_up_m2048", kind="linear", n=16384, k=3072, m=2048),
        # A whole 3B-class decoding step for one sequence: the framework's headline workload.
        dict(name="step_3b_m1", kind="step", layers=28, vocab=128256, m=1, **MODEL_3B),
        # A whole 8B-class decoding step for eight concurrent sequences.
        dict(name="step_8b_m8", kind="step", layers=32, vocab=128256, m=8, **MODEL_8B),
        # A 3B-class decoding step of a server with 48 sequences in flight.
        dict(name="step_3b_m48", kind="step", layers=28, vocab=128256, m=48, **MODEL_3B),
        # Every layer of the 3B-class model over a 512-token prompt (only the last token goes through the head).
        dict(name="prompt_3b_m512", kind="step", layers=28, vocab=0, m=512, **MODEL_3B),
        # One long conversation: 32768 cached tokens, 8B-class heads.
        dict(name="attn_8b_1x32768", kind="attn", seqs=1, min_len=32768, max_len=32768, q_heads=32, kv_heads=8, page=16),
        # A server's batch: 40 sequences of 100 to 6000 cached tokens, 3B-class heads.
        dict(name="attn_3b_40xmixed", kind="attn", seqs=40, min_len=100, max_len=6000, q_heads=24, kv_heads=8, page=16),
        # One token through the dependent 3B-class chain, up to the logits and the next token.
        dict(name="chain_3b", kind="chain", layers=28, vocab=128256, **MODEL_3B),
        # Quantizing the 8B-class gate/up projection when a model is loaded.
        dict(name="pack_8b_gate_up", kind="pack", n=28672, k=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    """Rough seconds of a pass, for bounding drawn cases."""
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 6e14)


def draw(rng: random.Random):
    kind = rng.choice(["linear", "linear", "linear", "step", "step", "attn", "attn", "chain", "pack"])
    while True:
        if kind == "linear":
            # One token, a small batch, or a prompt, a third of the draws each.
            m = rng.choice([1, _log_int(rng, 2, 64), _log_int(rng, 65, 4096)])
            case = dict(kind=kind, n=_log_int(rng, 256, 131072), k=32 * _log_int(rng, 16, 448), m=m)
        elif kind in ("step", "chain"):
            kv = rng.choice([2, 4, 8])
            q = kv * rng.randint(1, 32 // kv)
            hidden = 128 * rng.randint(8, 32)
            case = dict(kind=kind, layers=rng.randint(2, 32), vocab=rng.choice([0, _log_int(rng, 16000, 131072)]),
                        hidden=hidden, q_heads=q, kv_heads=kv, inter=32 * rng.randint(hidden // 16, hidden // 9))
            if kind == "step":
                case["m"] = rng.choice([1, _log_int(rng, 2, 64), _log_int(rng, 65, 1024)])
            elif not case["vocab"]:
                case["vocab"] = _log_int(rng, 16000, 131072)
        elif kind == "attn":
            kv = rng.choice([1, 2, 4, 8])
            top = _log_int(rng, 64, 32768)
            case = dict(kind=kind, seqs=_log_int(rng, 1, 64), min_len=max(1, top // rng.randint(1, 40)), max_len=top,
                        q_heads=kv * rng.randint(1, 8), kv_heads=kv, page=rng.choice([16, 16, 32, 64]))
        else:
            case = dict(kind=kind, n=_log_int(rng, 512, 32768), k=32 * _log_int(rng, 16, 448))
        if _cost(case) <= _cost(_LARGEST):
            return case


_LARGEST = dict(kind="step", layers=28, vocab=0, m=512, **MODEL_3B)


# ------------------------------------------------------------------ inputs


def _linears(case):
    """(layer, name, N, K) of every linear of a step or chain, in order."""
    q = case["q_heads"] * HEAD
    out = []
    for layer in range(case["layers"]):
        out += [(layer, "qkv", q + 2 * case["kv_heads"] * HEAD, case["hidden"]), (layer, "o", case["hidden"], q),
                (layer, "gate_up", 2 * case["inter"], case["hidden"]), (layer, "down", case["hidden"], case["inter"])]
    if case["vocab"]:
        out.append((0, "head", case["vocab"], case["hidden"]))
    return out


def _lens(case):
    """Sequence lengths, spread over their logarithm; the longest is max_len.  The same for every seed, as the case's work is."""
    rng = random.Random(case["seqs"] * 1000003 + case["max_len"])
    lens = [min(case["max_len"], max(case["min_len"], _log_int(rng, case["min_len"], case["max_len"]))) for _ in range(case["seqs"])]
    lens[rng.randrange(len(lens))] = case["max_len"]
    return lens


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _half(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(torch.float16)


def _weights(g, n, k):
    """A weight matrix as a program has it after loading a 4-bit model: N(0, 0.02^2) weights, quantized in groups of 32 along K
    (scale max/7 as fp16; codes offset by 8; eight to a word, the first in the lowest bits)."""
    packed = torch.empty((n, k // 8), dtype=torch.int32, device="cuda")
    scales = torch.empty((n, k // 32), dtype=torch.float16, device="cuda")
    rows = max(1, (1 << 27) // k)
    for r in range(0, n, rows):
        w = torch.randn((min(rows, n - r), k // 32, 32), generator=g, device="cuda").mul_(0.02)
        s = (w.abs().amax(-1) / 7.0).to(torch.float16)
        scales[r:r + rows] = s
        q = w.div_(s.float().unsqueeze(-1)).round_().add_(8.0).clamp_(0.0, 15.0).to(torch.uint8).view(w.shape[0], k // 2, 2)
        packed[r:r + rows] = (q[:, :, 0] | (q[:, :, 1] << 4)).view(torch.int32)
    return packed, scales


def _dequant(packed, scales):
    b = packed.view(torch.uint8)
    q = torch.stack((b & 15, b >> 4), dim=-1).view(b.shape[0], -1, 32).to(torch.float64).sub_(8.0)
    return q.mul_(scales.double().unsqueeze(-1)).view(b.shape[0], -1)


def _exact_linear(packed, scales, x):
    """x [M, K] (64 bits) times the dequantized matrix, in blocks of rows."""
    n = packed.shape[0]
    y = torch.empty((x.shape[0], n), dtype=torch.float64, device="cuda")
    rows = max(1, (1 << 26) // x.shape[1])
    for r in range(0, n, rows):
        y[:, r:r + rows] = x @ _dequant(packed[r:r + rows], scales[r:r + rows]).t()
    return y


def _inputs(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "linear":
        p, s = _weights(g, case["n"], case["k"])
        return dict(packed=p, scales=s, x=_half(g, case["m"], case["k"]))
    if kind == "step":
        return dict(weights=[_weights(g, n, k) for _, _, n, k in _linears(case)],
                    x=[_half(g, case["m"], k) for _, _, _, k in _linears(case)])
    if kind == "chain":
        norm = lambda: torch.rand(case["hidden"], generator=g, device="cuda").add_(0.5).to(torch.float16)  # noqa: E731
        return dict(weights=[_weights(g, n, k) for _, _, n, k in _linears(case)], embedded=_half(g, case["hidden"]),
                    norms=[norm() for _ in range(2 * case["layers"] + 1)])
    if kind == "attn":
        lens = _lens(case)
        need = [-(-n // case["page"]) for n in lens]
        pages = sum(need)
        # Pages in a random order, as in a cache that has served and freed many sequences; -1 past a sequence's last page.
        order = torch.randperm(pages, generator=g, device="cuda").to(torch.int32)
        table = torch.full((len(lens), max(need)), -1, dtype=torch.int32, device="cuda")
        at = 0
        for i, n in enumerate(need):
            table[i, :n] = order[at:at + n]
            at += n
        shape = (pages, case["kv_heads"], case["page"], HEAD)
        return dict(q=_half(g, len(lens), case["q_heads"], HEAD), k=_half(g, *shape), v=_half(g, *shape), table=table,
                    lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), lens_host=lens)
    return dict(w=torch.randn((case["n"], case["k"]), generator=g, device="cuda").mul_(0.02))


# ---------------------------------------------------------- prepare and run


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    d["kind"] = kind
    half = dict(dtype=torch.float16, device="cuda")
    if kind == "linear":
        d["y"] = torch.empty((case["m"], case["n"]), **half)
    elif kind == "step":
        d["y"] = {}
        sizes = {name: n for _, name, n, _ in _linears(case)}
        for name, n in sizes.items():
            d["y"][name] = torch.empty((1 if name == "head" else case["layers"], case["m"], n), **half)
        d["m"] = case["m"]
        d["linears"] = [(p, s, x, d["y"][name][layer])
                        for (layer, name, _, _), (p, s), x in zip(_linears(case), d["weights"], d["x"])]
        d["array"] = wq.make_linear_array(d["linears"], case["m"])  # descriptors are marshalled once, as a server does
    elif kind == "chain":
        layers, hid, q = case["layers"], case["hidden"], case["q_heads"] * HEAD
        d["qkv"] = torch.empty((layers, q + 2 * case["kv_heads"] * HEAD), **half)
        d["gate_up"] = torch.empty(2 * case["inter"], **half)
        d["stream"] = torch.empty((2 * layers, hid), **half)  # the residual stream after each half of a layer
        d["logits"] = torch.empty(case["vocab"], **half)
        d["token"] = torch.empty(1, dtype=torch.int32, device="cuda")
        d["linears"] = []
        h = d["embedded"]
        for (layer, name, _, _), (p, s) in zip(_linears(case), d["weights"]):
            one = dict(packed_w=p, scales=s, eps=EPS)
            if name == "qkv":
                one.update(x=h, y=d["qkv"][layer], prologue=wq.PROLOGUE_RMSNORM, norm_weight=d["norms"][2 * layer])
            elif name == "o":
                one.update(x=d["qkv"][layer][:q], y=d["stream"][2 * layer], residual=h)
                h = d["stream"][2 * layer]
            elif name == "gate_up":
                one.update(x=h, y=d["gate_up"], prologue=wq.PROLOGUE_RMSNORM, norm_weight=d["norms"][2 * layer + 1])
            elif name == "down":
                one.update(x=d["gate_up"], y=d["stream"][2 * layer + 1], prologue=wq.PROLOGUE_SILU_MUL, residual=h)
                h = d["stream"][2 * layer + 1]
            else:
                one.update(x=h, y=d["logits"], prologue=wq.PROLOGUE_RMSNORM, norm_weight=d["norms"][-1])
            d["linears"].append(one)
        d["array"] = wq.make_fused_array(d["linears"])
    elif kind == "attn":
        d["max_len"] = max(d["lens_host"])
        d["scale"] = 1.0 / math.sqrt(HEAD)
        d["out"] = torch.empty_like(d["q"])
        d["workspace"] = wq.paged_workspace(d["q"], d["max_len"], case["kv_heads"])  # one per server, kept
    else:
        d["packed"] = torch.empty((case["n"], case["k"] // 8), dtype=torch.int32, device="cuda")
        d["scales"] = torch.empty((case["n"], case["k"] // 32), **half)
    return d


def run(d):
    kind = d["kind"]
    if kind == "linear":
        wq.wq_gemv(d["packed"], d["scales"], d["x"], d["y"])
        return d["y"]
    if kind == "step":
        wq.wq_decode_linears(d["linears"], m=d["m"], _array=d["array"])
        return d["y"]
    if kind == "chain":
        # The token itself is not compared: it is the place of the largest logit, and two logits can lie one rounding apart.
        wq.wq_fused_linears(d["linears"], argmax=d["token"], _array=d["array"])
        return dict(logits=d["logits"], stream=d["stream"], qkv=d["qkv"])
    if kind == "attn":
        wq.paged_attention(d["q"], d["k"], d["v"], d["table"], d["lens"], d["out"], d["scale"], d["max_len"],
                           workspace=d["workspace"])
        return d["out"]
    wq.wq_pack(d["w"], d["packed"], d["scales"])
    return dict(packed=d["packed"], scales=d["scales"])


# ------------------------------------------------------- work and tolerance


def work(case):
    kind = case["kind"]
    if kind in ("step", "chain"):
        m = case.get("m", 1)
        shapes = [(n, k) for _, _, n, k in _linears(case)]
        return dict(bytes=sum(n * k // 2 + n * k // 16 + 2 * m * (n + k) for n, k in shapes),
                    flops=sum(2 * m * n * k for n, k in shapes))
    if kind == "attn":
        lens = _lens(case)
        tokens = sum(lens)
        pages = sum(-(-n // case["page"]) for n in lens)
        return dict(bytes=4 * tokens * case["kv_heads"] * HEAD + 4 * len(lens) * case["q_heads"] * HEAD + 4 * pages + 4 * len(lens),
                    flops=4 * tokens * case["q_heads"] * HEAD)
    n, k = case["n"], case["k"]
    if kind == "linear":
        m = case["m"]
        return dict(bytes=n * k // 2 + n * k // 16 + 2 * m * (n + k), flops=2 * m * n * k)
    return dict(bytes=4 * n * k + n * k // 2 + n * k // 16, flops=2 * n * k)


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return "exact"
    if kind == "chain":
        # Roundings of one layer travel through those that follow: 1.4e-3 to 2.7e-3 from the 64-bit result.
        return {"rel": 1e-2, "max": 6e-2}
    # fp16 results of 32-bit sums; from three rows of x on, each weight is rounded once to fp16 as well: 2.1e-4 to 2.8e-4 from the 64-bit result.
    return {"rel": 1.2e-3, "max": 6e-3}


# ----------------------------------------------------------------- 64 bits


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "linear":
        return _exact_linear(d["packed"], d["scales"], d["x"].double())
    if kind == "step":
        got = {}
        for (_, name, _, _), (p, s), x in zip(_linears(case), d["weights"], d["x"]):
            got.setdefault(name, []).append(_exact_linear(p, s, x.double()))
        return {name: torch.stack(v) for name, v in got.items()}
    if kind == "chain":
        norms = [t.double() for t in d["norms"]]
        rms = lambda h, w: (h / (h.square().mean() + EPS).sqrt() * w).unsqueeze(0)  # noqa: E731
        lin = lambda w, x: _exact_linear(w[0], w[1], x).squeeze(0)  # noqa: E731
        h, streams, qkvs, w = d["embedded"].double(), [], [], d["weights"]
        q = case["q_heads"] * HEAD
        for i in range(case["layers"]):
            qkvs.append(lin(w[4 * i], rms(h, norms[2 * i])))
            h = h + lin(w[4 * i + 1], qkvs[-1][:q].unsqueeze(0))
            streams.append(h)
            gate, up = lin(w[4 * i + 2], rms(h, norms[2 * i + 1])).chunk(2)
            h = h + lin(w[4 * i + 3], (gate * torch.sigmoid(gate) * up).unsqueeze(0))
            streams.append(h)
        return dict(logits=lin(w[-1], rms(h, norms[-1])), stream=torch.stack(streams), qkv=torch.stack(qkvs))
    if kind == "attn":
        kvh, group = case["kv_heads"], case["q_heads"] // case["kv_heads"]
        out = torch.empty(d["q"].shape, dtype=torch.float64, device="cuda")
        for i, n in enumerate(d["lens_host"]):
            pages = d["table"][i, :-(-n // case["page"])].long()
            k, v = (d[t][pages].transpose(0, 1).reshape(kvh, -1, HEAD)[:, :n].double() for t in ("k", "v"))
            q = d["q"][i].double().view(kvh, group, HEAD)
            for h in range(kvh):
                a = (q[h] @ k[h].t()) / math.sqrt(HEAD)
                out[i, h * group:(h + 1) * group] = torch.softmax(a, -1) @ v[h]
        return out
    amax = d["w"].view(case["n"], -1, 32).abs().amax(-1)
    return dict(packed=None, scales=amax.double() / 7.0)
