"""Performance cases of the verification step: what a serving program has this library do, by size and kind.

`listed()` names the cases, `draw()` gives further ones of the same ranges, `prepare()` makes what a program holds before a
call, `run()` is one pass through the public entry points, `work()` the traffic and operations it cannot do without,
`tolerance()` how far another correct implementation may be, `exact()` the same outputs in 64 bits by plain torch.

Kinds:
  attention   verify_attention of one layer, called directly (layers = 1), or of several layers with caches of their own,
              captured once in a HIP graph and replayed, as a decoder's step is
  accept      spec_accept on soft-maxed target and draft rows
  logits      spec_accept_logits on target and draft logits
  gemm        the four weight GEMMs of a decoder layer (QKV, O, gate+up, down) for one step's tokens
  step        verify_attention + spec_accept + majority_vote, the unit of the repository's benchmark
  stack       one verify step of a whole decoder held by latency_model.FullModel, replayed from a HIP graph
"""
import math

import torch

import paper_2505_19634_amd as lotts
from paper_2505_19634_amd import latency_model

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: one step of two short branches in fp32; launches and host calls are all there is to it
        {"name": "step_tiny_f32", "kind": "step", "B": 2, "k": 3, "Hq": 4, "Hkv": 4, "D": 64, "P": 32, "Lmax": 64,
         "ragged": False, "fused_q": False, "dtype": "f32", "V": 1000},
        # the benchmark's step: 16 branches of a 32B-shaped target, 3 drafts, 256 + 3840 tokens of context
        {"name": "step_32b_b16", "kind": "step", "B": 16, "k": 3, "Hq": 40, "Hkv": 8, "D": 128, "P": 256, "Lmax": 3840,
         "ragged": False, "fused_q": False, "dtype": "bf16", "V": 152064},
        # a single branch with drafts (no branch-wise parallelism), 3B-shaped: the attention of all 36 layers of a step
        {"name": "attn_3b_b1_layers", "kind": "attention", "B": 1, "k": 2, "Hq": 16, "Hkv": 2, "D": 128, "P": 1024,
         "Lmax": 7168, "ragged": False, "fused_q": True, "dtype": "bf16", "layers": 36},
        # 8 branches in mid generation, 3B-shaped, 4 drafts: one layer called directly
        {"name": "attn_3b_b8", "kind": "attention", "B": 8, "k": 4, "Hq": 16, "Hkv": 2, "D": 128, "P": 512,
         "Lmax": 2048, "ragged": False, "fused_q": True, "dtype": "bf16", "layers": 1},
        # few branches, long generations, long drafts, 32B-shaped
        {"name": "attn_32b_long", "kind": "attention", "B": 4, "k": 8, "Hq": 40, "Hkv": 8, "D": 128, "P": 512,
         "Lmax": 15872, "ragged": False, "fused_q": False, "dtype": "bf16", "layers": 1},
        # the widest branch sweep point, branches of different lengths, odd prefix: ragged tails everywhere
        {"name": "attn_3b_b64_ragged", "kind": "attention", "B": 64, "k": 2, "Hq": 16, "Hkv": 2, "D": 128, "P": 1003,
         "Lmax": 7168, "ragged": True, "fused_q": True, "dtype": "bf16", "layers": 1},
        # acceptance of 8 branches x 4 drafts on soft-maxed rows of a 3B-shaped vocabulary
        {"name": "accept_3b_b8", "kind": "accept", "B": 8, "k": 4, "V": 151936},
        # acceptance straight from the LM head's bf16 logits, 16 branches x 3 drafts, sampling temperature 0.7
        {"name": "logits_32b_b16", "kind": "logits", "B": 16, "k": 3, "V": 152064, "dtype": "bf16", "inv_temperature": 1.0 / 0.7},
        # fp32 logits of a vocabulary that is no multiple of anything, long drafts
        {"name": "logits_odd_f32", "kind": "logits", "B": 5, "k": 7, "V": 50257, "dtype": "f32", "inv_temperature": 1.0},
        # weight GEMMs of one 32B-shaped layer for the benchmark step's 64 tokens
        {"name": "gemm_32b_m64", "kind": "gemm", "M": 64, "hidden": 5120, "qkv": 7168, "attn": 5120, "mlp": 27648},
        # weight GEMMs of one 3B-shaped layer for the 64-branch sweep point's 192 tokens
        {"name": "gemm_3b_m192", "kind": "gemm", "M": 192, "hidden": 2048, "qkv": 2560, "attn": 2048, "mlp": 11008},
        # a whole verify step of a 3B-shaped decoder, every layer resident: 8 branches x (4 drafts + 1)
        {"name": "stack_3b_b8", "kind": "stack", "layers": 36, "hidden": 2048, "Hq": 16, "Hkv": 2, "D": 128, "mlp": 11008,
         "V": 151936, "P": 512, "private": 2044, "B": 8, "k": 4},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


HEADS = [(16, 2, 128), (40, 8, 128), (32, 8, 128), (28, 4, 128), (16, 16, 64), (32, 8, 64)]


def _draw_attention(rng):
    Hq, Hkv, D = rng.choice(HEADS)
    B, Lmax, P = _log(rng, 1, 64), _log(rng, 300, 16384), rng.choice([0, _log(rng, 17, 1100), _log(rng, 17, 1100), _log(rng, 500, 4096)])
    k = rng.randint(0, 8)
    while 4 * Hkv * D * (P + B * Lmax) > 480e6:  # at most the widest sweep point's caches
        if B > 4:
            B = B // 2
        else:
            Lmax = Lmax // 2
    return {"B": B, "k": k, "Hq": Hq, "Hkv": Hkv, "D": D, "P": P, "Lmax": Lmax, "ragged": rng.random() < 0.6,
            "fused_q": rng.random() < 0.5, "dtype": "bf16"}


def draw(rng):
    kind = rng.choice(["attention"] * 5 + ["accept"] + ["logits"] * 2 + ["gemm"] * 3 + ["step"] * 2 + ["stack"])
    if kind == "attention":
        c = _draw_attention(rng)
        kv = 4 * c["Hkv"] * c["D"] * (c["P"] + c["B"] * c["Lmax"])
        c["layers"] = rng.choice([1, 1, _log(rng, 4, 36)]) if kv < 20e6 else 1
        return dict(c, kind=kind)
    if kind == "step":
        if rng.random() < 0.4:
            Hq, Hkv, D = rng.choice([(4, 4, 64), (8, 2, 64), (4, 2, 128)])
            return {"kind": kind, "B": rng.randint(1, 8), "k": rng.randint(0, 6), "Hq": Hq, "Hkv": Hkv, "D": D, "P": rng.randint(0, 100),
                    "Lmax": rng.randint(20, 200), "ragged": True, "fused_q": False, "dtype": "f32", "V": rng.randint(500, 5000)}
        c = _draw_attention(rng)
        c["B"] = min(c["B"], 32)
        return dict(c, kind=kind, V=rng.choice([151936, 152064, _log(rng, 30000, 160000)]))
    if kind == "accept":
        return {"kind": kind, "B": _log(rng, 1, 32), "k": rng.randint(0, 8), "V": rng.choice([151936, 152064, 4 * _log(rng, 8000, 40000), _log(rng, 30000, 160000)])}
    if kind == "logits":
        return {"kind": kind, "B": _log(rng, 1, 32), "k": rng.randint(0, 8), "V": rng.choice([151936, 152064, 8 * _log(rng, 4000, 20000), _log(rng, 30000, 160000)]),
                "dtype": rng.choice(["bf16", "bf16", "f32"]), "inv_temperature": rng.choice([1.0, 1.0 / 0.7, 1.25, round(rng.uniform(0.5, 2.0), 3)])}
    if kind == "gemm":
        hidden = 128 * _log(rng, 8, 48)
        return {"kind": kind, "M": _log(rng, 1, 256), "hidden": hidden, "qkv": hidden + 128 * rng.randint(1, 20),
                "attn": 128 * _log(rng, 8, 48), "mlp": 128 * _log(rng, 24, 216)}
    Hq, Hkv, D = rng.choice([(16, 2, 128), (40, 8, 128), (32, 8, 64)])
    B = _log(rng, 1, 32)
    return {"kind": "stack", "layers": rng.randint(2, 4), "hidden": 128 * _log(rng, 8, 40), "Hq": Hq, "Hkv": Hkv, "D": D, "mlp": 128 * _log(rng, 24, 160),
            "V": rng.choice([151936, 8 * _log(rng, 4000, 20000)]), "P": rng.randint(17, 800), "private": _log(rng, 300, 3000), "B": B,
            "k": rng.randint(0, min(7, 256 // B - 1))}


# ------------------------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype):
    return (torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * std).to(dtype)


def _lengths(g, c):
    """Private tokens per branch, the new ones included: the whole cache, or branches at different points of it."""
    B, R, Lmax = c["B"], c["k"] + 1, c["Lmax"]
    if not c["ragged"]:
        return torch.full((B,), Lmax, dtype=torch.int32, device=DEV)
    lo = max(R, Lmax // 4)
    return torch.randint(lo, Lmax + 1, (B,), generator=g, device=DEV).to(torch.int32)


def _attention_inputs(g, c):
    """One layer: Q (a view of a QKV projection's output if fused_q), prefix and private caches.  Standard deviation
    0.5 (1 for the tiny fp32 case), as in the repository's benchmark."""
    dt, R = DTYPES[c["dtype"]], c["k"] + 1
    std = 0.5 if c["dtype"] == "bf16" else 1.0
    heads = c["Hq"] + (2 * c["Hkv"] if c["fused_q"] else 0)
    s = {"Q": _normal(g, (c["B"], R, heads, c["D"]), std, dt)[:, :, :c["Hq"]]}
    for n in ("Kpre", "Vpre"):
        s[n] = _normal(g, (c["Hkv"], c["P"], c["D"]), std, dt) if c["P"] else None
    for n in ("Kpriv", "Vpriv"):
        s[n] = _normal(g, (c["B"], c["Hkv"], c["Lmax"], c["D"]), std, dt)
    return s


def _attention_outputs(c, layers):
    """Output buffers of all layers, one block each; the layers get their slices."""
    R = c["k"] + 1
    return (torch.empty((layers, c["B"], R, c["Hq"], c["D"]), dtype=DTYPES[c["dtype"]], device=DEV),
            torch.empty((layers, c["B"], R, c["Hq"]), dtype=torch.float32, device=DEV))


def _logit_pair(g, B, k, V):
    """Target logits N(0, 2) and draft logits that are the target's plus N(0, 0.5): acceptance rate about 0.8."""
    zt = torch.randn((B, k + 1, V), generator=g, device=DEV) * 2.0
    zd = zt[:, :k] + torch.randn((B, k, V), generator=g, device=DEV) * 0.5 if k else None
    return zt, zd


def _drafts(g, q):
    B, k, V = q.shape
    return torch.multinomial(q.reshape(B * k, V), 1, generator=g).view(B, k).to(torch.int32)


def _uniforms(g, B, R):
    return torch.randint(0, 1 << 24, (B, R), generator=g, device=DEV).float() / float(1 << 24)


def _accept_inputs(g, B, k, V):
    zt, zd = _logit_pair(g, B, k, V)
    s = {"p": torch.softmax(zt.double(), -1).float(), "q": None, "draft": None}
    if k:
        s["q"] = torch.softmax(zd.double(), -1).float()
        s["draft"] = _drafts(g, s["q"])
    s["u"] = _uniforms(g, B, k + 1)
    for n in ("accept_len", "next_token"):
        s[n] = torch.empty((B,), dtype=torch.int32, device=DEV)
    return s


def _attend(s, lengths):
    lotts.verify_attention(s["Q"], s["Kpre"], s["Vpre"], s["Kpriv"], s["Vpriv"], lengths, out=s["O"], lse=s["lse"])


def _capture(call):
    """The call captured once; the warm-up outside the capture creates whatever is made lazily."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    return graph


GEMMS = (("qkv", "qkv", "hidden"), ("o", "hidden", "attn"), ("gate_up", "2mlp", "hidden"), ("down", "hidden", "mlp"))


def _gemm_sizes(c):
    d = dict(c)
    d["2mlp"] = 2 * c["mlp"]
    return [(n, d[rows], d[cols]) for n, rows, cols in GEMMS]


def _stack(g, c):
    """A decoder whose values keep their size from layer to layer: the library has no norms, so the O weights undo the averaging
    over the keys; logits come out as N(0, 2)."""
    shape = latency_model.ModelShape("decoder", c["layers"], c["hidden"], c["Hq"], c["Hkv"], c["D"], c["mlp"], c["V"])
    fm = latency_model.FullModel(shape, c["P"], c["private"], c["B"], c["k"], device=DEV)
    fm.h.copy_(_normal(g, fm.h.shape, 0.5, torch.bfloat16))
    caches = [torch.empty((c["layers"],) + fm.layers[0]["Kpriv"].shape, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    for i, L in enumerate(fm.layers):
        L["Kpriv"], L["Vpriv"] = caches[0][i], caches[1][i]
        for n in ("Kpre", "Vpre", "Kpriv", "Vpriv"):
            L[n].copy_(_normal(g, L[n].shape, 0.5, torch.bfloat16))
        L["o"].mul_(math.sqrt(c["P"] + c["private"]))
    fm.lm_head.mul_(4.0)
    if c["k"]:
        fm.zd.copy_(_normal(g, fm.zd.shape, 2.0, torch.bfloat16))
        fm.draft.copy_(_drafts(g, torch.softmax(fm.zd.float(), -1)))
    fm.u.copy_(_uniforms(g, c["B"], c["k"] + 1))
    return fm, [t[:, :, :, c["private"]:] for t in caches]


def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "attention":
        s = {"kind": kind, "lengths": _lengths(g, c), "layers": [_attention_inputs(g, c) for _ in range(c["layers"])], "graph": None}
        s["O"], s["lse"] = _attention_outputs(c, c["layers"])
        for i, L in enumerate(s["layers"]):
            L["O"], L["lse"] = s["O"][i], s["lse"][i]
        if c["layers"] > 1:
            s["graph"] = _capture(lambda: [_attend(L, s["lengths"]) for L in s["layers"]])
        return s
    if kind == "accept":
        return dict(_accept_inputs(g, c["B"], c["k"], c["V"]), kind=kind)
    if kind == "logits":
        zt, zd = _logit_pair(g, c["B"], c["k"], c["V"])
        dt = DTYPES[c["dtype"]]
        s = {"kind": kind, "zt": zt.to(dt), "zd": zd.to(dt) if c["k"] else None, "inv_temperature": c["inv_temperature"]}
        s["draft"] = _drafts(g, torch.softmax(s["zd"].float() * c["inv_temperature"], -1)) if c["k"] else None
        s["u"] = _uniforms(g, c["B"], c["k"] + 1)
        for n in ("accept_len", "next_token"):
            s[n] = torch.empty((c["B"],), dtype=torch.int32, device=DEV)
        return s
    if kind == "gemm":
        s = {"kind": kind, "calls": []}
        for _, N, K in _gemm_sizes(c):
            X, W = _normal(g, (c["M"], K), 1.0, torch.bfloat16), _normal(g, (N, K), K ** -0.5, torch.bfloat16)
            s["calls"].append((X, W, torch.empty((c["M"], N), dtype=torch.bfloat16, device=DEV)))
        return s
    if kind == "step":
        s = {"kind": kind, "lengths": _lengths(g, c), "attn": _attention_inputs(g, c), "accept": _accept_inputs(g, c["B"], c["k"], c["V"])}
        pmf = torch.arange(1, 51, device=DEV, dtype=torch.float32) ** -1.5
        (O, lse) = _attention_outputs(c, 1)
        s["attn"]["O"], s["attn"]["lse"] = O[0], lse[0]
        s["answers"] = torch.multinomial(pmf.expand(1, 50), c["B"], replacement=True, generator=g).to(torch.int32)
        s["vote"] = [torch.empty((1,), dtype=torch.int32, device=DEV) for _ in range(2)]
        return s
    fm, new_rows = _stack(g, c)
    return {"kind": kind, "model": fm, "new_rows": new_rows, "graph": _capture(fm.enqueue)}


def _accept(s):
    lotts.spec_accept(s["p"], s["q"], s["draft"], s["u"], accept_len=s["accept_len"], next_token=s["next_token"])


def run(s):
    kind = s["kind"]
    if kind == "attention":
        if s["graph"] is None:
            _attend(s["layers"][0], s["lengths"])
        else:
            s["graph"].replay()
        return s["O"], s["lse"]
    if kind == "accept":
        _accept(s)
        return s["accept_len"], s["next_token"]
    if kind == "logits":
        return lotts.spec_accept_logits(s["zt"], s["zd"], s["draft"], s["u"], inv_temperature=s["inv_temperature"],
                                        accept_len=s["accept_len"], next_token=s["next_token"])
    if kind == "gemm":
        return [lotts.skinny_gemm(X, W, out=Y) for X, W, Y in s["calls"]]
    if kind == "step":
        _attend(s["attn"], s["lengths"])
        _accept(s["accept"])
        lotts.majority_vote(s["answers"], winner=s["vote"][0], winner_count=s["vote"][1])
        return s["attn"]["O"], s["attn"]["lse"], s["accept"]["accept_len"], s["accept"]["next_token"], s["vote"][0], s["vote"][1]
    s["graph"].replay()
    # logits, accepted lengths and what the caches gained; the sampled token is left out: one step of bf16 in a logit moves
    # it, whoever computes the logits
    return s["model"].zt, s["model"].accept_len, s["new_rows"]


# ------------------------------------------------------------------------------------------------------------------------
def _attention_work(c):
    es, R = (2 if c["dtype"] == "bf16" else 4), c["k"] + 1
    private = c["B"] * (c["Lmax"] * 5 / 8 if c["ragged"] else c["Lmax"])  # lengths are even from a quarter to the whole
    rows = c["B"] * R * c["Hq"]
    return {"bytes": 2 * c["Hkv"] * c["D"] * es * (c["P"] + private) + rows * (2 * c["D"] * es + 4),
            "flops": 4.0 * R * c["Hq"] * c["D"] * (c["B"] * c["P"] + private)}


def _accept_work(c, es):
    """On soft-maxed rows only what is sampled has to be read: about half of the branches stop at a draft (two rows)."""
    return {"bytes": c["B"] * (2 if c["k"] else 1) * c["V"] * es, "flops": 2.0 * c["B"] * (2 if c["k"] else 1) * c["V"]}


def work(case):
    c = case
    if c["kind"] == "attention":
        w = _attention_work(c)
        return {n: v * c["layers"] for n, v in w.items()}
    if c["kind"] == "accept":
        return _accept_work(c, 4)
    if c["kind"] == "logits":  # every row's normaliser is needed
        n = c["B"] * (2 * c["k"] + 1) * c["V"]
        return {"bytes": n * (2 if c["dtype"] == "bf16" else 4), "flops": 16.0 * n}
    if c["kind"] == "gemm":
        return {"bytes": sum(2.0 * (N * K + c["M"] * (N + K)) for _, N, K in _gemm_sizes(c)),
                "flops": sum(2.0 * c["M"] * N * K for _, N, K in _gemm_sizes(c))}
    if c["kind"] == "step":
        a, b = _attention_work(c), _accept_work(c, 4)
        return {n: a[n] + b[n] for n in a}
    M, h = c["B"] * (c["k"] + 1), c["hidden"]
    att = _attention_work(dict(c, Lmax=c["private"] + c["k"] + 1, ragged=False, dtype="bf16"))
    mats = [((c["Hq"] + 2 * c["Hkv"]) * c["D"], h), (h, c["Hq"] * c["D"]), (2 * c["mlp"], h), (h, c["mlp"])]
    logits = c["B"] * (2 * c["k"] + 1) * c["V"]
    params = c["layers"] * sum(n * k for n, k in mats) + c["V"] * h
    acts = c["layers"] * sum(M * (n + k) for n, k in mats) + M * (h + c["V"])
    return {"bytes": 2.0 * (params + acts) + c["layers"] * att["bytes"] + 2.0 * logits,
            "flops": 2.0 * M * params + c["layers"] * att["flops"] + 16.0 * logits}


def tolerance(case):
    c = case
    if c["kind"] in ("accept", "logits"):
        return "exact"  # integers by definition
    if c["kind"] == "gemm":
        return {"rel": 7e-3}  # bf16 results: 1.7e-3 from 64 bits
    if c["kind"] == "stack":
        return {"rel": 2e-2, "differ": 0.26}  # bf16 between all layers: 5e-3 from 64 bits; an accept test may tip
    return {"rel": 1e-2} if c["dtype"] == "bf16" else {"rel": 2e-6}  # bf16: 2.4e-3 from 64 bits; fp32: 2e-7


# ------------------------------------------------------------------------------------------------------------------------
def _exact_attention(c, s, lengths):
    """Softmax attention of one layer in 64 bits, branch by branch."""
    G, R, O, E = c["Hq"] // c["Hkv"], c["k"] + 1, [], []
    for b, L in enumerate(lengths.tolist()):
        K, V = s["Kpriv"][b, :, :L].double(), s["Vpriv"][b, :, :L].double()
        if c["P"]:
            K, V = torch.cat([s["Kpre"].double(), K], 1), torch.cat([s["Vpre"].double(), V], 1)
        q = s["Q"][b].double().view(R, c["Hkv"], G, c["D"]).permute(1, 0, 2, 3).reshape(c["Hkv"], R * G, c["D"])
        z = torch.matmul(q, K.transpose(1, 2).contiguous()) / math.sqrt(c["D"])
        row = torch.arange(R * G, device=DEV) // G
        key = torch.arange(c["P"] + L, device=DEV)
        z = z.masked_fill(key[None, None, :] >= (c["P"] + L - c["k"] + row)[None, :, None], -math.inf)
        lse = torch.logsumexp(z, -1)
        o = torch.matmul(torch.exp(z - lse[..., None]), V)
        O.append(o.view(c["Hkv"], R, G, c["D"]).permute(1, 0, 2, 3).reshape(R, c["Hq"], c["D"]))
        E.append(lse.view(c["Hkv"], R, G).permute(1, 0, 2).reshape(R, c["Hq"]))
    return torch.stack(O), torch.stack(E)


def _exact_stack(c, s):
    fm, R, M = s["model"], c["k"] + 1, c["B"] * (c["k"] + 1)
    lengths = torch.full((c["B"],), c["private"] + R, device=DEV)
    x, rows = fm.h.double(), []
    for L in fm.layers:
        heads = (x @ L["qkv"].double().t()).view(c["B"], R, c["Hq"] + 2 * c["Hkv"], c["D"])
        Kp, Vp = L["Kpriv"].double(), L["Vpriv"].double()
        Kp[:, :, c["private"]:] = heads[:, :, c["Hq"]:c["Hq"] + c["Hkv"]].transpose(1, 2)
        Vp[:, :, c["private"]:] = heads[:, :, c["Hq"] + c["Hkv"]:].transpose(1, 2)
        a, _ = _exact_attention(c, {"Q": heads[:, :, :c["Hq"]].contiguous(), "Kpre": L["Kpre"], "Vpre": L["Vpre"], "Kpriv": Kp, "Vpriv": Vp}, lengths)
        x = a.reshape(M, c["Hq"] * c["D"]) @ L["o"].double().t()
        x = (x @ L["gate_up"][:c["mlp"]].double().t()) @ L["down"].double().t()
        rows.append((Kp[:, :, c["private"]:].clone(), Vp[:, :, c["private"]:].clone()))
    return (x @ fm.lm_head.double().t()).view(c["B"], R, c["V"]), None, [torch.stack(t) for t in zip(*rows)]


def exact(case, seed):
    c, s = case, prepare(case, seed)
    if c["kind"] == "attention":
        return [torch.stack(t) for t in zip(*(_exact_attention(c, L, s["lengths"]) for L in s["layers"]))]
    if c["kind"] == "step":
        return _exact_attention(c, s["attn"], s["lengths"]) + (None, None, None, None)
    if c["kind"] == "gemm":
        return [X.double() @ W.double().t() for X, W, _ in s["calls"]]
    if c["kind"] == "stack":
        return _exact_stack(c, s)
    return None  # integers: compared as they are
