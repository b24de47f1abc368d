"""verify_attention where the items deal a KV head's tiles by the branches' lengths, on the device.  A build of the library that does so for
calls of any length, wherever lengths differ (liblotts_flat.so), runs small geometries against the CPU oracle; which plans they reach is
checked on the host (test_plans.py).  Long calls run in the library itself, which deals where that gains."""
import os

import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import DEV, attn_to_dev
from test_gpu_no_patience import lotts as no_polls  # noqa: F401  (a fixture)
from test_gpu_parity import BF, run_attention

pytestmark = pytest.mark.gpu
NAMES = ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")

CASES = [
    # branches with several items each (merge workgroups): one row tile and two, both head dims, a prefix and none
    BF.with_(B=20, Hq=32, Hkv=8, k=5, P=30, L=400), BF.with_(B=17, Hq=40, Hkv=8, k=8, P=60, L=500), BF.with_(B=12, Hq=80, Hkv=16, k=6, D=64, P=31, L=333),
    BF.with_(B=9, Hq=16, Hkv=2, k=1, D=64, P=100, L=900),
    BF.with_(B=2, Hq=2, Hkv=1, k=1, D=64, P=0, L=9000),     # up to 512 items for two branches: partials beyond a wavefront's lanes
    BF.with_(B=33, Hq=9, Hkv=3, k=2, D=64, P=0, L=700),     # heads that do not divide the units
    # several items each, few bytes of partials in fixed shares: one share a branch, and more
    BF.with_(B=20, Hq=32, Hkv=8, k=3, P=30, L=400), BF.with_(B=12, Hq=16, Hkv=16, k=2, D=64, P=22, L=700), BF.with_(B=10, Hq=32, Hkv=8, k=0, P=11, L=900),
    # items with several branches each (the last arriver)
    BF.with_(B=40, Hq=8, Hkv=8, k=0, P=0, L=300), BF.with_(B=64, Hq=40, Hkv=8, k=7, P=33, L=260),
    BF.with_(B=35, Hq=16, Hkv=16, k=2, D=64, P=40, L=200), BF.with_(B=34, Hq=80, Hkv=16, k=7, D=64, P=0, L=130),
    BF.with_(B=18, Hq=16, Hkv=16, k=0, D=64, P=20, L=230),  # a few more items of whole rows than units
]
# those where equal lengths are not dealt; the last ones have two shares, which the later of two items merges
SHARED = [c for i, c in enumerate(CASES) if i not in (5, 13)] + [BF.with_(B=14, Hq=32, Hkv=8, k=1, D=64, P=0, L=900),
                                                                 BF.with_(B=12, Hq=32, Hkv=8, k=5, P=30, L=900)]
# merge workgroups and the last arriver, one row tile and two; lengths uneven enough to be dealt
LONG = [BF.with_(B=64, Hq=16, Hkv=2, k=3, P=70, L=4608), BF.with_(B=40, Hq=16, Hkv=2, k=4, P=0, L=7400),
        BF.with_(B=40, Hq=32, Hkv=8, k=3, P=0, L=2000), BF.with_(B=33, Hq=72, Hkv=8, k=3, P=0, L=2300),
        BF.with_(B=30, Hq=2, Hkv=2, k=1, P=58, L=10030)]
LONG_IDS = ["groups", "groups_two_row_tiles", "last_arriver", "last_arriver_two_row_tiles", "groups_few_bytes"]


def lengths(cfg, pattern):
    lo, B = cfg.k + 1, cfg.B
    if pattern == "equal":
        return np.full(B, cfg.L, np.int32)
    if pattern == "ragged":
        return np.linspace(lo, cfg.L, B).astype(np.int32)
    if pattern == "shuffled":
        return np.random.default_rng(B).permutation(np.linspace(lo, cfg.L, B)).astype(np.int32)
    if pattern == "uneven":
        return np.random.default_rng(B).permutation(lo + (cfg.L - lo) * np.linspace(0, 1, B) ** 6).astype(np.int32)
    out = np.full(B, lo, np.int32)  # all but one hold the new tokens only, or all but one token more
    out[{"first": 0, "last": B - 1, "one": B // 2, "none": B // 3}[pattern]] = cfg.L if pattern != "none" else lo + 1
    return out


@pytest.fixture
def flat():
    """The package on top of that build, with workspaces of its own, for one test: the others are about the library itself."""
    import paper_2505_19634_amd as m
    from paper_2505_19634_amd import binding
    usual, workspaces = m.load(), binding._workspaces
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(binding, "LIB_PATH", os.path.join(os.path.dirname(binding.LIB_PATH), "liblotts_flat.so"))
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_workspaces", {})
        mp.setattr(binding, "_sized", {})
        assert m.load() is not usual
        yield m
        torch.cuda.synchronize()
    assert m.load() is usual and binding._workspaces is workspaces


def without_dealing(m, d):
    """(O, lse) of the library itself, whose plan for a short call has fixed shares."""
    from paper_2505_19634_amd import binding
    torch.cuda.synchronize()
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(binding, "LIB_PATH", os.path.join(os.path.dirname(binding.LIB_PATH), "liblotts.so"))
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_workspaces", {})
        mp.setattr(binding, "_sized", {})
        out = m.verify_attention(*(d[n] for n in NAMES), return_lse=True)
        torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "B%d_k%d_Hq%d_Hkv%d_D%d_P%d_L%d" % (c.B, c.k, c.Hq, c.Hkv, c.D, c.P, c.L))
@pytest.mark.parametrize("pattern", ["equal", "ragged", "shuffled", "first", "last", "one", "none"])
def test_lengths(flat, oracle, cfg, pattern):
    run_attention(flat, oracle, cfg, priv_len=lengths(cfg, pattern))


@pytest.mark.parametrize("cfg", SHARED, ids=lambda c: "B%d_k%d_Hq%d_Hkv%d_D%d_P%d_L%d" % (c.B, c.k, c.Hq, c.Hkv, c.D, c.P, c.L))
@pytest.mark.parametrize("share", [1.0, 0.6])
def test_equal_lengths_have_the_bits_of_fixed_shares(flat, cfg, share):
    """Nothing is dealt where all lengths are alike: the shares and the merge of the plan without them, as the library itself takes it for calls
    this short."""
    d = attn_to_dev(cfg, S.attention_inputs(cfg, priv_len=np.full(cfg.B, max(cfg.k + 1, int(cfg.L * share)), np.int32)))
    got = [t.clone() for t in flat.verify_attention(*(d[n] for n in NAMES), return_lse=True)]
    want = without_dealing(flat, d)
    assert all(torch.equal(g, w) for g, w in zip(got, want))


@pytest.mark.parametrize("cfg", [CASES[0], CASES[1], CASES[6], CASES[9]], ids=["groups", "two_row_tiles", "few_bytes", "last_arriver"])
def test_replays_with_other_lengths(flat, cfg):
    """What a captured call deals follows the lengths it finds, and every cell is down again when it ends."""
    sets = [attn_to_dev(cfg, S.attention_inputs(cfg, salt=i, priv_len=lengths(cfg, p))) for i, p in enumerate(("equal", "shuffled", "one"))]
    want = [flat.verify_attention(*(d[n] for n in NAMES)).clone() for d in sets]
    buf = {n: sets[0][n].clone() for n in NAMES}
    out = torch.empty_like(buf["Q"])
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device=DEV)
    call = lambda: flat.verify_attention(*(buf[n] for n in NAMES), out=out, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (1, 2, 0, 1):
        for n in NAMES:
            buf[n].copy_(sets[i][n])
        for again in (graph.replay, call, graph.replay):
            out.zero_()
            again()
            torch.cuda.synchronize()
            assert torch.equal(out, want[i]), i
            assert int(ws[:131072].to(torch.int32).sum()) == 0


@pytest.mark.parametrize("cfg", [CASES[0], CASES[1], CASES[3]], ids=["D128", "two_row_tiles", "D64"])
def test_strided_operands(flat, cfg):
    """Caches [B][L][Hkv][D], padded prefix rows, Q as columns of a wider projection: the same result, bit for bit."""
    d = attn_to_dev(cfg, S.attention_inputs(cfg, priv_len=lengths(cfg, "shuffled")))
    want = flat.verify_attention(*(d[n] for n in NAMES)).clone()
    for n in ("Kpriv", "Vpriv"):
        d[n] = d[n].transpose(1, 2).contiguous().transpose(1, 2)
    for n in ("Kpre", "Vpre"):
        wide = torch.full((cfg.Hkv, cfg.P, cfg.D + 24), float("nan"), dtype=torch.bfloat16, device=DEV)
        wide[..., :cfg.D].copy_(d[n])
        d[n] = wide[..., :cfg.D]
    wide = torch.full((cfg.B, cfg.k + 1, cfg.Hq + 3, cfg.D), float("nan"), dtype=torch.bfloat16, device=DEV)
    wide[:, :, :cfg.Hq].copy_(d["Q"])
    d["Q"] = wide[:, :, :cfg.Hq]
    assert torch.equal(flat.verify_attention(*(d[n] for n in NAMES)), want)


def test_rows_behind_the_lengths_do_not_count(flat):
    """NaN in every cache row at or beyond a branch's length: those rows are read as zeros or not at all."""
    cfg = CASES[0]
    d = attn_to_dev(cfg, S.attention_inputs(cfg, priv_len=lengths(cfg, "shuffled")))
    want = flat.verify_attention(*(d[n] for n in NAMES)).clone()
    for b, L in enumerate(d["priv_len"].tolist()):
        for n in ("Kpriv", "Vpriv"):
            d[n][b, :, L:] = float("nan")
    assert torch.equal(flat.verify_attention(*(d[n] for n in NAMES)), want)


def test_calls_side_by_side(flat):
    cfgs = [CASES[0], CASES[1], CASES[6]]
    sets = [attn_to_dev(c, S.attention_inputs(c, priv_len=lengths(c, "shuffled"))) for c in cfgs]
    for d, c in zip(sets, cfgs):
        if c.P == 0:
            d["Kpre"] = d["Vpre"] = None
    want = [flat.verify_attention(*(d[n] for n in NAMES)).clone() for d in sets]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    got = [[flat.verify_attention(*(d[n] for n in NAMES), stream=s) for d, s in zip(sets, streams)] for _ in range(20)]
    torch.cuda.synchronize()
    for round_ in got:
        assert all(torch.equal(o, w) for o, w in zip(round_, want))


@pytest.fixture
def itself():
    """The package on top of the library itself, whatever other fixtures are alive."""
    import paper_2505_19634_amd as m
    assert os.path.basename(m.load()._name) == "liblotts.so"
    return m


def long_inputs(cfg):
    g = torch.Generator(device=DEV)
    g.manual_seed(cfg.B)
    t = lambda *shape: (torch.randn(shape, generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    d = {"Q": t(cfg.B, cfg.k + 1, cfg.Hq, cfg.D), "Kpriv": t(cfg.B, cfg.Hkv, cfg.L, cfg.D), "Vpriv": t(cfg.B, cfg.Hkv, cfg.L, cfg.D)}
    for n in ("Kpre", "Vpre"):
        d[n] = t(cfg.Hkv, cfg.P, cfg.D) if cfg.P else None
    d["priv_len"] = torch.from_numpy(lengths(cfg, "uneven")).to(DEV)
    return d


def fixed_shares(m, d):
    """(O, lse) of a call whose workspace holds the partials of fixed shares and not those of dealt tiles."""
    import ctypes
    O, lse = torch.empty_like(d["Q"]), torch.empty(d["Q"].shape[:3], dtype=torch.float32, device=DEV)
    lib, desc = m.load(), m.make_attn_desc(d["Q"], d["Kpre"], d["Kpriv"], O)
    ws = torch.zeros(lib.verify_attention_workspace_bytes(ctypes.byref(desc)) - 256, dtype=torch.uint8, device=DEV)
    m.verify_attention(*(d[n] for n in NAMES), out=O, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    return O, lse


@pytest.mark.parametrize("cfg", [BF.with_(B=14, Hq=32, Hkv=8, k=1, D=64, P=0, L=12491), BF.with_(B=7, Hq=16, Hkv=16, k=7, D=64, P=0, L=15408)],
                         ids=["14x8", "7x16"])
@pytest.mark.parametrize("shortest,dealt", [(1, False), (7 / 8, False), (1 / 2, True), (1 / 16, True)])
def test_nearly_equal_lengths_are_not_dealt(itself, cfg, shortest, dealt):
    """Two shares a branch and most of the units with one item fill the memory already: 14 x 8 heads x 12491 tokens down to 10930 51.5 us in fixed
    shares, dealt 54.5.  What was dealt shows in the low bits."""
    d = long_inputs(cfg)
    d["priv_len"] = torch.from_numpy(np.linspace(cfg.L * shortest, cfg.L, cfg.B).astype(np.int32)).to(DEV)
    got = [t.clone() for t in itself.verify_attention(*(d[n] for n in NAMES), return_lse=True)]
    want = fixed_shares(itself, d)
    assert all(torch.equal(g, w) for g, w in zip(got, want)) != dealt
    assert torch.allclose(got[1], want[1], rtol=0, atol=1e-4)


def test_a_workspace_for_more_branches_serves_fewer(itself):
    """128 branches ask for fewer bytes than 64, whose tiles are dealt by their lengths; the 64 then take fixed shares."""
    import ctypes
    d = long_inputs(LONG[0])
    want, lse = (t.clone() for t in itself.verify_attention(*(d[n] for n in NAMES), return_lse=True))
    desc = itself.make_attn_desc(d["Q"], d["Kpre"], d["Kpriv"], want)
    need = lambda: itself.load().verify_attention_workspace_bytes(ctypes.byref(desc))
    most = need()
    desc.B = 128
    fewer = need()
    assert 0 < fewer < most
    guard = torch.zeros(most, dtype=torch.uint8, device=DEV)
    guard[fewer:] = 7
    for _ in range(2):
        O, got = itself.verify_attention(*(d[n] for n in NAMES), return_lse=True, workspace=guard[:fewer])
        torch.cuda.synchronize()
        assert torch.allclose(got, lse, rtol=0, atol=1e-4) and ((O - want).float().norm() / want.float().norm()).item() <= 8e-3
        assert bool((guard[fewer:] == 7).all())


@pytest.mark.parametrize("cfg", LONG, ids=LONG_IDS)
def test_long_calls(itself, cfg):
    """The library itself, against plain fp32 attention of some branches; the lengths are dealt."""
    d = long_inputs(cfg)
    O, lse = (t.clone() for t in itself.verify_attention(*(d[n] for n in NAMES), return_lse=True))
    assert not torch.equal(lse, fixed_shares(itself, d)[1])
    G = cfg.Hq // cfg.Hkv
    for b in range(0, cfg.B, 7):
        L = int(d["priv_len"][b])
        K, V = (torch.cat(([d[p].float()] if cfg.P else []) + [d[n][b, :, :L].float()], 1) for p, n in (("Kpre", "Kpriv"), ("Vpre", "Vpriv")))
        for r in range(cfg.k + 1):
            q = d["Q"][b, r].float().view(cfg.Hkv, G, cfg.D)
            n = cfg.P + L - cfg.k + r
            z = torch.matmul(q, K[:, :n].transpose(1, 2).contiguous()) / cfg.D ** 0.5
            ref = torch.matmul(torch.softmax(z, -1), V[:, :n]).view(cfg.Hq, cfg.D)
            err = ((O[b, r].float() - ref).norm() / ref.norm()).item()
            assert err <= 8e-3, (b, r, err)  # one row of few: twice the band of whole outputs (4e-3)


@pytest.mark.parametrize("cfg", LONG, ids=LONG_IDS)
def test_long_calls_without_patience(no_polls, cfg):  # noqa: F811
    """Merge workgroups that leave at once: the items merge in their place, in the same order."""
    from paper_2505_19634_amd import binding
    d = long_inputs(cfg)
    got = [no_polls.verify_attention(*(d[n] for n in NAMES)).clone() for _ in range(3)]
    torch.cuda.synchronize()
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(binding, "LIB_PATH", os.path.join(os.path.dirname(binding.LIB_PATH), "liblotts.so"))
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_workspaces", {})
        want = no_polls.verify_attention(*(d[n] for n in NAMES))
        torch.cuda.synchronize()
    assert all(torch.equal(o, want) for o in got)
