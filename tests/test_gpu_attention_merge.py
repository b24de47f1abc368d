"""verify_attention over the ways its partials meet: whole rows stored by one item, pairs, merge workgroups (one to eight rows each,
up to 64 key shares), a launch of its own.  Against the CPU oracle, and replayed from a captured graph."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import DEV, attn_to_dev
from test_gpu_parity import BF, run_attention

pytestmark = pytest.mark.gpu

CASES = [
    # one item per (KV head, branch): the output straight from it; also with two row tiles, several row groups, head_dim 64
    BF.with_(B=32, Hq=16, Hkv=8, k=3, P=40, L=170), BF.with_(B=33, Hq=16, Hkv=8, k=7, P=0, L=133),
    BF.with_(B=16, Hq=48, Hkv=16, k=23, P=0, L=70), BF.with_(B=64, Hq=16, Hkv=8, D=64, k=1, P=20, L=90),
    BF.with_(B=3, Hq=8, Hkv=2, k=1, P=0, L=32),                        # a single tile
    # pairs; a pair whose second share is empty for the short branches
    BF.with_(B=16, Hq=16, Hkv=8, k=3, P=33, L=300), BF.with_(B=1, Hq=4, Hkv=4, D=64, k=2, P=0, L=200),
    # merge workgroups: 1, 2, 4 and 8 rows each; one and two row tiles; odd shares; the most shares
    BF.with_(B=1, Hq=16, Hkv=2, k=2, P=1024, L=7168), BF.with_(B=5, Hq=5, Hkv=1, k=0, P=7, L=5000),
    BF.with_(B=8, Hq=16, Hkv=2, k=4, P=512, L=2048), BF.with_(B=12, Hq=40, Hkv=8, k=3, P=100, L=900),
    BF.with_(B=4, Hq=40, Hkv=8, k=8, P=64, L=1500), BF.with_(B=11, Hq=16, Hkv=4, D=64, k=6, P=65, L=1000),
    BF.with_(B=12, Hq=16, Hkv=8, D=64, k=2, P=50, L=2100), BF.with_(B=7, Hq=8, Hkv=4, D=64, k=15, P=31, L=700),
    BF.with_(B=2, Hq=16, Hkv=2, k=7, P=60, L=9000),                    # as many cells as there are: two rows each instead of one
    BF.with_(B=1, Hq=8, Hkv=4, k=2, P=96, L=4000),                     # few pairs, up to 4096 tokens
    # the last arriver: three to eight partials of few bytes; prefix items of the smallest batches
    BF.with_(B=10, Hq=32, Hkv=8, D=64, k=2, P=95, L=510), BF.with_(B=7, Hq=32, Hkv=8, k=1, P=84, L=562),
    BF.with_(B=5, Hq=16, Hkv=16, D=64, k=0, P=195, L=2021), BF.with_(B=15, Hq=16, Hkv=2, k=0, P=336, L=6487),
    BF.with_(B=4, Hq=16, Hkv=8, D=64, k=1, P=200, L=300), BF.with_(B=1, Hq=16, Hkv=8, k=4, P=300, L=900),
    # few branches and few tiles: one share, two
    BF.with_(B=5, Hq=16, Hkv=8, D=64, k=2, P=0, L=150), BF.with_(B=6, Hq=32, Hkv=8, D=64, k=3, P=51, L=256),
    # a launch of its own: prefix items; several row groups
    BF.with_(B=2, Hq=8, Hkv=1, k=8, P=0, L=539), BF.with_(B=24, Hq=32, Hkv=8, D=64, k=3, P=900, L=2000),
    BF.with_(B=37, Hq=4, Hkv=4, k=1, P=300, L=65), BF.with_(B=16, Hq=40, Hkv=8, k=3, P=1100, L=1500),
    BF.with_(B=2, Hq=16, Hkv=2, k=4, P=1000, L=3000),
    BF.with_(B=3, Hq=24, Hkv=2, k=7, P=100, L=1400),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "B%d_k%d_Hq%d_Hkv%d_D%d_P%d_L%d" % (c.B, c.k, c.Hq, c.Hkv, c.D, c.P, c.L))
@pytest.mark.parametrize("ragged", [False, True])
def test_every_merge(oracle, cfg, ragged):
    import paper_2505_19634_amd as lotts
    lens = None
    if ragged:  # the shortest branch holds the new tokens only
        lens = np.linspace(cfg.k + 1, cfg.L, cfg.B).astype(np.int32) if cfg.B > 1 else np.array([max(cfg.k + 1, cfg.L // 3)], np.int32)
    run_attention(lotts, oracle, cfg, priv_len=lens)


def test_merge_flags_are_cleared_for_a_replay(oracle):
    """A captured launch keeps its tag, so its flags have to be down again when it ends: replays on changing inputs, with eager
    calls of other geometries on the same workspace in between, equal the eager result."""
    import paper_2505_19634_amd as lotts
    cfg, other = BF.with_(B=8, Hq=16, Hkv=2, k=4, P=512, L=2048), BF.with_(B=1, Hq=16, Hkv=2, k=2, P=64, L=7000)
    sets = [attn_to_dev(cfg, S.attention_inputs(cfg, salt=i)) for i in range(3)]
    d2 = attn_to_dev(other, S.attention_inputs(other))
    names = ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")
    want = [lotts.verify_attention(*(d[n] for n in names)).clone() for d in sets]
    want2 = lotts.verify_attention(*(d2[n] for n in names)).clone()
    buf = {n: sets[0][n].clone() for n in names}
    out = torch.empty_like(buf["Q"])
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device=DEV)
    call = lambda: lotts.verify_attention(*(buf[n] for n in names), out=out, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (1, 2, 0, 1):
        for n in names:
            buf[n].copy_(sets[i][n])
        out.zero_()
        graph.replay()
        got2 = lotts.verify_attention(*(d2[n] for n in names), workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, want[i]), i
        assert torch.equal(got2, want2)
    assert int(ws[:131072].to(torch.int32).sum()) == 0  # every cell is down again


def test_merge_workgroups_side_by_side():
    """Calls on several streams overlap, and the merge workgroups of one may hold the places that the items of another need (with two
    row tiles a workgroup fills a compute unit): every call ends with the result it has alone."""
    import paper_2505_19634_amd as lotts
    cfgs = [BF.with_(B=8, Hq=16, Hkv=2, k=4, P=512, L=2048), BF.with_(B=4, Hq=40, Hkv=8, k=8, P=64, L=1500),
            BF.with_(B=1, Hq=16, Hkv=2, k=7, P=0, L=7000)]
    sets = [attn_to_dev(c, S.attention_inputs(c)) for c in cfgs]
    call = lambda d, **kw: lotts.verify_attention(*(d[n] for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")), **kw)
    sets[2]["Kpre"] = sets[2]["Vpre"] = None
    want = [call(d).clone() for d in sets]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    got = [[call(d, stream=s) for d, s in zip(sets, streams)] for _ in range(20)]
    torch.cuda.synchronize()
    for round_ in got:
        assert all(torch.equal(o, w) for o, w in zip(round_, want))


@pytest.mark.parametrize("D", [64, 128])
def test_fp32_keeps_nan_and_infinities(D):
    """NaN in all keys that a group of lanes sees in its first chunk stays NaN; an infinite value in the last row is that
    infinity, not NaN from the rows that stand in for absent keys."""
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C1"].with_(B=1, Hq=2, Hkv=2, D=D, k=0, P=0, L=70)
    d = attn_to_dev(cfg, S.attention_inputs(cfg))
    call = lambda: lotts.verify_attention(*(d[n] for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")))
    K = d["Kpriv"].clone()
    for step in (2, 4, 8, 16):
        d["Kpriv"].copy_(K)
        d["Kpriv"][0, 0, 0:4 * step:step] = float("nan")
        O = call()
        assert torch.isnan(O[0, 0, 0]).all() and torch.isfinite(O[0, 0, 1]).all()
    d["Kpriv"].copy_(K)
    d["Vpriv"][0, 0, 69] = float("inf")
    O = call()
    assert (O[0, 0, 0] == float("inf")).all() and torch.isfinite(O[0, 0, 1]).all()
