"""The library built so that nothing waits (every poll limit is 0): whatever a workgroup would get from another one in the same
launch it works out itself, or leaves to the one that comes last.  Same results, against the CPU oracle, with words of the
ordinary way arriving or not; nothing stays behind that a replay of a captured call could trip over."""
import os

import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import DEV, attn_to_dev, to_dev
from test_gpu_attention_merge import CASES
from test_gpu_parity import BF, logit_inputs, run_attention

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lotts():
    """The package on top of the other build, with workspaces of its own, for the tests of this file."""
    import paper_2505_19634_amd as m
    from paper_2505_19634_amd import binding
    usual, workspaces = m.load(), binding._workspaces
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(binding, "LIB_PATH", os.path.join(os.path.dirname(binding.LIB_PATH), "liblotts_no_polls.so"))
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_workspaces", {})
        assert m.load() is not usual
        yield m
        torch.cuda.synchronize()
    assert m.load() is usual and binding._workspaces is workspaces


LOGITS = [(3, 2, 1), (4, 3, 8193), (5, 0, 50257), (1, 8, 16385), (16, 3, 152064), (2, 1, 524288), (2, 1, 600001),
          (1, 256, 9000), (1, 40, 152064), (2, 100, 60001), (2, 1, 786433)]   # pieces of every size


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B,k,V", LOGITS)
def test_logits(lotts, oracle, B, k, V, bf16):
    cfg = S.CONFIGS["C1"].with_(B=B, V=V, k=k)
    print("logits without patience", cfg, bf16, flush=True)
    zt, zd, draft, u = logit_inputs(cfg, 1.0, salt=V + B, bf16=bf16)
    n_ref, t_ref = oracle.spec_accept_logits(zt, zd, draft, u, 0.7)
    for _ in range(3):
        n, t = lotts.spec_accept_logits(to_dev(zt, bf16), to_dev(zd, bf16), to_dev(draft), to_dev(u), inv_temperature=0.7)
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)


def test_logits_replayed(lotts, oracle):
    cfg = S.CONFIGS["C2"].with_(B=6, V=70001, k=3)
    sets = [logit_inputs(cfg, 1.0, salt=i, bf16=True) for i in range(3)]
    want = [oracle.spec_accept_logits(*s) for s in sets]
    buf = [to_dev(sets[0][0], True).clone(), to_dev(sets[0][1], True).clone(), to_dev(sets[0][2]), to_dev(sets[0][3])]
    n, t = (torch.empty(cfg.B, dtype=torch.int32, device=DEV) for _ in range(2))
    ws = torch.empty(lotts.load().spec_accept_logits_workspace_bytes(cfg.B, cfg.k, cfg.V), dtype=torch.uint8, device=DEV)
    call = lambda: lotts.spec_accept_logits(*buf, accept_len=n, next_token=t, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (1, 2, 0, 1):
        for dst, src, bf in zip(buf, sets[i], (True, True, False, False)):
            dst.copy_(to_dev(src, bf))
        for again in (graph.replay, call, graph.replay):
            again()
            torch.cuda.synchronize()
            assert np.array_equal(n.cpu().numpy(), want[i][0]) and np.array_equal(t.cpu().numpy(), want[i][1]), i


def accept_on_dev(s):
    return [to_dev(s[n]) for n in ("p", "q", "draft", "u")]


@pytest.mark.parametrize("B,k,V", [(3, 2, 1), (2, 1, 255), (6, 3, 1025), (4, 2, 16385), (5, 0, 50257), (32, 8, 30000), (3, 3, 151936),
                                   (2, 2, 262143)])
def test_accept(lotts, oracle, B, k, V):
    cfg = S.CONFIGS["C2"].with_(B=B, V=V, k=k)
    print("acceptance without patience", cfg, flush=True)
    s = S.accept_inputs(cfg, salt=V)
    for u_last in (None, 0.0, 1.0 - 2.0 ** -24):          # the first and the last token of the row among them
        if u_last is not None:
            s["u"][:, -1] = u_last
        n_ref, t_ref = oracle.spec_accept(s["p"], s["q"], s["draft"], s["u"])
        n, t = lotts.spec_accept(*accept_on_dev(s))
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)


def test_accept_replayed(lotts, oracle):
    cfg = S.CONFIGS["C2"].with_(B=6, V=70001, k=3)
    sets = [S.accept_inputs(cfg, salt=i) for i in range(3)]
    want = [oracle.spec_accept(s["p"], s["q"], s["draft"], s["u"]) for s in sets]
    buf = [x.clone() for x in accept_on_dev(sets[0])]
    n, t = (torch.empty(cfg.B, dtype=torch.int32, device=DEV) for _ in range(2))
    ws = torch.zeros(lotts.load().spec_accept_workspace_bytes(cfg.B, cfg.k, cfg.V), dtype=torch.uint8, device=DEV)
    call = lambda: lotts.spec_accept(*buf, accept_len=n, next_token=t, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (1, 2, 0, 1):
        for dst, src in zip(buf, accept_on_dev(sets[i])):
            dst.copy_(src)
        for again in (graph.replay, call, graph.replay):
            again()
            torch.cuda.synchronize()
            assert np.array_equal(n.cpu().numpy(), want[i][0]) and np.array_equal(t.cpu().numpy(), want[i][1]), i
            assert int(ws.to(torch.int32).sum()) == 0     # every word is down again, taken or marked


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "B%d_k%d_Hq%d_Hkv%d_D%d_P%d_L%d" % (c.B, c.k, c.Hq, c.Hkv, c.D, c.P, c.L))
def test_attention(lotts, oracle, cfg):
    lens = np.linspace(cfg.k + 1, cfg.L, cfg.B).astype(np.int32) if cfg.B > 1 else None
    run_attention(lotts, oracle, cfg, priv_len=lens)


def test_attention_replayed(lotts):
    """Whoever merges takes the flags and the words of the merge workgroups that left down again, and adds in the same order."""
    cfg = BF.with_(B=8, Hq=16, Hkv=2, k=4, P=512, L=2048)
    sets = [attn_to_dev(cfg, S.attention_inputs(cfg, salt=i)) for i in range(3)]
    names = ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")
    want = [lotts.verify_attention(*(d[n] for n in names)).clone() for d in sets]
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
        for again in (graph.replay, call, graph.replay):
            out.zero_()
            again()
            torch.cuda.synchronize()
            assert torch.equal(out, want[i]), i
            assert int(ws[:131072].to(torch.int32).sum()) == 0
