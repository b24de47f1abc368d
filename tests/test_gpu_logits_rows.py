"""spec_accept_logits on rows that start anywhere and end anywhere: vocabularies around the sizes of groups, chunks and pieces,
tensors that begin off a 16-byte boundary, more than 2^19 logits, replays of a captured call.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import DEV, to_dev
from test_gpu_parity import logit_inputs

pytestmark = pytest.mark.gpu


def shifted(x, bf16, off):
    """The same values in a tensor whose first element lies `off` elements past a 16-byte boundary."""
    t = to_dev(x, bf16)
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device=DEV)
    out = buf[off:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V,off", [(1, 0), (3, 1), (7, 3), (8, 0), (2047, 0), (2049, 5), (8191, 0), (8192, 2), (8193, 0), (16384, 1),
                                   (16385, 7), (50257, 0), (50257, 3), (151936, 1), (524288, 0), (524289, 0), (600001, 1)])
def test_rows_anywhere(oracle, V, off, bf16):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C1"].with_(B=2 if V > 100000 else 4, V=V, k=3 if V < 100000 else 1)
    print("logits rows case", cfg, off, bf16, flush=True)
    zt, zd, draft, u = logit_inputs(cfg, 1.0, salt=V + off, bf16=bf16)
    for inv_temp in (1.0, 0.7):
        n_ref, t_ref = oracle.spec_accept_logits(zt, zd, draft, u, inv_temp)
        n, t = lotts.spec_accept_logits(shifted(zt, bf16, off), shifted(zd, bf16, off), to_dev(draft), to_dev(u),
                                        inv_temperature=inv_temp)
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)


def test_captured_call_replayed_on_changing_logits(oracle):
    import paper_2505_19634_amd as lotts
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
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(n.cpu().numpy(), want[i][0]) and np.array_equal(t.cpu().numpy(), want[i][1]), i
        call()                                    # an eager call on the same workspace in between
        torch.cuda.synchronize()
        assert np.array_equal(n.cpu().numpy(), want[i][0]) and np.array_equal(t.cpu().numpy(), want[i][1]), i


def test_calls_side_by_side(oracle):
    """Calls on several streams overlap, and their launches may find any part of the chip taken by the others' waiting workgroups:
    every one ends with the right result."""
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=16, V=152064, k=3)
    sets = [logit_inputs(cfg, 1.0, salt=i, bf16=True) for i in range(3)]
    want = [oracle.spec_accept_logits(*s) for s in sets]
    d = [[to_dev(x, bf) for x, bf in zip(s, (True, True, False, False))] for s in sets]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    got = [[lotts.spec_accept_logits(*x, stream=s) for x, s in zip(d, streams)] for _ in range(20)]
    torch.cuda.synchronize()
    for i, (n_ref, t_ref) in enumerate(want):
        for round_ in got:
            assert np.array_equal(round_[i][0].cpu().numpy(), n_ref) and np.array_equal(round_[i][1].cpu().numpy(), t_ref), i
