"""fp32 rows that start at any multiple of 4 bytes, through 16-byte loads: spec_accept on vocabularies that are no multiple of 4 and
on tensors off a 16-byte boundary, fp32 verify_attention on caches with odd strides.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import DEV, TOL, attn_errors, to_dev

pytestmark = pytest.mark.gpu


def shifted(x, off):
    t = to_dev(x)
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device=DEV)
    out = buf[off:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("V,off", [(1, 0), (2, 1), (255, 0), (257, 2), (1003, 3), (16383, 0), (50257, 0), (50257, 1), (65537, 2),
                                   (151938, 3), (151936, 1), (262143, 0), (262144, 1)])
def test_accept_rows_anywhere(oracle, V, off):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=3 if V > 100000 else 6, V=V, k=2)
    print("accept rows case", cfg, off, flush=True)
    s = S.accept_inputs(cfg, salt=V + off)
    for u_last in (None, 0.0, 1.0 - 2.0 ** -24):          # the first and the last token of the row among them
        u = s["u"].copy()
        if u_last is not None:
            u[:, -1] = u_last
        n_ref, t_ref = oracle.spec_accept(s["p"], s["q"], s["draft"], u)
        n, t = lotts.spec_accept(shifted(s["p"], off), shifted(s["q"], off), to_dev(s["draft"]), to_dev(u))
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)


@pytest.mark.parametrize("B,k,Hq,Hkv,D,P,L", [(1, 0, 1, 1, 64, 0, 1), (2, 3, 4, 4, 64, 32, 64), (1, 2, 4, 2, 128, 15, 17), (3, 1, 6, 3, 128, 0, 33),
                                              (2, 0, 8, 2, 64, 63, 65), (5, 4, 4, 1, 128, 130, 500)])
@pytest.mark.parametrize("pad", [0, 1, 3])
def test_fp32_attention_rows_anywhere(oracle, B, k, Hq, Hkv, D, P, L, pad):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C1"].with_(B=B, k=k, Hq=Hq, Hkv=Hkv, D=D, P=P, L=L)
    lens = np.linspace(k + 1, L, B).astype(np.int32) if B > 1 else np.array([L], np.int32)
    a = S.attention_inputs(cfg, priv_len=lens)

    def padded(x):                                         # rows `pad` elements further apart than they are long
        t = to_dev(x)
        buf = torch.full(t.shape[:-1] + (D + pad,), 1e30, dtype=t.dtype, device=DEV)
        buf[..., :D] = t
        return buf[..., :D]
    d = {n: padded(a[n]) if a[n].size else None for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv")}
    O, lse = lotts.verify_attention(d["Q"], d["Kpre"], d["Vpre"], d["Kpriv"], d["Vpriv"], to_dev(a["priv_len"]), return_lse=True)
    Oref, lref = oracle.verify_attention(a["Q"], a["Kpre"], a["Vpre"], a["Kpriv"], a["Vpriv"], a["priv_len"])
    e_abs, e_fro, _ = attn_errors(O, Oref)
    assert e_abs <= TOL["f32"]["abs"] and e_fro <= TOL["f32"]["fro_band"]
    assert np.abs(lse.cpu().numpy().astype(np.float64) - lref).max() <= TOL["f32"]["lse"]


@pytest.mark.parametrize("V", [1000, 262144, 262145, 600004])
def test_accept_on_a_workspace_of_the_size_asked_for(oracle, V):
    """One launch up to 2^18, two beyond: each within the bytes that the query names for that vocabulary."""
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=3, V=V, k=2)
    s = S.accept_inputs(cfg, salt=V)
    n_ref, t_ref = oracle.spec_accept(s["p"], s["q"], s["draft"], s["u"])
    need = lotts.load().spec_accept_workspace_bytes(cfg.B, cfg.k, V)
    buf = torch.full((need + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
    n, t = lotts.spec_accept(*(to_dev(s[x]) for x in ("p", "q", "draft", "u")), workspace=buf[:need])
    assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)
    assert bool((buf[need:] == 0x5a).all())
