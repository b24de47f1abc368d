"""verify_attention's work items at the edges of what they assume: key rows far apart."""
import pytest
import torch

import synth_inputs as S
from gpu_util import attn_to_dev
from test_gpu_parity import BF

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("far", ["private", "prefix"])
@pytest.mark.parametrize("stride", [(1 << 25) - 8, 1 << 25])   # the last stride whose tiles use 32-bit offsets, the first beyond
def test_key_rows_far_apart(far, stride):
    """The same values with 2^25 elements from key to key and densely stored: the same result, bit for bit."""
    import paper_2505_19634_amd as lotts
    cfg = BF.with_(B=1, Hq=4, Hkv=1, k=2, P=9, L=37)
    d = attn_to_dev(cfg, S.attention_inputs(cfg))
    want = lotts.verify_attention(*(d[n] for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")))
    for n in ("Kpriv", "Vpriv") if far == "private" else ("Kpre", "Vpre"):
        dense = d[n]
        rows = dense.shape[-2]
        buf = torch.empty((rows - 1) * stride + cfg.D, dtype=torch.bfloat16, device=dense.device)
        shape = tuple(dense.shape)
        d[n] = buf.as_strided(shape, ((rows * stride,) * (len(shape) - 2)) + (stride, 1))
        d[n].copy_(dense)
    got = lotts.verify_attention(*(d[n] for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len")))
    torch.cuda.synchronize()
    assert torch.equal(got, want)
