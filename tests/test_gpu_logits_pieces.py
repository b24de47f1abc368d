"""spec_accept_logits with every size of piece (8192 to 16384 logits): vocabularies at the pieces' edges, drafted tokens on both sides
of an edge.  Against the CPU oracle."""
import numpy as np
import pytest

import synth_inputs as S
from gpu_util import to_dev
from test_gpu_parity import logit_inputs

pytestmark = pytest.mark.gpu

# pieces of 4, 5, 6 and 8 x 2048 logits, by the sizes (checked on the host, test_plans.py)
CASES = [(4, 8, 3, 16385), (4, 1, 0, 8193), (5, 5, 4, 40961), (5, 5, 4, 51200), (6, 7, 4, 49152), (6, 17, 3, 24576), (5, 2, 1, 600001),
         (8, 2, 1, 786433), (8, 1, 0, 1048575)]


@pytest.mark.parametrize("loads,B,k,V", CASES, ids=lambda x: str(x))
@pytest.mark.parametrize("bf16", [False, True])
def test_pieces(oracle, loads, B, k, V, bf16):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=B, V=V, k=k)
    zt, zd, draft, u = logit_inputs(cfg, 1.0, salt=V, bf16=bf16)
    size = loads * 2048
    edges = [x for x in (0, size - 1, size, V - 1, (V - 1) // size * size, size + 2047) if x < V]
    draft = draft.copy()
    for i in range(B * k):
        if i % 3:
            draft.flat[i] = edges[i % len(edges)]
    n, t = lotts.spec_accept_logits(to_dev(zt, bf16), to_dev(zd, bf16) if k else None, to_dev(draft) if k else None, to_dev(u), inv_temperature=1.3)
    n_ref, t_ref = oracle.spec_accept_logits(zt, zd, draft, u, 1.3)
    assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)
