"""spec_accept with one, two and four wavefronts to a sub-chunk: vocabularies around the sizes of groups and sub-chunks, thresholds at
both ends of the row.  Against the CPU oracle."""
import numpy as np
import pytest

import synth_inputs as S
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 255, 257, 1023, 1025, 16384, 16385, 49153, 151937, 196609, 262144])
@pytest.mark.parametrize("parts,B,k", [(4, 2, 3), (2, 9, 2), (1, 19, 1)])   # (for vocabularies of 60 to 64 sub-chunks)
def test_parts(oracle, parts, B, k, V):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=B, V=V, k=k)
    s = S.accept_inputs(cfg, salt=V)
    for u_last in (None, 0.0, 1.0 - 2.0 ** -24):          # the first and the last token of the row among them
        if u_last is not None:
            s["u"][:, -1] = u_last
        n_ref, t_ref = oracle.spec_accept(s["p"], s["q"], s["draft"], s["u"])
        n, t = lotts.spec_accept(*(to_dev(s[x]) for x in ("p", "q", "draft", "u")))
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)


# sub-chunks of one to three groups of 256 tokens: (groups, wavefronts to a sub-chunk, B, V)
SHORT = [(1, 1, 2, 1), (1, 1, 2, 1000), (1, 1, 130, 1024), (1, 4, 2, 1025), (1, 4, 1, 16384), (1, 2, 5, 16200), (1, 1, 17, 16384), (1, 1, 130, 5001),
         (2, 4, 2, 16385), (2, 2, 6, 32768), (2, 1, 17, 32767), (2, 1, 40, 20001), (3, 4, 2, 32769), (3, 2, 14, 40000), (3, 1, 33, 49152)]


@pytest.mark.parametrize("groups,parts,B,V", SHORT)
@pytest.mark.parametrize("k", [0, 2])
def test_short_sub_chunks(oracle, groups, parts, B, V, k):
    import paper_2505_19634_amd as lotts
    cfg = S.CONFIGS["C2"].with_(B=B, V=V, k=k)
    s = S.accept_inputs(cfg, salt=V + k)
    for u_last in (None, 0.0, 1.0 - 2.0 ** -24):
        if u_last is not None:
            s["u"][:, -1] = u_last
        n_ref, t_ref = oracle.spec_accept(s["p"], s["q"], s["draft"], s["u"])
        n, t = lotts.spec_accept(*(to_dev(s[x]) for x in ("p", "q", "draft", "u")))
        assert np.array_equal(n.cpu().numpy(), n_ref) and np.array_equal(t.cpu().numpy(), t_ref)
