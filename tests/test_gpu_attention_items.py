"""verify_attention's work items at the edges of what they assume: key rows far apart, one tile for every wavefront and just more.  Which
plans the lists reach is checked on the host (test_plans.py)."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import attn_to_dev
from test_gpu_parity import BF, run_attention

pytestmark = pytest.mark.gpu


# whole 32-key tiles and ragged ones in both segments; the prefix in items of its own, and folded into the private ones
@pytest.mark.parametrize("far,P,L", [("private", 45, 37), ("prefix", 45, 37), ("prefix", 45, 181)])
@pytest.mark.parametrize("stride", [(1 << 25) - 8, 1 << 25])   # the last stride whose tiles use 32-bit offsets, the first beyond
def test_key_rows_far_apart(far, P, L, stride):
    """The same values with 2^25 elements from key to key and densely stored: the same result, bit for bit."""
    import paper_2505_19634_amd as lotts
    cfg = BF.with_(B=1, Hq=4, Hkv=1, k=2, P=P, L=L)
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


ONE_TILE = [
    # one row tile, at most four tiles an item: whole rows
    BF.with_(B=20, Hq=32, Hkv=8, k=3, P=0, L=128), BF.with_(B=20, Hq=32, Hkv=8, k=7, P=9, L=65), BF.with_(B=33, Hq=8, Hkv=8, k=0, P=0, L=1),
    # pairs, with and without a folded prefix tile; the last arriver, also with a prefix item; merge workgroups
    BF.with_(B=16, Hq=24, Hkv=8, k=3, P=31, L=193), BF.with_(B=16, Hq=24, Hkv=8, k=3, P=0, L=225), BF.with_(B=9, Hq=16, Hkv=8, k=1, P=0, L=353),
    BF.with_(B=1, Hq=4, Hkv=1, k=2, P=45, L=37), BF.with_(B=1, Hq=16, Hkv=2, k=2, P=225, L=961),
    # a launch of its own
    BF.with_(B=5, Hq=16, Hkv=2, k=3, P=100, L=120), BF.with_(B=4, Hq=16, Hkv=2, k=3, P=240, L=120),
    # two row tiles, five to eight tiles an item; 33, 40 and 64 rows: whole rows, merge workgroups, a launch of its own
    BF.with_(B=20, Hq=40, Hkv=8, k=7, P=0, L=256), BF.with_(B=17, Hq=24, Hkv=8, k=10, P=0, L=161), BF.with_(B=16, Hq=64, Hkv=8, k=7, P=60, L=385),
    BF.with_(B=8, Hq=16, Hkv=2, k=4, P=511, L=2047), BF.with_(B=3, Hq=16, Hkv=2, k=4, P=900, L=801),
]
# the merges of those, by row tiles (see kMergeLast .. kMergePair)
ONE_TILE_MERGES = {1: {0, 1, 2, 3, 4}, 2: {1, 2, 3}}
# more tiles to a wavefront than those
SEVERAL_TILES = [
    BF.with_(B=20, Hq=32, Hkv=8, k=7, P=9, L=97), BF.with_(B=16, Hq=24, Hkv=8, k=3, P=31, L=225), BF.with_(B=5, Hq=16, Hkv=2, k=3, P=300, L=120),
    BF.with_(B=6, Hq=16, Hkv=2, k=3, P=1500, L=320), BF.with_(B=16, Hq=64, Hkv=8, k=7, P=60, L=449),
]
# two row tiles at D = 64, whose Q rows do not pass through LDS: 36, 40 and 64 rows, folded, stacked, whole rows, several row groups
TWO_ROW_TILES_D64 = [
    BF.with_(B=4, Hq=32, Hkv=8, D=64, k=8, P=113, L=643), BF.with_(B=2, Hq=16, Hkv=2, D=64, k=4, P=217, L=386),
    BF.with_(B=20, Hq=16, Hkv=8, D=64, k=19, P=0, L=170), BF.with_(B=3, Hq=16, Hkv=2, D=64, k=7, P=40, L=1000),
    BF.with_(B=2, Hq=16, Hkv=2, D=64, k=9, P=33, L=333),
]


@pytest.mark.parametrize("cfg", ONE_TILE + SEVERAL_TILES + TWO_ROW_TILES_D64,
                         ids=lambda c: "B%d_k%d_Hq%d_Hkv%d_D%d_P%d_L%d" % (c.B, c.k, c.Hq, c.Hkv, c.D, c.P, c.L))
@pytest.mark.parametrize("ragged", [False, True])
def test_one_tile_per_wavefront(oracle, cfg, ragged):
    import paper_2505_19634_amd as lotts
    lens = None
    if ragged:  # wavefronts, and whole items, without a tile
        lens = np.linspace(cfg.k + 1, cfg.L, cfg.B).astype(np.int32) if cfg.B > 1 else np.array([max(cfg.k + 1, cfg.L // 3)], np.int32)
    run_attention(lotts, oracle, cfg, priv_len=lens)
