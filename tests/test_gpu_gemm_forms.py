"""skinny_gemm at the edges of each form that its plan can take: single-workgroup K ranges straight from memory, 64-, 128- and
256-row streaming blocks, split and unsplit, short row tiles, ragged last tiles, staggered starts.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    # direct: one tile shape each (16 * RN weight rows x 16 * TT tokens), ragged in rows and tokens
    (1, 8, 128), (16, 2040, 256), (17, 2056, 384), (33, 1544, 1536), (64, 2560, 1920), (129, 2568, 640), (193, 2048, 128),
    (192, 2504, 1152), (256, 2560, 1024), (1, 4096, 4096), (15, 3848, 4096), (9, 5000, 2048), (39, 2568, 2048), (27, 4104, 896),
    (60, 2568, 1024), (45, 5128, 1024), (192, 2048, 2048), (15, 3080, 2048), (30, 3912, 1024),
    # either side of the direct form's lines: 8192 rows, K = 4096
    (8, 8192, 512), (8, 8200, 512), (24, 4736, 1280), (2, 2048, 4096), (2, 2048, 4224),
    # 64-row blocks: split K, odd chunk counts, M in every token tile count
    (1, 2056, 8320), (31, 72, 4480), (40, 2048, 11008), (65, 520, 4352), (97, 4608, 4224), (129, 2056, 5248), (161, 64, 4224),
    (193, 264, 4480), (225, 136, 8192), (256, 4600, 4352),
    # 128-row blocks: split; unsplit with 20 .. 32 rows per wavefront
    (24, 4616, 5120), (100, 5000, 4480), (170, 6152, 4224), (5, 18440, 256), (70, 20608, 256), (96, 24584, 256), (33, 28680, 128),
    (90, 32768, 128), (128, 18440, 256), (224, 18448, 128), (256, 20488, 128),
    # 256-row blocks: 20 .. 32 rows per wavefront, more than one round of workgroups
    (1, 32776, 256), (40, 49160, 128), (96, 57352, 128), (64, 65544, 128), (66, 98312, 128), (97, 33032, 128), (200, 33000, 256),
    # W rows a multiple of 4 KB apart (blocks start at different k): each form, split and unsplit, uneven splits
    (40, 2056, 8192), (33, 2056, 6144), (96, 1032, 10240), (193, 520, 6144), (70, 10248, 2048), (7, 5128, 6144), (130, 4744, 4096),
    (40, 36872, 2048), (100, 33032, 2048),
])
def test_every_form(oracle, M, N, K):
    import paper_2505_19634_amd as lotts
    print("gemm form case", M, N, K, flush=True)
    g = S.rng_for(7, 33, salt=M + N + K)
    X = S.f32_to_bf16_bits(g.standard_normal((M, K), dtype=np.float32))
    W = S.f32_to_bf16_bits(g.standard_normal((N, K), dtype=np.float32) * np.float32(K ** -0.5))
    out = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device="cuda:0")  # a margin that has to stay as it is
    lotts.skinny_gemm(to_dev(X, True), to_dev(W, True), out=out[:M, :N])
    torch.cuda.synchronize()
    ref = oracle.skinny_gemm(X, W)
    y = out[:M, :N].float().cpu().numpy().astype(np.float64)
    # the bf16 result is within half a unit in the last place (2^-9 relative) of the fp32 sum, which is within about
    # K * 2^-24 of the exact one for terms of this size
    assert (np.abs(y - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-3).all(), np.abs(y - ref).max()
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) <= 3e-3
    assert bool((out[M:] == 7.0).all()) and bool((out[:, N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K", [
    # two token parts: tokens of the parts in 3 and 4 tiles, odd tokens (the parts overlap by one), blocks 1 .. 36, ragged rows, short K splits
    (129, 8, 4224), (130, 136, 4480), (161, 264, 5248), (191, 1288, 4352), (192, 2048, 4224), (193, 2056, 4480), (223, 520, 6144), (255, 4600, 4224),
    (256, 4608, 4352), (256, 128, 8320), (157, 1032, 2944), (251, 1344, 3072), (129, 3592, 1536), (247, 2304, 2048),
    # either side of K = 12288 and 160 tokens
    (160, 264, 12288), (160, 264, 12416), (161, 264, 12416),
    # more than 5 MB of X, the XCDs with runs of the list: two parts, staggered and not; one part, staggered
    (256, 72, 10368), (255, 1160, 10368), (250, 264, 12288), (193, 520, 14336), (177, 136, 16384), (128, 264, 22528), (97, 72, 28672), (150, 520, 18432),
])
def test_token_parts_and_runs_by_xcd(oracle, M, N, K):
    test_every_form(oracle, M, N, K)
