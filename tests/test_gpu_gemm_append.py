"""skinny_gemm_append against skinny_gemm followed by kv_append: the same bits in Y and in the caches, and nothing else touched, in each form
that writes Y (direct tiles, the reduce launch of split K, a product that streams W unsplit), with the first K column inside a tile, lengths
that put tokens outside the cache, and padded caches and rows; and when replayed from a graph with other lengths."""
import numpy as np
import pytest
import torch

import synth_inputs as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def lotts():
    import paper_2505_19634_amd as m
    return m


def _inputs(B, k, Hq, Hkv, D, K, Lmax):
    g = torch.Generator(device=DEV)
    g.manual_seed(B + 7 * k + Hq * D + K)
    mk = lambda *sh: torch.randn(*sh, generator=g, device=DEV).to(torch.bfloat16)
    N = (Hq + 2 * Hkv) * D
    caches = [mk(B, Hkv + 1, Lmax + 3, D + 8)[:, :Hkv, :Lmax, :D] for _ in range(2)]
    rng = S.rng_for(7, 55, salt=B * K + N)
    lengths = rng.integers(k + 1, Lmax + 1, size=B).astype(np.int32)
    lengths[0] = Lmax
    if B > 2:
        lengths[1], lengths[2] = k, Lmax + 2   # the first token below the cache, the last two beyond it
    return mk(B * (k + 1), K), mk(N, K) * K ** -0.5, caches, torch.from_numpy(lengths).to(DEV)


def _apart(lotts, X, W, caches, lengths, Y, Hkv, D):
    B, R = lengths.numel(), X.shape[0] // lengths.numel()
    lotts.skinny_gemm(X, W, out=Y)
    new = [Y[:, Y.shape[1] - n * Hkv * D:][:, :Hkv * D].unflatten(0, (B, R)).unflatten(2, (Hkv, D)) for n in (2, 1)]
    lotts.kv_append(new[0], new[1], caches[0], caches[1], lengths)


def _whole(t):
    """Everything behind a padded view."""
    return t._base if t._base is not None else t


SIZES = [
    (1, 0, 1, 1, 8, 128), (1, 0, 16, 2, 128, 2048), (5, 2, 3, 2, 24, 1024), (8, 4, 16, 2, 128, 2048), (16, 3, 32, 8, 128, 4096),
    (3, 8, 28, 4, 128, 3584), (13, 2, 0, 4, 64, 640), (64, 3, 16, 16, 64, 1024), (1, 255, 16, 2, 128, 2048), (27, 7, 32, 8, 64, 1152),
    (4, 4, 40, 8, 128, 5120), (16, 3, 40, 8, 128, 5120), (32, 5, 33, 3, 72, 4480), (7, 0, 8, 1, 8, 8320), (85, 2, 64, 8, 128, 8192),
    (43, 2, 20, 4, 128, 8192), (51, 4, 12, 2, 64, 12288),   # K split and the tokens in two parts
    (5, 0, 2299, 3, 8, 256), (32, 7, 2555, 3, 8, 128),   # W streamed with K unsplit
    (40, 3, 12, 2, 128, 2048), (21, 2, 24, 4, 128, 2048), (47, 3, 8, 2, 128, 1536), (21, 2, 4, 2, 128, 4096),   # direct tiles with several workgroups over the tokens
]


@pytest.mark.parametrize("B,k,Hq,Hkv,D,K", SIZES)
def test_append_in_the_projection(lotts, B, k, Hq, Hkv, D, K):
    print("projection with append", B, k, Hq, Hkv, D, K, flush=True)
    Lmax = k + 40
    X, W, caches, lengths = _inputs(B, k, Hq, Hkv, D, K, Lmax)
    M, N = X.shape[0], W.shape[0]
    pad = lambda: torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device=DEV)
    want, got = pad(), pad()
    mine = [_whole(t).clone()[:, :Hkv, :Lmax, :D] for t in caches]
    _apart(lotts, X, W, caches, lengths, want[:M, :N], Hkv, D)
    lotts.skinny_gemm_append(X, W, mine[0], mine[1], lengths, out=got[:M, :N])
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    for a, b in zip(mine, caches):
        assert torch.equal(_whole(a).view(torch.int16), _whole(b).view(torch.int16))


@pytest.mark.parametrize("B,k,Hq,Hkv,D,K", [(8, 4, 16, 2, 128, 2048), (16, 3, 40, 8, 128, 5120), (5, 0, 2299, 3, 8, 256)])
def test_replays_with_other_lengths(lotts, B, k, Hq, Hkv, D, K):
    print("captured projection with append", B, k, Hq, Hkv, D, K, flush=True)
    Lmax = k + 40
    X, W, caches, lengths = _inputs(B, k, Hq, Hkv, D, K, Lmax)
    mine = [_whole(t).clone()[:, :Hkv, :Lmax, :D] for t in caches]
    want, got = (torch.zeros((X.shape[0], W.shape[0]), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = torch.zeros(max(256, lotts.load().skinny_gemm_workspace_bytes(X.shape[0], W.shape[0], K)), dtype=torch.uint8, device=DEV)
    call = lambda: lotts.skinny_gemm_append(X, W, mine[0], mine[1], lengths, out=got, workspace=ws)
    call()
    _apart(lotts, X, W, caches, lengths, want, Hkv, D)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for shift in (0, 1, 3):
        lengths.copy_(torch.arange(B, device=DEV, dtype=torch.int32) * 5 % (Lmax - k) + k + shift)
        X.mul_(0.5)
        got.zero_()
        graph.replay()
        _apart(lotts, X, W, caches, lengths, want, Hkv, D)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        for a, b in zip(mine, caches):
            assert torch.equal(_whole(a).view(torch.int16), _whole(b).view(torch.int16)), shift


def test_binding_refuses_what_the_kernels_cannot_address(lotts):
    X, W, (K, V), lengths = _inputs(4, 1, 4, 2, 64, 256, 41)
    call = lambda **kw: lotts.skinny_gemm_append(*[kw.get(n, v) for n, v in (("X", X), ("W", W), ("K", K), ("V", V), ("len", lengths))],
                                                 out=kw.get("out"))
    for bad in ({"X": X.float()}, {"W": W.t()}, {"K": K.transpose(2, 3)}, {"len": lengths.long()}, {"len": lengths[:3]},
                {"out": torch.empty((8, 7), dtype=torch.bfloat16, device=DEV)}):
        with pytest.raises((TypeError, ValueError)):
            call(**bad)
    for bad in ({"X": X[:7]}, {"V": V.contiguous()}, {"X": X[:, :128]}, {"K": K[:1].expand_as(K), "V": V[:1].expand_as(V)}):
        with pytest.raises(ValueError):
            call(**bad)
    for bad in ({"W": W[:64]}, {"K": K[:, :, :1], "V": V[:, :, :1]}):   # fewer columns than K and V take; a cache shorter than the new tokens
        with pytest.raises(lotts.LottsError):
            call(**bad)
