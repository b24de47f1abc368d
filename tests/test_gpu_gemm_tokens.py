"""skinny_gemm where a workgroup's share of the tokens is no multiple of anything: even shares of the direct form, one to several workgroups
over the tokens, next to rows of the output that stay as they are.  Against the float32 product."""
import pytest
import torch

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 2048, 2048), (17, 1024, 512), (20, 2048, 2048), (33, 2560, 2048), (40, 2048, 2048), (41, 2048, 2048),
                                   (72, 2048, 2048), (100, 2560, 2048), (191, 2048, 1024), (5, 64, 128), (255, 512, 256)])
def test_even_shares_of_tokens(M, N, K):
    import paper_2505_19634_amd as lotts
    g = torch.Generator(device=DEV).manual_seed(M * 7 + N)
    X = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    W = (torch.randn(N, K, generator=g, device=DEV) * K ** -0.5).bfloat16()
    Y = torch.full((M + 3, N), 7.0, dtype=torch.bfloat16, device=DEV)
    lotts.skinny_gemm(X, W, out=Y[:M])
    ref = X.float() @ W.float().t()
    # one rounding to bf16 (2^-9 relative, a bit more for the order of the sums)
    assert ((Y[:M].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-3).all()
    assert (Y[M:] == 7.0).all()
