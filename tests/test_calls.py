"""The binding's extension against stand-ins for the library: what a call hands over, and that a call whose tensors do not hold what the
kernels would address is refused before the library is reached."""
import ctypes

import pytest
import torch

I32, I64, VP, SZ, F32 = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float
NEED = 4096


class Library:
    """Stand-ins for the entry points; `made` holds the arguments of the calls that reached them."""
    SIGNATURES = [  # result, arguments
        (SZ, [VP]), (ctypes.c_int, [VP] * 10 + [SZ, VP]), (SZ, [I32] * 3), (ctypes.c_int, [I32] * 3 + [VP] * 7 + [SZ, VP]),
        (ctypes.c_int, [I32, I32] + [VP] * 4), (SZ, [I32] * 3), (ctypes.c_int, [I32] * 3 + [VP, I64] * 3 + [VP, SZ, VP]),
        (ctypes.c_int, [VP] * 10)]

    def __init__(self):
        try:
            from paper_2505_19634_amd import binding
        except ImportError:
            import __graft_entry__
            __graft_entry__.build()
            from paper_2505_19634_amd import binding
        self.made, self.answer = [], 0

        def query(*args):
            return NEED

        def call(*args):
            self.made.append(args)
            return self.answer

        def attend(desc, *args):   # the descriptor lives as long as the call
            return call(binding.AttnDesc.from_buffer_copy(binding.AttnDesc.from_address(desc)), *args)
        self.keep = [ctypes.CFUNCTYPE(res, *args)(query if res is SZ else attend if args[0] is VP else call)
                     for res, args in self.SIGNATURES]
        self.calls = type(binding.load().calls)(*(ctypes.cast(f, VP).value for f in self.keep))


@pytest.fixture()
def library():
    return Library()


WS = torch.zeros(NEED, dtype=torch.uint8)


def attention(**other):
    B, k, Hq, Hkv, D, P, L = 3, 2, 4, 2, 64, 5, 9
    bf = torch.bfloat16
    t = dict(Q=torch.zeros(B, k + 1, Hq, D, dtype=bf), Kpre=torch.zeros(Hkv, P, D, dtype=bf), Vpre=torch.zeros(Hkv, P, D, dtype=bf),
             Kpriv=torch.zeros(B, Hkv, L, D, dtype=bf), Vpriv=torch.zeros(B, Hkv, L, D, dtype=bf),
             priv_len=torch.full((B,), L, dtype=torch.int32), scale=0.0, out=torch.zeros(B, k + 1, Hq, D, dtype=bf), lse=None,
             workspace=None, cached=WS, stream=0)
    t.update(other)
    return t


def accept(**other):
    t = dict(p=torch.zeros(3, 3, 8), q=torch.zeros(3, 2, 8), draft=torch.zeros(3, 2, dtype=torch.int32), u=torch.zeros(3, 3),
             accept_len=torch.zeros(3, dtype=torch.int32), next_token=torch.zeros(3, dtype=torch.int32), workspace=None, cached=WS, stream=0)
    t.update(other)
    return t


def vote(**other):
    t = dict(answers=torch.zeros(2, 5, dtype=torch.int32), winner=torch.zeros(2, dtype=torch.int32),
             count=torch.zeros(2, dtype=torch.int32), stream=0)
    t.update(other)
    return t


def gemm(**other):
    bf = torch.bfloat16
    t = dict(X=torch.zeros(3, 128, dtype=bf), W=torch.zeros(16, 128, dtype=bf), out=torch.zeros(3, 16, dtype=bf), workspace=None, cached=WS, stream=0)
    t.update(other)
    return t


def test_what_a_call_hands_over(library):
    a = attention(lse=torch.zeros(3, 3, 4), stream=77)
    assert library.calls.verify_attention(*a.values()) == 0
    (d, *ptrs, nbytes, stream), = library.made
    assert (d.B, d.k, d.Hq, d.Hkv, d.D, d.P, d.Lmax, d.dtype, d.scale) == (3, 2, 4, 2, 64, 5, 9, 1, 0.0)
    assert (d.q_stride_b, d.q_stride_r, d.q_stride_h, d.kpre_stride_h, d.kpre_stride_t) == (768, 256, 64, 320, 64)
    assert (d.kpriv_stride_b, d.kpriv_stride_h, d.kpriv_stride_t, d.o_stride_b, d.o_stride_r, d.o_stride_h) == (1152, 576, 64, 768, 256, 64)
    assert ptrs == [a[n].data_ptr() for n in ("Q", "Kpre", "Vpre", "Kpriv", "Vpriv", "priv_len", "out", "lse")] + [WS.data_ptr()]
    assert nbytes == NEED and stream == 77
    without = {n: v for n, v in a.items() if n not in ("workspace", "cached")}
    assert library.calls.verify_attention_noalloc(*without.values()) == 0
    assert list(library.made[1][1:]) == ptrs[:-1] + [77]
    g = gemm()
    assert library.calls.skinny_gemm(*g.values()) == 0
    assert library.made[2] == (3, 16, 128, g["X"].data_ptr(), 128, g["W"].data_ptr(), 128, g["out"].data_ptr(), 16, WS.data_ptr(), NEED, None)
    s = accept()
    assert library.calls.spec_accept(*s.values()) == 0
    assert library.made[3] == (3, 2, 8, *(s[n].data_ptr() for n in ("p", "q", "draft", "u", "accept_len", "next_token")), WS.data_ptr(), NEED, None)
    assert library.calls.spec_accept(*accept(p=torch.zeros(3, 1, 8), u=torch.zeros(3, 1), q=None, draft=None).values()) == 0
    assert library.made[4][:3] == (3, 0, 8) and library.made[4][4:6] == (None, None)
    v = vote()
    assert library.calls.majority_vote(*v.values()) == 0
    assert library.made[5] == (2, 5, *(v[n].data_ptr() for n in ("answers", "winner", "count")), None)
    library.answer = -5
    assert library.calls.majority_vote(*v.values()) == -5


@pytest.mark.parametrize("name,make", [("verify_attention", attention), ("spec_accept", accept), ("skinny_gemm", gemm)])
def test_workspaces(library, name, make):
    call = getattr(library.calls, name)
    small = torch.zeros(NEED - 1, dtype=torch.uint8)
    assert call(*make(cached=None).values()) == NEED and call(*make(cached=small).values()) == NEED   # made again with that many bytes
    assert not library.made
    assert call(*make(workspace=small, cached=None).values()) == 0     # the caller's own goes to the library as it is
    assert library.made[0][-2] == NEED - 1 and library.made[0][-3] == small.data_ptr()


BF, FL = torch.bfloat16, torch.float32
LARGER = [  # more than a call needs stays accepted
    dict(out=torch.zeros(5, 4, 6, 64, dtype=BF)), dict(priv_len=torch.zeros(8, dtype=torch.int32)), dict(lse=torch.zeros(100)),
    dict(Kpre=torch.zeros(3, 5, 64, dtype=BF), Vpre=torch.zeros(4, 5, 64, dtype=BF)), dict(Kpre=None, Vpre=None),
    dict(Kpre=torch.zeros(2, 0, 64, dtype=BF), Vpre=None),
    dict(Kpriv=torch.zeros(3, 9, 2, 64, dtype=BF).transpose(1, 2), Vpriv=torch.zeros(3, 9, 2, 64, dtype=BF).transpose(1, 2)),
    dict(Q=torch.zeros(3, 3, 8, 64, dtype=BF)[:, :, :4])]
UNFIT = [
    (ValueError, dict(out=torch.zeros(2, 3, 4, 64, dtype=BF))), (ValueError, dict(out=torch.zeros(3, 2, 4, 64, dtype=BF))),
    (ValueError, dict(out=torch.zeros(3, 3, 3, 64, dtype=BF))), (ValueError, dict(out=torch.zeros(3, 3, 256, dtype=BF))),
    (ValueError, dict(Vpriv=torch.zeros(3, 2, 9, 64, dtype=BF)[:, :, :8])), (ValueError, dict(Vpriv=torch.zeros(3, 2, 9, 64, dtype=BF)[:2])),
    (ValueError, dict(Vpriv=torch.zeros(3, 2, 9, 64, dtype=BF)[:, :1])), (ValueError, dict(Vpriv=torch.zeros(3, 2, 8, 64, dtype=BF))),
    (ValueError, dict(Kpriv=torch.zeros(2, 2, 9, 64, dtype=BF), Vpriv=torch.zeros(2, 2, 9, 64, dtype=BF))),
    (ValueError, dict(Kpre=torch.zeros(1, 5, 64, dtype=BF), Vpre=torch.zeros(1, 5, 64, dtype=BF))),
    (ValueError, dict(Vpre=torch.zeros(2, 5, 64, dtype=BF)[:, :4])), (ValueError, dict(Vpre=torch.zeros(2, 5, 64, dtype=BF)[:1])),
    (ValueError, dict(Kpre=torch.zeros(2, 5, 64, dtype=BF)[:, :, :32], Vpre=torch.zeros(2, 5, 64, dtype=BF)[:, :, :32])),
    (ValueError, dict(Q=torch.zeros(1, 3, 4, 64, dtype=BF).expand(3, -1, -1, -1))), (ValueError, dict(Q=torch.zeros(3, 3, 64, dtype=BF))),
    (ValueError, dict(Kpriv=torch.zeros(1, 2, 9, 64, dtype=BF).expand(3, -1, -1, -1), Vpriv=torch.zeros(1, 2, 9, 64, dtype=BF).expand(3, -1, -1, -1))),
    (ValueError, dict(Q=torch.zeros(3, 3, 64, 4, dtype=BF).transpose(2, 3))),
    (ValueError, dict(priv_len=torch.zeros(2, dtype=torch.int32))), (ValueError, dict(priv_len=torch.zeros(6, dtype=torch.int32)[::2])),
    (ValueError, dict(lse=torch.zeros(35))), (TypeError, dict(lse=torch.zeros(36, dtype=BF))), (TypeError, dict(lse=torch.zeros(72)[::2])),
    (TypeError, dict(priv_len=torch.zeros(3, dtype=torch.int64))), (TypeError, dict(Q=torch.zeros(3, 3, 4, 64, dtype=torch.float16))),
    (TypeError, dict(Q=torch.zeros(3, 3, 4, 64))), (TypeError, dict(out=torch.zeros(3, 3, 4, 64))), (TypeError, dict(Vpriv=torch.zeros(3, 2, 9, 64))),
    (TypeError, dict(Kpre=torch.zeros(2, 5, 64))), (TypeError, dict(Vpre=torch.zeros(2, 5, 64))), (TypeError, dict(Vpre=None)),
    (TypeError, dict(Q=[1.0])), (TypeError, dict(scale="large")), (TypeError, dict(lse=3))]


@pytest.mark.parametrize("other", LARGER)
def test_attention_takes_larger_tensors(library, other):
    a = attention(**other)
    assert library.calls.verify_attention(*a.values()) == 0
    del a["workspace"], a["cached"]
    assert library.calls.verify_attention_noalloc(*a.values()) == 0 and len(library.made) == 2


@pytest.mark.parametrize("error,other", UNFIT)
def test_attention_refuses_tensors_that_do_not_fit(library, error, other):
    a = attention(**other)
    with pytest.raises(error):
        library.calls.verify_attention(*a.values())
    del a["workspace"], a["cached"]
    with pytest.raises(error):
        library.calls.verify_attention_noalloc(*a.values())
    assert not library.made


@pytest.mark.parametrize("name,make,error,other", [
    ("spec_accept", accept, ValueError, dict(q=None)), ("spec_accept", accept, ValueError, dict(draft=None)),
    ("spec_accept", accept, ValueError, dict(q=torch.zeros(3, 3, 8))), ("spec_accept", accept, ValueError, dict(draft=torch.zeros(2, 2, dtype=torch.int32))),
    ("spec_accept", accept, ValueError, dict(u=torch.zeros(3, 2))), ("spec_accept", accept, ValueError, dict(p=torch.zeros(9, 8))),
    ("spec_accept", accept, TypeError, dict(p=torch.zeros(3, 3, 8, dtype=BF))), ("spec_accept", accept, TypeError, dict(q=torch.zeros(3, 2, 8, dtype=BF))),
    ("spec_accept", accept, TypeError, dict(draft=torch.zeros(3, 2, dtype=torch.int64))), ("spec_accept", accept, TypeError, dict(p=torch.zeros(3, 8, 3).transpose(1, 2))),
    ("spec_accept", accept, ValueError, dict(accept_len=torch.zeros(2, dtype=torch.int32))), ("spec_accept", accept, TypeError, dict(next_token=torch.zeros(3))),
    ("spec_accept", accept, TypeError, dict(next_token=torch.zeros(6, dtype=torch.int32)[::2])),
    ("majority_vote", vote, TypeError, dict(answers=torch.zeros(2, 5))), ("majority_vote", vote, ValueError, dict(answers=torch.zeros(1, 2, 5, dtype=torch.int32))),
    ("majority_vote", vote, ValueError, dict(winner=torch.zeros(1, dtype=torch.int32))), ("majority_vote", vote, TypeError, dict(count=torch.zeros(2, dtype=torch.int64))),
    ("skinny_gemm", gemm, ValueError, dict(W=torch.zeros(16, 256, dtype=BF))), ("skinny_gemm", gemm, ValueError, dict(X=torch.zeros(128, 3, dtype=BF).t())),
    ("skinny_gemm", gemm, ValueError, dict(out=torch.zeros(2, 16, dtype=BF))), ("skinny_gemm", gemm, ValueError, dict(out=torch.zeros(3, 16, dtype=BF)[:, :8])),
    ("skinny_gemm", gemm, ValueError, dict(out=torch.zeros(16, 3, dtype=BF).t())), ("skinny_gemm", gemm, ValueError, dict(out=torch.zeros(48, dtype=BF))),
    ("skinny_gemm", gemm, TypeError, dict(out=torch.zeros(3, 16))), ("skinny_gemm", gemm, TypeError, dict(X=None)),
])
def test_refused(library, name, make, error, other):
    with pytest.raises(error):
        getattr(library.calls, name)(*make(**other).values())
    assert not library.made


@pytest.mark.parametrize("other", [dict(out=torch.zeros(4, 32, dtype=BF)[:, :16]), dict(out=torch.zeros(3, 1, 16, dtype=BF)),
                                   dict(X=torch.zeros(3, 256, dtype=BF)[:, :128])])
def test_gemm_takes_views(library, other):
    assert library.calls.skinny_gemm(*gemm(**other).values()) == 0 and len(library.made) == 1


def test_wrong_number_of_arguments(library):
    for call in ("verify_attention", "verify_attention_noalloc", "spec_accept", "majority_vote", "skinny_gemm"):
        with pytest.raises(TypeError):
            getattr(library.calls, call)(1, 2)
