"""spec_accept_logits on workspaces that hold what earlier calls leave there: row sums and maxima of other sizes, and words made
to look like a piece maximum of the very call.  In a child process, whose calls draw the first tags; against the CPU oracle."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import sys
import numpy as np, torch
sys.path[:0] = [%(root)r, %(root)r + "/tests"]
import oracle
import paper_2505_19634_amd as lotts
import synth_inputs as S
from gpu_util import DEV, to_dev
from test_gpu_parity import logit_inputs

def case(B, V, k, salt):
    zt, zd, draft, u = logit_inputs(S.CONFIGS["C2"].with_(B=B, V=V, k=k), 1.0, salt=salt, bf16=True)
    n, t = oracle.spec_accept_logits(zt, zd, draft, u)
    return [to_dev(zt, True), to_dev(zd, True), to_dev(draft), to_dev(u)], n, t

def check(c, what, **kw):
    n, t = lotts.spec_accept_logits(*c[0], **kw)
    assert np.array_equal(n.cpu().numpy(), c[1]) and np.array_equal(t.cpu().numpy(), c[2]), what

# Two tags a call, drawn from the first on, the maxima's before the chunk sums'.  Planted in turn: the bare counter, the maxima's
# tag, its complement; the low half is a number above every logit.
small = case(3, 40000, 2, 1)
ws = torch.empty(8 << 20, dtype=torch.uint8, device=DEV)
for call in range(6):
    upper = (1 + 2 * call, 0x80000000 + 2 * call, 0x7fffffff - 2 * call)[call %% 3]
    word = (upper << 32) | 0x7f000000
    ws.view(torch.int64).fill_(word - (1 << 64) if word >> 63 else word)
    print("planted words, call", call, hex(word), flush=True)
    check(small, hex(word), workspace=ws)

# Falling branch counts on one workspace: the words of the later call lie where the row sums of the earlier ones lay.
many, one = case(16, 152064, 3, 2), case(1, 152064, 3, 3)
for calls in range(1, 13):
    print("16 branches", calls, "times, then one", flush=True)
    for _ in range(calls):
        lotts.spec_accept_logits(*many[0])
    check(one, calls)
check(many, "16 branches")
print("LEFTOVERS OK", flush=True)
"""


def test_leftovers_are_not_taken_for_piece_maxima():
    res = subprocess.run([sys.executable, "-u", "-c", CHILD % {"root": ROOT}], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                         text=True, timeout=110)
    print(res.stdout[-4000:], flush=True)
    assert res.returncode == 0 and "LEFTOVERS OK" in res.stdout
