"""A head's results next to few and to many other heads (marked ``gpu``).

Launches with few tiles split a row's keys over waves, larger ones do not, so the number of heads
decides the order of a head's fp32 sums.  It must not decide how P~ is rounded to bf16: that
takes the same reference max for any number of splits.  fp32 sums in another order move a value
by about 2^-23, so a bf16 result changes where it lies that close to a rounding boundary, for one
value in 2^13 or so: relative L2 of 2^-8 / 2^6.5 = 4e-5 (measured 3e-5 to 5e-5, and up to 2e-4 in
the gradients, which take O and LSE from the forward).  Another rounding of P~ shows as 2.5e-3.  In fp32 the bits are the same for any number of heads.
"""
import sys

import pytest
import torch

from paper_2606_25473_amd import attn_bwd, attn_fwd, attn_jvp_fwd
from paper_2606_25473_amd.workloads import (MASK_BLOCK_CAUSAL, MASK_FULL, MASK_TEACHER_FORCING, custom_workload,
                                            make_inputs)

pytestmark = pytest.mark.gpu


def _calls(x, w, offs, B):
    g = {k: v.cuda().repeat(B, 1, 1, 1) for k, v in x.items()}
    o, do, lse = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind, offs)
    of, lf = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    assert torch.equal(o, of) and torch.equal(lse, lf)
    gq, gk, gv, _ = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    return {"O": o, "dO": do, "LSE": lse, "gQ": gq, "gK": gk, "gV": gv}


@pytest.mark.parametrize("kind,L,offs,H,D,B", [(MASK_FULL, 1560, None, 12, 64, 15), (MASK_FULL, 1100, None, 2, 128, 110),
                                               (MASK_TEACHER_FORCING, 0, (0, 1560, 3120), 3, 128, 15),
                                               (MASK_TEACHER_FORCING, 0, (0, 487, 974, 1461), 2, 64, 50),
                                               (MASK_BLOCK_CAUSAL, 0, (0, 251, 1001, 1751), 4, 128, 40)], ids=str)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_results_do_not_depend_on_the_other_heads(dtype, kind, L, offs, H, D, B):
    w = custom_workload("head_count", 1, H, D, dtype, kind, L=L, offsets=offs, tangent_std=0.5)
    print(f"[head-count] {dtype} {kind} L={w.L} D={D}: {H} and {H * B} heads", file=sys.stderr, flush=True)
    x = make_inputs(w, "cpu", 12)
    few, many = _calls(x, w, offs and list(offs), 1), _calls(x, w, offs and list(offs), B)
    for name, a in few.items():
        b = many[name][-1:]
        err = float((a.double() - b.double()).norm() / b.double().norm())
        print(f"[head-count] {name} rel-L2 {err:.1e}", file=sys.stderr, flush=True)
        assert torch.equal(many[name][0], many[name][-1]), name
        assert torch.equal(a, b) if dtype == "f32" else err <= 3e-4, (name, err)
