"""fp32 over the whole range of exponents (marked ``gpu``).

The fp32 kernels form products from three bf16 parts of each operand.  Operands near the smallest
normal number, the results of a key that no query attends to, and scores beyond 2^80 take the
parts or the sums to the ends of their range.  Every output is compared with the fp64 oracle at
the 1e-4 relative L2 that holds for fp32 elsewhere, over all its elements or over the row or column
in question (results below 2^-126 keep multiples of 2^-149: at 2^-122 that is 2^-28).
"""
import sys

import numpy as np
import pytest
import torch

from oracle import attention_fwd, attention_jvp, attention_vjp
from paper_2606_25473_amd import attn_bwd, attn_fwd, attn_jvp_fwd, attn_jvp_fwd_zero_clean
from paper_2606_25473_amd.workloads import MASK_FULL, MASK_TEACHER_FORCING, custom_workload, make_inputs

pytestmark = pytest.mark.gpu

TOL = 1e-4
OFFS = (0, 40, 41, 149)


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _close(name, got, want):
    err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    print(f"[f32-range] {name} rel-L2 {err:.2e}", file=sys.stderr, flush=True)
    assert np.isfinite(got).all() and err <= TOL, (name, err)


def _case(D, H, scales, seed=8, kind=MASK_TEACHER_FORCING):
    """Inputs with some tensors multiplied by a power of two: on the GPU and in 64 bits."""
    w = custom_workload("f32_range", 1, H, D, "f32", kind, L=300 if kind == MASK_FULL else 0,
                        offsets=None if kind == MASK_FULL else OFFS)
    print(f"[f32-range] H={H} L={w.L} D={D} {scales}", file=sys.stderr, flush=True)
    x = make_inputs(w, "cpu", seed)
    for k, e in scales.items():
        x[k] = x[k] * 2.0 ** e
    return w, {k: v.cuda() for k, v in x.items()}, {k: _np(v) for k, v in x.items()}


# (44 heads: 128-row tiles; 2: 64-row tiles)
@pytest.mark.parametrize("D,H", [(64, 2), (64, 44), (128, 2), (128, 44)])
@pytest.mark.parametrize("scales", [{"V": -122, "dV": -122}, {"V": -122, "dQ": -122, "dV": -118, "dK": -100},
                                    {"dQ": -122, "dK": -122, "dV": -122}, {"dQ": -116, "dK": -116, "dV": -139},
                                    {"V": -100, "dV": -118, "dQ": -18, "dK": -18}], ids=str)
def test_small_tangents_and_values(D, H, scales):
    w, g, n = _case(D, H, scales)
    offs = list(OFFS)
    o, do, lse = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind, offs)
    of, _ = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    assert torch.equal(o, of)
    want = attention_jvp(*[n[k] for k in ("Q", "K", "V", "dQ", "dK", "dV")], w.kind, offs)
    for name, a, b in zip(("O", "dO", "LSE"), (o, do, lse), want):
        _close(name, _np(a), b)
    half = w.L // 2
    t = [g[k].clone() for k in ("dQ", "dK", "dV")]
    for x in t:
        x[:, :, :half] = 0
    _, dz, _ = attn_jvp_fwd(g["Q"], g["K"], g["V"], *t, w.kind, offs)
    _, dn, _ = attn_jvp_fwd_zero_clean(g["Q"], g["K"], g["V"], *[x[:, :, half:].contiguous() for x in t], offs)
    assert torch.equal(dn, dz[:, :, half:])


@pytest.mark.parametrize("D,H", [(64, 2), (64, 44), (128, 2), (128, 44)])
@pytest.mark.parametrize("scales", [{"dV": -122}, {"dV": -60, "V": -62}, {"V": -122, "dV": 10}, {"K": -100, "Q": 90, "dV": -20}], ids=str)
def test_small_cotangents(D, H, scales):
    w, g, n = _case(D, H, scales)  # (dV is the cotangent of O)
    offs = list(OFFS)
    o, lse = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    got = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    want = attention_vjp(n["Q"], n["K"], n["V"], n["dV"], w.kind, offs)
    for name, a, b in zip(("gQ", "gK", "gV"), got, want):
        _close(name, _np(a), b)


@pytest.mark.parametrize("D,H", [(64, 2), (128, 44)])
def test_key_that_no_query_attends_to(D, H):
    """Scores 74 below the row's others (P of 2^-109 to 2^-121): the key's own gK and gV rows."""
    w, g, n = _case(D, H, {}, kind=MASK_FULL)
    for x in (g, n):  # a feature that only separates the key
        x["Q"][..., 0] = 10.0
        x["K"][..., 0] = 0.0
        x["K"][:, :, 77, 0] = -7.4 * D ** 0.5
    o, lse = attn_fwd(g["Q"], g["K"], g["V"], w.kind)
    _, gk, gv, _ = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind)
    _, rk, rv, _ = attention_vjp(n["Q"], n["K"], n["V"], n["dV"], w.kind, None)
    assert 0 < np.abs(rv[:, :, 77]).max() < 2.0 ** -98
    _close("gV of the key", _np(gv)[:, :, 77], rv[:, :, 77])
    _close("gK of the key", _np(gk)[:, :, 77], rk[:, :, 77])


@pytest.mark.parametrize("D,H", [(64, 2), (128, 2), (128, 44)])
def test_scores_beyond_the_scaled_sums(D, H):
    """Scores of -2^95 and less in every row: the first key, with the largest, takes all weight."""
    w, g, n = _case(D, H, {}, kind=MASK_FULL)
    for x in (g, n):
        x["Q"][:] = 2.0 ** 45
        x["K"][:] = -2.0 ** 45
        x["K"][:, :, 1:] *= 1.5
    o, lse = attn_fwd(g["Q"], g["K"], g["V"], w.kind)
    want, wl = attention_fwd(n["Q"], n["K"], n["V"], w.kind, None)
    _close("O", _np(o), want)
    _close("LSE", _np(lse), wl)


def test_column_of_small_values():
    """One column of V at 2^-122 beside ordinary ones: its outputs keep their precision."""
    w, g, n = _case(128, 2, {}, kind=MASK_FULL)
    for x in (g, n):
        x["V"][..., 5] *= 2.0 ** -122
        x["dV"][..., 5] *= 2.0 ** -122
    o, do, _ = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind)
    want = attention_jvp(*[n[k] for k in ("Q", "K", "V", "dQ", "dK", "dV")], w.kind, None)
    _close("O column", _np(o)[..., 5], want[0][..., 5])
    _close("dO column", _np(do)[..., 5], want[1][..., 5])
