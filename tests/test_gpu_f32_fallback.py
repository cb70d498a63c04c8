"""fp32 tiles that are computed again with fp32 matrix instructions (marked ``gpu``).

A tile whose result is not finite under the three-part products goes to the bodies of
f32_plain.hpp: an element of 1e33 has no three-part sum in the range of the scaled products, but a
finite result, which the oracle gives.  One element is set in the first and in the last head; the
other heads must keep their bits.  Two heads take 64-row tiles (4 waves), 100 and 44 heads 128-row
ones (8 waves); the masks have partial blocks, chunk bounds inside a tile and tiles cut at them,
and the range mask a group without keys.  Relative L2 <= 1e-4 per output, as for fp32 elsewhere,
and <= 1e-2 for each row (key): the element enters some of them only, and its terms cancel to a
thousandth in a few.  Where the element is in Q (K), the other tensor is zero in its column, since
scores of 1e33 have no exponentials.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import attention_fwd, attention_jvp, attention_vjp
from paper_2606_25473_amd import attn_bwd, attn_fwd, attn_jvp_fwd, attn_jvp_fwd_zero_clean
from paper_2606_25473_amd.workloads import MASK_RANGES, MASK_TEACHER_FORCING, custom_workload, make_inputs

pytestmark = pytest.mark.gpu

TF = (0, 40, 41, 149)
RANGES = [(0, 50, [(0, 50)]), (50, 60, []), (60, 331, [(0, 50), (60, 331)]), (331, 700, [(0, 7), (20, 50), (300, 700)])]
SHAPES = [(MASK_TEACHER_FORCING, TF, H, D) for H in (2, 100) for D in (64, 128)]
SHAPES += [(MASK_RANGES, RANGES, H, D) for H in (2, 44) for D in (64, 128)]
BIG = 1e33


def _ids(x):
    return f"{x[0]}_H{x[2]}_D{x[3]}" if isinstance(x, tuple) else str(x)


def _inputs(shape, seed=9):
    kind, offs, H, D = shape
    w = custom_workload("f32_fallback", 1, H, D, "f32", kind, offsets=offs)
    return w, list(offs), make_inputs(w, "cpu", seed)


def _put(x, name, row, value, H):
    """x on the GPU, with one element of the first and the last head set; and unchanged"""
    g = {k: v.cuda() for k, v in x.items()}
    if name in "QK":
        g["QK"[name == "Q"]][..., 5] = 0
    clean = {k: v.clone() for k, v in g.items()}
    for h in (0, H - 1):
        g[name][0, h, row, 5] = value
    return g, clean


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _check(name, got, want, clean, H):
    """The two heads against the oracle, whole and row by row; the others equal to the clean call's."""
    for h in {0, H - 1}:
        a, b = _np(got[0, h]), want[0, 0 if h == 0 else -1]
        fin = np.isfinite(b)
        assert np.array_equal(np.isfinite(a), fin), name
        a, b = np.where(fin, a, 0.0), np.where(fin, b, 0.0)
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        rows = np.linalg.norm(np.atleast_2d(a - b), axis=-1) / np.maximum(np.linalg.norm(np.atleast_2d(b), axis=-1), 1e-3)
        print(f"[f32-fallback] head {h} {name} rel-L2 {err:.2e}, worst row {rows.max():.2e}", file=sys.stderr, flush=True)
        assert err <= 1e-4 and rows.max() <= 1e-2, (name, h, err, rows.max())
    assert torch.equal(got[:, 1:H - 1], clean[:, 1:H - 1]), name


def _ends(g, names):
    return [_np(g[k][:, [0, -1]]) for k in names]


@pytest.mark.parametrize("shape", SHAPES, ids=_ids)
@pytest.mark.parametrize("name,row", [("V", 3), ("K", 30), ("Q", 100), ("Q", 297)])
def test_forward(shape, name, row):
    w, offs, x = _inputs(shape)
    print(f"[f32-fallback] forward {_ids(shape)} {name}[{row}]", file=sys.stderr, flush=True)
    g, c = _put(x, name, row, BIG, w.H)
    o, lse = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    oc, lc = attn_fwd(c["Q"], c["K"], c["V"], w.kind, offs)
    want = attention_fwd(*_ends(g, ("Q", "K", "V")), w.kind, offs)
    _check("O", o, want[0], oc, w.H)
    for h in (0, w.H - 1):
        assert np.allclose(_np(lse[0, h]), want[1][0, 0 if h == 0 else -1], rtol=1e-5, atol=1e-5)
    assert torch.equal(lse[:, 1:-1], lc[:, 1:-1])


@pytest.mark.parametrize("shape", SHAPES, ids=_ids)
@pytest.mark.parametrize("name,row", [("V", 3), ("dQ", 200), ("dK", 33), ("dV", 297)])
def test_tangent(shape, name, row):
    w, offs, x = _inputs(shape)
    print(f"[f32-fallback] JVP {_ids(shape)} {name}[{row}]", file=sys.stderr, flush=True)
    names = ("Q", "K", "V", "dQ", "dK", "dV")
    g, c = _put(x, name, row, BIG, w.H)
    got = attn_jvp_fwd(*[g[k] for k in names], w.kind, offs)
    clean = attn_jvp_fwd(*[c[k] for k in names], w.kind, offs)
    want = attention_jvp(*_ends(g, names), w.kind, offs)
    _check("O", got[0], want[0], clean[0], w.H)
    _check("dO", got[1], want[1], clean[1], w.H)


@pytest.mark.parametrize("shape", SHAPES[:4], ids=_ids)
@pytest.mark.parametrize("name,row", [("V", 3), ("V", 160), ("dQ", 150), ("dK", 190), ("dV", 260)])
def test_zero_clean(shape, name, row):
    """The element in a clean and in noisy rows; tiles of clean rows run the primal only."""
    w, offs, x = _inputs(shape)
    print(f"[f32-fallback] zero clean {_ids(shape)} {name}[{row}]", file=sys.stderr, flush=True)
    half = w.L // 2
    for k in ("dQ", "dK", "dV"):
        x[k][:, :, :half] = 0
    g, c = _put(x, name, row, BIG, w.H)
    call = lambda t: attn_jvp_fwd_zero_clean(t["Q"], t["K"], t["V"], *[t[k][:, :, half:].contiguous() for k in ("dQ", "dK", "dV")], offs)
    got, clean = call(g), call(c)
    want = attention_jvp(*_ends(g, ("Q", "K", "V", "dQ", "dK", "dV")), w.kind, offs)
    _check("O", got[0], want[0], clean[0], w.H)
    _check("dO", got[1], want[1][:, :, half:], clean[1], w.H)


@pytest.mark.parametrize("shape", SHAPES, ids=_ids)
@pytest.mark.parametrize("name,row", [("V", 3), ("Q", 60), ("K", 20), ("dV", 45), ("dV", 297)])
def test_backward(shape, name, row):
    """(dV is the cotangent of O)"""
    w, offs, x = _inputs(shape)
    print(f"[f32-fallback] backward {_ids(shape)} {name}[{row}]", file=sys.stderr, flush=True)

    def call(t):
        o, lse = attn_fwd(t["Q"], t["K"], t["V"], w.kind, offs)
        return attn_bwd(t["Q"], t["K"], t["V"], o, t["dV"], lse, w.kind, offs)

    g, c = _put(x, name, row, BIG, w.H)
    got, clean = call(g), call(c)
    want = attention_vjp(*_ends(g, ("Q", "K", "V", "dV")), w.kind, offs)
    for what, a, b, cl in zip(("gQ", "gK", "gV"), got, want, clean):
        _check(what, a, b, cl, w.H)


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3]], ids=_ids)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_elements(shape, value):
    """They reach the rows (keys) that see them, in V their own column only, and no other head nor
    the tiles that do not visit them.  (Masked rows of a tile that does take 0 inf = NaN from it.)"""
    w, offs, x = _inputs(shape)
    print(f"[f32-fallback] {value} {_ids(shape)}", file=sys.stderr, flush=True)
    names = ("Q", "K", "V", "dQ", "dK", "dV")
    half, row = w.L // 2, w.L // 2 + 60  # (a noisy key of the last chunk: its own chunk sees it)
    rows, cols = torch.arange(w.L), torch.arange(w.D)
    close = lambda a, b: torch.allclose(a, b, rtol=1e-4, atol=1e-5)
    for name in ("V", "dV", "dK", "dQ"):
        g, c = _put(x, name, row, value, w.H)
        o, do, lse = attn_jvp_fwd(*[g[k] for k in names], w.kind, offs)
        oc, doc, lc = attn_jvp_fwd(*[c[k] for k in names], w.kind, offs)
        sees = rows >= half + 41 if name != "dQ" else rows == row
        assert close(lse, lc)
        for out, ref in ((o, oc), (do, doc), (lse, lc)):
            assert torch.equal(out[:, 1:-1], ref[:, 1:-1])
            assert close(out[0, 0, :128], ref[0, 0, :128])
        if name == "V":
            assert bool((torch.isnan(o[0, 0, sees, 5]) if value != value else torch.isposinf(o[0, 0, sees, 5])).all())
            assert close(o[0, 0][:, cols != 5], oc[0, 0][:, cols != 5])
        else:
            assert close(o, oc)
            assert not bool(torch.isfinite(do[0, 0, sees, 5]).any())
    g, c = _put(x, "dV", row, value, w.H)  # as the cotangent: gQ of its row, gK and gV of the keys it sees
    o, lse = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    got = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    ref = attn_bwd(g["Q"], g["K"], g["V"], o, c["dV"], lse, w.kind, offs)
    seen = (rows < 41) | (rows >= half + 41)
    for what, a, b, hit in zip(("gQ", "gK", "gV"), got, ref, (rows == row, seen, seen)):
        assert torch.equal(a[:, 1:-1], b[:, 1:-1]), what
        assert not bool(torch.isfinite(a[0, 0, hit, 5]).any()), what
    assert close(got[0][0, 0, rows != row], ref[0][0, 0, rows != row])
