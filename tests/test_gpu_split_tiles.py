"""GPU parity of the split-tile kernels (marked ``gpu``), and the rule that selects them.

Small launches give each work-group 64 or 128 query rows (64 keys in the backward's key-tile
pass) and split the other side's blocks over its waves; larger ones keep the full-size tiles.
The shapes below sit at the edges of those tiles (one row more or less, rounds that leave some
splits idle, a clean/noisy boundary inside a tile and inside a block) and on each side of the
rule; every output is compared with the fp64 oracle by relative L2 error <= 1e-2 (bf16 operands
and results: 2^-9 per rounding, a few of them per output).
"""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import attention_jvp, attention_jvp_zero_clean, attention_vjp
from paper_2606_25473_amd import attn_bwd, attn_fwd, attn_jvp_fwd, attn_jvp_fwd_zero_clean
from paper_2606_25473_amd.workloads import (MASK_FULL, MASK_RANGES, MASK_TEACHER_FORCING, custom_workload,
                                            make_inputs)

TF = MASK_TEACHER_FORCING
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _full(L, H, D):
    return custom_workload(f"full_{L}_{H}_{D}", 1, H, D, "bf16", MASK_FULL, L=L, tangent_std=0.5)


def _tf(offs, H, D):
    return custom_workload(f"tf_{offs[-1]}_{H}_{D}", 1, H, D, "bf16", TF, offsets=offs, tangent_std=0.5)


# (workload, key splits of the forward, tangent and query-tile pass; query splits of the key-tile pass)
SHAPES = [(_full(L, 2, D), 4, 4) for D in (64, 128) for L in (1, 33, 63, 65, 129)]
SHAPES += [(_full(1500, 12, 64), 2, 1), (_full(1537, 12, 128), 2, 1), (_full(1100, 2, 128), 4, 4)]
SHAPES += [(_tf((0, 70, 117, 297), 2, 128), 4, 4), (_tf((0, 40, 41, 208), 3, 64), 4, 4),
           (_tf((0, 500, 777), 12, 128), 2, 4), (_tf((0, 333, 1001), 14, 64), 2, 4)]
SHAPES += [(custom_workload("window", 1, 3, 128, "bf16", MASK_RANGES, tangent_std=0.5, offsets=[
    (0, 50, [(0, 50)]), (50, 60, []), (60, 331, [(0, 50), (60, 331)]),
    (331, 700, [(0, 7), (20, 50), (300, 700)])]), 4, 4)]


def _np(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def _close(name, got, want):
    assert got.shape == want.shape
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin), name  # (LSE = -inf of rows without keys)
    err = float(np.linalg.norm(got[fin] - want[fin]) / max(np.linalg.norm(want[fin]), 1e-3 * want.size ** 0.5))
    print(f"[split] {name} rel-L2 {err:.2e}", file=sys.stderr, flush=True)
    assert err <= 1e-2, (name, err)


@pytest.mark.gpu
@pytest.mark.parametrize("w,ks,qs", SHAPES, ids=lambda x: getattr(x, "name", str(x)))
def test_split_tiles_match_the_oracle(w, ks, qs):
    offs = list(w.offsets) or None
    x = make_inputs(w, "cpu", 3)
    g = {k: v.cuda() for k, v in x.items()}
    n = {k: _np(v) for k, v in x.items()}
    print(f"[split] {w.name} B={w.B} H={w.H} L={w.L} D={w.D} splits {ks}/{qs}", file=sys.stderr, flush=True)
    o, do, lse = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind, offs)
    of, lf = attn_fwd(g["Q"], g["K"], g["V"], w.kind, offs)
    assert torch.equal(o, of) and torch.equal(lse, lf)  # the same tiles, splits and merge order
    for name, got, want in zip(("O", "dO", "LSE"), (o, do, lse),
                               attention_jvp(*[n[k] for k in ("Q", "K", "V", "dQ", "dK", "dV")], w.kind, offs)):
        _close(name, _np(got), want)
    if w.kind == TF:
        half = w.L // 2
        t = [g[k][:, :, half:].contiguous() for k in ("dQ", "dK", "dV")]
        oz, dz, lz = attn_jvp_fwd_zero_clean(g["Q"], g["K"], g["V"], *t, offs)
        assert torch.equal(oz, o) and torch.equal(lz, lse)
        want = attention_jvp_zero_clean(n["Q"], n["K"], n["V"], *[n[k][:, :, half:] for k in ("dQ", "dK", "dV")], offs)
        _close("dO (zero clean)", _np(dz), want[1][:, :, half:])
    got = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    again = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    want = attention_vjp(n["Q"], n["K"], n["V"], n["dV"], w.kind, offs)
    for name, a, b in zip(("gQ", "gK", "gV"), got, want):
        _close(name, _np(a), b)


def test_split_rule(tmp_path):
    """choose_ksplit / choose_qsplit (plain C++) on the shapes above, and on full launches."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    big = [(_full(4680, 12, 128), 1, 1), (_full(32760, 12, 128), 1, 1),
           (_tf(tuple(4680 * i for i in range(8)), 12, 128), 1, 1),
           (_tf(tuple(1560 * i for i in range(22)), 80, 128), 1, 1)]
    lines = []
    for w, ks, qs in SHAPES + big:
        if w.kind == MASK_RANGES:
            continue
        o = ",".join(map(str, w.offsets)) or "0"
        kind = 0 if w.kind == MASK_FULL else 2
        lines.append(f"  {{ int32_t o[] = {{{o}}}; attn_chunk_layout l{{{kind}, {max(0, len(w.offsets) - 1)}, o, nullptr, nullptr}};"
                     f" check(l, {w.L}, {w.B * w.H}, {ks}, {qs}); }}")
    src = tmp_path / "rule.cpp"
    src.write_text('#include <cstdio>\n#include "layout.hpp"\nstatic int bad = 0;\n'
                   'static void check(const attn_chunk_layout& l, int L, int nbh, int ks, int qs) {\n'
                   '  attn::GroupTable gt; std::string err;\n'
                   '  if (!attn::build_groups(&l, L, &gt, &err)) { std::puts(err.c_str()); bad = 1; return; }\n'
                   '  const int k = attn::choose_ksplit(gt, L, nbh), q = attn::choose_qsplit(gt, L, nbh);\n'
                   '  if (k != ks || q != qs) { std::printf("L=%d heads=%d: %d/%d, expected %d/%d\\n", L, nbh, k, q, ks, qs); bad = 1; }\n'
                   '  // cut tiles cover every row once, in order, and never span a group bound unless uncut\n'
                   '  for (int br : {64, 128}) {\n'
                   '    attn::TileOrder o = attn::make_tile_order(&l, L, br);\n'
                   '    attn::cut_tiles(&o, gt, L, br);\n'
                   '    int at = 0;\n'
                   '    for (int t = 0; t < o.nt; ++t) {\n'
                   '      int a, b;\n'
                   '      attn::tile_rows(o, t, br, L, &a, &b);\n'
                   '      const bool one = attn::find_group(gt, a) == attn::find_group(gt, b - 1);\n'
                   '      if (a != at || b <= a || b > a + br || (o.nseg > 0 && !one)) { std::printf("tile %d L=%d br=%d\\n", t, L, br); bad = 1; }\n'
                   '      at = b;\n'
                   '    }\n'
                   '    if (at != L) { std::printf("tiles end at %d, L=%d\\n", at, L); bad = 1; }\n'
                   '    if (L == 2002 && br == 64 && o.nseg == 0) { std::puts("not cut"); bad = 1; }\n'
                   '  }\n'
                   '}\nint main() {\n' + "\n".join(lines) + "\n  return bad;\n}\n")
    csrc = os.path.join(ROOT, "paper_2606_25473_amd", "csrc")
    exe = str(tmp_path / "rule")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(csrc, "layout.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def _special(w, name, value, seed=5):
    """Inputs of w on the GPU with one element of tensor `name` set to value."""
    g = {k: v.cuda() for k, v in make_inputs(w, "cpu", seed).items()}
    g[name][0, 0, 3, 5] = value
    return g


F32 = [custom_workload(f"f32_{kind}_{L}_{D}", 1, H, D, "f32", kind, L=L if kind == MASK_FULL else 0,
                       offsets=None if kind == MASK_FULL else (0, 40, 41, L // 2))
       for kind, L, H, D in ((MASK_FULL, 1, 1, 128), (MASK_FULL, 65, 2, 64), (MASK_FULL, 127, 2, 128),
                             (MASK_FULL, 1030, 15, 64), (MASK_FULL, 1030, 15, 128), (TF, 298, 2, 128),
                             (TF, 298, 44, 64))]


@pytest.mark.gpu
@pytest.mark.parametrize("w", F32, ids=lambda w: f"{w.name}_H{w.H}")
def test_f32_three_part_products(w):
    """fp32 by bf16 part products, 64- and 128-row tiles: relative L2 <= 2e-6 against the oracle.
    Per product the parts left out are below 2^-24 (0.09 2^-24 rms, either sign) and an element
    takes at most L / 32 + 8 roundings of 2^-24 at the size of its result, random in sign:
    sqrt(40) 2^-24 = 4e-7, and as much again for exp2 and the scores (measured 2e-7 to 6e-7); a
    dropped part would show as 2^-17."""
    offs = list(w.offsets) or None
    x = make_inputs(w, "cpu", 4)
    g, n = {k: v.cuda() for k, v in x.items()}, {k: _np(v) for k, v in x.items()}
    print(f"[split] {w.name} H={w.H} L={w.L} D={w.D}", file=sys.stderr, flush=True)
    o, do, lse = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind, offs)
    want = attention_jvp(*[n[k] for k in ("Q", "K", "V", "dQ", "dK", "dV")], w.kind, offs)
    got = attn_bwd(g["Q"], g["K"], g["V"], o, g["dV"], lse, w.kind, offs)
    ref = attention_vjp(n["Q"], n["K"], n["V"], n["dV"], w.kind, offs)
    floor = 1e-3 * np.linalg.norm(n["dV"])  # (gradients that cancel exactly, as for L = 1)
    for name, a, b in list(zip(("O", "dO", "LSE"), (o, do, lse), want)) + list(zip(("gQ", "gK", "gV"), got, ref)):
        err = float(np.linalg.norm(_np(a) - b) / max(np.linalg.norm(b), floor))
        print(f"[split] {name} rel-L2 {err:.2e}", file=sys.stderr, flush=True)
        assert err <= (1e-4 if w.L == 1 else 2e-6), (name, err)


@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_operands_without_three_parts(D, value):
    """An infinite V makes infinite outputs, not NaN (no 0 inf products of parts); a NaN stays NaN;
    a V that rounds to an infinite bf16 gives the finite result.  Other columns and heads are
    untouched."""
    w = custom_workload("f32_special", 1, 2, D, "f32", MASK_FULL, L=70)
    print(f"[split] f32 D={D} V element {value}", file=sys.stderr, flush=True)
    g, clean = _special(w, "V", value), _special(w, "V", 0.25)
    run = lambda t: attn_jvp_fwd(t["Q"], t["K"], t["V"], t["dQ"], t["dK"], t["dV"], w.kind, None)
    o, do, lse = run(g)
    oc, doc, lsec = run(clean)
    assert torch.allclose(lse, lsec, rtol=1e-6, atol=1e-6)
    col = o[0, 0, :, 5]
    if value == 3.4e38:
        p = torch.softmax(g["Q"][0, 0].double() @ g["K"][0, 0].double().t().contiguous() / D ** 0.5, 1)[:, 3]
        assert torch.allclose(col.double(), p * g["V"][0, 0, 3, 5].double(), rtol=1e-4)
    else:
        assert bool((torch.isnan(col) if value != value else torch.isposinf(col)).all())
    keep = torch.ones(D, dtype=torch.bool)
    keep[5] = False
    assert torch.allclose(o[0, 0][:, keep], oc[0, 0][:, keep], rtol=1e-4, atol=1e-5)
    assert torch.allclose(o[0, 1], oc[0, 1], rtol=1e-4, atol=1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("offs,H,D", [((0, 40, 41, 149), 44, 64), ((0, 40, 41, 149), 44, 128), ((0, 500, 1013), 9, 128),
                                      ((0, 500, 1013), 2, 64), ((0, 640, 1280), 8, 64), ((0, 1), 3, 128), ((0, 31, 97), 2, 128),
                                      ((0, 100, 200), 100, 128), ((0, 40, 41, 149), 100, 128)],
                         ids=str)
def test_f32_zero_clean_drops_only_zero_products(offs, H, D):
    """fp32 with zero clean tangents, 64- and 128-row tiles, cut at the clean/noisy boundary or
    spanning it, the boundary inside a key block or at its end: equal to the dense call on padded
    tangents, and relative L2 <= 2e-6 against the oracle (as test_f32_three_part_products)."""
    w = custom_workload("f32_zc", 1, H, D, "f32", TF, offsets=offs)
    print(f"[split] f32 zero clean H={H} L={w.L} D={D}", file=sys.stderr, flush=True)
    half = w.L // 2
    x = make_inputs(w, "cpu", 6)
    for k in ("dQ", "dK", "dV"):
        x[k][:, :, :half] = 0
    g, n = {k: v.cuda() for k, v in x.items()}, {k: _np(v) for k, v in x.items()}
    t = [g[k][:, :, half:].contiguous() for k in ("dQ", "dK", "dV")]
    got = attn_jvp_fwd_zero_clean(g["Q"], g["K"], g["V"], *t, list(offs))
    o, do, lse = attn_jvp_fwd(g["Q"], g["K"], g["V"], g["dQ"], g["dK"], g["dV"], w.kind, list(offs))
    assert torch.equal(got[0], o) and torch.equal(got[1], do[:, :, half:]) and torch.equal(got[2], lse)
    want = attention_jvp(*[n[k] for k in ("Q", "K", "V", "dQ", "dK", "dV")], w.kind, list(offs))
    floor = 1e-3 * np.linalg.norm(n["dV"])
    for name, a, b in zip(("O", "dO", "LSE"), got, (want[0], want[1][:, :, half:], want[2])):
        err = float(np.linalg.norm(_np(a) - b) / max(np.linalg.norm(b), floor))
        print(f"[split] {name} rel-L2 {err:.2e}", file=sys.stderr, flush=True)
        assert err <= (1e-4 if w.L == 2 else 2e-6), (name, err)
