"""The bf16 tile rules against measured launches (CPU; the rules are plain C++).

Each row: (batch, head) pairs, head size, mask, first chunk, other chunks' size, chunks, and the
times in us on one MI355X of the forward and of the JVP with full tiles, 2 and 4 key splits, and
of the backward with (query-tile splits, key-tile splits) = (1, 1), (2, 1), (4, 1), (1, 4).  What
the rules choose may be at most 6 % slower than full tiles in each of the three calls (the
backward's two passes are taken as independent), and on the small launches has to be within 10 %
of the best tiling on average.
"""
import math
import os
import shutil
import subprocess

import pytest

from paper_2606_25473_amd.workloads import WORKLOADS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# launches that fill the chip with full tiles, or nearly, and tiles of a few blocks
FULL = [
    (5, 128, "full", 73, 73, 1, [10.26, 10.29, 10.27], [12.88, 13.72, 12.95], [21.79, 23.16, 25.02, 21.5]),
    (10, 128, "full", 3346, 3346, 1, [95.21, 114.76, 112.5], [181.14, 271.7, 249.32], [290.01, 337.95, 325.0, 275.18]),
    (12, 128, "full", 2753, 2753, 1, [80.71, 98.14, 95.22], [153.94, 225.9, 210.45], [245.39, 286.14, 277.37, 234.18]),
    (6, 128, "full", 5590, 5590, 1, [154.26, 183.05, 179.11], [295.14, 438.16, 399.78], [475.26, 544.61, 518.81, 451.25]),
    (6, 64, "full", 11762, 11762, 1, [300.84, 392.58, 358.59], [874.22, 763.73, 740.41], [1088.21, 1045.32, 991.74, 1048.68]),
    (40, 64, "block_causal", 420, 420, 2, [25.33, 31.7, 27.11], [40.13, 50.04, 40.07], [59.67, 67.64, 63.21, 61.34]),
    (5, 128, "full", 13174, 13174, 1, [503.38, 623.19, 666.5], [1608.18, 1539.59, 1530.24], [1919.46, 1873.34, 1833.58, 1896.91]),
    (40, 64, "block_causal", 6, 28, 60, [42.88, 52.94, 57.76], [99.37, 82.22, 85.52], [136.48, 126.05, 131.13, 139.08]),
    (12, 64, "block_causal", 440, 463, 12, [102.93, 124.93, 109.75], [205.24, 218.36, 197.94], [285.38, 300.03, 285.15, 278.13]),
    (24, 64, "teacher_forcing", 118, 151, 7, [34.58, 39.26, 38.45], [56.23, 59.84, 56.27], [97.52, 101.05, 100.39, 91.75]),
    (40, 128, "block_causal", 34, 65, 21, [46.37, 52.29, 58.09], [93.03, 104.23, 105.18], [128.15, 139.63, 144.65, 132.75]),
    (24, 128, "teacher_forcing", 55, 57, 21, [51.19, 57.67, 66.12], [103.81, 106.87, 113.08], [154.0, 159.91, 170.82, 152.41]),
    (4, 64, "full", 8230, 8230, 1, [145.65, 184.74, 155.81], [272.33, 348.28, 306.02], [439.49, 484.99, 446.65, 400.76]),
]
# launches with few tiles
SMALL = [
    (8, 64, "block_causal", 75, 75, 40, [53.95, 41.81, 29.11], [106.25, 67.45, 46.57], [123.26, 101.69, 88.77, 104.9]),
    (10, 128, "block_causal", 36, 36, 21, [23.98, 21.3, 16.25], [55.76, 39.49, 28.62], [68.26, 57.17, 50.7, 60.52]),
    (3, 64, "teacher_forcing", 2637, 2637, 2, [179.37, 72.1, 65.07], [315.45, 124.21, 117.04], [376.01, 229.18, 221.09, 317.05]),
    (4, 64, "block_causal", 2199, 2199, 5, [189.28, 135.02, 133.01], [377.37, 250.12, 256.94], [424.87, 338.51, 334.68, 426.08]),
    (4, 128, "block_causal", 130, 422, 16, [137.58, 101.25, 75.04], [334.9, 240.01, 166.75], [346.67, 287.74, 248.17, 306.52]),
    (12, 64, "block_causal", 852, 937, 2, [38.82, 27.1, 27.25], [71.5, 44.29, 44.72], [90.52, 71.7, 71.69, 87.89]),
    (4, 128, "teacher_forcing", 1311, 1311, 3, [142.7, 69.31, 77.45], [317.32, 161.51, 171.24], [367.85, 262.32, 266.48, 308.81]),
    (6, 64, "block_causal", 316, 316, 5, [32.37, 25.76, 16.94], [61.98, 40.35, 26.35], [76.82, 63.96, 53.86, 64.11]),
    (5, 64, "teacher_forcing", 843, 843, 2, [62.07, 27.25, 22.67], [108.08, 43.58, 36.28], [136.57, 88.34, 85.03, 111.3]),
    (12, 64, "teacher_forcing", 383, 696, 3, [65.84, 41.0, 43.35], [102.88, 64.3, 66.4], [141.87, 113.62, 115.51, 135.0]),
    (16, 128, "teacher_forcing", 98, 98, 12, [46.37, 41.76, 43.13], [97.69, 73.74, 75.76], [132.74, 120.82, 123.04, 120.6]),
    (5, 128, "teacher_forcing", 2319, 2319, 2, [208.82, 123.62, 135.76], [432.38, 289.91, 295.74], [482.04, 376.45, 378.46, 469.38]),
    (3, 64, "full", 8119, 8119, 1, [133.22, 98.95, 107.2], [269.93, 171.64, 200.41], [296.14, 240.73, 249.47, 316.08]),
]
# the bf16 workloads that bench.py runs: all full tiles (its ratio of computed pairs counts those)
BENCH = [(w.B * w.H, w.D, w.kind, w.offsets[1] if w.offsets else w.L, w.offsets[1] if w.offsets else w.L,
          max(1, len(w.offsets) - 1)) for w in WORKLOADS.values() if w.dtype == "bf16"]
KIND = {"full": 0, "block_causal": 1, "teacher_forcing": 2}


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    """row -> (key splits of the forward and JVP, of the query-tile pass, query splits)"""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    rows, calls = FULL + SMALL + BENCH, []
    for nbh, D, kind, first, chunk, n, *_ in rows:
        o = [0] + [first + i * chunk for i in range(n)]
        L = o[-1] * (2 if kind == "teacher_forcing" else 1)
        calls.append(f"  {{ int32_t o[] = {{{','.join(map(str, o))}}}; attn_chunk_layout l{{{KIND[kind]}, {n}, o, nullptr, nullptr}};"
                     f" show(l, {L}, {nbh}, {D}); }}")
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", str(d / "rules")
    src.write_text('#include <cstdio>\n#include "layout.hpp"\n'
                   'static void show(const attn_chunk_layout& l, int L, int nbh, int D) {\n'
                   '  attn::GroupTable gt; std::string err;\n'
                   '  if (!attn::build_groups(&l, L, &gt, &err)) std::puts(err.c_str());\n'
                   '  else std::printf("%d %d %d\\n", attn::choose_ksplit(gt, L, nbh, D), attn::choose_bwd_ksplit(gt, L, nbh, D),'
                   ' attn::choose_qsplit(gt, L, nbh, D));\n'
                   '}\nint main() {\n' + "\n".join(calls) + "\n}\n")
    csrc = os.path.join(ROOT, "paper_2606_25473_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, "-I", os.path.join(ROOT, "include"), str(src),
                    os.path.join(csrc, "layout.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n")
    return {id(r): tuple(map(int, line.split())) for r, line in zip(rows, out)}


def _ratios(row, k, b, q):
    """(chosen time over full tiles' time, best time over it) of the forward, the JVP and the backward"""
    fwd, jvp, bwd = row[6:]
    i, j = {1: 0, 2: 1, 4: 2}[k], {1: 0, 2: 1, 4: 2}[b]
    keys = bwd[3] - bwd[0]
    return [(fwd[i] / fwd[0], min(fwd) / fwd[0]), (jvp[i] / jvp[0], min(jvp) / jvp[0]),
            ((bwd[j] + (keys if q > 1 else 0)) / bwd[0], (min(bwd[:3]) + min(keys, 0)) / bwd[0])]


@pytest.mark.parametrize("row", FULL + SMALL, ids=lambda r: f"{r[2]}_{r[3]}_{r[4]}x{r[5]}_H{r[0]}_D{r[1]}")
def test_no_launch_is_slower_than_with_full_tiles(row, chosen):
    for name, (got, _) in zip(("forward", "JVP", "backward"), _ratios(row, *chosen[id(row)])):
        assert got <= 1.06, (name, chosen[id(row)], got)


def test_small_launches_are_near_the_best_tiling(chosen):
    logs = [math.log(got / best) for r in SMALL for got, best in _ratios(r, *chosen[id(r)])]
    assert math.exp(sum(logs) / len(logs)) <= 1.10


def test_bench_workloads_take_full_tiles(chosen):
    assert len(BENCH) >= 4
    for row in BENCH:
        assert chosen[id(row)] == (1, 1, 1), row
