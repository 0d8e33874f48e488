"""Which kernels the attention passes launch for a call, and what these give
against the fp64 oracle (tolerances of parity_util), at sizes where the rules
that choose them change.  The kernels' names come from the profiler; where the
bench model mirrors a rule, the mirror is checked against them too."""
import os
import sys

import pytest
import torch

from tests.parity_util import compare, gpu_run, kernels_run, make_inputs, oracle_run, to_device

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

pytestmark = pytest.mark.gpu


def run_named(x, rpb):
    """(results, kernel names of the forward and the backward)"""
    names = kernels_run(lambda: gpu_run(x, "bf16", rpb))
    return gpu_run(x, "bf16", rpb), names


# The dQ/dBias pass where few rows share a bias plane: (N, L, H, d, rows per
# plane, kernel).  qbias_kernel (8 waves up to 256 keys, 16 past them) where the
# cost rule finds it no slower, with one row chunk per plane (it then writes
# dBias itself) and with several; never at lengths that are no multiple of 8.
FEW = [
    (3, 136, 2, 16, 1, "qbias_kernel<16, 8, true>"),
    (6, 160, 2, 32, 3, "qbias_kernel<32, 8, true>"),
    (4, 256, 1, 32, 2, "qbias_kernel<32, 8, true>"),
    (4, 216, 3, 16, 2, "qbias_kernel<16, 8, true>"),
    (3, 264, 2, 8, 3, "qbias_kernel<8, 16, true>"),
    (2, 512, 1, 32, 1, "qbias_kernel<32, 16, true>"),
    (4, 376, 1, 16, 2, "qbias_kernel<16, 16, true>"),
    (104, 136, 2, 16, 4, "qbias_kernel<16, 8, true>"),
    (16, 256, 2, 32, 16, "qbias_kernel<32, 8, true>"),   # four row chunks
    (27, 200, 5, 32, 9, "qbias_kernel<32, 8, true>"),    # two, the second with fewer rows
    (100, 136, 2, 16, 4, "rows_qbias_kernel<"),
    (8, 160, 2, 32, 4, "rows_qbias_kernel<"),
    (70, 136, 2, 32, 70, "rows_qbias_kernel<"),
    (3, 140, 2, 32, 1, "rows_qbias_kernel<"),
]


@pytest.mark.parametrize("case", FEW, ids=lambda c: "N%dL%dH%dd%drpb%d" % c[:5])
def test_few_rows_per_bias_plane(case):
    N, L, H, d, rpb, kernel = case
    w, x = make_inputs(N, L, H, d, "bf16", rpb=rpb, mask="length", seed=60 + L)
    print("\n[case]", case, flush=True)
    got, names = run_named(x, rpb)
    compare(got, oracle_run(x, "bf16", rpb), "bf16", label=str(case))
    ran = [n for n in names if "qbias_kernel" in n]
    assert len(ran) == 1 and ran[0].startswith(kernel), names
    assert kernel.startswith(bench.dq_kernel(w, 2) + "<")


def test_few_rows_without_a_workspace():
    """The no-alloc entry point gives the same bits."""
    from paper_2404_11068_amd import evo_attn as ea
    w, x = make_inputs(6, 200, 2, 32, "bf16", rpb=2, seed=3)
    dev = {n: to_device(x[n], "bf16") for n in ("q", "k", "v", "gate", "bias", "dout")}
    args = (dev["q"], dev["k"], dev["v"], dev["gate"], dev["bias"], torch.from_numpy(x["mask"]).cuda())
    out, lse = ea.evo_attn_fwd(*args, rows_per_bias=2)
    a = ea.evo_attn_bwd(*args, out, lse, dev["dout"], rows_per_bias=2)
    b = ea.evo_attn_bwd_noalloc(*args, out, lse, dev["dout"], rows_per_bias=2)
    torch.cuda.synchronize()
    assert all(torch.equal(s, t) for s, t in zip(a, b))


# Tile counts that split into odd numbers of groups, at the unit counts (rows
# times heads) where the split or the tile count of the kernel changes: (N, L, H,
# d, forward kernel, dK/dV kernel).  fwd_kernel<d, tiles, 1, even length, query
# groups>, kv_kernel<d, tiles, even length, key groups, waves per key tile>.
SPLITS = [
    (20, 72, 4, 8, "fwd_kernel<8, 3, 1, true, 1>", None),             # three tiles: never split
    (17, 67, 3, 16, "fwd_kernel<16, 3, 1, false, 1>", None),
    (17, 160, 3, 32, "fwd_kernel<32, 5, 1, true, 5>", "kv_kernel<32, 5, true, 5, 2>"),
    (13, 157, 4, 16, "fwd_kernel<16, 6, 1, false, 3>", "kv_kernel<16, 6, false, 3, 2>"),
    (32, 134, 4, 8, "fwd_kernel<8, 6, 1, true, 2>", "kv_kernel<8, 5, true, 1, 1>"),
    (43, 160, 3, 16, "fwd_kernel<16, 5, 1, true, 1>", "kv_kernel<16, 5, true, 1, 1>"),
    (17, 319, 3, 8, "fwd_kernel<8, 10, 1, false, 5>", "kv_kernel<8, 10, false, 5, 2>"),
    (16, 290, 4, 16, "fwd_kernel<16, 12, 1, true, 4>", "kv_kernel<16, 12, true, 4, 2>"),
    (12, 421, 3, 16, "fwd_kernel<16, 14, 1, false, 7>", "kv_kernel<16, 14, false, 7, 2>"),
    (16, 448, 4, 8, "fwd_kernel<8, 16, 1, true, 4>", "kv_kernel<8, 16, true, 4, 2>"),
]


@pytest.mark.parametrize("case", SPLITS, ids=lambda c: "N%dL%dH%dd%d" % c[:4])
def test_splits_of_small_calls(case):
    N, L, H, d, fwd, kv = case
    w, x = make_inputs(N, L, H, d, "bf16", mask="length", seed=70 + L)
    print("\n[case]", case, flush=True)
    got, names = run_named(x, N)
    compare(got, oracle_run(x, "bf16", N), "bf16", label=str(case))
    assert fwd in names, names
    assert kv is None or kv in names, names


# The dQ/dBias kernel's variants, rows_qbias_kernel<d, key tiles per wave, waves
# per row>: (N, L, H, d, rows per plane, tiles, waves).  Every one that the plan
# can take, with rows that leave the last chunk's row slots partly empty.
ROWS_QBIAS = [
    # one wave per row (eight rows in flight, no barrier in the row loop)
    (49, 131, 4, 8, 49, 5, 1), (41, 163, 4, 8, 41, 6, 1), (73, 197, 2, 8, 73, 7, 1), (41, 229, 3, 8, 41, 8, 1),
    (49, 142, 4, 16, 49, 5, 1), (41, 179, 4, 16, 41, 6, 1), (73, 222, 2, 16, 73, 7, 1), (41, 250, 3, 16, 41, 8, 1),
    (49, 157, 4, 32, 49, 5, 1), (41, 190, 4, 32, 41, 6, 1), (73, 198, 2, 32, 73, 7, 1),
    # two
    (5, 163, 1, 8, 5, 3, 2), (6, 229, 2, 8, 3, 4, 2), (5, 290, 1, 8, 5, 5, 2), (4, 350, 2, 8, 2, 6, 2),
    (5, 389, 2, 8, 5, 7, 2), (3, 490, 1, 8, 1, 8, 2),
    (5, 190, 1, 16, 5, 3, 2), (6, 250, 2, 16, 3, 4, 2), (5, 261, 1, 16, 5, 5, 2), (4, 383, 2, 16, 2, 6, 2),
    (5, 418, 2, 16, 5, 7, 2), (3, 511, 1, 16, 1, 8, 2),
    (5, 131, 1, 32, 5, 3, 2), (6, 197, 2, 32, 3, 4, 2), (5, 319, 1, 32, 5, 5, 2), (4, 322, 2, 32, 2, 6, 2),
    # four
    (5, 389, 1, 32, 5, 4, 4), (3, 453, 2, 32, 1, 4, 4),
]


@pytest.mark.parametrize("case", ROWS_QBIAS, ids=lambda c: "d%d_tiles%d_waves%d_N%dL%d" % (c[3], c[5], c[6], c[0], c[1]))
def test_rows_qbias_variants(case):
    N, L, H, d, rpb, tiles, waves = case
    w, x = make_inputs(N, L, H, d, "bf16", rpb=rpb, mask="length" if L % 2 else "bernoulli", seed=90 + L)
    print("\n[case]", case, flush=True)
    got, names = run_named(x, rpb)
    compare(got, oracle_run(x, "bf16", rpb), "bf16", label=str(case))
    assert "rows_qbias_kernel<%d, %d, %d>" % (d, tiles, waves) in names, names


# The one-unit forward and the dK/dV pass with two groups per unit (65 to 511
# units) and with one (from 512), at every tile count that has a kernel of its own:
# (N, L, H, d, tiles, forward groups, dK/dV tiles, groups).  Planes of eight rows,
# compared in the first, a middle and the last plane.
GROUPS = [
    (32, 163, 4, 16, 6, 2, 6, 2), (32, 197, 4, 32, 8, 2, 8, 2), (32, 290, 4, 8, 10, 2, 10, 2),
    (32, 347, 4, 16, 12, 2, 12, 2), (32, 418, 4, 8, 14, 2, 14, 2), (32, 511, 4, 16, 16, 2, 16, 2),
    (24, 317, 4, 32, 10, 2, 10, 2), (24, 384, 4, 32, 12, 2, 12, 2),
    (128, 131, 4, 16, 5, 1, 5, 1), (128, 162, 4, 32, 6, 1, 6, 1), (128, 251, 4, 8, 8, 1, 8, 1),
    (128, 319, 4, 8, 10, 1, 10, 1), (128, 322, 4, 16, 12, 1, 12, 1), (128, 447, 4, 8, 14, 1, 14, 1),
    (128, 490, 4, 8, 16, 1, 16, 1), (136, 317, 4, 32, 10, 1, 10, 1), (136, 384, 4, 32, 12, 1, 12, 1),
]


@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "N%dL%dH%dd%d" % c[:4])
def test_group_variants(case):
    N, L, H, d, ft, fg, kt, kg = case
    w, x = make_inputs(N, L, H, d, "bf16", rpb=8, mask="length", seed=30 + L)
    print("\n[case]", case, flush=True)
    got, names = run_named(x, 8)
    for plane in (0, N // 16, N // 8 - 1):
        r = slice(plane * 8, plane * 8 + 8)
        sub = {n: v[r] if n != "bias" else v[plane:plane + 1] for n, v in x.items()}
        cut = {n: v[r] if n != "dbias" else v[plane:plane + 1] for n, v in got.items()}
        compare(cut, oracle_run(sub, "bf16", 8), "bf16", label=str((case, plane)))
    even = "true" if L % 2 == 0 else "false"
    assert "fwd_kernel<%d, %d, 1, %s, %d>" % (d, ft, even, fg) in names, names
    assert "kv_kernel<%d, %d, %s, %d, 1>" % (d, kt, even, kg) in names, names
