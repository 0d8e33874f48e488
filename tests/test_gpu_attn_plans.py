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
