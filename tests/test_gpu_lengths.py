"""Attention forward and backward at the row lengths where the kernels' tile
counts, key parts and bias loads change, against the fp64 oracle (tolerances of
parity_util: bf16 inputs, fp32 sums).

* one key tile more or less around every tile count that has a kernel of its
  own (bf16, 65..512 keys);
* odd lengths (bias rows on 2-byte boundaries, the last element in half a
  dword of the plane) and even ones that are no multiple of 8, with odd head
  counts and several planes so that planes start on odd elements;
* row counts that leave row steps of the dQ / dBias pass partly empty, one and
  several row chunks per plane.
"""
import numpy as np
import pytest
import torch

from tests.parity_util import compare, gpu_run, make_inputs, oracle_run, to_device

pytestmark = pytest.mark.gpu

CASES = [
    # N, L, H, d, kwargs
    (3, 67, 3, 16, dict(rpb=1)),                   # single pass, three key tiles, odd planes
    (5, 95, 1, 32, dict()),
    (2, 131, 3, 8, dict(rpb=1)),                   # two passes at head_dim 8, odd length past 128 keys
    (9, 190, 1, 8, dict(mask="length")),
    (2, 193, 2, 8, dict(bias=False)),
    (9, 130, 2, 32, dict()),                       # two passes from here: 5, 6, 7 and 8 key tiles
    (1, 161, 3, 32, dict(mask="none")),
    (17, 222, 1, 32, dict(mask="length")),
    (6, 225, 2, 16, dict(rpb=3)),
    (5, 254, 2, 32, dict(p=0.4)),
    (70, 249, 1, 32, dict()),                      # several row chunks, odd rows of partial planes
    (4, 255, 3, 16, dict(rpb=1, gate=False)),
    (3, 257, 1, 32, dict(rpb=1)),                  # two waves to a row: 9 .. 12 key tiles
    (7, 290, 2, 8, dict(mask="length")),
    (11, 321, 1, 32, dict()),
    (2, 383, 1, 32, dict(bias=False)),
    (4, 385, 1, 16, dict(rpb=2)),                  # 13 .. 16 key tiles
    (5, 418, 1, 32, dict(mask="length")),
    (3, 511, 1, 32, dict()),
    (2, 481, 2, 8, dict(mask="none", rpb=1)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%dL%dH%dd%d" % c[:4])
def test_lengths_against_the_oracle(case):
    N, L, H, d, kw = case
    w, x = make_inputs(N, L, H, d, "bf16", seed=900 + L, **kw)
    print("\n[case]", case, flush=True)
    got = gpu_run(x, "bf16", w.rows_per_bias)
    compare(got, oracle_run(x, "bf16", w.rows_per_bias), "bf16", label=str(case))


@pytest.mark.parametrize("N,L,H,d", [(1100, 157, 1, 32), (600, 223, 1, 8), (700, 90, 3, 16), (1030, 33, 2, 32)])
def test_row_walking_forward_at_odd_tile_counts(N, L, H, d, monkeypatch):
    """The row-walking forward gives the one-unit kernel's bits (odd lengths, tile
    counts between the powers of two)."""
    from paper_2404_11068_amd import evo_attn as ea
    w, x = make_inputs(N, L, H, d, "bf16", seed=12 + L)
    print("\n[case] row-walking", (N, L, H, d), flush=True)
    dev = {n: to_device(x[n], "bf16") for n in ("q", "k", "v", "gate", "bias")}
    args = (dev["q"], dev["k"], dev["v"], dev["gate"], dev["bias"], torch.from_numpy(x["mask"]).cuda())
    res = []
    for rows in ("0", "1"):
        monkeypatch.setenv("EVO_ATTN_FWD_ROWS", rows)
        out, lse = ea.evo_attn_fwd(*args, rows_per_bias=N)
        torch.cuda.synchronize()
        res.append((out.view(torch.int16).cpu(), lse.cpu()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


def test_values_after_the_plane_do_not_matter():
    """An odd plane ends in half a dword: whatever lies in the other half (here a
    NaN) must not reach any output."""
    from paper_2404_11068_amd import evo_attn as ea
    for L, d in ((33, 16), (131, 8), (163, 32), (321, 32)):
        N, H = 3, 1
        w, x = make_inputs(N, L, H, d, "bf16", seed=5 + L)
        print("\n[case] tail", L, d, flush=True)
        ref = gpu_run(x, "bf16", w.rows_per_bias)
        dev = {n: to_device(x[n], "bf16") for n in ("q", "k", "v", "gate", "bias", "dout")}
        buf = torch.full((L * L + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")
        buf[:L * L] = dev["bias"].reshape(-1)
        bias = buf[:L * L].view(1, H, L, L)
        mask = torch.from_numpy(x["mask"]).cuda()
        args = (dev["q"], dev["k"], dev["v"], dev["gate"], bias, mask)
        out, lse = ea.evo_attn_fwd(*args, rows_per_bias=N)
        grads = ea.evo_attn_bwd(*args, out, lse, dev["dout"], rows_per_bias=N)
        torch.cuda.synchronize()
        for name, t in zip(("out", "lse", "dq", "dk", "dv", "dgate", "dbias"), (out, lse) + tuple(grads)):
            assert np.array_equal(t.double().cpu().numpy(), ref[name]), (L, d, name)


@pytest.mark.parametrize("L,d", [(131, 8), (190, 8), (254, 8), (163, 16), (222, 32), (317, 32), (418, 16)])
def test_minus_inf_bias_leaves_a_pair_out(L, d):
    """A bias of -inf gives the bits of a very low finite one (P = 0 either way), at
    the lengths past 128 keys that are no multiple of 8, forward and backward."""
    from paper_2404_11068_amd import evo_attn as ea
    N, H = 5, 2
    w, x = make_inputs(N, L, H, d, "bf16", seed=40 + L)
    print("\n[case] -inf bias", L, d, flush=True)
    dev = {n: to_device(x[n], "bf16") for n in ("q", "k", "v", "gate", "bias", "dout")}
    mask = torch.from_numpy(x["mask"]).cuda()
    drop = torch.rand(dev["bias"].shape, generator=torch.Generator().manual_seed(L)).cuda() < 0.1
    res = []
    for low in (-1e30, float("-inf")):
        args = (dev["q"], dev["k"], dev["v"], dev["gate"], dev["bias"].masked_fill(drop, low), mask)
        out, lse = ea.evo_attn_fwd(*args, rows_per_bias=N)
        res.append((out, lse) + tuple(ea.evo_attn_bwd(*args, out, lse, dev["dout"], rows_per_bias=N)))
    torch.cuda.synchronize()
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv", "dgate", "dbias"), *res):
        assert torch.isfinite(b).all() and torch.equal(a, b), (L, d, name)


@pytest.mark.parametrize("L,d", [(18, 16), (34, 32), (66, 8), (90, 16), (122, 32), (126, 8)])
def test_minus_inf_stays_in_its_row(L, d):
    """Up to 128 keys a pair bias of -inf gives NaN in its own query row's tile (the
    bias enters through a matrix product).  At lengths that are no multiple of 8 it
    must not reach the row before it, whose padded keys lie where it is stored: with -inf at the first key of every
    other row, the rows between them and the keys of the last tile give the bits of
    a very low finite bias."""
    from paper_2404_11068_amd import evo_attn as ea
    N, H = 3, 2
    w, x = make_inputs(N, L, H, d, "bf16", seed=80 + L, mask="none")
    print("\n[case] -inf in the next row", L, d, flush=True)
    dev = {n: to_device(x[n], "bf16") for n in ("q", "k", "v", "gate", "bias", "dout")}
    last = (L - 1) // 32 * 32
    res = []
    for low in (-1e30, float("-inf")):
        bias = dev["bias"].clone()
        bias[..., 1::2, 0] = low
        args = (dev["q"], dev["k"], dev["v"], dev["gate"], bias, None)
        out, lse = ea.evo_attn_fwd(*args, rows_per_bias=N)
        dq, dk, dv, dg, db = ea.evo_attn_bwd(*args, out, lse, dev["dout"], rows_per_bias=N)
        tiles = (dk[:, last:], dv[:, last:]) if last else ()
        res.append((out, lse, dg, dq[:, ::2], db[..., ::2, :]) + tiles)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(*res)):
        assert torch.isfinite(b).all() and torch.equal(a, b), (L, d, i)
