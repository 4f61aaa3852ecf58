"""GPU rows from any element boundary: 16-byte accesses that never leave the row, the last
slots of a row moved back so that they end with it, duplicates counted once. Widths around every
slot edge of the register tiles, the workgroup-held rows and the rows read twice; in place and on
buffers that are not 16-byte aligned; against the fp64 oracle (bounds of gpu_util)."""

import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import (backward_inputs, bits_to_f64, compare, compare_backward, covered_mask, run_plan,
                      run_plan_backward, to_device, to_host_bits)

pytestmark = pytest.mark.gpu

# remainders of every size at one vector, one slot and just past it, per kernel class
EDGES = {
    "f32": [[4, 5, 6, 7, 61, 65, 127], [129, 257, 258, 511], [513, 641, 1023], [1025, 1281, 2047],
            [2049, 2565, 3071, 3073, 4097, 8191], [8193, 16383], [16385, 32767, 32769, 40001]],
    "bf16": [[8, 9, 11, 15, 121, 129, 255], [257, 513, 515, 1023], [1025, 2047], [2049, 2571, 4095],
             [4097, 5125, 6143, 6145, 8191], [8193, 10241, 12289, 16383], [16385, 32767, 32771, 40003]],
}


@pytest.mark.parametrize("kclass", range(7))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_slot_edges_in_place_and_unaligned(dtype, kclass):
    cols = EDGES[dtype][kclass]
    rows = [(5, 3, 4, 2, 3, 1, 2)[i % 7] for i in range(len(cols))]
    w = workloads.custom(rows, cols, dtype=dtype, sigma=3.0, seed=50 + kclass, gap=1, base=1)
    n = int(w.offsets[-1])
    offs = w.offsets[: w.batch]
    mask = covered_mask(offs, w.rows, w.cols, n)
    ref = oracle.softmax(w.x, dtype, offs, w.rows, w.cols)
    first = None
    for start in (0, 1, 3):  # elements past a 16-byte boundary where the buffer begins
        print(f"[slot edges {dtype} class {kclass} start {start}] {cols}", flush=True)
        buf = to_device(np.concatenate([np.zeros(start, w.x.dtype), w.x]), dtype)
        y = buf[start:]
        _, st = run_plan(w, "balanced", x=y, out=y)
        assert st["kernel_class"] == kclass
        bits = to_host_bits(y)
        compare(bits, ref, dtype, mask)
        assert np.array_equal(bits[~mask], to_host_bits(to_device(w.x, dtype))[~mask]), "a gap was written"
        first = bits if first is None else first
        assert np.array_equal(bits, first)
    yb, dyb = backward_inputs(w)
    bref = oracle.softmax_backward(yb, dyb, dtype, offs, w.rows, w.cols, nthreads=16)
    for start in (0, 1):
        buf = to_device(np.concatenate([np.zeros(start, dyb.dtype), dyb]), dtype)
        dx = buf[start:]
        run_plan_backward(w, to_device(yb, dtype), dx, "balanced", dx=dx)  # in place over dy
        compare_backward(to_host_bits(dx), bref, yb, dyb, dtype, offs, w.rows, w.cols, mask)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_special_values_among_duplicates(dtype):
    """Rows whose duplicated elements are masked, the largest of the row, or NaN."""
    cols = [77, 333, 1001, 2051, 8193]
    w = workloads.custom([4] * len(cols), cols, dtype=dtype, sigma=1.0, seed=60, gap=1, base=1)
    x = bits_to_f64(w.x) if dtype == "bf16" else w.x.astype(np.float64)
    epv = 4 if dtype == "f32" else 8
    nan_rows = np.zeros(x.size, bool)
    for o, c in zip(w.offsets, cols):
        r = x[o:o + 4 * c].reshape(4, c)
        r[0, :] = -np.inf            # fully masked
        r[1, c - epv:] = -np.inf     # the last vector masked
        r[2, c - epv:] = 9.0         # ... or holding nearly the whole sum
        r[3, max(0, c - epv)] = np.nan
        nan_rows[o + 3 * c:o + 4 * c] = True
    t = torch.from_numpy(x.astype(np.float32)).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    host = t.numpy() if dtype == "f32" else t.view(torch.int16).numpy().view(np.uint16)
    ref = oracle.softmax(host, dtype, w.offsets[: w.batch], w.rows, w.cols)
    mask = covered_mask(w.offsets[: w.batch], w.rows, w.cols, x.size)
    out, _ = run_plan(w, "balanced", x=t.cuda())
    bits = to_host_bits(out)
    compare(bits, ref, dtype, mask & ~nan_rows)
    assert np.all(np.isnan(bits_to_f64(bits)[nan_rows]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_nan_anywhere_in_rows_read_twice(dtype):
    """Rows of more than 32768 elements, aligned and shifted: a NaN in a lane's first vectors, in
    its last ones, or after vectors that are all masked makes the whole row NaN, and only that row."""
    cols = [32776, 32769, 40001]
    w = workloads.custom([5] * len(cols), cols, dtype=dtype, sigma=1.0, seed=61, gap=1, base=8)
    x = bits_to_f64(w.x) if dtype == "bf16" else w.x.astype(np.float64)
    nan_rows = np.zeros(x.size, bool)
    for o, c in zip(w.offsets, cols):
        r = x[o:o + 5 * c].reshape(5, c)
        r[0, 5] = np.nan
        r[0, 6] = 30.0               # the row's maximum, in the same lane
        r[1, c - 1] = np.nan
        r[2, :32768] = -np.inf
        r[2, c - 1] = np.nan
        r[3, :32768] = -np.inf       # no NaN: the probabilities of the rest
        nan_rows[o:o + 3 * c] = True
    t = torch.from_numpy(x.astype(np.float32)).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    host = t.numpy() if dtype == "f32" else t.view(torch.int16).numpy().view(np.uint16)
    ref = oracle.softmax(host, dtype, w.offsets[: w.batch], w.rows, w.cols)
    mask = covered_mask(w.offsets[: w.batch], w.rows, w.cols, x.size)
    out, st = run_plan(w, "balanced", x=t.cuda())
    assert st["kernel_class"] == 6
    bits = to_host_bits(out)
    compare(bits, ref, dtype, mask & ~nan_rows)
    assert np.all(np.isnan(bits_to_f64(bits)[nan_rows]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_y_among_duplicates(dtype):
    """Backward rows with one infinite y where slots meet: every other dx follows from the row's
    infinite sum (an element that two lanes hold must not add inf * 0 to it)."""
    epv = 4 if dtype == "f32" else 8
    cols = [77, 333, 1001, 1999, 2051, 8193, 33001]  # every tile, workgroup-held, read twice
    at = [[p for p in [c - epv, c - 1] + [g * epv - 1 for g in (8, 16, 32, 64, 256, 512)] if p < c] for c in cols]
    w = workloads.custom([len(a) for a in at], cols, dtype=dtype, sigma=1.0, seed=62, gap=1, base=1)
    yb, dyb = backward_inputs(w)
    inf = np.inf if dtype == "f32" else 0x7F80
    one = 1.0 if dtype == "f32" else 0x3F80
    for o, c, ps in zip(w.offsets, cols, at):
        for r, p in enumerate(ps):
            yb[o + r * c + p] = inf
            dyb[o + r * c + p] = one
    ref = oracle.softmax_backward(yb, dyb, dtype, w.offsets[: w.batch], w.rows, w.cols, nthreads=16)
    mask = covered_mask(w.offsets[: w.batch], w.rows, w.cols, yb.size)
    dx, st = run_plan_backward(w, to_device(yb, dtype), to_device(dyb, dtype), "balanced")
    assert st["kernel_class"] == 6
    got = bits_to_f64(to_host_bits(dx))
    assert np.count_nonzero(np.isinf(ref[mask])) > mask.sum() // 2
    assert np.array_equal(got[mask], ref[mask], equal_nan=True)
