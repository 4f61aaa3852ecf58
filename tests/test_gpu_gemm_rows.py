"""GPU parity of the products by row-tile workgroups, and of the general forms on the shapes they
take, against the fp64 oracle.  The score softmax (k <= 128, n <= 2048): both workgroup sizes at the edges of their columns, reductions that do and do not
fill their slices, partial row tiles, several rounds per workgroup, operands at any element
boundary, negative and zero scale, and infinities in columns that are not there."""

import numpy as np
import pytest
import torch

import paper_2002_07062_amd as bsm
from gpu_util import bits_to_f64
from test_gpu_gemm import _check as check_product
from test_gpu_gemm import _dev_bf16, _operands
from test_gpu_gemm_forms import SHAPES as FORM_SHAPES
from test_gpu_gemm_forms import _product
from test_gpu_gemm_softmax import _check

pytestmark = pytest.mark.gpu

SHAPES = [(2, 33, 513, 1), (3, 31, 700, 72), (2, 65, 1024, 64), (1, 40, 1025, 128), (2, 32, 2048, 65),
          (1, 1, 1999, 100), (1, 5, 2047, 127), (9, 200, 600, 8)]


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_row_tiles_against_the_oracle(shape, out):
    batch, m, n, k = shape
    print(f"[rows {shape} {out}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=500 + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    for alpha in (0.125, -0.125, 0.0):
        got = _product(shape, "nt_softmax", out, a_d, b_d, alpha)
        _check(got, a, b, batch, m, n, k, alpha, out)
    want = _product(shape, "nt_softmax", out, a_d, b_d, 0.125)
    for schedule in ("rr", "xcd"):
        assert np.array_equal(_product(shape, "nt_softmax", out, a_d, b_d, 0.125, schedule=schedule), want)
    few = {"n_cu": 3, "n_xcd": 1, "flags": bsm.BSM_FLAG_TEMPORAL}  # many rounds per workgroup
    assert np.array_equal(_product(shape, "nt_softmax", out, a_d, b_d, 0.125, topology=few), want)
    odd = [torch.cat([torch.zeros(3, device="cuda", dtype=torch.bfloat16), t])[3:] for t in (a_d, b_d)]
    assert np.array_equal(_product(shape, "nt_softmax", out, *odd, 0.125), want)


@pytest.mark.parametrize("topology", [None, {"wg_threads": 256}], ids=["row tiles", "two passes"])
@pytest.mark.parametrize("n,k", [(520, 72), (1100, 64)])
def test_infinite_operands(n, k, topology):
    """-inf, +inf and NaN in one row of B reach the row's column only as the softmax says: a
    logit of -inf is a probability of 0, one of +inf or NaN makes its row NaN; the last row of B,
    that stands in for rows past n, is -inf."""
    m = 40
    a = np.abs(_operands(1, m, n, k, seed=7)[0].astype(np.int32) & 0x7FFF).astype(np.uint16)  # positive
    b = _operands(1, m, n, k, seed=8)[1].copy()
    b.reshape(n, k)[[3, n - 1]] = 0xFF80
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    got = bits_to_f64(_product((1, m, n, k), "nt_softmax", "f32", a_d, b_d, 0.01, topology=topology)).reshape(m, n)
    assert np.all(got[:, [3, n - 1]] == 0.0) and np.allclose(got.sum(1), 1.0, atol=1e-5)
    for special in (0x7F80, 0x7FC0):
        for row in (5, n // 2, n - 2):  # the first, a middle and the last column block
            c = b.copy()
            c.reshape(n, k)[row, 0] = special
            got = bits_to_f64(_product((1, m, n, k), "nt_softmax", "f32", a_d, _dev_bf16(c), 0.01, topology=topology))
            assert np.all(np.isnan(got))


def test_plan_takes_the_row_tiles():
    """Workgroups of four waves up to 1024 columns, of eight up to 2048; a topology that names
    a workgroup size or more workgroups, longer rows and longer reductions keep the general form."""
    def describe(n, k, topology=None):
        p = bsm.bsm_gemm_plan_create(8, 64, n, k, "nt_softmax", "bf16", topology=topology, device=0)
        st = bsm.bsm_plan_describe(p)
        p.destroy()
        return st["wg_threads"], st["n_wg"] // torch.cuda.get_device_properties(0).multi_processor_count

    assert describe(513, 64) == (256, 2) and describe(1024, 128) == (256, 2)
    assert describe(1025, 64) == (512, 1) and describe(2048, 128) == (512, 1)
    assert describe(2049, 128) == (256, 2) and describe(1100, 136) == (256, 3)
    assert describe(600, 64, {"wg_threads": 256}) == (256, 3) and describe(1100, 64, {"wg_threads": 256}) == (256, 3)
    assert describe(1100, 64, {"wg_per_cu": 2}) == (256, 2)


# row tiles of one and several rounds, columns split over several workgroups, reductions of fewer
# slices than waves and of more, the operand's last piece
PLAIN = [("nt", (2, 33, 65, 72)), ("nt", (1, 1, 2050, 128)), ("nt", (5, 40, 300, 1)), ("nt", (3, 97, 511, 127)),
         ("nt", (900, 3, 130, 40)), ("nn", (2, 33, 65, 130)), ("nn", (1, 31, 513, 64)), ("nn", (4, 70, 96, 333)),
         ("nn", (3, 5, 7, 600)), ("nn", (1, 64, 128, 8)), ("nn", (700, 2, 64, 65))]


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("layout,shape", PLAIN, ids=lambda s: s if isinstance(s, str) else "x".join(map(str, s)))
def test_plain_row_tiles_against_the_oracle(layout, shape, out):
    batch, m, n, k = shape
    print(f"[plain rows {layout} {shape} {out}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=600 + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    want = _product(shape, layout, out, a_d, b_d, 0.25)
    check_product(want, a, b, batch, m, n, k, layout, out, 0.25)
    for topology in ({"n_cu": 3, "n_xcd": 1, "flags": bsm.BSM_FLAG_TEMPORAL}, {"wg_per_cu": 3}):
        assert np.array_equal(_product(shape, layout, out, a_d, b_d, 0.25, topology=topology), want)
    for schedule in ("rr", "xcd"):
        assert np.array_equal(_product(shape, layout, out, a_d, b_d, 0.25, schedule=schedule), want)
    odd = [torch.cat([torch.zeros(3, device="cuda", dtype=torch.bfloat16), t])[3:] for t in (a_d, b_d)]
    assert np.array_equal(_product(shape, layout, out, *odd, 0.25), want)


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 512, 512, 200), (1, 256, 400, 72), (8, 500, 256, 133)], ids=lambda s: "x".join(map(str, s)))
def test_context_column_parts_under_every_schedule(shape, out):
    """Two or three workgroups to a CU, by how many the busiest XCD has (the balanced order deals few
    row tiles to one XCD, the XCD order to all): the same bits."""
    batch, m, n, k = shape
    print(f"[context parts {shape} {out}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=800 + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    want = _product(shape, "nn", out, a_d, b_d, 0.5)
    check_product(want, a, b, batch, m, n, k, "nn", out, 0.5)
    for schedule in ("rr", "xcd"):
        assert np.array_equal(_product(shape, "nn", out, a_d, b_d, 0.5, schedule=schedule), want)
    assert np.array_equal(_product(shape, "nn", out, a_d, b_d, 0.5, topology={"wg_per_cu": 3}), want)
    assert np.array_equal(_product(shape, "nn", out, a_d, b_d, 0.5, topology={"n_cu": 5, "n_xcd": 4}), want)


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["nt", "nn", "nt_softmax"])
@pytest.mark.parametrize("shape", FORM_SHAPES + [(2, 70, 520, 128), (2, 70, 700, 72)], ids=lambda s: "x".join(map(str, s)))
def test_general_forms_on_small_shapes(shape, layout, out):
    """A topology that names the workgroup size keeps the general forms: the small shapes that
    row tiles take by default, through every one of them."""
    batch, m, n, k = shape
    print(f"[general {layout} {shape} {out}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=700 + m + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    alpha = 1.0 / np.sqrt(k)
    got = _product(shape, layout, out, a_d, b_d, alpha, topology={"wg_threads": 256})
    if layout == "nt_softmax":
        _check(got, a, b, batch, m, n, k, alpha, out)
    else:
        check_product(got, a, b, batch, m, n, k, layout, out, alpha)
    assert np.array_equal(_product(shape, layout, out, a_d, b_d, alpha, topology={"wg_threads": 256}, schedule="rr"), got)
    if layout == "nt":  # the same sums in the same order
        assert np.array_equal(_product(shape, layout, out, a_d, b_d, alpha), got)


def test_default_topology_is_no_topology():
    """bsm_default_topology's own values give the plan, and the bits, that NULL gives."""
    shape = (2, 70, 1100, 72)
    a, b = _operands(*shape, seed=9)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    stats = []
    for topo in (None, bsm.bsm_default_topology(0)):
        p = bsm.bsm_gemm_plan_create(*shape, "nt_softmax", "bf16", topology=topo, device=0)
        st = bsm.bsm_plan_describe(p)
        stats.append((st["wg_threads"], st["n_wg"], st["n_items"]))
        p.destroy()
    assert stats[0] == stats[1] and stats[0][0] == 512
    assert np.array_equal(_product(shape, "nt_softmax", "bf16", a_d, b_d, 0.125, topology=bsm.bsm_default_topology(0)),
                          _product(shape, "nt_softmax", "bf16", a_d, b_d, 0.125))


@pytest.mark.parametrize("layout,shape", [("nt", (1, 40, 2050, 128)), ("nn", (2, 64, 500, 130)), ("nt", (40, 200, 300, 64))])
def test_trace_has_every_column_part(layout, shape):
    """Column parts leave a record per wave each, with the times of their own work; the rows are
    counted once."""
    batch, m, n, k = shape
    print(f"[trace parts {layout} {shape}]", flush=True)
    a, b = _operands(*shape, seed=10)
    p = bsm.bsm_gemm_plan_create(*shape, layout, "f32", device=0)
    st = bsm.bsm_plan_describe(p)
    waves = st["wg_threads"] // 64
    assert st["n_wg"] > st["n_workers"]
    c = torch.empty(batch * m * n, device="cuda")
    trace = torch.full((st["trace_bytes"] + 32,), 255, dtype=torch.uint8, device="cuda")
    bsm.bsm_gemm_execute(p, _dev_bf16(a), _dev_bf16(b), c, 0.25, trace=trace)
    torch.cuda.synchronize()
    p.destroy()
    rec = trace.cpu().numpy().view(bsm.TRACE_DTYPE)
    assert rec["wg"][-1] == 0xFFFFFFFF, "written past the trace"
    rec = rec[:-1]
    assert np.array_equal(rec["wg"], np.repeat(np.arange(st["n_wg"], dtype=np.uint32), waves))
    assert np.all(rec["t_start"] > 0) and np.all(rec["t_end"] >= rec["t_start"])
    assert int(rec["rows"].sum()) == batch * m
