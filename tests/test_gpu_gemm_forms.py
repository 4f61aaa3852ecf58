"""GPU parity of the matrix products' forms at the edges of their dispatch, against the fp64
oracle and, bit for bit, between launches that cut the rows differently: operands whose rows are
not whole 16-byte pieces (any element boundary, the operand's last piece, operands shorter than
one piece), A held in registers for 64 < k <= 128, and NN in 128-column blocks."""

import numpy as np
import pytest
import torch

import paper_2002_07062_amd as bsm
from gpu_util import bits_to_f64, to_host_bits
from test_gpu_gemm import _check as check_product
from test_gpu_gemm import _dev_bf16, _operands
from test_gpu_gemm_softmax import _check as check_softmax

pytestmark = pytest.mark.gpu


def _product(shape, layout, out, a_d, b_d, alpha, topology=None, schedule="balanced", pad=5):
    batch, m, n, k = shape
    c = torch.full((batch * m * n + pad,), float("nan"), device="cuda",
                   dtype=torch.float32 if out == "f32" else torch.bfloat16)
    p = bsm.bsm_gemm_plan_create(batch, m, n, k, layout, out, schedule, topology=topology, device=0)
    bsm.bsm_gemm_execute(p, a_d, b_d, c, alpha)
    torch.cuda.synchronize()
    p.destroy()
    bits = to_host_bits(c)
    assert np.all(np.isnan(bits_to_f64(bits[batch * m * n:]))), "written past C"
    return bits[: batch * m * n]


# n and k just inside and outside each form (blocks of 64 and 128 columns, reductions of 64 and
# 128), odd lengths whose rows start at every element boundary, and operands of 1..9 elements
SHAPES = [(2, 130, 65, 72), (1, 33, 129, 128), (3, 31, 200, 120), (2, 129, 64, 136), (2, 64, 66, 65),
          (3, 37, 96, 333), (1, 128, 128, 200), (2, 50, 130, 64), (1, 70, 81, 77), (1, 1, 7, 1),
          (1, 1, 1, 9), (1, 3, 3, 3), (3, 5, 511, 127)]


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["nt", "nn", "nt_softmax"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forms_against_the_oracle_and_each_other(shape, layout, out):
    batch, m, n, k = shape
    print(f"[forms {layout} {shape} {out}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=300 + m + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    alpha = 1.0 / np.sqrt(k)
    got = _product(shape, layout, out, a_d, b_d, alpha)
    if layout == "nt_softmax":
        check_softmax(got, a, b, batch, m, n, k, alpha, out)
    else:
        check_product(got, a, b, batch, m, n, k, layout, out, alpha)
    assert np.array_equal(_product(shape, layout, out, a_d, b_d, alpha, schedule="rr"), got)
    if layout != "nt_softmax" and out == "bf16":
        # the general forms (a named workgroup size keeps row tiles out); four workgroups per CU
        # leave no room for the 128-wide ones: the same bits without them
        general = _product(shape, layout, out, a_d, b_d, alpha, topology={"wg_threads": 256})
        assert np.array_equal(_product(shape, layout, out, a_d, b_d, alpha, topology={"wg_threads": 256, "wg_per_cu": 4}), general)


@pytest.mark.parametrize("n,k", [(520, 128), (700, 72), (513, 64), (600, 136), (513, 100), (64, 40)])
def test_two_pass_softmax_forms(n, k):
    """A named workgroup size keeps the two passes: A in registers for one and for two slices
    of k, A staged at every step, operands at any boundary, and one column block."""
    batch, m = 2, 70
    a, b = _operands(batch, m, n, k, seed=400 + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    for alpha in (0.125, -0.125):
        for out in ("f32", "bf16"):
            got = _product((batch, m, n, k), "nt_softmax", out, a_d, b_d, alpha, topology={"wg_threads": 256})
            check_softmax(got, a, b, batch, m, n, k, alpha, out)
            for topology in ({"wg_threads": 256, "flags": bsm.BSM_FLAG_TEMPORAL}, {"wg_threads": 256, "n_cu": 3}):
                assert np.array_equal(_product((batch, m, n, k), "nt_softmax", out, a_d, b_d, alpha, topology=topology,
                                               schedule="xcd"), got)


@pytest.mark.parametrize("shape", [(2, 128, 65, 72), (3, 512, 256, 128), (1, 512, 260, 96), (1, 512, 260, 104)],
                         ids=lambda s: "x".join(map(str, s)))
def test_both_forms_of_the_plain_scores(shape):
    """fp32 scores of whole rounds, 64 < k <= 128: with A staged at every step, where that is faster, and
    (two workgroups per CU) with A in registers the same sums in the same order."""
    batch, m, n, k = shape
    print(f"[plain scores, both forms {shape}]", flush=True)
    a, b = _operands(batch, m, n, k, seed=900 + n)
    a_d, b_d = _dev_bf16(a), _dev_bf16(b)
    got = _product(shape, "nt", "f32", a_d, b_d, 0.25, topology={"wg_threads": 256})
    check_product(got, a, b, batch, m, n, k, "nt", "f32", 0.25)
    assert np.array_equal(_product(shape, "nt", "f32", a_d, b_d, 0.25, topology={"wg_threads": 256, "wg_per_cu": 2}), got)
