"""What the numeric forms of the kernels promise, at bounds that a wrong form
would miss: complex64 products from exact bfloat16 parts are as accurate as
FP32 products, and the interpreter's two kernels give the same bits."""
import json
import os

import numpy as np
import pytest

import paper_1805_01450_amd as q
from workload import generate_circuit, random_bitstrings

pytestmark = pytest.mark.gpu
PLANS = os.path.join(os.path.dirname(q.__file__), "plans")


@pytest.fixture(scope="module", autouse=True)
def cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def test_exact_parts_are_as_accurate_as_fp32_products(cuda):
    """Single slices of 64 bitstrings of 8x8x40: the 2-norm error against the
    complex128 plan on the vector ALUs.  Bound: twice the error of the
    complex64 plan on the vector ALUs, whose products are FP32 (a plan's sums
    differ in order, which moves it by a few percent).  Without one of the six
    part products the error is that of BF16x3 or worse, about eight times as
    large."""
    with open(os.path.join(PLANS, "8x8x40.json")) as f:
        rec = json.load(f)
    cz = rec["circuit"]
    c = q.Circuit(generate_circuit(cz["n"], cz["depth"], cz["seed"]))
    bits = random_bitstrings(64, 64, 17)

    def values(prec, vector_only):
        p = q.Plan(c, rec["sliced"], rec["order"], prec=prec, engine=q.QGM_ENGINE_WIDE, vector_only=vector_only)
        print("[forms]", prec, vector_only, flush=True)
        v = np.stack([p.amplitudes_range(bits, None, s, s + 1) for s in (5, 2970, 8190)])
        p.release_workspace()
        cuda.cuda.empty_cache()
        return v[..., 0] + 1j * v[..., 1]

    want = values(q.QGM_C128, True)
    error = lambda v: np.linalg.norm(v - want) / np.linalg.norm(want)
    parts, fp32 = error(values(q.QGM_C64, False)), error(values(q.QGM_C64, True))
    print("[forms] error: exact parts", parts, "fp32 products", fp32, flush=True)
    assert parts <= 2 * fp32


@pytest.mark.parametrize("prec", [q.QGM_C128, q.QGM_C64, q.QGM_BF16X3])
@pytest.mark.parametrize("n,depth,k", [(4, 10, 3), (5, 12, 5)])
def test_both_interpreter_kernels_give_the_same_bits(n, depth, k, prec):
    """Level kernel up to 32768 items (128 per compute unit), one wavefront
    per 64 items beyond."""
    c = q.Circuit(generate_circuit(n, depth, 0))
    sl, order = c.plan_slices(k_req=k, time_budget_s=0.1, flags=q.QGM_PLAN_DETERMINISTIC)
    p = q.Plan(c, sl, order, prec=prec, engine=q.QGM_ENGINE_INTERPRETER)
    per = 1 << len(sl)
    bits = random_bitstrings(n * n, 32768 // per + 9, 3)
    print("[forms] interpreter", n, prec, flush=True)
    every = p.amplitudes(bits)
    for count in (1, 4096 // per + 1, 32768 // per):
        assert np.array_equal(p.amplitudes(bits[:count]), every[:count]), count
