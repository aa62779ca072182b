"""The fp16 output is the product Y * scale rounded once to binary16, on every
tile: bit for bit the oracle's value (one rounding of the exact product).  |Y|
stays below 2^24, so its binary32 value is exact and no other rounding enters.
A product rounded to binary32 first lands on the middle between two codes, and
then on the wrong one, for about one output in 50 000: the 2^20 outputs of a
case hold about 20 of those."""
import numpy as np
import pytest

import oracle
from paper_2607_12505_amd import nmspmm
from paper_2607_12505_amd import workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu

M_, N_, K_ = 2048, 512, 512


@pytest.mark.parametrize("plan", [None] + [(t, s) for t in range(12) for s in (1, 2)], ids=str)
def test_fp16_output_is_rounded_once(plan):
    print(f"fp16 rounding plan={plan}", flush=True)
    rng = np.random.default_rng(16)
    X = rng.integers(-128, 128, (M_, K_)).astype(np.int8)
    W = wl.random_nm(N_, K_, 2, 4, rng, full=True)
    W[::37] = 0                                                  # zero sums: the product's sign is the scale's
    scale = rng.uniform(1e-5, 1e-2, N_).astype(np.float32)
    scale[1::2] *= -1
    scale[3::16] *= 1e-6                                         # subnormal results
    scale[5::16] *= 1e3                                          # overflow to infinity
    packed = nmspmm.compress(W, 2, 4)
    ref = oracle.matmul_i8(X, W)
    assert np.abs(ref).max() < 2 ** 24
    p = None if plan is None else nmspmm.make_plan(packed.desc.kind, *plan)
    _, Yh = gu.run_sparse(X, packed, scale, want_i32=False, want_f16=True, plan=p)
    want = oracle.dequant_f16(ref, scale).view(np.uint16)
    bad = np.flatnonzero(Yh.ravel() != want.ravel())
    assert bad.size == 0, f"{bad.size} of {want.size} differ, first {Yh.ravel()[bad[:3]]} for {want.ravel()[bad[:3]]}"
