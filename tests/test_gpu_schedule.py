"""GPU parity of calls without a plan on the tiles that no plan names: the
outputs against the oracle (int32 and int8 equal, fp16 within the rounding of
assert_f16_close), with guard bands after them."""
import numpy as np
import pytest

import oracle
from paper_2607_12505_amd import nmspmm
from paper_2607_12505_amd import workloads as wl
from schedule_cases import CASES, PATTERN
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", CASES, ids=str)
def test_unplanned_tile_matches_oracle(case):
    import torch
    m, n, k, kind, mode, _ = case
    print(f"schedule case {case}", flush=True)
    rng = np.random.default_rng(m + n + k)
    X = rng.integers(-128, 128, (m, k)).astype(np.int8)
    W = wl.random_nm(n, k, *PATTERN[kind], rng)
    scale = rng.uniform(1e-6, 1e-3, n).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    sd = torch.from_numpy(scale).cuda()
    Yb, Yhb = gu.device_outputs(m, n, mode == nmspmm.NM_OUT_I32, mode == nmspmm.NM_OUT_F16)
    Yqb = torch.full((m * n + gu.GUARD,), -128, dtype=torch.int8, device="cuda")
    Yq = gu.view2d(Yqb, m, n) if mode == nmspmm.NM_OUT_I8 else None
    kw = dict(Y=gu.view2d(Yb, m, n), scale=sd if Yhb is not None else None, Yh=gu.view2d(Yhb, m, n), Yq=Yq,
              qscale=sd if Yq is not None else None)
    if kind == nmspmm.NM_KIND_DENSE:
        nmspmm.gemm_i8_dense(Xd, torch.from_numpy(W).cuda(), **kw)
    else:
        nmspmm.spmm(Xd, nmspmm.DeviceWeight.from_packed(nmspmm.compress(W, *PATTERN[kind])), **kw)
    torch.cuda.synchronize()
    ref = oracle.matmul_i8(X, W)
    if Yb is not None:
        assert np.array_equal(gu.fetch(Yb, m, n), ref)
    if Yhb is not None:
        gu.assert_f16_close(gu.fetch(Yhb, m, n), oracle.dequant_f16(ref, scale))
    if Yq is not None:
        h = Yqb.cpu().numpy()
        assert (h[m * n:] == -128).all(), "write past the end of Yq"
        assert np.array_equal(h[:m * n].reshape(m, n), oracle.requant_i8(ref, scale))
