"""GPU parity of calls without a plan on the tiles that no plan names: the
outputs against the oracle (int32 and int8 equal, fp16 within the rounding of
assert_f16_close), with guard bands after them."""
import numpy as np
import pytest

import oracle
from paper_2607_12505_amd import nmprobe, nmspmm
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


ALL_PATTERNS = ((2, 4), (1, 4), (1, 8), (2, 8), (3, 8), (4, 8), (5, 8), (8, 8))


def _run_all_outputs(m, n, k, N, M, call, nthreads=1):
    """Random operands, the three outputs and a carried expansion through
    call(Xd, w, outputs and job): everything against the oracle, guards intact."""
    import torch
    rng = np.random.default_rng(m + n + k + 8 * N + M)
    X = rng.integers(-128, 128, (m, k)).astype(np.int8)
    W = wl.random_nm(n, k, N, M, rng)
    scale = rng.uniform(1e-6, 1e-3, n).astype(np.float32)
    sd = torch.from_numpy(scale).cuda()
    Yb, Yhb = gu.device_outputs(m, n, True, True)
    Yqb = torch.full((m * n + gu.GUARD,), -128, dtype=torch.int8, device="cuda")
    Wj = wl.random_nm(96, 1024, 2, 8, rng, full=True)
    dj = nmspmm.DeviceWeight.from_packed(nmspmm.compress(Wj, 2, 8))
    nbytes = nmspmm.expand_size(dj.desc)[1]
    want = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    nmspmm.expand(dj, out=want)
    out = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    job, _ = nmspmm.expand_job(dj, out)
    call(torch.from_numpy(X).cuda(), nmspmm.DeviceWeight.from_packed(nmspmm.compress(W, N, M)),
         dict(Y=gu.view2d(Yb, m, n), scale=sd, Yh=gu.view2d(Yhb, m, n), Yq=gu.view2d(Yqb, m, n), qscale=sd, job=job))
    torch.cuda.synchronize()
    ref = oracle.matmul_i8(X, W, nthreads=nthreads)
    assert np.array_equal(gu.fetch(Yb, m, n), ref)
    gu.assert_f16_close(gu.fetch(Yhb, m, n), oracle.dequant_f16(ref, scale))
    h = Yqb.cpu().numpy()
    assert (h[m * n:] == -128).all(), "write past the end of Yq"
    assert np.array_equal(h[:m * n].reshape(m, n), oracle.requant_i8(ref, scale))
    assert torch.equal(out[:nbytes], want) and (out[nbytes:] == 0xA5).all().item()


# more k-steps than any ring holds (every slot refilled, several times), whole
# and ragged reductions, rows of outputs on and off 128-byte lines (the last k
# with int32 alone stored non-temporally), partial last tiles both ways
@pytest.mark.parametrize("n,k", [(524, 1040), (512, 1152), (524, 1424)])
@pytest.mark.parametrize("pattern", ALL_PATTERNS, ids=str)
@pytest.mark.parametrize("tile", range(12, 16))
def test_every_kind_on_the_unplanned_tiles(tile, pattern, n, k):
    print(f"tile {tile} {pattern} n={n} k={k}", flush=True)
    if (tile == 13 and pattern not in ((2, 4), (8, 8))) or (tile == 14 and pattern in ((3, 8), (4, 8), (5, 8))):
        # not built for this kind (the estimate never chooses it): refused
        with pytest.raises(nmspmm.NmError) as e:
            _run_all_outputs(700, n, k, *pattern, lambda X, w, kw: nmprobe.probe_spmm_tile(X, w, tile, **kw))
        assert e.value.status == nmspmm.NM_ERR_ARG
        return
    _run_all_outputs(700, n, k, *pattern, lambda X, w, kw: nmprobe.probe_spmm_tile(X, w, tile, **kw))


@pytest.mark.parametrize("pattern", [(1, 8), (2, 8), (4, 8)], ids=str)
def test_unplanned_tile_on_an_expanded_weight(pattern):
    m, n, k = 4200, 2048, 1040
    print(f"expanded weight {pattern} m={m} n={n} k={k}", flush=True)
    d = nmspmm.compress_size(n, k, *pattern)
    mode = nmspmm.NM_OUT_I32 | nmspmm.NM_OUT_F16 | nmspmm.NM_OUT_I8
    p = nmspmm.spmm_plan(d, m, mode)
    assert p.expand == 1
    assert nmprobe.schedule_tile(nmspmm.expand_size(d)[0].kind, m, n, k, mode, p.tile) >= nmspmm.num_tiles()
    _run_all_outputs(m, n, k, *pattern, lambda X, w, kw: nmspmm.spmm(X, w, **kw), nthreads=16)
