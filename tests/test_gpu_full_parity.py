"""Element-by-element GPU parity of every GEMM of the five benchmark
workloads at full size, against the oracle's plain product run on the host
threads: with the planner's plan, and, where the library runs another tile
without a plan, that call too:

* int32 outputs bit-exact everywhere;
* the fp16 dequantisation output of the DeiT-Small workload within
  |g - r| <= 1e-3 |r| or 2^-24, infinities exact;
* every sparse GEMM of configs 0-4 (all 96 linears of the ViT-L chain,
  dense layers included) and the dense baseline of every distinct shape.

Every output is prefilled with a sentinel and followed by a guard band, so an
unwritten element or a write past the end fails too.  One test per GEMM keeps
each test to a few seconds of oracle time."""
import os

import numpy as np
import pytest

import oracle
from paper_2607_12505_amd import nmprobe, nmspmm
from paper_2607_12505_amd import workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu

THREADS = max(1, min(len(os.sched_getaffinity(0)), 16))


def _cases():
    cases, dense_seen = [], set()
    for cfg in range(5):
        w = wl.workload(cfg)
        for i, g in enumerate(w.gemms):
            cases.append(pytest.param(cfg, i, False, id=f"cfg{cfg}-{i}-{g.name.replace(' ', '_')}"))
            shape = (cfg, g.m, g.k, g.n)
            if shape not in dense_seen and g.N != g.M:
                dense_seen.add(shape)
                cases.append(pytest.param(cfg, i, True, id=f"cfg{cfg}-{i}-dense-baseline-{g.m}x{g.k}x{g.n}"))
    return cases


@pytest.mark.parametrize("cfg,idx,baseline", _cases())
def test_workload_gemm_full(cfg, idx, baseline):
    w = wl.workload(cfg)
    g = w.gemms[idx]
    X, W, scale = wl.inputs_for(cfg, g)
    want_f16 = w.out_f16
    kind = "dense baseline" if baseline or g.N == g.M else f"{g.N}:{g.M}"
    print(f"cfg{cfg} {g.name} m={g.m} k={g.k} n={g.n} {kind}", flush=True)
    mode = nmspmm.NM_OUT_I32 | (nmspmm.NM_OUT_F16 if want_f16 else 0)
    dense = baseline or g.N == g.M
    if dense:
        plan, ran = nmspmm.dense_plan(g.m, g.n, g.k, mode), nmspmm.NM_KIND_DENSE
    else:
        packed = nmspmm.compress(W, g.N, g.M)
        plan = nmspmm.spmm_plan(packed.desc, g.m, mode)
        ran = nmspmm.expand_size(packed.desc)[0].kind if plan.expand else plan.kind
    tile = nmprobe.schedule_tile(ran, g.m, g.n, g.k, mode, plan.tile)
    ref = oracle.matmul_i8(X, W, nthreads=THREADS)
    for p in [plan] if tile == plan.tile else [plan, None]:
        if dense:
            Y, Yh = gu.run_dense(X, W, scale, want_i32=True, want_f16=want_f16, plan=p)
        else:
            Y, Yh = gu.run_sparse(X, packed, scale, want_i32=True, want_f16=want_f16, plan=p)
        bad = np.flatnonzero(Y != ref)
        assert bad.size == 0, (f"tile {tile if p is None else plan.tile}: {bad.size} int32 mismatches of {ref.size}, "
                               f"first at {np.unravel_index(bad[:5], ref.shape)}")
        if want_f16:
            gu.assert_f16_close(Yh, oracle.dequant_f16(ref, scale))
