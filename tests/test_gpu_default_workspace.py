"""Calls that take a workspace for themselves, on the GPU: captured in a graph
and replayed among other work, on several streams at once, and on a stream that
is not the current one, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2607_12505_amd import nmspmm
from paper_2607_12505_amd import workloads as wl

pytestmark = pytest.mark.gpu

M_, N_, K_ = 197, 768, 1024


def _linear(seed, N, M, split, expand, n=N_, k=K_):
    import torch
    rng = np.random.default_rng(seed)
    X = rng.integers(-127, 128, (M_, k), dtype=np.int8)
    W = wl.random_nm(n, k, N, M, rng, full=True)
    w = nmspmm.DeviceWeight.from_packed(nmspmm.compress(W, N, M))
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((M_, n), -1, dtype=torch.int32, device="cuda")
    plan = nmspmm.make_plan(w.desc.kind, 3, split, expand)
    return lambda stream=None: nmspmm.spmm(Xd, w, Y=Y, plan=plan, stream=stream), Y, oracle.matmul_i8(X, W)


def test_captured_calls_keep_their_workspace():
    import torch
    linears = [_linear(1, 2, 8, 1, 1), _linear(2, 2, 4, 4, 0), _linear(3, 4, 8, 2, 1)]
    for call, _, _ in linears:
        call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for call, _, _ in linears:
            call()
    bigger, Yb, ref_b = _linear(4, 2, 8, 8, 1, n=2048, k=4096)
    for rep in range(3):
        bigger()                                     # more than the captured calls needed
        others = [torch.full((1 << 20,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(64)]
        for _, Y, _ in linears:
            Y.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for _, Y, ref in linears:
            assert np.array_equal(Y.cpu().numpy(), ref), f"replay {rep}"
        assert all((o == 0x5A).all().item() for o in others), f"replay {rep} wrote into other memory"
        assert np.array_equal(Yb.cpu().numpy(), ref_b)


@pytest.mark.parametrize("current", [True, False])
def test_calls_on_several_streams(current):
    import torch
    linears = [_linear(10 + i, N, M, split, expand)
               for i, (N, M, split, expand) in enumerate([(2, 8, 1, 1), (4, 8, 1, 1), (2, 4, 4, 0), (1, 8, 2, 1)])]
    streams = [torch.cuda.Stream() for _ in linears]
    torch.cuda.synchronize()
    for _ in range(8):
        for (call, _, _), s in zip(linears, streams):
            if current:
                with torch.cuda.stream(s):
                    call()
            else:
                call(stream=s)
    torch.cuda.synchronize()
    for _, Y, ref in linears:
        assert np.array_equal(Y.cpu().numpy(), ref)
