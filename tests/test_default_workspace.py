"""Calls without a workspace take one for themselves (CPU, the library's entry
points replaced by recorders): a call issued while another is being issued, as
a second host thread does, gets other memory; memory for another stream than
the current one is taken on that stream; counters are cleared where split-K
reads them."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2607_12505_amd import nmspmm

M_, N_, K_ = 100, 64, 256


class _Library:
    """The real library with its launching entry points replaced."""

    def __init__(self, real, log, nested):
        self._real, self._log, self._nested = real, log, nested

    def __getattr__(self, name):
        if name == "nm_spmm_ex":
            return self._spmm
        if name == "nm_gemm_i8_dense_ex":
            return lambda *a: self._log.append(("dense", a[8], a[9], a[10])) or 0
        if name == "nm_workspace_init":
            return lambda ws, n, stream: self._log.append(("clear", ws, n, stream)) or 0
        return getattr(self._real, name)

    def _spmm(self, *a):
        if self._nested:
            self._nested.pop()()          # another thread's call while this one is being issued
        self._log.append(("spmm", a[8], a[9], a[10]))
        return 0


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


@pytest.fixture
def calls(monkeypatch):
    log, nested = [], []
    fake = _Library(nmspmm.lib(), log, nested)
    monkeypatch.setattr(nmspmm, "lib", lambda: fake)
    monkeypatch.setattr(nmspmm, "_on_device", lambda *a, **k: None)
    monkeypatch.setattr(nmspmm, "_stream", lambda s: 7 if s is None else s.cuda_stream)
    return log, nested


def _call(split=1, expand=1, N=2, M=8, stream=None):
    W = np.zeros((N_, K_), np.int8)
    W[:, ::8] = 1
    w = nmspmm.DeviceWeight.from_packed(nmspmm.compress(W, N, M), device="cpu")
    X = torch.zeros((M_, K_), dtype=torch.int8)
    plan = nmspmm.make_plan(w.desc.kind, 3, split, expand)
    return lambda: nmspmm.spmm(X, w, Y=torch.empty((M_, N_), dtype=torch.int32), plan=plan, stream=stream)


def test_a_call_issued_meanwhile_gets_memory_of_its_own(calls):
    log, nested = calls
    nested.append(_call())
    _call()()
    (_, inner, inner_bytes, _), (_, outer, outer_bytes, _) = log
    assert inner and outer and (outer + outer_bytes <= inner or inner + inner_bytes <= outer)


def test_memory_is_taken_on_the_calls_stream(calls, monkeypatch):
    log, _ = calls
    entered = []

    @contextlib.contextmanager
    def on(stream):
        entered.append(stream.cuda_stream)
        yield

    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device=None: _Stream(handle))
    monkeypatch.setattr(torch.cuda, "stream", on)
    _call(stream=_Stream(9))()
    assert entered == [9] and log[-1][3] == 9
    _call(stream=_Stream(7))()            # the current stream
    _call()()
    assert entered == [9]


@pytest.mark.parametrize("split,expand", [(1, 1), (2, 0), (2, 1)])
def test_counters_are_cleared_for_split_k_on_the_calls_stream(calls, split, expand):
    log, _ = calls
    _call(split, expand)()
    _, ws, nbytes, stream = log[-1]
    assert nbytes >= 16384 and stream == 7
    assert log[:-1] == ([("clear", ws, 16384, 7)] if split > 1 else [])


def test_no_workspace_where_none_is_needed(calls):
    log, _ = calls
    _call(1, 0)()
    assert log == [("spmm", None, 0, 7)]


def test_dense_calls_do_the_same(calls):
    log, _ = calls
    X, W = torch.zeros((M_, K_), dtype=torch.int8), torch.zeros((N_, K_), dtype=torch.int8)
    nmspmm.gemm_i8_dense(X, W, Y=torch.empty((M_, N_), dtype=torch.int32),
                         plan=nmspmm.make_plan(nmspmm.NM_KIND_DENSE, 3, 2))
    (what, ws, n, stream), (_, used, _, _) = log
    assert what == "clear" and ws == used and (n, stream) == (16384, 7)
