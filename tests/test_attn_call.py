"""The compiled marshalling of the attention call against the general path: it takes the same calls with the same arguments,
and leaves everything it does not take, errors above all, to the general path."""
import os
import sys
import sysconfig

import numpy as np
import pytest
import torch

import paper_2412_16434_amd as S
from paper_2412_16434_amd import binding, build


def _call(dev, dtype=torch.bfloat16, d=128):
    """Arguments of a call: two sessions of 20 and 0 cached tokens, 3 and 2 new ones, 4 / 2 heads."""
    g = torch.Generator().manual_seed(5)
    rand = lambda *shape: torch.randn(shape, generator=g).to(dtype).to(dev)
    cache = S.KVCache(rand(2, 4, 16, 2, d), rand(2, 4, 16, 2, d))
    q = rand(5, 4, d)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)
    return dict(cache=cache, layer=1, q=q, k_new=rand(5, 2, d), v_new=rand(5, 2, d), out=torch.zeros_like(q),
                cu_new_lens=i32([0, 3, 5]), prefix_lens=i32([20, 0]), block_table=i32([[3, 1], [-1, -1]]), max_new_len=3,
                max_prefix_len=20, scale=0.125)


def _compiled(a, workspace=None):
    return binding._load_attn_call()(a["cache"].k_pool, a["cache"].v_pool, *list(a.values())[1:], workspace)


def test_calls_on_the_host_are_left_to_the_general_path():
    a = _call("cpu")
    assert _compiled(a) is None
    with pytest.raises(ValueError, match="must be a device tensor"):
        S.prefix_prefill_attn(**a)
    assert binding._load_attn_call()() is None and binding._load_attn_call()(*range(14)) is None


def test_a_cache_that_describes_itself_takes_the_general_path(monkeypatch):
    """The compiled marshalling reads the pools; what a subclass says in ``struct()`` it does not see."""
    class LastBlocks(S.KVCache):
        def struct(self):
            st = super().struct()
            st.n_blocks = 2
            return st

    taken = []
    monkeypatch.setattr(binding, "_attn_call", lambda *args: taken.append(args) or 0)
    a = _call("cpu")
    S.prefix_prefill_attn(**a)
    assert len(taken) == 1
    a["cache"] = LastBlocks(a["cache"].k_pool, a["cache"].v_pool)
    with pytest.raises(ValueError, match="must be a device tensor"):
        S.prefix_prefill_attn(**a)
    assert len(taken) == 1


@pytest.fixture
def without_the_module(monkeypatch):
    """The compiled marshalling as if it had not been built."""
    monkeypatch.setattr(binding, "_attn_call", None)
    monkeypatch.delattr(S, "_attn_call", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2412_16434_amd._attn_call", None)


def test_without_the_module_the_general_path_decides(without_the_module):
    with pytest.raises(ValueError, match="must be a device tensor"):
        S.prefix_prefill_attn(**_call("cpu"))
    assert binding._attn_call is not None, "the import is tried again by every call"


def test_without_the_library_the_checks_come_first(monkeypatch):
    monkeypatch.setattr(binding, "_attn_call", None)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", "/nonexistent/libsymph.so")
    with pytest.raises(ValueError, match="must be a device tensor"):
        S.prefix_prefill_attn(**_call("cpu"))


def test_the_file_is_for_one_interpreter(monkeypatch, tmp_path, capsys):
    assert build.CALL_LIB.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    # where gcc or the interpreter's headers are absent there is none, and building goes on
    monkeypatch.setattr(build, "CALL_LIB", str(tmp_path / "call.so"))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    with monkeypatch.context() as m:
        m.setenv("PATH", str(tmp_path))
        assert build.build_attn_call() is False and not os.listdir(tmp_path)
        assert "gcc" in capsys.readouterr().err
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_attn_call() is False and not os.listdir(tmp_path)
    assert "Python.h" in capsys.readouterr().err


def _workspace(a):
    n = S.prefix_prefill_attn_workspace_bytes(a["cache"], 2, 4, 5, a["max_new_len"], a["max_prefix_len"])
    return torch.empty(n, dtype=torch.uint8, device="cuda:0") if n else None


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 64)])
def test_same_call_both_ways(dtype, d):
    a = _call("cuda:0", dtype, d)
    ws = _workspace(a)
    assert _compiled(a, ws) == 0
    torch.cuda.synchronize()
    by_c = a["out"].clone()
    a["out"] = torch.zeros_like(by_c)
    S.prefix_prefill_attn(**a, workspace=ws, stream=torch.cuda.current_stream())   # (a stream: the general path)
    torch.cuda.synchronize()
    assert torch.equal(by_c, a["out"]) and bool(by_c.float().abs().sum() > 0)


@pytest.mark.gpu
def test_the_call_goes_to_the_current_stream():
    """On a side stream: a delay, the queries copied over other values, the call.  Launched anywhere else it would not wait for the
    copy and read the other values."""
    a = _call("cuda:0")
    ws = _workspace(a)
    S.prefix_prefill_attn(**a, workspace=ws)
    torch.cuda.synchronize()
    want, q = a["out"].clone(), a["q"]
    a["q"] = torch.ones_like(q)
    a["out"].zero_()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)   # (10 to 200 ms)
        a["q"].copy_(q)
        assert _compiled(a, ws) == 0
    side.synchronize()
    assert torch.equal(want, a["out"])


@pytest.mark.gpu
def test_same_call_without_the_module(without_the_module, monkeypatch):
    a = _call("cuda:0")
    ws = _workspace(a)
    S.prefix_prefill_attn(**a, workspace=ws)
    torch.cuda.synchronize()
    by_python = a["out"].clone()
    monkeypatch.undo()
    a["out"].zero_()
    assert _compiled(a, ws) == 0
    torch.cuda.synchronize()
    assert torch.equal(by_python, a["out"])


@pytest.mark.gpu
@pytest.mark.parametrize("change,error", [
    (dict(layer=2), S.SymphError),                       # statuses of the entry point
    (dict(scale=0.0), S.SymphError),
    (dict(max_new_len=6), S.SymphError),
    (dict(workspace=None), S.SymphError),
    (dict(scale=np.float32(0.125)), None),               # not of the plain types: converted by the general path
    (dict(layer=np.int64(1)), None),
    (dict(prefix_lens=lambda t: t.long()), ValueError),  # what the C side cannot see
    (dict(q=lambda t: t.float()), ValueError),
    (dict(k_new=lambda t: t.cpu()), ValueError),
    (dict(out=lambda t: t[:4]), ValueError),
    (dict(v_new=lambda t: torch.empty(5, 4, 128, dtype=t.dtype, device=t.device)[:, ::2]), ValueError),
    (dict(block_table=lambda t: t[0]), ValueError),
])
def test_what_is_not_taken_ends_as_it_did(change, error):
    a = _call("cuda:0")
    a["workspace"] = _workspace(a)
    for k, v in change.items():
        a[k] = v(a[k]) if callable(v) else v
    results = []
    for stream in (None, torch.cuda.current_stream()):   # (a stream: the general path)
        try:
            S.prefix_prefill_attn(**a, stream=stream)
            torch.cuda.synchronize()
            results.append(a["out"].clone())
        except Exception as e:
            results.append((type(e), str(e)))
    if error is None:
        assert torch.equal(*results)
    else:
        assert results[0] == results[1] and results[0][0] is error
