"""The two decisions called through the extension and through ctypes: the same C call for every form of arguments (a recorder in
place of the library's entry points; nothing is launched)."""
import ctypes as C
import os
import sysconfig

import numpy as np
import pytest
import torch

from paper_2604_15750_amd import api, build

I32, F32, VP = C.c_int32, C.c_float, C.c_void_p
BOUNDARY = C.CFUNCTYPE(C.c_int, VP, VP, VP, VP, VP, C.c_int, VP, VP, VP, VP, VP)
SELECT = C.CFUNCTYPE(C.c_int, VP, C.c_int, C.c_int, VP, VP, VP, VP, VP, VP, VP, C.c_int, C.c_int, VP, C.c_int, VP, VP, VP, VP)


class Calls:
    """Calling it runs a function through both ways, the extension first, and gives the recorded calls of each (or the exception's type);
    `taken` then says whether the extension took the call itself, and `status` is what the recorder returns."""


@pytest.fixture
def calls(monkeypatch):
    ext = api._decisions()
    assert ext is not None, "the extension has not been built"
    seen, self = [], Calls()
    self.status = 0

    def ints(p, n):
        return None if not p else tuple((I32 * n).from_address(p))

    def boundary(I, H, ws, wl, cold, n, p, L, S, m, st):
        q = C.cast(p, C.POINTER(api.dlm_boundary_params))[0]
        seen.append((I, H, ints(ws, n), ints(wl, n), ints(cold, n), n, q.lam, q.l_min, q.smooth_radius, q.norm_mode, q.rule, L, S, m, st))
        return self.status

    def select(z, V, dt, lse, cf, am, tok, rs, ts, bl, n, mask, p, ap, sel, ns, m, st):
        q = C.cast(p, C.POINTER(api.dlm_select_params))[0]
        seen.append((z, V, dt, lse, cf, am, tok, ints(rs, n), ints(ts, n), ints(bl, n), n, mask, q.tau_low, q.tau_high, q.gamma, q.mode, ap, sel, ns, m, st))
        return self.status

    cb, cs, L = BOUNDARY(boundary), SELECT(select), api.lib()
    real = [C.cast(f, VP).value for f in (L.block_boundary, L.select_parallel)]

    class Recorder:
        block_boundary, select_parallel, dlm_last_error = cb, cs, L.dlm_last_error

    class Spy:
        """The extension; a call that it takes has reached the library when it returns, one that it declines has not."""
        @staticmethod
        def ask(f, args):
            before = len(seen)
            rc = f(*args)
            assert rc in (None, self.status) and len(seen) - before == (rc is not None)
            self.taken = rc is not None
            return rc

        boundary = staticmethod(lambda *a: Spy.ask(ext.boundary, a))
        select = staticmethod(lambda *a: Spy.ask(ext.select, a))

    def run(f):
        out = []
        for through_ext in (True, False):
            seen.clear()
            monkeypatch.setattr(api, "_decisions", (lambda: Spy) if through_ext else (lambda: None))
            try:
                f()
                out.append(list(seen))
            except Exception as e:
                out.append(type(e))
        return out

    Calls.__call__ = lambda self, f: run(f)

    monkeypatch.setattr(api, "lib", lambda: Recorder)
    monkeypatch.setattr(api, "_stream", lambda: 0x1230)
    ext.bind(C.cast(cb, VP).value, C.cast(cs, VP).value, torch.float32, torch.bfloat16)
    yield self
    ext.bind(*real, torch.float32, torch.bfloat16)


f = torch.zeros(64)
i = torch.zeros(64, dtype=torch.int32)
ARRAYS = [[0, 8], (0, 8), [True, 8], np.array([0, 8], dtype=np.int32), [np.int64(0), 8], torch.tensor([0, 8]), [0.0, 8.9], [0, 2**31], [], ["a", 1], None, list(range(33))]


def plain(v, n=None):
    """Whether a host array (n None: the first, else one beside a first of n entries) is one that the extension takes."""
    return type(v) in (list, tuple) and (len(v) <= 32 if n is None else len(v) >= n) and all(number(x) for x in v[:n])


def number(x):
    """... a whole number or a real one of a parameter struct."""
    if isinstance(x, int):
        return -2**31 <= x < 2**31
    return type(x) is float and (abs(x) < 3.4e38 or x - x != 0)


@pytest.mark.parametrize("arr", range(len(ARRAYS)))
@pytest.mark.parametrize("lam,l_min", [(1.2, 8), (np.float32(1.2), 8), (1, True), (1e300, 8), (float("inf"), 8), (1.2, 2**40), (1.2, 8.0)])
def test_block_boundary_forms(calls, arr, lam, l_min):
    for cold in (None, [0, 1] * 17, (True,) * 34):
        for S in (None, f):
            a, b = calls(lambda: api.block_boundary(f, f, ARRAYS[arr], [8] * 40, i, lam, l_min, 1, 0, 1, cold=cold, S_out=S))
            assert a == b
            assert calls.taken == (plain(ARRAYS[arr]) and not any(type(x) is float for x in ARRAYS[arr]) and type(lam) is float and number(lam) and
                                   isinstance(l_min, int) and number(l_min))


@pytest.mark.parametrize("arr", range(len(ARRAYS)))
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_select_parallel_forms(calls, arr, dtype):
    z = torch.zeros((8, 16), dtype=dtype)
    for tau in (0.5, 1, np.float64(0.5), -1e39):
        for apply, mask in ((True, 15), (0, np.int32(15)), (2, 2**33), ("x", 15)):
            a, b = calls(lambda: api.select_parallel(z, f, f, i, i, ARRAYS[arr], [0, 8] * 17, [8, 8] * 17, mask, tau, 0.9, -16.0, 0, i, i, apply, margin_out=None))
            assert a == b
            assert calls.taken == (plain(ARRAYS[arr]) and not any(type(x) is float for x in ARRAYS[arr]) and dtype != torch.float16 and
                                   type(tau) is float and number(tau) and isinstance(apply, int) and isinstance(mask, int) and number(mask))
    for bad in (None, 3, "x"):
        a, b = calls(lambda: api.select_parallel(bad, f, f, i, i, [0], [0], [8], 15, 0.5, 0.9, -16.0, 0, i, i))
        assert a == b
        a, b = calls(lambda: api.select_parallel(z, bad, f, i, i, [0], [0], [8], 15, 0.5, 0.9, -16.0, 0, i, i))
        assert a == b


@pytest.mark.parametrize("form", [list, tuple, lambda v: np.array(v, dtype=np.int32)])
def test_short_host_arrays_are_refused(calls, form):
    """The library reads an entry per sequence (of dlm_step's row_offsets one more): no call with fewer reaches it."""
    full, short = form([0, 8]), form([8])
    for ws, wl, cold in ((full, short, None), (full, full, short), (full, form([]), None)):
        assert calls(lambda: api.block_boundary(f, f, ws, wl, i, 1.2, 8, cold=cold)) == [ValueError, ValueError]
    for rs, ts, bl in ((full, short, full), (full, full, short), (full, form([]), full)):
        assert calls(lambda: api.select_parallel(torch.zeros(8, 16), f, f, i, i, rs, ts, bl, 15, 0.5, 0.9, -16.0, 0, i, i)) == [ValueError, ValueError]


STEP = dict(row_offsets=[0, 1, 2], commit_len=[0, 0], tok_start=[0, 4], slot=[0, 1], kl_first=[0, 0], kl_count=[0, 0], save_first=[0, 0], save_count=[0, 0],
            suffix_len=[0, 0])


@pytest.mark.parametrize("short", [None, *STEP])
def test_short_host_arrays_of_a_step_are_refused(monkeypatch, short):
    seen = []

    class Recorder:
        dlm_step = staticmethod(lambda *a: seen.append(a) or 0)

    class Buffers:
        handle = None
        logits = max_logit = lse = entropy = kl = conf = argmax = f

    monkeypatch.setattr(api, "lib", lambda: Recorder)
    monkeypatch.setattr(api, "_stream", lambda: None)
    args = {k: v[:-1] if k == short else v for k, v in STEP.items()}
    step = lambda: api.dlm_step(Buffers, i, Buffers, span_start=[0, 0], **args)  # noqa: E731
    if short is None:
        step()
    else:
        with pytest.raises(ValueError, match="entries"):
            step()
    assert len(seen) == (short is None)


def test_a_refused_call_raises_either_way(calls):
    boundary = lambda: api.block_boundary(f, f, [0, 8], [8, 8], i, 1.2, 8)  # noqa: E731
    z = torch.zeros(8, 16)
    select = lambda: api.select_parallel(z, f, f, i, i, [0], [0], [8], 15, 0.5, 0.9, -16.0, 0, i, i)  # noqa: E731
    for call in (boundary, select):
        calls.status = 0
        a, b = calls(call)
        assert a == b and len(a) == 1 and calls.taken
        calls.status = -2
        assert calls(call) == [api.DlmError, api.DlmError] and calls.taken


def test_the_extension_is_the_interpreters_own_and_the_library_builds_without_it(monkeypatch, tmp_path, capsys):
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert suffix != ".so" and os.path.basename(api._decisions().__file__) == "_decisions" + suffix
    monkeypatch.setattr(build, "OUT_PY", str(tmp_path / ("_decisions" + suffix)))
    (tmp_path / "_decisions.so").touch()  # of an earlier build
    assert build.build_extension() == build.OUT_PY and os.listdir(tmp_path) == ["_decisions" + suffix]
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.build_extension() is None and os.listdir(tmp_path) == [] and "ctypes" in capsys.readouterr().err
