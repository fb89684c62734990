"""The callables of _entry.so against the functions that they stand for: the same results, errors and statuses for arguments of every kind
(statuses from calls that the host refuses or that have no rows: nothing is launched)."""
import copy
import inspect
import os
import pickle
import shutil
import subprocess
import sys
import threading
import weakref

import numpy as np
import pytest

from paper_2407_13885_amd import binding

BF16, F32 = binding.ATTNW_BF16, binding.ATTNW_F32
A, B, C, D = 0x10000000, 0x20000000, 0x40000000, 0x60000000


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(binding.library_path()) or not os.path.exists(binding._ENTRY):
        binding.build()
    assert binding._entry is not None
    binding.load_library()


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Stream:
    cuda_stream = 0


class Number:
    def __int__(self):
        return A + 4

    def __index__(self):
        return 1


def _outcome(f, args, kwargs):
    try:
        return f(*args, **kwargs)
    except Exception as e:                        # noqa: BLE001
        return type(e), str(e), getattr(e, "status", None)


CALLS = [("attnw_fused", (A, B, C, 1, 1, 128, 64, 0.125, BF16)), ("attnw_gemm_scores", (A, B, C, 1, 1, 128, 64, 0.125, F32)),
         ("attnw_attention", (A, B, C, D, 1, 1, 128, 64, 0.125, BF16)), ("attnw_softmax", (A, C, 4, 8, BF16)),
         ("attnw_softmax_cast", (A, C, 4, 8, F32, BF16)), ("attnw_scale", (A, C, 8, 0.5, F32))]


@pytest.mark.parametrize("name,good", CALLS)
def test_same_as_the_function(name, good):
    entry = getattr(binding, name)
    plain = entry.__wrapped__
    assert entry is binding._entries[name] and entry.__name__ == name and entry.__doc__ == plain.__doc__
    assert inspect.signature(entry) == inspect.signature(plain)
    odd = [None, 0, -1, 1 << 40, 1 << 64, True, 1.5, "x", np.int64(4), np.float32(0.5), Tensor(A + 8), Tensor("x"), Number(), float("nan")]
    for i in range(len(good)):
        for v in odd:
            if i >= len(good) - 1 or not isinstance(v, (int, np.integer)) or v in (0, -1) or i < 2:
                # the output at an address that no call accepts, so that nothing is launched whatever v is
                args = list(good)
                args[3 if name == "attnw_attention" else 2 if name in ("attnw_fused", "attnw_gemm_scores") else 1] = C + 2
                args[i] = v
                if (i == 1 and len(good) < 7) or (name == "attnw_attention" and i == 3) or (i == 2 and len(good) == 9):
                    args[0] = A + 2               # (that address was replaced itself)
                assert _outcome(entry, args, {}) == _outcome(plain, args, {}), (i, v)
    bad = list(good)
    bad[0] = A + 2
    for stream in (None, 0, Stream(), Number(), "x", 1 << 64):
        assert _outcome(entry, bad + [stream], {}) == _outcome(plain, bad + [stream], {}), stream
        assert _outcome(entry, bad, {"stream": stream}) == _outcome(plain, bad, {"stream": stream}), stream
    names = list(inspect.signature(plain).parameters)
    assert _outcome(entry, [], dict(zip(names, bad))) == _outcome(plain, bad, {})
    for wrong in (good[:-1], tuple(good) + (None, None)):
        assert _outcome(entry, wrong, {}) == _outcome(plain, wrong, {})


@pytest.mark.parametrize("name,good", CALLS)
def test_functions_like_any_other(name, good):
    f = getattr(binding, name)
    assert inspect.isfunction(f) and copy.deepcopy(f) is f and pickle.loads(pickle.dumps(f)) is f and weakref.ref(f)() is f
    assert f.__defaults__ == (None,) and f.__code__.co_varnames[:len(good)] == tuple(inspect.signature(f).parameters)[:len(good)]
    assert f.__module__ == binding.__name__ and name in repr(f)

    class Holder:
        call = f
    assert Holder().call.__func__ is f


def test_no_rows():
    assert binding.attnw_fused(None, None, None, 0, 4, 128, 64, 0.125, BF16) is None
    assert binding.attnw_softmax(None, None, 0, 128, F32, Stream()) is None
    assert binding.attnw_scale(None, None, 0, 2.0, F32) is None


def test_an_error_of_data_ptr_is_its_own():
    class Bad:
        def data_ptr(self):
            raise ValueError("mine")
    with pytest.raises(ValueError, match="mine"):
        binding.attnw_softmax(Bad(), C, 4, 4, BF16)


def test_threads():
    seen = []

    def work():
        for _ in range(2000):
            with pytest.raises(binding.AttnwError):
                binding.attnw_softmax(A + 1, C, 4, 4, BF16)
        seen.append(1)
    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(seen) == 4


def test_calls_after_a_build_reach_the_library_built(monkeypatch, tmp_path):
    """build() without its compilers, the library that it would have made in place of the one loaded: every entry point returns 77."""
    source = tmp_path / "lib.c"
    source.write_text("".join(f"int {name}() {{ return 77; }}\n" for name in binding.EXPORTS if name != "attnw_status_string")
                      + 'const char* attnw_status_string(int s) { return "the new one"; }\n')
    other = tmp_path / "libother.so"
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", str(source), "-o", str(other)], check=True)
    bad = {name: (A + 2,) + tuple(good[1:]) for name, good in CALLS}
    for name, args in bad.items():                # (refused by the library loaded now)
        with pytest.raises(binding.AttnwError, match="aligned"):
            getattr(binding, name)(*args)
    try:
        with monkeypatch.context() as m:
            m.setattr(subprocess, "run", lambda cmd, **_: subprocess.CompletedProcess(cmd, 0, "", ""))
            m.setattr(shutil, "move", lambda *_: None)
            m.setattr(binding, "_LIB", str(other))
            binding.build()
            for name, args in bad.items():
                with pytest.raises(binding.AttnwError, match="the new one") as e:
                    getattr(binding, name)(*args)
                assert e.value.status == 77
            assert binding.attnw_version() == 77
    finally:
        binding._lib = None
        binding.load_library()
    for name, args in bad.items():
        with pytest.raises(binding.AttnwError, match="aligned"):
            getattr(binding, name)(*args)


def _child(tmp_path, entry, then):
    """Runs `then` in a process of its own, on a copy of the package's Python files with the given bytes for _entry.so (None: no such file)."""
    package = tmp_path / "paper_2407_13885_amd"
    package.mkdir()
    for f in os.listdir(binding._PKG):
        if f.endswith(".py"):
            shutil.copy(os.path.join(binding._PKG, f), package / f)
    if entry is not None:
        (package / "_entry.so").write_bytes(entry)
    return subprocess.run([sys.executable, "-W", "always", "-c", then], cwd=tmp_path, capture_output=True, text=True,
                          env={**os.environ, "PYTHONPATH": str(tmp_path)})


def test_an_extension_that_does_not_load_is_heard_of(tmp_path):
    done = _child(tmp_path, b"not a library", "from paper_2407_13885_amd import binding as b; assert b._entry is None; b.attnw_fused")
    assert done.returncode == 0 and "RuntimeWarning" in done.stderr and "_entry.so does not load" in done.stderr, done.stderr


def test_an_extension_built_after_the_import_is_taken(tmp_path):
    done = _child(tmp_path, None, f"""if True:
        import shutil, subprocess
        from paper_2407_13885_amd import binding as b
        f = b.attnw_softmax
        assert b._entry is None and not b._direct
        def run(cmd, **_):
            if "entry.cpp" in " ".join(cmd): shutil.copy({binding._ENTRY!r}, cmd[-1])
            return subprocess.CompletedProcess(cmd, 0, "", "")
        b.subprocess = type("S", (), {{"run": staticmethod(run)}})
        b.sources = lambda: []
        b.build()
        assert b._entry is not None and len(b._direct) == 6 and f is b.attnw_softmax and f.__globals__["direct"] is b._direct["attnw_softmax"]
        """)
    assert done.returncode == 0 and "Warning" not in done.stderr, done.stderr
