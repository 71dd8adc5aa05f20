"""The launch calls through the CPython module against the ctypes route: the same statuses, and the same
conversions and refusals for arguments that are not plain integers (CPU: nothing is launched)."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2402_10876_amd as tw
from paper_2402_10876_amd import binding


@pytest.fixture()
def weights():
    p = tw.tw_pack_host(np.ones((64, 128), np.float16), np.ones((64, 128), np.uint8), 128, tw.PATTERN_TW)
    q = tw.tw_pack_i8_host(np.ones((64, 128), np.int8), np.ones((64, 128), np.uint8), 128)
    yield p, q
    p.free()
    q.free()


def _outcome(f, *a):
    try:
        return f(*a)
    except Exception as e:      # the class and the status are what a caller sees
        return type(e), getattr(e, "status", None)


ODD = [None, True, 8.0, "8", np.int64(8), -1, 1 << 31, 1 << 40, 1 << 64, -(1 << 70), C.c_void_p(0x10000)]


def test_odd_arguments_end_as_with_ctypes(weights):
    p, q = weights
    good = [0x10000, 8, 8, tw.LAYOUT_KM, p, 0x20000, 8, 0]
    good8 = [0x10000, 16, 16, q, 0x20000, 16, 1, 0.5, 0]
    for good, f in ((good, tw.tw_gemm), (good8, tw.tw_gemm_i8)):
        for i, w in enumerate(good):
            if w is p or w is q:
                continue
            for v in [w, *ODD]:
                a = list(good)
                a[i] = v
                got = _outcome(f, *a)
                call, binding._call = binding._call, binding._Unbound
                try:
                    want = _outcome(f, *a)
                finally:
                    binding._call = call
                assert got == want, (f.__name__, i, v)
    assert _outcome(tw.tw_gemm, *([0x10000, 8, 8, 0, q, 0x20000, 8])) == (tw.TwError, 1)    # int8 weight
    assert binding._call is not binding._Unbound


def test_freed_weight_is_refused(weights):
    p, _ = weights
    p.free()
    with pytest.raises(ValueError):
        tw.tw_gemm(0x10000, 8, 8, tw.LAYOUT_KM, p, 0x20000, 8)
    with pytest.raises(ValueError):
        tw.tw_gemm_i8(0x10000, 16, 16, p, 0x20000, 16)


def test_module_takes_plain_numbers_only():
    tw.lib()
    m = binding._call
    assert m.gemm(0, 1, 1, 0, 0, 0, 1, 0) == 1 and m.conv(0, 0, 0, 8, 0) == 1          # refused by the library
    assert m.gemm_i8(0, 1, 1, 0, 0, 1, 0, 1.0, 0) == 1 and m.conv_i8(0, 0, 0, 8, 0, 1.0, 0) == 1
    assert m.gemm(0, 1, 1, 0, None, 0, 1, 0) is None and m.gemm(0, 1, 1) is None
    assert m.gemm_i8(0, 1, 1, 0, 0, 1, 0, 1, 0) is None and m.conv(0, 1 << 64, 0, 8, 0) is None
    with pytest.raises(TypeError):
        m.bind(1, 2, 3)


def _copy_of_the_package(tmp_path, module):
    """The package as a tree that was never built (module: with the CPython module all the same)."""
    from paper_2402_10876_amd import build
    dst = tmp_path / "tree"
    shutil.copytree(build.PKG, dst / "paper_2402_10876_amd", ignore=shutil.ignore_patterns("*.so", "*.srchash", "__pycache__", "*.tmp"))
    shutil.copytree(os.path.join(build.ROOT, "include"), dst / "include")
    if module:
        shutil.copy(build.CALL, dst / "paper_2402_10876_amd")
    return dst


USE = """
import numpy as np, paper_2402_10876_amd as tw
from paper_2402_10876_amd import binding, build
assert build.ensure_built() == {lib!r}
p = tw.tw_pack_host(np.ones((64, 128), np.float16), np.ones((64, 128), np.uint8), 128, tw.PATTERN_TW)
try:
    tw.tw_gemm(0x10000, 8, 8, tw.LAYOUT_KM, p, 0x20000, 8)
except tw.TwError as e:
    assert e.status == 6           # not uploaded: the call reached the library
else:
    raise SystemExit("no error")
assert (binding._call is binding._Unbound) == {unbound}
"""


@pytest.mark.parametrize("module", [False, True])
def test_another_library_in_a_tree_that_was_not_built(tmp_path, module):
    from paper_2402_10876_amd import build
    lib = build.ensure_built()
    dst = _copy_of_the_package(tmp_path, module)
    r = subprocess.run([sys.executable, "-c", USE.format(lib=lib, unbound=not module)], cwd=dst, env=dict(os.environ, TWGEMM_LIB=lib),
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]


def test_module_that_cannot_be_built(tmp_path, monkeypatch):
    """No host compiler: the library is built all the same, and a module of older sources does not stay."""
    from paper_2402_10876_amd import build
    old = tmp_path / "_twcall.so"
    old.write_bytes(b"old")
    monkeypatch.setattr(build, "CALL", str(old))
    for cxx in (str(tmp_path / "no-such-compiler"), shutil.which("false")):
        old.write_bytes(b"old")
        monkeypatch.setenv("CXX", cxx)
        with pytest.warns(UserWarning, match="ctypes"):
            assert build.build_call() is None
        assert not old.exists()
