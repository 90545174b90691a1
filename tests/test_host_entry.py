"""The launching calls' own argument conversion (the module _sventry, and ctypes for an interpreter that has none) against plain ctypes
on the same C functions: same statuses for the same arguments, the same things refused.  Every call ends before a launch.  And where the
module comes from: it is built for one interpreter and says so in its name."""
import ctypes
import importlib.machinery
import os
import shutil
import subprocess
import sys

import pytest

import paper_2509_24695_amd as sv
from paper_2509_24695_amd import binding

FAKE, BIG = 0x10000, 1 << 33


@pytest.fixture(params=["module", "ctypes"])
def route(request, monkeypatch):
    lib = sv.load_library()
    calls = binding._load_entry(lib) if request.param == "module" else binding._CtypesCalls(lib)
    assert isinstance(calls, binding._CtypesCalls) == (request.param == "ctypes")
    monkeypatch.setattr(binding, "_entry", calls)


class _Tensor:
    def data_ptr(self):
        return FAKE

    def numel(self):
        return 1 << 10

    def element_size(self):
        return 4


class _Index:
    def __index__(self):
        return 0


def _desc(**kw):
    return sv.TensorDesc(**{**dict(B=1, H=2, N=128, d=64, stride_b=2 * 128 * 64, stride_h=128 * 64, stride_n=64, dtype=sv.SV_BF16), **kw})


def _rope(**kw):
    return sv.Rope3D(**{**dict(frames=2, rows=8, cols=8, n_t=12, n_h=10, n_w=10, cs_t=FAKE, cs_h=FAKE, cs_w=FAKE), **kw})


def _status(f, *a, **kw):
    try:
        f(*a, **kw)
    except sv.SvError as e:
        return e.status
    return 0


@pytest.mark.parametrize("desc,rope,t0,t1,eps,ws,wb", [
    (_desc(), _rope(), 0, 0, 1e-6, FAKE, BIG), (_desc(d=48), _rope(), 0, 0, 1e-6, FAKE, BIG), (None, _rope(), 0, 0, 1e-6, FAKE, BIG),
    (_desc(), None, 0, 0, 1e-6, FAKE, BIG), (_desc(), _rope(rows=7), 0, 0, 1e-6, FAKE, BIG), (_desc(), _rope(cs_h=None), 0, 0, 1e-6, FAKE, BIG),
    (_desc(), _rope(cs_w=_Tensor()), 0, 0, 0, _Tensor(), BIG), (_desc(), _rope(), -1, 4, 1e-6, FAKE, BIG), (_desc(), _rope(), 0, 129, 1e-6, FAKE, BIG),
    (_desc(stride_n=1 << 40), _rope(), 0, 0, 1e-6, FAKE, BIG), (_desc(), _rope(), 0, 0, -1.0, FAKE, BIG), (_desc(), _rope(), 0, 0, 1e-6, FAKE + 8, BIG),
    (_desc(), _rope(), 0, 0, 1e-6, None, BIG), (_desc(), _rope(), 0, 0, 1e-6, FAKE, 1000),
])
def test_statuses_are_those_of_the_c_functions(route, desc, rope, t0, t1, eps, ws, wb):
    lib = sv.load_library()
    d, r, p = desc._c() if desc else None, rope._c() if rope else None, binding._ptr
    dp, rp = ctypes.byref(d) if d else None, ctypes.byref(r) if r else None
    x = _Tensor()
    assert _status(sv.sv_linattn_state, x, FAKE, desc, t0, t1, True, FAKE, x, ws, wb) == lib.sv_linattn_state(FAKE, FAKE, dp, t0, t1, 1, FAKE, FAKE, p(ws), wb, None)
    assert _status(sv.sv_linattn_apply, x, desc, t0, t1, FAKE, FAKE, eps, x, stream=0) == lib.sv_linattn_apply(FAKE, dp, t0, t1, FAKE, FAKE, eps, FAKE, None)
    assert _status(sv.sv_linattn_state_rope3d, x, x, desc, rope, t0, t1, 1, FAKE, FAKE, ws, wb) == lib.sv_linattn_state_rope3d(FAKE, FAKE, dp, rp, t0, t1, 1, FAKE, FAKE, p(ws), wb, None)
    assert _status(sv.sv_linattn_apply_rope, x, desc, x, t0, t1, FAKE, FAKE, eps, ws) == lib.sv_linattn_apply_rope(FAKE, dp, FAKE, t0, t1, FAKE, FAKE, eps, p(ws), None)
    # block steps launch on valid arguments: a workspace that is too small ends every call
    for name, extra_py, extra_c in (("step", (), ()), ("lookahead", (), ()), ("step_rope", (x,), (FAKE,)), ("lookahead_rope", (None,), (None,)),
                                    ("step_rope3d", (rope,), (rope and ctypes.byref(rope._c()),)), ("lookahead_rope3d", (rope,), (rope and ctypes.byref(rope._c()),))):
        got = _status(getattr(sv, "sv_block_linattn_" + name), x, x, x, desc, *extra_py, FAKE, FAKE, eps, x, ws, min(wb, 4096))
        assert got == getattr(lib, "sv_block_linattn_" + name)(FAKE, FAKE, FAKE, dp, *extra_c, FAKE, FAKE, eps, FAKE, p(ws), min(wb, 4096), None) != 0


def test_conversion_of_single_arguments(route):
    d, x = _desc(), _Tensor()
    assert _status(sv.sv_linattn_apply, x, d, _Index(), False, FAKE, FAKE, 0, x) == 0
    assert _status(sv.sv_linattn_state, x, x, d, 0, 0, 1.5, FAKE, FAKE, x) == 6          # the workspace's own 4 KiB are too few
    for bad in (dict(tok_begin=0.0), dict(tok_begin="0"), dict(tok_begin=None)):
        with pytest.raises(ctypes.ArgumentError):
            sv.sv_linattn_apply(x, d, bad["tok_begin"], 0, FAKE, FAKE, 1e-6, x)
    with pytest.raises(AttributeError):
        sv.sv_linattn_apply(object(), d, 0, 0, FAKE, FAKE, 1e-6, x)
    with pytest.raises(AttributeError):
        sv.sv_linattn_state(x, x, d, 0, 0, 1, FAKE, FAKE, FAKE)                             # an address has no size of its own
    with pytest.raises(AttributeError):
        sv.sv_linattn_apply(x, d, 0, 0, FAKE, FAKE, 1e-6, x, stream=object())
    with pytest.raises(TypeError):
        sv.sv_linattn_apply(x, _desc(B=1.0), 0, 0, FAKE, FAKE, 1e-6, x)
    with pytest.raises((TypeError, ValueError)):
        sv.sv_linattn_apply(x, d, 0, 0, FAKE, FAKE, "eps", x)
    assert _status(sv.sv_tconv_block_step, x, FAKE, None, x, None, 1, 1, 1, 12) == 3
    with pytest.raises(ctypes.ArgumentError):
        sv.sv_tconv_block_step(x, FAKE, None, x, None, 1, 1, 1.0, 16)


def test_the_module_is_for_one_interpreter():
    """Its name carries the interpreter's ABI, so that another Python does not load it."""
    from paper_2509_24695_amd import build
    assert build.ENTRY == binding._ENTRY_PATH and os.path.exists(build.ENTRY)
    assert os.path.basename(build.ENTRY) == "_sventry" + importlib.machinery.EXTENSION_SUFFIXES[0]
    assert "cpython" in importlib.machinery.EXTENSION_SUFFIXES[0]
    assert not os.path.exists(os.path.join(os.path.dirname(build.ENTRY), "_sventry.so"))


def test_a_package_with_another_interpreters_module_works(tmp_path):
    """The library as another Python's build leaves it: no module with this one's suffix, one that is no module at all."""
    pkg = tmp_path / "paper_2509_24695_amd"
    pkg.mkdir()
    for name in ("__init__.py", "binding.py", "libsvlinattn.so"):
        shutil.copy(os.path.join(os.path.dirname(binding.__file__), name), pkg / name)
    (pkg / "_sventry.cpython-399-x86_64-linux-gnu.so").write_bytes(b"not this interpreter's")
    (pkg / "_sventry.so").write_bytes(b"of no interpreter in particular")
    code = ("import paper_2509_24695_amd as sv\n"
            "d = sv.TensorDesc(1, 2, 128, 64, 16384, 8192, 64, sv.SV_BF16)\n"
            "sv.sv_linattn_apply(65536, d, 0, 0, 65536, 65536, 1e-6, 65536)\n"
            "try:\n    sv.sv_linattn_state(65536, 65536, d, 0, 999, 0, 65536, 65536, 65536, 1 << 33)\n"
            "except sv.SvError as e:\n    print(sv.__file__, e.status)\n")
    res = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path)}, stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.split() == [str(pkg / "__init__.py"), "5"], res.stdout


@pytest.mark.parametrize("lacking", ["headers", "compiler"])
def test_builds_without_what_the_module_needs(lacking, tmp_path, monkeypatch):
    from paper_2509_24695_amd import build
    monkeypatch.setattr(build, "ENTRY", str(tmp_path / os.path.basename(build.ENTRY)))
    stale = tmp_path / "_sventry.so"
    stale.write_bytes(b"of other sources")
    if lacking == "headers":
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    else:
        monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert build.build_entry() is None and os.listdir(tmp_path) == []
