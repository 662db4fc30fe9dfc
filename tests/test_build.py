"""The two built files belong together, and the package works without the second one."""
import os
import subprocess
import sys

import pytest

from paper_2508_06133_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def places(tmp_path, monkeypatch):
    lib, host = tmp_path / "libkvsched.so", tmp_path / "kvsched_host.so"
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "HOST", str(host))
    return lib, host


def test_stale_by_the_older_file(places):
    lib, host = places
    assert build.is_stale()
    lib.write_text("built")
    assert build.is_stale()
    host.write_text("built")
    assert not build.is_stale()
    os.utime(host, (1, 1))  # (a module left over from an earlier build)
    assert build.is_stale()
    os.utime(host)
    os.utime(lib, (1, 1))
    assert build.is_stale()


@pytest.mark.parametrize("fails", ["host.cpp", "-shared", "check", None])
def test_all_or_nothing(places, monkeypatch, fails):
    lib, host = places
    lib.write_text("old"), host.write_text("old")

    def run(cmd, **_):
        out = cmd[cmd.index("-o") + 1]
        if fails and any(os.path.basename(a) == fails for a in cmd):
            raise subprocess.CalledProcessError(1, cmd)
        with open(out, "w") as f:
            f.write("new")

    def check(*_):
        if fails == "check":
            raise RuntimeError("registers")

    monkeypatch.setattr(build.subprocess, "check_call", run)
    monkeypatch.setattr(build, "check_reserved_vgprs", check)
    if fails:
        with pytest.raises((subprocess.CalledProcessError, RuntimeError)):
            build.build()
    else:
        assert build.build() == str(lib)
    assert lib.read_text() == host.read_text() == ("old" if fails else "new")
    assert sorted(p.name for p in lib.parent.iterdir()) == ["kvsched_host.so", "libkvsched.so"]


def test_name_of_the_module_is_one_interpreters():
    import importlib.machinery

    suffix = os.path.basename(build.HOST)[len("kvsched_host"):]
    assert suffix in importlib.machinery.EXTENSION_SUFFIXES and sys.implementation.cache_tag.split("-")[1] in suffix


def _import_with(stand_in):
    """Imports the binding in a process of its own where `stand_in` takes the native module's place."""
    code = ("import sys, types, warnings\n" + stand_in + "\n"
            "with warnings.catch_warnings(record=True) as seen:\n"
            "    warnings.simplefilter('always')\n"
            "    from paper_2508_06133_amd import kvsched\n"
            "print(kvsched._host is None, any(issubclass(w.category, RuntimeWarning) and 'kvsched_host' in str(w.message) for w in seen))\n")
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr
    return done.stdout.split()


def test_import_without_the_module():
    assert _import_with("sys.modules['paper_2508_06133_amd.kvsched_host'] = None") == ["True", "True"]
    assert _import_with("m = types.ModuleType('kvsched_host'); m.torch_version = '1.0.0'\n"
                        "import paper_2508_06133_amd as package; package.kvsched_host = m\n"
                        "sys.modules['paper_2508_06133_amd.kvsched_host'] = m") == ["True", "True"]
    assert _import_with("") == ["False", "False"]


@pytest.mark.gpu
def test_calls_without_the_module(monkeypatch):
    import numpy as np
    import torch

    import oracle
    from paper_2508_06133_amd import kvsched

    monkeypatch.setattr(kvsched, "_host", None)
    rng = np.random.default_rng(2)
    n, M = 90, 700
    s, o = rng.integers(1, 60, n).astype(np.int32), rng.integers(1, 90, n).astype(np.int32)
    rows = np.stack([rng.permutation(n) for _ in range(5)]).astype(np.int32)
    ds, do, dr = (torch.from_numpy(x).to("cuda:0") for x in (s, o, rows))
    ctx = kvsched.Context(0)
    print(f"calls of a planning step through ctypes: n={n}", flush=True)
    order = ctx.sortedF(ds, do, M)[0]
    tel, comp = ctx.simulate(dr, ds, do, M)
    best = ctx.argmin(tel)
    tel_o, comp_o = oracle.simulate_many(s, o, M, rows)
    assert (order.cpu().numpy() == oracle.sortedF(s, o, M)[0]).all()
    assert (tel.cpu().numpy() == tel_o).all() and (comp.cpu().numpy() == comp_o).all()
    assert best.tolist() == [int(tel_o.argmin()), int(tel_o.min())]
    ctx.close()
