"""C-ABI library checks that need no GPU: it loads, exports every function
declared in include/chns.h, and rejects bad descriptions before touching the
device."""
import ctypes
import os
import re

import pytest

import paper_2009_06628_amd as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    src = open(os.path.join(ROOT, "include", "chns.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(chns_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    lib = P.load_library()
    names = declared_functions()
    assert "chns_step" in names and "chns_solve_pressure" in names
    for name in names:
        assert hasattr(lib, name), name
    assert set(P.EXPORTS) >= set(names)


def test_error_strings():
    lib = P.load_library()
    for code in (0, 1, -1, -2, -3, -4):
        assert lib.chns_error_string(code)


@pytest.mark.parametrize("n,bc", [((64, 64), ("periodic", "periodic")), ((256, 512), ("periodic", "wall")),
                                  ((96, 96), ("periodic", "periodic")), ((128, 128, 128), ("periodic",) * 3),
                                  ((20, 20), ("wall", "wall"))])
def test_workspace_size_supported(n, bc):
    b = P.workspace_size(n, 1.0 / n[0], bc)
    cells = 1
    for x in n:
        cells *= x
    assert b > 8 * cells * 10


@pytest.mark.parametrize("n", [(50, 50), (1, 8), (0, 0), (100, 100)])
def test_workspace_size_rejects_unsupported(n):
    with pytest.raises(P.CHNSError) as ei:
        P.workspace_size(n, 0.1, ("periodic", "periodic"))
    assert ei.value.code == P.CHNS_EINVAL


def test_create_rejects_small_workspace_before_device_use():
    lib = P.load_library()
    d = P.make_desc((64, 64), 1 / 64, ("periodic", "periodic"))
    h = ctypes.c_void_p()
    rc = lib.chns_create_grid(ctypes.byref(d), ctypes.c_void_p(4096), ctypes.c_size_t(1024), None, ctypes.byref(h))
    assert rc == P.CHNS_ENOMEM
    rc = lib.chns_create_grid(ctypes.byref(d), ctypes.c_void_p(4097), ctypes.c_size_t(1 << 30), None, ctypes.byref(h))
    assert rc == P.CHNS_EINVAL
    d.dim = 4
    rc = lib.chns_create_grid(ctypes.byref(d), ctypes.c_void_p(4096), ctypes.c_size_t(1 << 30), None, ctypes.byref(h))
    assert rc == P.CHNS_EINVAL


def test_binding_fails_loudly_without_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    with pytest.raises(RuntimeError):
        P.create_grid((64, 64), 1 / 64, ("periodic", "periodic"))


@pytest.mark.parametrize("n,bc", [((128, 128), ("periodic", "periodic")), ((16, 16, 16), ("wall", "wall", "periodic"))])
def test_adjoint_workspace_size(n, bc):
    lib = P.load_library()
    d = P.make_desc(n, 1.0 / n[0], bc)
    out = ctypes.c_size_t(0)
    assert lib.chns_adjoint_workspace_size(ctypes.byref(d), ctypes.byref(out)) == P.CHNS_OK
    cells = 1
    for x in n:
        cells *= x
    dim = len(n)
    # 11 cell arrays and 8 face arrays per axis, plus partials
    assert out.value >= 8 * cells * (11 + 8 * dim)
    d.dim = 5
    assert lib.chns_adjoint_workspace_size(ctypes.byref(d), ctypes.byref(out)) == P.CHNS_EINVAL
    assert lib.chns_adjoint_step(None, None, None, None, None) == P.CHNS_EINVAL


def test_batch_workspace_size_and_validation():
    lib = P.load_library()
    descs = (P.chns_grid_desc * 3)()
    for i, n in enumerate((64, 96, 256)):
        descs[i] = P.make_desc((n, n), 1.0 / n, ("periodic", "periodic"))
    out = ctypes.c_size_t(0)
    assert lib.chns_batch_workspace_size(3, descs, ctypes.byref(out)) == P.CHNS_OK
    cells = 64 * 64 + 96 * 96 + 256 * 256
    assert out.value >= 8 * cells * 20
    descs[1].precision = P.CHNS_FP32_REFINE      # mixed precision is rejected
    assert lib.chns_batch_workspace_size(3, descs, ctypes.byref(out)) == P.CHNS_EINVAL
    descs[1].precision = P.CHNS_FP64
    descs[2].n[0] = 50                           # unsupported size
    assert lib.chns_batch_workspace_size(3, descs, ctypes.byref(out)) == P.CHNS_EINVAL
    h = ctypes.c_void_p()
    props = (P.chns_props * 3)()
    assert lib.chns_create_batch(3, descs, props, ctypes.c_void_p(4096), ctypes.c_size_t(1 << 30), None,
                                 ctypes.byref(h)) == P.CHNS_EINVAL


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU: --gpus N > 1 (or a multi-rank launch) exits
    with a message before touching torch or the device."""
    import subprocess
    import sys
    for extra_env, args in (({}, ["--gpus", "2"]), ({"WORLD_SIZE": "2"}, [])):
        env = dict(os.environ, **extra_env)
        r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py")] + args, capture_output=True, text=True,
                           env=env, timeout=120)
        assert r.returncode == 2
        assert "one GPU only" in r.stderr
        assert r.stdout == ""


def test_workspace_carries_no_vector_that_no_solve_uses():
    """A z of the one-reduction CG is carved only where solves take that form
    (4096 x 128: 1024 tiles; 4096 x 256 has 2048): one array per velocity
    component less per cell.  (No direct Cahn-Hilliard solve on these axes, so
    all else is per cell or smaller on the larger grid.)"""
    per_cell = [P.workspace_size((4096, m), 1.0 / 4096, ("periodic", "wall")) / (4096 * m) for m in (128, 256)]
    assert per_cell[0] - per_cell[1] >= 16.0
