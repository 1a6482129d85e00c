"""Builds and loads host_plans.cpp: the library's host-side planning."""
import ctypes as C
import os
import subprocess
import tempfile

from paper_2506_03747_amd import _native
from paper_2506_03747_amd.build import CSRC, HIPCC, LIB, ROOT

HERE = os.path.dirname(os.path.abspath(__file__))
_lib = None


def lib():
    global _lib
    if _lib is None:
        _native.lib()
        with tempfile.TemporaryDirectory() as tmp:
            so = os.path.join(tmp, "host_plans.so")
            subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-shared", "-fPIC",
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(HERE, "host_plans.cpp"),
                            "-o", so, "-Wl,-Bsymbolic", "-x", "none", LIB, f"-Wl,-rpath,{os.path.dirname(LIB)}"],
                           check=True)
            _lib = C.CDLL(so)
    return _lib


def params(nx, ny, T, bin_ps=8.0, fwhm_ps=50.0, laser=(0, 0), cosines=True):
    G, half = _native.Grid, 1.0
    return _native.Params(G(nx, ny, half, half, 0.0, 0.0), G(*laser, half if laser[0] else 0.0, half if laser[0] else 0.0,
                                                             0.0, 0.0),
                          0.0, bin_ps, T, _native.NLOS_F_COSINES if cosines else 0, fwhm_ps)


FORWARD = ("tl", "tx", "ty", "pair", "one", "groups", "n_split", "n_windows", "workgroups", "lds_bytes")


def forward_plan(prm, n_patches, target=256, solo=True):
    out = (C.c_int64 * len(FORWARD))()
    rc = lib().host_forward_plan(C.byref(prm), n_patches, C.c_int64(target), int(solo), out)
    assert rc == 0, rc
    return dict(zip(FORWARD, out))


SMOOTH = ("moments", "tx", "ty", "tiles", "split", "workgroups", "per_cu", "table_bytes")
ADJOINT = ("moments", "rows", "split", "patch_blocks", "two_buffers", "head_bytes", "lds_bytes")


def smooth_plan(prm, n_patches):
    out = (C.c_int64 * len(SMOOTH))()
    rc = lib().host_smooth_plan(C.byref(prm), n_patches, out)
    assert rc == 0, rc
    return dict(zip(SMOOTH, out))


def adjoint_plan(prm, n_patches):
    out = (C.c_int64 * len(ADJOINT))()
    rc = lib().host_adjoint_plan(C.byref(prm), n_patches, out)
    assert rc == 0, rc
    return dict(zip(ADJOINT, out))


def moment_fit(sigma, adjoint):
    """(nodes, coefficients [m][j]) of the smooth kernels' polynomials, or None: by taps."""
    node, coef = (C.c_double * 16)(), (C.c_double * 256)()
    n = lib().host_moment_fit(C.c_double(sigma), int(adjoint), node, coef)
    return (list(node)[:n], [list(coef)[m * n:(m + 1) * n] for m in range(n)]) if n else None
