"""The library's kernels and their launchers on the CPU, lane by lane, under an address sanitizer
(tests/host_lanes): every buffer is allocated to the byte and filled with NaN, so a read or write
outside it ends the program, a read of what nobody wrote shows in the result, and so does a barrier
or a wave operation that part of a workgroup does not reach.  The cases are the lattices and widths at which
the kernels, site maps, column groups and block layouts change: partial tiles, more
than one tile per workgroup, one column to sixteen.

Results are compared with the oracle at the tolerances of the GPU tests (tests/test_gpu_parity.py,
tests/test_gpu_lowp.py, tests/test_gpu_learned.py)."""

import importlib.util
import os
import platform
import subprocess

import numpy as np
import pytest

import wdinputs as wi
from oracle import WilsonClover
from oracle import learned as ln
from oracle.bbicggr import true_residual
from oracle.jacobi import jacobi_apply
from oracle.lowp import apply_lowp, jacobi_sweeps_lowp

HERE = os.path.dirname(os.path.abspath(__file__))
PREC = {"f64": 0, "f32": 1, "bf16": 2, "f64c32": 3, "f64cbf16": 4}
KAPPA, CSW = 0.12, 1.6


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    spec = importlib.util.spec_from_file_location("host_lanes_build", os.path.join(HERE, "host_lanes", "build.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    if not os.path.exists(m.CLANG) or platform.machine() != "x86_64":
        pytest.skip("needs the ROCm clang++ on x86-64")
    return m.build(str(tmp_path_factory.mktemp("host_lanes")))


def _theta(seed, scale=0.2):
    rng = np.random.default_rng(seed)
    th = ln.identity_theta()
    th += scale * (rng.standard_normal(th.shape) + 1j * rng.standard_normal(th.shape))
    return th.astype(np.complex64)


def _tiled(X, V):
    """Rows k V + s of each column in the order (s // 64, k, s % 64)."""
    L = X.shape[0]
    return np.ascontiguousarray(X.reshape(L, 12, V // 64, 64).transpose(0, 2, 1, 3)).reshape(L, 12, V)


def _standard(X, V):
    L = X.shape[0]
    return np.ascontiguousarray(X.reshape(L, V // 64, 12, 64).transpose(0, 2, 1, 3)).reshape(L, 12, V)


class Case:
    def __init__(self, dims, L, bc=1, max_L=None, layout=0, kind=0, seed=900):
        self.dims, self.L, self.bc, self.layout, self.kind = dims, L, bc, layout, kind
        self.max_L = max_L or L
        self.U = wi.random_links(dims, 0.3, seed)
        self.op = WilsonClover(dims, self.U, KAPPA, CSW, bc_t=bc)
        self.V = self.op.V
        self.theta = _theta(seed + 1)
        self.A = wi.gaussian_block(self.V, L, seed + 2)
        self.B = wi.gaussian_block(self.V, L, seed + 3)

    def run(self, exe, tmp, call, prec="f64", j=0, loss=0):
        fin, fout = os.path.join(tmp, "in"), os.path.join(tmp, "out")
        with open(fin, "wb") as f:
            f.write(self.U.tobytes())
            f.write(self.theta.tobytes())
            for X in (self.A, self.B):
                f.write((_tiled(X, self.V) if self.layout else X).tobytes())
        args = [*self.dims, self.bc, self.max_L, self.layout, self.kind, KAPPA, CSW, call, PREC[prec], self.L, j, loss]
        r = subprocess.run([exe, *map(str, args), fin, fout], capture_output=True, text=True, timeout=300,
                           env={**os.environ, "ASAN_OPTIONS": "detect_leaks=0:detect_stack_use_after_return=0"})
        assert r.returncode == 0, f"{args}: {r.returncode}\n{r.stderr[:3000]}"
        return np.fromfile(fout) if call == "grad" else np.fromfile(fout, dtype=np.complex128)

    def block(self, out):
        X = out.reshape(self.L, 12, self.V)
        return _standard(X, self.V) if self.layout else X


def _rel(a, b):
    assert np.all(np.isfinite(a))
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


def _lowp_close(Z, Zo, prec):
    err = _rel(Z, Zo)
    if prec == "f32":
        assert err < 2e-6
    else:
        assert err < 2.0 ** -7 and np.linalg.norm(Z - Zo) < 1e-3 * np.linalg.norm(Zo)


# dims, L, bc, layout: partial tiles in the linear map, in planes, whole tiles, the tiled layout, an
# XCD split that leaves workgroups without sites
SHAPES = [((2, 2, 2, 2), 1, 0, 0), ((5, 3, 3, 5), 2, 1, 0), ((5, 3, 3, 5), 3, 1, 0), ((3, 4, 5, 6), 7, 0, 0),
          ((2, 3, 5, 7), 16, 1, 0), ((4, 4, 4, 4), 4, 1, 1), ((16, 4, 2, 2), 13, 0, 1), ((2, 2, 2, 32), 5, 1, 0),
          ((8, 6, 4, 10), 6, 1, 1), ((7, 9, 8, 3), 5, 0, 0), ((8, 16, 8, 3), 2, 1, 1)]


@pytest.mark.parametrize("dims,L,bc,layout", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_apply(exe, tmp_path, dims, L, bc, layout, prec):
    c = Case(dims, L, bc, layout=layout)
    Y = c.block(c.run(exe, tmp_path, "apply", prec))
    x = c.op.from_block(c.A)
    if prec == "f64":
        assert _rel(Y, c.op.to_block(c.op.apply_A(x))) < 1e-13
    else:
        _lowp_close(Y, c.op.to_block(apply_lowp(c.op, x, prec)), prec)


@pytest.mark.parametrize("dims,L,bc,layout", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_jacobi(exe, tmp_path, dims, L, bc, layout, prec):
    c = Case(dims, L, bc, max_L=min(16, L + 2), layout=layout)
    Y = c.block(c.run(exe, tmp_path, "jacobi", prec, j=4))
    x = c.op.from_block(c.A)
    if prec == "f64":
        assert _rel(Y, c.op.to_block(jacobi_apply(c.op, x, 4))) < 1e-13
    else:
        _lowp_close(Y, c.op.to_block(jacobi_sweeps_lowp(c.op, x, 4, prec)), prec)


@pytest.mark.parametrize("dims,L", [((5, 3, 3, 5), 1), ((5, 3, 3, 5), 7), ((4, 4, 4, 4), 2)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16", "f64c32", "f64cbf16"])
@pytest.mark.parametrize("kind,j", [(1, 3), (0, 1)])
def test_jacobi_forms_stay_in_bounds(exe, tmp_path, dims, L, prec, kind, j):
    c = Case(dims, L, kind=kind)
    assert np.all(np.isfinite(c.run(exe, tmp_path, "jacobi", prec, j=j)))


@pytest.mark.parametrize("dims,L,bc,layout", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_learned_apply(exe, tmp_path, dims, L, bc, layout, prec):
    c = Case(dims, L, bc, layout=layout)
    Y = c.block(c.run(exe, tmp_path, "learned", prec))
    Yo = c.op.to_block(ln.forward(c.op, c.theta.astype(np.complex128), c.op.from_block(c.A)))
    assert _rel(Y, Yo) < {"f32": 1e-4, "f64": 1e-13}[prec]


# 17 x 10 x 10 x 10: 265 whole tiles and a partial one, so that some of the weight gradient's 256
# workgroups take two
@pytest.mark.parametrize("dims,L,layout,loss", [((5, 3, 3, 5), 1, 0, "error"), ((5, 3, 3, 5), 3, 0, "residual"),
                                                ((2, 3, 5, 7), 5, 0, "error"), ((4, 4, 4, 4), 12, 1, "residual"),
                                                ((17, 10, 10, 10), 1, 0, "error")])
def test_gradient(exe, tmp_path, dims, L, layout, loss):
    c = Case(dims, L, max_L=min(16, L + 1), layout=layout)
    out = c.run(exe, tmp_path, "grad", loss=int(loss == "residual"))
    lv, G = out[0], out[1:].view(np.complex128).reshape(3, 9, 4, 4)
    th = c.theta.astype(np.complex128)
    if loss == "error":
        lo, Go = ln.grad(c.op, th, c.op.from_block(c.A), c.op.from_block(c.B))
    else:
        lo, Go = ln.grad_residual(c.op, th, c.op.from_block(c.A))
    assert abs(lv - lo) / lo < 1e-5 and _rel(G, Go) < 1e-5


# rows: fewer than one chunk of 256, a last partial one, and more chunks than the 384 workgroups
@pytest.mark.parametrize("dims,L", [((2, 2, 2, 2), 16), ((3, 4, 5, 6), 5), ((3, 3, 7, 131), 2)])
def test_gram(exe, tmp_path, dims, L):
    c = Case(dims, L)
    out = c.run(exe, tmp_path, "gram").reshape(2, L, L)
    P, Q = c.A.reshape(L, -1).T, c.B.reshape(L, -1).T
    want = P.conj().T @ Q
    assert _rel(out[0], want) < 1e-12 and _rel(out[1], want) < 1e-12


@pytest.mark.parametrize("call,prec,dims,L,layout", [("solve", "f64", (5, 3, 3, 5), 1, 0),
                                                    ("solve", "f64", (3, 4, 5, 2), 10, 0),
                                                    ("solve", "bf16", (4, 4, 2, 2), 3, 1),
                                                    ("solve", "f32", (3, 2, 5, 2), 5, 0),
                                                    ("stab", "f64", (4, 4, 2, 2), 3, 1)])
def test_solve(exe, tmp_path, call, prec, dims, L, layout):
    c = Case(dims, L, bc=0, layout=layout)
    X = c.block(c.run(exe, tmp_path, call, prec, j=3))
    tr = true_residual(c.op.A_mat, c.op.block_to_mat(c.A), c.op.block_to_mat(X))
    assert np.max(tr) < 1e-10
