"""The library's own FP32 / BF16 blocks (tiles of 64 sites, the last one padded, planes
interleaved in 16-byte words) and the kernels chosen by width and size.

Against the oracle's emulation of the storage where a tile is partial, with the tolerances of
tests/test_gpu_lowp.py (only the order of the float32 operations differs: 2e-6; a BF16 iterate
may flip an element by one ulp: 2^-7 of the largest element, 1e-3 in the Frobenius norm).  Columns
are independent, so a column has the same value, bit for bit, in a BF16 block of any width, whichever
kernel the width selects (one column per wave, pairs of columns, LDS-staged).  In FP32 this holds
from three columns on: the kernel of one and two columns rounds the rebuilt third row of a link
in another order (with BF16 rows the products are exact)."""

import numpy as np
import pytest

import wdinputs as wi
from oracle import WilsonClover
from oracle.lowp import jacobi_sweeps_lowp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0907_3261_amd as p
    p.load()
    return p


def _ctx(pkg, dims, U, kappa, csw, bc_t, max_L, kind=0):
    c = pkg.Context(dims, bc_t=bc_t, max_L=max_L)
    c.set_links(U)
    c.set_params(kappa, csw, kind)
    return c


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("dims,L", [((5, 3, 3, 5), 2), ((5, 3, 3, 5), 7), ((3, 4, 5, 6), 16), ((2, 2, 2, 2), 3)])
def test_partial_tiles_against_emulated_storage(pkg, dims, L, prec):
    U = wi.random_links(dims, 0.3, 311)
    op = WilsonClover(dims, U, 0.12, 1.6, bc_t=1)
    c = _ctx(pkg, dims, U, 0.12, 1.6, 1, L)
    R = wi.gaussian_block(op.V, L, 312)
    Z = c.jacobi(torch.from_numpy(R).cuda(), 4, prec=prec).cpu().numpy()
    Zo = op.to_block(jacobi_sweeps_lowp(op, op.from_block(R), 4, prec))
    err = np.max(np.abs(Z - Zo)) / np.max(np.abs(Zo))
    if prec == "f32":
        assert err < 2e-6
    else:
        assert err < 2.0 ** -7 and np.linalg.norm(Z - Zo) < 1e-3 * np.linalg.norm(Zo)
    c.close()


# 1024 tiles is where BF16 blocks of three to six columns change kernels; 16 x 16 x 16 x 15 is
# below it, 20 x 20 x 20 x 9 above it with partial tiles in every plane
@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (16, 16, 16, 15), (20, 20, 20, 9), (5, 3, 3, 5)])
def test_a_column_does_not_depend_on_the_width(pkg, dims, kind, prec):
    U = wi.random_links(dims, 0.3, 313)
    c = _ctx(pkg, dims, U, 0.12, 1.6, 1, 12, kind)
    V = wi.volume(dims)
    R = torch.from_numpy(wi.gaussian_block(V, 12, 314)).cuda()
    Z = c.jacobi(R, 3, prec=prec)
    Y = c.apply(R, prec=prec)
    assert torch.isfinite(torch.view_as_real(Z)).all()
    for lo, L in [(0, 1), (1, 2), (2, 3), (4, 4), (0, 5), (5, 6), (3, 7)]:
        if prec == "f32" and L < 3:
            continue
        part = R[lo:lo + L].contiguous()
        assert torch.equal(c.jacobi(part, 3, prec=prec), Z[lo:lo + L]), L
        assert torch.equal(c.apply(part, prec=prec), Y[lo:lo + L]), L
    c.close()
