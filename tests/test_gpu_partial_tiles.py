"""The learned layers, their gradient and the BF16 pairs of columns where the library's own blocks
(tiles of 64 sites, the last one padded) end in a partial tile, and where the weight gradient's
workgroups take more than one tile.  Against the FP64 oracle and the oracle's emulated storage, with
the tolerances of tests/test_gpu_learned.py (1e-4 for an application, 1e-13 in FP64, 1e-5 for the
gradient and the loss) and tests/test_gpu_lowp.py (BF16: 2^-7 of the largest element, 1e-3 in the
Frobenius norm)."""

import numpy as np
import pytest

import wdinputs as wi
from oracle import WilsonClover
from oracle import learned as ln
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


def _ctx(pkg, dims, max_L, seed):
    U = wi.random_links(dims, 0.3, seed)
    c = pkg.Context(dims, bc_t=1, max_L=max_L)
    c.set_links(U)
    c.set_params(0.12, 1.6)
    rng = np.random.default_rng(seed + 1)
    th = ln.identity_theta()
    th += 0.2 * (rng.standard_normal(th.shape) + 1j * rng.standard_normal(th.shape))
    th = th.astype(np.complex64).astype(np.complex128)
    c.set_learned(th)
    return c, WilsonClover(dims, U, 0.12, 1.6, bc_t=1), th


def _maxrel(a, b):
    assert np.all(np.isfinite(a))
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", [2, 3, 7])
def test_learned_apply(pkg, L, prec):
    c, op, th = _ctx(pkg, (5, 3, 3, 5), 9, 321)
    R = wi.gaussian_block(op.V, L, 322)
    Z = c.learned_apply(torch.from_numpy(R).cuda(), prec=prec).cpu().numpy()
    assert _maxrel(Z, op.to_block(ln.forward(op, th, op.from_block(R)))) < {"f32": 1e-4, "f64": 1e-13}[prec]
    c.close()


# 17 x 10 x 10 x 10: 265 whole tiles and a partial one over 256 workgroups
@pytest.mark.parametrize("loss", ["error", "residual"])
@pytest.mark.parametrize("dims,L", [((5, 3, 3, 5), 1), ((5, 3, 3, 5), 3), ((5, 3, 3, 5), 5), ((17, 10, 10, 10), 3)])
def test_gradient(pkg, dims, L, loss):
    c, op, th = _ctx(pkg, dims, 6, 323)
    R = wi.gaussian_block(op.V, L, 324)
    E = wi.gaussian_block(op.V, L, 325)
    lv, G = c.learned_grad(torch.from_numpy(R).cuda(), torch.from_numpy(E).cuda(), loss=loss)
    if loss == "error":
        lo, Go = ln.grad(op, th, op.from_block(R), op.from_block(E))
    else:
        lo, Go = ln.grad_residual(op, th, op.from_block(R))
    assert abs(lv - lo) / lo < 1e-5
    assert _maxrel(G, Go) < 1e-5
    c.close()


# 21 x 15 x 15 x 14 = 1033 whole tiles and a partial one: BF16 blocks of three to six columns take pairs
@pytest.mark.parametrize("L", [3, 4, 5, 6])
def test_bf16_pairs(pkg, L):
    c, op, _ = _ctx(pkg, (21, 15, 15, 14), 8, 326)
    R = wi.gaussian_block(op.V, L, 327)
    Z = c.jacobi(torch.from_numpy(R).cuda(), 3, prec="bf16").cpu().numpy()
    Zo = op.to_block(jacobi_sweeps_lowp(op, op.from_block(R), 3, "bf16"))
    assert _maxrel(Z, Zo) < 2.0 ** -7 and np.linalg.norm(Z - Zo) < 1e-3 * np.linalg.norm(Zo)
    c.close()


# the conversion of a block streams where block and copy exceed 256 MB: sixteen columns of these
# lattices do, four do not.  A column's value does not depend on the width of its block
@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("dims,layout", [((21, 17, 16, 13), "standard"), ((16, 16, 16, 20), "tiled")])
def test_apply_on_streamed_blocks(pkg, dims, layout, prec):
    c, op, _ = _ctx(pkg, dims, 16, 328)
    c.set_layout(layout)
    R = torch.from_numpy(wi.gaussian_block(op.V, 16, 329)).cuda()
    Y = c.apply(R, prec=prec)
    assert torch.isfinite(torch.view_as_real(Y)).all()
    for lo in (0, 7, 12):
        assert torch.equal(c.apply(R[lo:lo + 4].contiguous(), prec=prec), Y[lo:lo + 4])
    c.close()
