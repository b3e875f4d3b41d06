"""The one-workgroup eigensolver behind the preconditioner at the edges of its size classes (20, 44, 64, 154 and 200
rows, odd and even, and the first size of the multi-launch path), against the oracle's eigh-based preconditioner.
Tolerance: the bound of the other preconditioner tests (1e-10), which leaves the eigensolver's 1e-15 relative
off-diagonal norm five orders of magnitude for the regularised inverse at delta = 0.05."""
import numpy as np
import pytest

from gpu_helpers import rel, require_gpu, to_np
from oracle import manifold as mf
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 20, 21, 44, 45, 64, 65, 154, 155, 199, 200, 201]


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


def _case(sizes, seed):
    W = [inputs.haar_params(seed + i, [(p + 3, p)])[0] for i, p in enumerate(sizes)]
    X = [mf.project(w, d) for w, d in zip(W, inputs.normal_like(seed + 50, W))]
    return W, X


def _check(got, W, X, rho, tag):
    for w, x, r, g in zip(W, X, rho, got):
        err = rel(to_np(g), mf.precondition(w, x, r, 0.05))
        print(f"{tag} p={w.shape[1]}: {err:.2e}", flush=True)
        assert err < 1e-10


@pytest.mark.parametrize("p", SIZES)
def test_single_matrix(ctx, p):
    W, X = _case([p], 400 + p)
    rho = [inputs.density_matrix(500 + p, p)]
    _check(ctx.stiefel_precondition(W, X, rho, 0.05), W, X, rho, "alone")


def test_all_sizes_in_one_call(ctx):
    """Every class at once, more matrices than one launch takes (18 of up to 20 rows), a diagonal matrix, a multiple of
    the identity, one of rank 5 and one with eigenvalues of both signs."""
    sizes = [4] * 18 + SIZES + [30, 60, 100, 100]
    W, X = _case(sizes, 700)
    rho = [inputs.density_matrix(800 + i, p) for i, p in enumerate(sizes)]
    rho[-4] = np.diag(np.linspace(0.0, 1.0, 30))
    rho[-3] = 0.25 * np.eye(60)
    g = inputs.normal_like(900, [np.zeros((100, 5))])[0]
    rho[-2] = g @ g.T / 500.0
    rho[-1] = inputs.symmetric_operator(901, 100) / 20.0
    _check(ctx.stiefel_precondition(W, X, rho, 0.05), W, X, rho, "batch")


@pytest.mark.parametrize("p", [20, 21, 64, 155, 200])
def test_warm_start(ctx, p):
    """lbfgs.step with an empty history gives -P G; its second call decomposes the changed rho in the kept basis."""
    W, X = _case([p], 1000 + p)
    rho = inputs.density_matrix(1100 + p, p)
    q = inputs.symmetric_operator(1200 + p, p)
    lb = ctx.lbfgs([w.shape for w in W], m=4)
    for r in (rho, rho + 1e-3 * np.max(np.abs(rho)) * q / np.max(np.abs(q))):
        d, _ = lb.step(W, X, [r])
        err = rel(to_np(d[0]), -mf.precondition(W[0], X[0], r))
        print(f"warm p={p}: {err:.2e}", flush=True)
        assert err < 1e-10
