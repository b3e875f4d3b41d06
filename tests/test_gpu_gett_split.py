"""FP32 and split-bf16 contractions on the bf16 matrix cores from split operands, against the FP64 oracle: layer maps
of the ternary geometry (two-site operators: dense oracle contractions in seconds) at bond dimensions whose squares
are, against the 128 and 192-wide tiles, below one tile (144), whole tiles (256, 576) and a tile with a remainder of
16 (400); split-K reductions run in the derivative programs.

Tolerances: each output is a sum of a few thousand products in a chain of four contractions; FP32 rounding of the
stored intermediates (2^-24 each) and of the accumulation stays below 2e-6 of the largest element (the bound of the
other FP32 layer maps), the 16-bit mantissas of the split-bf16 form below 1e-4."""
import numpy as np
import pytest

from gpu_helpers import rel, require_gpu, to_np
from oracle import ternary as ot
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp32": 2e-6, "bf16x3": 1e-4}


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


def _layer(chi):
    u, w = inputs.mera_init(300 + chi, [(chi, chi)], 3)[0]
    return u, w, inputs.symmetric_operator(301, chi * chi), inputs.density_matrix(302, chi * chi)


@pytest.mark.parametrize("chi", [12, 16, 20, 24])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_split_layer_maps(ctx, chi, prec):
    u, w, h, rho = _layer(chi)
    kw = dict(prec=prec, d=chi, geometry="ternary")
    A = ctx.ascend(1, chi, 1, u, w, h, **kw)
    D = ctx.descend(1, chi, 1, u, w, rho, **kw)
    ea, ed = rel(to_np(A), ot.ascend(h, u, w, chi, chi)), rel(to_np(D), ot.descend(rho, u, w, chi, chi))
    print(f"chi={chi} {prec}: ascend {ea:.2e} descend {ed:.2e}", flush=True)
    assert ea < TOL[prec] and ed < TOL[prec]


@pytest.mark.parametrize("chi", [12, 20])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_split_layer_grad(ctx, chi, prec):
    u, w, h, rho = _layer(chi)
    Du, Dw, ro, _ = ctx.layer_grad(1, chi, 1, u, w, h, rho, prec=prec, d=chi, geometry="ternary")
    ref = ot.layer_environments(h, rho, u, w, chi, chi)
    errs = [rel(to_np(Du), ref[0]), rel(to_np(Dw), ref[1]), rel(to_np(ro), ot.descend(rho, u, w, chi, chi))]
    print(f"chi={chi} {prec}: " + " ".join(f"{e:.2e}" for e in errs), flush=True)
    assert max(errs[:2]) < 5 * TOL[prec] and errs[2] < TOL[prec]  # the environments chain eight contractions


@pytest.mark.parametrize("scale", [2.0 ** 100, 2.0 ** -60])
def test_power_of_two_scaling_is_exact(ctx, scale):
    """Splitting scales with its operand: the map of 2^k h is 2^k times the map of h, bit by bit, far from the ends
    of the exponent range."""
    u, w, h, _ = _layer(12)
    kw = dict(prec="fp32", d=12, geometry="ternary")
    A, B = ctx.ascend(1, 12, 1, u, w, h, **kw), ctx.ascend(1, 12, 1, u, w, scale * h, **kw)
    assert np.array_equal(scale * to_np(A), to_np(B))


def test_elements_that_bf16_rounds_to_infinity(ctx):
    """c 1 with c = 3.4e38, below the largest FP32 number but above the largest bf16 one: the map of the identity is
    the identity, and, as in plain FP32 arithmetic, no contraction gives a NaN. (The closing symmetrisation adds
    x + x before halving, which is beyond FP32 on the diagonal: +inf there.)"""
    u, w, _, _ = _layer(12)
    c = 3.4e38
    A = to_np(ctx.ascend(1, 12, 1, u, w, c * np.eye(144), prec="fp32", d=12, geometry="ternary"))
    assert not np.any(np.isnan(A)) and np.all(np.diag(A) == np.inf)
    off = A[~np.eye(144, dtype=bool)]
    assert np.max(np.abs(off / c)) < TOL["fp32"]


def test_nan_stays_nan(ctx):
    u, w, h, _ = _layer(12)
    h[5, 7] = h[7, 5] = np.nan
    A = to_np(ctx.ascend(1, 12, 1, u, w, h, prec="fp32", d=12, geometry="ternary"))
    assert np.all(np.isnan(A))  # dense u and w spread it over every output
