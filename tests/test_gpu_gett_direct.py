"""Contractions in 32 x 32 tiles read straight from global memory, against the FP64 oracle: maps and derivatives at bond
dimensions whose powers lie below one tile (16, 25), at whole tiles (64, 256, 512) and at remainders of 4 (36, 100),
1 (81, 225), 17 and 11 (49, 343); the ternary ones also hold the split reductions and, from chi = 8, launches on either
side of the line to the LDS tiles.

Tolerances: FP64 roundings of at most 1e4 products in a chain of at most eight contractions, 1e-12; FP32 as for the other
FP32 layer maps, 2e-6 (derivatives, which chain eight contractions, five times that); the split-bf16 form, whose larger
contractions have 16-bit mantissas, 1e-4."""
import pytest

from gpu_helpers import rel, require_gpu, to_np
from oracle import mera as om
from oracle import ternary as ot
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-6, "bf16x3": 1e-4}


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


@pytest.mark.parametrize("chi", [4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("geometry", ["binary", "ternary"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_small_maps_and_derivatives(ctx, chi, geometry, prec):
    ter = geometry == "ternary"
    o, sites = (ot, 2) if ter else (om, 3)
    u, w = inputs.mera_init(400 + chi, [(chi, chi)], 3 if ter else 2)[0]
    h, rho = inputs.symmetric_operator(401, chi ** sites), inputs.density_matrix(402, chi ** sites)
    kw = dict(prec=prec, d=chi, geometry=geometry)
    got = [to_np(ctx.ascend(1, chi, 1, u, w, h, **kw)), to_np(ctx.descend(1, chi, 1, u, w, rho, **kw))]
    ref = [o.ascend(h, u, w, chi, chi), o.descend(rho, u, w, chi, chi)]
    errs = [rel(a, b) for a, b in zip(got, ref)]
    grads = ctx.layer_grad(1, chi, 1, u, w, h, rho, **kw)
    genv = [rel(to_np(a), b) for a, b in zip(grads[:2], o.layer_environments(h, rho, u, w, chi, chi)[:2])]
    print(f"{geometry} chi={chi} {prec}: " + " ".join(f"{e:.1e}" for e in errs + genv), flush=True)
    assert max(errs) < TOL[prec] and max(genv) < 5 * TOL[prec]
