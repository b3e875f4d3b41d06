"""FP32 and split-bf16 contractions on the bf16 matrix cores where the layouts allow no 16-byte loads (bond dimensions that
are no multiple of 4), against the FP64 oracle: ternary maps and derivatives with odd and even legs, whose squares leave
remainders of 41, 68, 97 and 100 against the 128 tiles, k ranges that end inside a tile of 16 and four k's that lie side by
side as well as across two legs; a binary map whose chi^3 extents pass 192-wide tiles.

Tolerances: those of the FP32 and split-bf16 layer maps with 16-byte loads (2e-6 and 1e-4 of the largest element; five
times that for derivatives, which chain eight contractions), since the split and the order of sums are the same."""
import pytest

from gpu_helpers import rel, require_gpu, to_np
from oracle import mera as om
from oracle import ternary as ot
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp32": 2e-6, "bf16x3": 1e-4}


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


@pytest.mark.parametrize("chi", [13, 14, 15, 18, 22])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_ternary(ctx, chi, prec):
    u, w = inputs.mera_init(500 + chi, [(chi, chi)], 3)[0]
    h, rho = inputs.symmetric_operator(501, chi * chi), inputs.density_matrix(502, chi * chi)
    kw = dict(prec=prec, d=chi, geometry="ternary")
    A, D = ctx.ascend(1, chi, 1, u, w, h, **kw), ctx.descend(1, chi, 1, u, w, rho, **kw)
    errs = [rel(to_np(A), ot.ascend(h, u, w, chi, chi)), rel(to_np(D), ot.descend(rho, u, w, chi, chi))]
    genv = []
    if chi <= 15:
        Du, Dw, _, _ = ctx.layer_grad(1, chi, 1, u, w, h, rho, **kw)
        genv = [rel(to_np(a), b) for a, b in zip((Du, Dw), ot.layer_environments(h, rho, u, w, chi, chi)[:2])]
    print(f"chi={chi} {prec}: " + " ".join(f"{e:.1e}" for e in errs + genv), flush=True)
    assert max(errs) < TOL[prec] and max(genv, default=0.0) < 5 * TOL[prec]


@pytest.mark.parametrize("chi", [9, 10])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_binary(ctx, chi, prec):
    u, w = inputs.mera_init(510 + chi, [(chi, chi)])[0]
    h, rho = inputs.symmetric_operator(511, chi ** 3), inputs.density_matrix(512, chi ** 3)
    A, D = ctx.ascend(1, chi, 1, u, w, h, prec=prec, d=chi), ctx.descend(1, chi, 1, u, w, rho, prec=prec, d=chi)
    errs = [rel(to_np(A), om.ascend(h, u, w, chi, chi)), rel(to_np(D), om.descend(rho, u, w, chi, chi))]
    print(f"chi={chi} {prec}: " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) < TOL[prec]
