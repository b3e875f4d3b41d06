"""FP32 contractions on the bf16 matrix cores over the whole range of FP32, against 64 bits: operands of every magnitude
from FP32 denormals to 2^120 keep the 24 bits that FP32 arithmetic gives them.

The tensors route elements instead of mixing them: u = 1 and w[xyz, p] = 1 where y = p, x = z = 0, so that each result is
a third of the sum of at most three elements of h (or a partial trace of it), all positive. Every element is compared with
the FP64 oracle relative to itself: eight FP32 roundings (the stored intermediates, alpha = 1/3, three accumulations, the
symmetrisation), 8 * 2^-24, plus as many halves of the smallest denormal."""
import numpy as np
import pytest

from gpu_helpers import require_gpu, to_np
from oracle import ternary as ot
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

RTOL, ATOL = 8 * 2.0 ** -24, 8 * 2.0 ** -149


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


def _routing(chi):
    w = np.zeros((chi, chi, chi, chi))
    for p in range(chi):
        w[0, p, 0, p] = 1.0
    return np.eye(chi * chi), w.reshape(chi ** 3, chi)


def _wide(seed, n, lo, hi):
    """Symmetric, positive, exponents uniform in [lo, hi), exactly FP32."""
    rng = np.random.default_rng(seed)
    x = np.triu(np.ldexp(rng.uniform(1.0, 2.0, (n, n)), rng.integers(lo, hi, (n, n))))
    x = (x + np.triu(x, 1).T).astype(np.float32).astype(np.float64)
    return x


@pytest.mark.parametrize("chi", [12, 13, 14, 20])
@pytest.mark.parametrize("lo,hi", [(-126, -100), (-149, -126), (-140, 90), (-140, 120), (100, 120)])
def test_every_magnitude_keeps_its_bits(ctx, chi, lo, hi):
    u, w = _routing(chi)
    h = _wide(17 + chi, chi * chi, lo, hi)
    ref = ot.ascend(h, u, w, chi, chi)
    got = to_np(ctx.ascend(1, chi, 1, u, w, h, prec="fp32", d=chi, geometry="ternary"))
    ref = 0.5 * (ref + ref.T)
    err = np.abs(got - ref)
    worst = np.max(err / (RTOL * np.abs(ref) + ATOL))
    print(f"chi={chi} 2^{lo}..2^{hi}: {worst:.2f} of the bound, {np.count_nonzero(ref)} of {ref.size} nonzero", flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("scale", [2.0 ** -80, 2.0 ** -100])
@pytest.mark.parametrize("chi", [12, 14])
def test_small_operands_scale_exactly(ctx, chi, scale):
    """The map of 2^k h is 2^k times the map of h, bit by bit, while every element stays a normal FP32 number."""
    u, w = inputs.mera_init(300 + chi, [(chi, chi)], 3)[0]
    h = inputs.symmetric_operator(301, chi * chi)
    kw = dict(prec="fp32", d=chi, geometry="ternary")
    A, B = ctx.ascend(1, chi, 1, u, w, h, **kw), ctx.ascend(1, chi, 1, u, w, scale * h, **kw)
    assert np.array_equal(scale * to_np(A), to_np(B))


@pytest.mark.parametrize("geometry,chi", [("ternary", 16), ("binary", 12)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_operators_take_a_few_passes(ctx, geometry, chi, value):
    """A NaN or an infinity in h spreads over every result. Bound: the ordinary pass, one with unscaled operands and one on
    the FP32 matrix instructions (1.4 times as long), the last two with operands that are not staged for the whole tile
    (three times the loads): 1 + 3 + 3 * 1.4, half as much again for the scatter of short launches."""
    ter = geometry == "ternary"
    u, w = inputs.mera_init(320 + chi, [(chi, chi)], 3 if ter else 2)[0]
    h = inputs.symmetric_operator(321, chi ** (2 if ter else 3))
    bad = h.copy()
    bad[3, 3] = value

    def seconds(x):
        best = np.inf
        for _ in range(4):
            ctx.profile(True)
            A = ctx.ascend(1, chi, 1, u, w, x, prec="fp32", d=chi, geometry=geometry)
            best = min(best, sum(s["seconds"] for s in ctx.kernel_stats()))
            ctx.profile(False)
        return best, to_np(A)

    t, _ = seconds(h)
    tb, A = seconds(bad)
    print(f"{geometry} chi={chi} {value}: {1e3 * t:.3f} ms, {1e3 * tb:.3f} ms, {tb / t:.1f} times", flush=True)
    assert np.all(np.isnan(A))
    assert tb < 12.3 * t
