"""Where an operand lies in memory changes how it is loaded and nothing else: factors that start 8 bytes past a 16-byte
boundary give the same bits as aligned ones, and a factor gives the same bits alone as beside an unaligned one of its
shape. Sizes: single tiles and many, k ranges within one chunk and split ones, on both sides of the lines between the
small-step and the LDS-tiled kernels (1024 x 576 crosses the lower line, 4096 x 576 lies beyond both), and one whose
fastest contracted leg is no multiple of 4.

Tolerance: none, the same arithmetic in the same order."""
import pytest
import torch

from gpu_helpers import require_gpu
from paper_2007_03638_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(20, 20), (36, 18), (144, 144), (400, 64), (576, 576), (1024, 576), (4096, 576)]


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_2007_03638_amd import api
    return api.Context(0)


def _pair(shape, seed):
    """A factor and a tangent-sized matrix, aligned."""
    W = torch.as_tensor(inputs.haar_params(seed, [shape])[0]).cuda()
    D = torch.as_tensor(inputs.normal_like(seed + 1, [W.cpu().numpy()])[0]).cuda()
    return W, D / torch.linalg.norm(D)


def _odd(x):
    """The same matrix one element past a 16-byte boundary, as it lies behind an odd-sized one in a flat buffer."""
    flat = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
    v = flat[1:].view(x.shape)
    v.copy_(x)
    assert x.data_ptr() % 16 == 0 and v.data_ptr() % 16 == 8 and v.is_contiguous()
    return v


@pytest.mark.parametrize("shape", SHAPES)
def test_unaligned_factor_gives_the_same_bits(ctx, shape):
    W, D = _pair(shape, 30 + shape[0])
    Wu, Du = _odd(W), _odd(D)
    X = ctx.stiefel_project([W], [D])[0]
    Xu = _odd(X)
    calls = [("project", lambda w, d, x: ctx.stiefel_project([w], [d])),
             ("transport", lambda w, d, x: ctx.stiefel_transport([w], [d])),
             ("grassmann", lambda w, d, x: ctx.grassmann_project([w], [d])),
             ("retract", lambda w, d, x: sum(ctx.stiefel_retract([w], [x], 0.5), []))]
    differ = []
    for name, f in calls:
        ref = f(W, D, X)
        for got in (f(Wu, Du, Xu), f(W, Du, X), f(Wu, D, X)):
            if not all(torch.equal(a, b) for a, b in zip(ref, got)):
                differ.append(name)
    assert not differ


@pytest.mark.parametrize("shape", SHAPES[:5])
def test_factor_beside_an_unaligned_one_gives_the_same_bits(ctx, shape):
    n, p = shape
    W, D = _pair(shape, 60 + n)
    W2, D2 = _pair(shape, 90 + n)
    G, G2 = ctx.stiefel_project([W], [D])[0], ctx.stiefel_project([W2], [D2])[0]
    rho = [torch.as_tensor(inputs.density_matrix(7 + i, p)).cuda() for i in range(2)]
    alone = ctx.lbfgs([shape], m=4).step([W], [G], [rho[0]])[0][0]
    both = ctx.lbfgs([shape, shape], m=4).step([W, _odd(W2)], [G, _odd(G2)], rho)[0]
    assert torch.equal(both[0], alone)
    assert torch.equal(both[1], ctx.lbfgs([shape], m=4).step([W2], [G2], [rho[1]])[0][0])
