"""The tiled kernels of a single network (planes, folds, packed C) at sizes
past the rule that sends small networks to kernels of their own, and the paths
of a context that only those networks take.  Tolerances as derived at each test."""
import numpy as np
import pytest

from paper_1507_07039_amd import inputs as I

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.fixture(scope="module")
def pd(torch):
    from paper_1507_07039_amd import panda
    panda.load_library()
    return panda


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


def gpu_net(torch, seed, Ne, Na):
    """A network of normal entries, P and C symmetric, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn(Ne, Na, generator=g, device="cuda")

    def sym(n):
        a = torch.randn(n, n, generator=g, device="cuda").triu()
        return a + a.triu(1).T
    return W, sym(Ne), sym(Na)


def t64(torch, X, Y):
    dot = X @ Y
    den = (X * X).sum(1)[:, None] + (Y * Y).sum(0)[None, :] - dot.abs()
    return torch.where(den > 0, dot / den.clamp_min(1e-300).sqrt(), torch.zeros_like(dot))


# as many tiles of 256 x 128 as CUs, so that each is summed over all of K in
# one block; K at and either side of the longest sum without a fold
@pytest.mark.parametrize("Na", [1000, 1024, 1100])
def test_packed_equals_full_whole_k(torch, pd, Na):
    """Two iterations on packed C equal those on C stored whole bit for bit,
    and the first W is the FP64 one within 1e-5 of its largest entry."""
    Ne = 8000
    W, P, C = gpu_net(torch, Na, Ne, Na)
    out = []
    for packed in (0, 1):
        c = pd.Context(Ne, Na, pd.default_options(tol=0.0, packed_c=packed))
        c.load(W, P, C)
        c.iterate()
        first = c.state()[0]
        c.iterate()
        out.append((first,) + c.state()[:3])
        c.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    W, P, C = W.double(), P.double(), C.double()
    want = 0.9 * W + 0.05 * (t64(torch, P, W) + t64(torch, W, C))
    assert (out[1][0].double() - want).abs().max() <= 1e-5 * want.abs().max()
