"""Kernels at the sizes where their tilings, chunks and dispatch rules change,
against FP64 references (numpy or the oracle).  Tolerances as derived at each
test."""
import numpy as np
import pytest

from oracle import warmstart as WS
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


def f32r(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


def cuda(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


# one edge, a partial chunk, one block of slots, more chunks than slots
@pytest.mark.parametrize("n", [1, 33, 128, 65536 + 33])
def test_mlp_grad_slots(torch, pd, n):
    """The reduction over every count of slots.  The bf16 rounding points are
    the oracle's; what is left is FP32 accumulation (relative 1e-2 of a block's
    norm and 1e-4 of the loss, as for the other sizes)."""
    rng = np.random.default_rng(n)
    p = f32r(WS.init_params(4) + rng.normal(scale=0.05, size=WS.NPARAM))
    X, t = f32r(rng.normal(size=(n, 16))), f32r(rng.normal(size=n))
    g, loss = pd.mlp_grad(cuda(torch, p), cuda(torch, X), cuda(torch, t))
    lw, gw = WS.loss_grad(p, X, t, bf16_mode=True)
    assert abs(loss.item() - lw) <= 1e-4 * lw
    for got, want in zip(WS.unpack(host(g)), WS.unpack(gw)):
        got, want = np.asarray(got), np.asarray(want)
        assert np.linalg.norm(got - want) <= 1e-2 * max(np.linalg.norm(want), 1e-30)
