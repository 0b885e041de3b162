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


# ------------------------------------------------ iterations past the small rule --
ALPHA = 0.1


def tiled(pd, Ne, Na):
    """Whether a network of this size iterates in the tiled kernels: asked of
    the library, so that a change of its rule cannot empty these tests."""
    import ctypes as ct
    f = pd.load_library()._ZN5panda9small_netEll
    f.restype, f.argtypes = ct.c_bool, [ct.c_int64, ct.c_int64]
    return not f(Ne, Na)


def damp64(torch, M, T, n, t, kw):
    """Eq. 5 off the diagonal, Eq. 6 on it, with the readings kw."""
    d, k = M.diagonal().clone(), M.shape[0]
    M = (1 - ALPHA) * M + ALPHA * T
    S = (T if kw.get("sigma_from_T") else M).clone()
    S.fill_diagonal_(0.0)
    m = max(k - 1, 1)
    q = (S - (S.sum(1) / m)[:, None]).square()
    q.fill_diagonal_(0.0)
    dof = k - 1 - kw.get("sigma_ddof", 0)
    sd = (q.sum(1) / dof).sqrt() if dof >= 1 else torch.zeros_like(d)
    mult = k if kw.get("n_own") else n
    f = ALPHA if kw.get("diag_alpha", 1) else 1.0
    M.diagonal().copy_((1 - ALPHA) * d + f * mult * sd * np.exp(2 * ALPHA * t))
    return M


def step64(torch, W, P, C, t, kw):
    """One iteration in 64 bits: (W, P, C, h)."""
    Ne, Na = W.shape
    pred = 0.5 * (t64(torch, P, W) + t64(torch, W, C))
    new = (1 - ALPHA) * W + ALPHA * pred
    h = ((pred if kw.get("h_undamped") else new) - W).abs().mean().item()
    return (new, damp64(torch, P, t64(torch, new, new.T.contiguous()), Na, t, kw),
            damp64(torch, C, t64(torch, new.T.contiguous(), new), Ne, t, kw), h)


def close(got, want, tol):
    """Off the diagonal to tol of the largest entry there (or of 1), the
    diagonal of a square matrix to 0.1 tol of each entry's size."""
    got = got.double()
    if got.shape[0] == got.shape[1]:
        g, w = got.diagonal(), want.diagonal()
        assert ((g - w).abs() <= 0.1 * tol * w.abs().clamp_min(1.0)).all()
        got, want = got.clone(), want.clone()
        got.fill_diagonal_(0.0)
        want.fill_diagonal_(0.0)
        assert (got == got.T).all()
    assert (got - want).abs().max() <= tol * max(1.0, want.abs().max().item())


# one tile row and one past it; either side of a padded row tile; more TFs than
# an unfolded sum takes (the C update and R fold in LDS); so many that the
# partials of W W^T fold as well
SIZES = [(3, 2100), (64, 2176), (65, 2060), (129, 2100), (257, 2200), (1100, 2100), (2900, 2300)]


@pytest.mark.parametrize("Ne,Na", SIZES)
@pytest.mark.parametrize("packed", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kw", [{}, {"sigma_from_T": 1, "sigma_ddof": 1, "n_own": 1},
                                {"h_undamped": 1, "diag_alpha": 0, "update_last": 1}])
def test_tiled_steps(torch, pd, Ne, Na, packed, precision, kw):
    """Three iterations one at a time against 64 bits, each from the library's
    own state before it, then a resume of the stored state bit for bit.

    FP32 form: |dT| <= 2 K u sum |x y| / sqrt(den), which for these normal
    entries is below 1e-4 of T's largest; it enters W, P and C damped by 0.1 (or
    0.05).  Split form: 2^-16 sum |x y| / sqrt(den) is below 1e-3 on W, damped
    like it on P and C (the targets of both forms elsewhere)."""
    assert tiled(pd, Ne, Na)
    tol = 1e-3 if precision else 1e-4
    o = pd.default_options(tol=0.0, packed_c=packed, precision=precision, **kw)
    c = pd.Context(Ne, Na, o)
    c.load(*gpu_net(torch, Ne + Na, Ne, Na))
    mid = None
    for t in range(1, 4):
        before = c.state()[:3]
        h, tt = c.iterate()
        want = step64(torch, *(M.double() for M in before), t, kw)
        after = c.state()[:3]
        assert tt == t and abs(h - want[3]) <= 0.1 * tol * want[3]
        for g, w in zip(after, want):
            close(g, w, tol)
        if t == 2:
            mid = after
    r = pd.Context(Ne, Na, o)
    r.load(*mid, t=2)
    r.iterate()
    assert all(torch.equal(a, b) for a, b in zip(r.state()[:3], after))


@pytest.mark.parametrize("precision", [0, 1])
def test_grouped_batch_steps(torch, pd, precision):
    """The grouped kernels over ragged networks past the small rule, the bounds
    of test_tiled_steps."""
    shapes = [(3, 2100), (64, 2176), (130, 2300), (1100, 2100)]
    assert all(tiled(pd, *s) for s in shapes)
    tol = 1e-3 if precision else 1e-4
    b = pd.Batch(shapes, pd.default_options(tol=0.0, precision=precision))
    for i, s in enumerate(shapes):
        b.load(i, *gpu_net(torch, 7 + i, *s))
    for t in range(1, 4):
        before = [b.state(i)[:3] for i in range(len(shapes))]
        b.iterate(1, graph=t > 1)
        for i, net in enumerate(before):
            for g, w in zip(b.state(i)[:3], step64(torch, *(M.double() for M in net), t, {})):
                close(g, w, tol)


@pytest.mark.parametrize("where", ["W", "C", "P"])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3.4e38])
@pytest.mark.parametrize("packed", [0, 1])
def test_tiled_extreme_entry(torch, pd, where, bad, packed):
    """One extreme entry of a prior: W keeps its infinity (or NaN), T is 0
    where its denominator is not positive, and no entry whose sums do not
    hold the extreme one is lost."""
    Ne, Na = 40, 2100
    assert tiled(pd, Ne, Na)
    net = dict(zip("WPC", gpu_net(torch, 3, Ne, Na)))
    i, j = (4, 7)
    net[where][i, j] = bad
    if where != "W":
        net[where][j, i] = bad
    c = pd.Context(Ne, Na, pd.default_options(tol=0.0, packed_c=packed))
    c.load(*(net[k] for k in "WPC"))
    c.iterate()
    got = c.state()[0].double()
    d = {k: M.double() for k, M in net.items()}
    rest = torch.ones(Ne, Na, dtype=torch.bool, device="cuda")
    if where == "W":
        rest[i, :] = rest[:, j] = False
    elif where == "P":
        rest[i, :] = rest[j, :] = False
    else:
        rest[:, i] = rest[:, j] = False
    want = 0.9 * d["W"] + 0.05 * (t64(torch, d["P"], d["W"]) + t64(torch, d["W"], d["C"]))
    assert torch.isfinite(got[rest]).all()
    assert (got[rest] - want[rest]).abs().max() <= 1e-4
    if where == "W":
        g = got[i, j].item()
        assert g == bad or (g != g and bad != bad) or abs(g - 0.9 * bad) <= 0.06 * abs(bad)
    else:  # W itself is finite: so is every T of it (or 0)
        assert torch.isfinite(got).all()


# the line past which a network that could take the small kernels iterates in
# the tiled ones (more than 256 tiles of W, and more than 1900 genes in the FP32
# form or 1600 in the split one), and the longest such networks
@pytest.mark.parametrize("Ne,Na,precision", [(129, 1901, 0), (192, 2048, 0), (161, 1601, 1), (192, 2048, 1)])
@pytest.mark.parametrize("packed", [0, 1])
def test_tiled_steps_within_the_small_rule(torch, pd, Ne, Na, precision, packed):
    """As test_tiled_steps (the same bounds), with features taken after two
    iterations, which leave the run as it was."""
    import ctypes as ct
    f = pd.load_library()._ZN5panda9small_runElli
    f.restype, f.argtypes = ct.c_bool, [ct.c_int64, ct.c_int64, ct.c_int32]
    assert not tiled(pd, Ne, Na) and not f(Ne, Na, precision)
    tol = 1e-3 if precision else 1e-4
    o = pd.default_options(tol=0.0, packed_c=packed, precision=precision)
    net = gpu_net(torch, Ne + Na, Ne, Na)
    a, b = pd.Context(Ne, Na, o), pd.Context(Ne, Na, o)
    a.load(*net)
    b.load(*net)
    for t in range(1, 4):
        before = a.state()[:3]
        h, tt = a.iterate()
        want = step64(torch, *(M.double() for M in before), t, {})
        assert tt == t and abs(h - want[3]) <= 0.1 * tol * want[3]
        for g, w in zip(a.state()[:3], want):
            close(g, w, tol)
        assert b.iterate() == (h, tt)
        if t == 2 and not packed:
            b.features(*(torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
                         for x in I.sketch_matrices(5, Ne, Na)))
    assert all(torch.equal(x, y) for x, y in zip(a.state()[:3], b.state()[:3]))


# ------------------------------------------------------- warm start, tiled context --
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("steps", [0, 2])
def test_tiled_features(torch, pd, precision, steps):
    """Features of a tiled context just loaded and after iterations (where the
    FP32 form holds R in W's buffer) equal the oracle's on its stored state
    within 1e-4 (z-scored O(1) values; the one-step similarity in FP32), and
    the run goes on bit for bit as one left alone."""
    from oracle import warmstart as WS
    Ne, Na = 70, 2100
    assert tiled(pd, Ne, Na)
    o = pd.default_options(tol=0.0, precision=precision)
    a, b = pd.Context(Ne, Na, o), pd.Context(Ne, Na, o)
    for c in (a, b):
        c.load(*gpu_net(torch, 11, Ne, Na))
        for _ in range(steps):
            c.iterate()
    Op, Oc = I.sketch_matrices(5, Ne, Na)
    F, tau = a.features(*(torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
                          for x in (Op, Oc)))
    W, P, C = (host(M) for M in b.state()[:3])
    want = WS.features(W, P, C, Op.astype(np.float32).astype(np.float64),
                       Oc.astype(np.float32).astype(np.float64))
    assert np.abs(host(F) - want).max() <= 1e-4
    S = WS.one_step(W, P, C)
    assert abs(tau - WS.target_scale(W, S)) <= 1e-5 * WS.target_scale(W, S)
    assert all(torch.equal(x, y) for x, y in zip(a.state()[:3], b.state()[:3]))
    for _ in range(2):
        assert a.iterate() == b.iterate()
    assert all(torch.equal(x, y) for x, y in zip(a.state()[:3], b.state()[:3]))


@pytest.mark.parametrize("precision,packed", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_tiled_warm_state(torch, pd, precision, packed):
    """The warm state of a tiled context against the oracle's, and two
    iterations from it against 64 bits (the bounds of test_tiled_steps)."""
    from oracle import warmstart as WS
    Ne, Na, t0 = 70, 2100, 6
    assert tiled(pd, Ne, Na)
    tol = 1e-3 if precision else 1e-4
    W, P, C = gpu_net(torch, 12, Ne, Na)
    Wp = W + 0.05 * torch.randn(W.shape, generator=torch.Generator(device="cuda").manual_seed(1),
                                device="cuda")
    c = pd.Context(Ne, Na, pd.default_options(tol=0.0, precision=precision, packed_c=packed))
    c.load(W, P, C)
    c.ws_init(Wp, t0)
    for g, w in zip(c.state()[:3], WS.warm_state(*(host(M) for M in (Wp, P, C)), t0)):
        close(g, torch.from_numpy(w).cuda(), tol)
    for t in (t0 + 1, t0 + 2):
        before = c.state()[:3]
        assert c.iterate()[1] == t
        for g, w in zip(c.state()[:3], step64(torch, *(M.double() for M in before), t, {})):
            close(g, w, tol)


# two networks that the small kernels run three to four times faster, and a
# batch that they run three times slower
@pytest.mark.parametrize("n,Ne,Na,small", [(2, 500, 500, True), (32, 100, 2000, False)])
def test_autotune_keeps_the_faster_kernels(torch, pd, n, Ne, Na, small):
    """A tuned batch goes on in whichever kernels are faster: bit for bit as one
    that takes the small ones by rule, or one given the tuned tiles."""
    shapes = [(Ne, Na)] * n
    net = gpu_net(torch, 5, Ne, Na)
    tuned, given = (pd.Batch(shapes, pd.default_options(tol=0.0)) for _ in range(2))
    best = tuned.autotune(reps=2)
    assert all(v > 0 for v in best.values())
    with pytest.raises(pd.PandaError):
        tuned.iterate(1)
    if small:
        assert tuned.tiles == [0, 0, 0, 0]
    else:
        given.tiles = tuned.tiles
    for b in (tuned, given):
        for i in range(n):
            b.load(i, *net)
        b.iterate(2, graph=True)
    assert all(torch.equal(x, y) for x, y in zip(tuned.state(n - 1)[:3], given.state(n - 1)[:3]))
    want = [M.double() for M in net]
    for t in (1, 2):
        want = step64(torch, *want[:3], t, {})
    assert (tuned.state(0)[0].double() - want[0]).abs().max() <= 1e-4


# ------------------------------------------------------------- sums of few terms --
# With the products of a few terms rounded once to FP32, |dT| <= 1.5 u |T| from
# the product (T moves by at most 1.5 d / sqrt(den) with it, and |dot| <= den)
# and u |T| from storing T.
@pytest.mark.parametrize("K", [1, 2, 3, 5, 7, 8])
@pytest.mark.parametrize("M,N", [(1, 1), (129, 130), (500, 900)])
def test_tanimoto_few_terms(torch, pd, M, K, N):
    g = torch.Generator(device="cuda").manual_seed(K * M)
    X, Y = (torch.randn(s, generator=g, device="cuda") for s in ((M, K), (K, N)))
    want = t64(torch, X.double(), Y.double())
    err = (pd.tanimoto(X, Y).double() - want).abs()
    assert (err <= 2.51 * U * want.abs() + 1e-30).all()


@pytest.mark.parametrize("S", [2, 3, 5, 8])
def test_pearson_few_samples(torch, pd, S):
    """Two factors and the result each rounded once: 3 u of |c| <= 1."""
    E = np.random.default_rng(S).normal(size=(300, S)).astype(np.float32)
    got = host(pd.pearson(torch.from_numpy(E).cuda()))
    assert np.abs(got - np.corrcoef(E.astype(np.float64))).max() <= 3.01 * U
    assert np.array_equal(got, got.T)


def few_bounds(torch, before, after, what, steps=1):
    """With alpha = 1 and products rounded `steps` times (once where they are
    summed in FP64, at each term of an FP32 accumulation): C is T of the new W (the product 1.5 u, its FP32
    denominator, root and quotient 2.5 u); P is it with an FP64 quotient; W is
    (A + R) / 2, R stored.  The diagonal of P or C enters A's and R's sums in
    FP64 after the rounded rest, so there the product's error is 1.5 u of that
    rest over sqrt(den)."""
    W, P, C = (M.double() for M in before)
    W1, P1, C1 = (M.double() for M in after)
    if "C" in what:
        T = t64(torch, W1.T.contiguous(), W1)
        err = (C1 - T).abs()
        err.fill_diagonal_(0.0)
        assert (err <= 4.05 * U * T.abs() + 1e-30).all()

    def rounding(X, Y, diagonal=None):
        """Of a sum of whole products; `diagonal`: their part added in FP64."""
        dot, mag = X @ Y, X.abs() @ Y.abs()
        den = (X * X).sum(1)[:, None] + (Y * Y).sum(0)[None, :] - dot.abs()
        if diagonal is not None:
            dot, mag = dot - diagonal, mag - diagonal.abs()
        return 1.5 * U * (dot.abs() if steps == 1 else steps * mag) / den.clamp_min(1e-300).sqrt()
    if "P" in what:
        T = t64(torch, W1, W1.T.contiguous())
        err = (P1 - T).abs()
        err.fill_diagonal_(0.0)
        assert (err <= 1.01 * (rounding(W1, W1.T.contiguous()) + U * T.abs()) + 1e-30).all()
    A, R = t64(torch, W, C), t64(torch, P, W)
    eA = rounding(W, C, W * C.diagonal()[None, :])
    eR = rounding(P, W, P.diagonal()[:, None] * W) + U * R.abs()
    want = 0.5 * (A + R)
    assert ((W1 - want).abs() <= 1.01 * (0.5 * (eA + eR) + U * want.abs()) + 1e-30).all()


def diagonal(torch, M):
    return torch.diag(M.diagonal().clone()).contiguous()


@pytest.mark.parametrize("Ne", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("packed", [0, 1])
def test_few_factors(torch, pd, Ne, packed):
    """N_e terms in R and the C update of a tiled network."""
    Na = 2100
    assert tiled(pd, Ne, Na)
    W, P, C = gpu_net(torch, Ne, Ne, Na)
    before = (W, P, diagonal(torch, C))
    c = pd.Context(Ne, Na, pd.default_options(tol=0.0, alpha=1.0, packed_c=packed))
    c.load(*before)
    c.iterate()
    few_bounds(torch, before, c.state()[:3], "C")


@pytest.mark.parametrize("Na", [1, 3, 8])
def test_few_genes(torch, pd, Na):
    """N_a terms in A and the P update, of as many TFs as take the tiled kernels
    with more genes: whole FP32 products in the small kernels, accumulated in FP32."""
    Ne = 2100
    W, P, C = gpu_net(torch, Na, Ne, Na)
    before = (W, diagonal(torch, P), C)
    c = pd.Context(Ne, Na, pd.default_options(tol=0.0, alpha=1.0))
    c.load(*before)
    c.iterate()
    few_bounds(torch, before, c.state()[:3], "P", steps=Na)


@pytest.mark.parametrize("tiles", [0, 1, 2])
@pytest.mark.parametrize("sigma_from_T", [0, 1])
def test_few_terms_in_a_grouped_batch(torch, pd, tiles, sigma_from_T):
    """The same in the grouped kernels, beside a network of long sums."""
    shapes = [(1, 2100), (3, 2100), (8, 2300), (2100, 1), (2100, 8), (1100, 2100)]
    nets = []
    for i, s in enumerate(shapes):
        W, P, C = gpu_net(torch, 20 + i, *s)
        nets.append((W, diagonal(torch, P), C) if s[1] <= 8 else (W, P, diagonal(torch, C)))
    b = pd.Batch(shapes, pd.default_options(tol=0.0, alpha=1.0, sigma_from_T=sigma_from_T))
    b.tiles = [tiles] * 4
    for i, net in enumerate(nets):
        b.load(i, *net)
    b.iterate(1)
    for i, s in enumerate(shapes[:-1]):
        few_bounds(torch, nets[i], b.state(i)[:3], "P" if s[1] <= 8 else "C")
    W, P, C = (M.double() for M in nets[-1])
    assert (b.state(5)[0].double() - 0.5 * (t64(torch, P, W) + t64(torch, W, C))).abs().max() <= 1e-4


# ------------------------------------------------------------ W held as its planes --
@pytest.mark.parametrize("packed", [0, 1])
def test_w_keeps_every_bit(torch, pd, packed):
    """With P = C = 0 both similarities are 0 and W is damped alone: what comes
    back is 0.9 W rounded once, bit for bit, down to the subnormals."""
    Ne, Na = 70, 2100
    assert tiled(pd, Ne, Na)
    rng = np.random.default_rng(9)
    W = (rng.choice([-1.0, 1.0], (Ne, Na)) * rng.uniform(1.0, 2.0, (Ne, Na))
         * np.exp2(-rng.integers(0, 149, (Ne, Na)))).astype(np.float32)
    assert ((np.abs(W) < 2.0 ** -126) & (W != 0)).any()
    c = pd.Context(Ne, Na, pd.default_options(tol=0.0, packed_c=packed))
    c.load(torch.from_numpy(W).cuda(), torch.zeros(Ne, Ne, device="cuda"),
           torch.zeros(Na, Na, device="cuda"))
    c.iterate()
    got = c.state()[0].cpu().numpy()
    want = (0.9 * W.astype(np.float64)).astype(np.float32)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
