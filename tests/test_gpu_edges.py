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


# ------------------------------------------------------------------- z-score --
# entries of one 1024-entry chunk and either side; a matrix past the size from
# which chunks hold 8192 entries; both also off 16-byte alignment
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 2), (3, 341), (32, 32), (25, 41), (1, 4097),
                                       (2900, 2900)])
@pytest.mark.parametrize("off", [0, 1])
def test_normalize_chunks(torch, pd, rows, cols, off):
    """Against numpy's moments; one FP32 rounding of an FP64 value."""
    rng = np.random.default_rng(rows * 7 + cols)
    M = f32r(rng.normal(3.0, 2.0, size=rows * cols))
    buf = torch.zeros(rows * cols + off + 3, device="cuda")
    buf[off:off + M.size] = cuda(torch, M)
    t = buf[off:off + M.size].view(rows, cols)
    if M.size == 1:
        with pytest.raises(pd.PandaError) as e:
            pd.normalize(t)
        assert e.value.code == pd.ERR_DEGENERATE
        return
    pd.normalize(t)
    want = ((M - M.mean()) / M.std()).reshape(rows, cols)
    assert np.abs(host(t) - want).max() <= 2e-7 * max(1.0, np.abs(want).max())
    assert not buf[:off].any() and not buf[off + M.size:].any()


@pytest.mark.parametrize("rows,cols", [(1, 7), (300, 300), (2900, 2900)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_normalize_refuses_equal_entries(torch, pd, rows, cols, mode):
    t = torch.full((rows, cols), 0.1, device="cuda")
    with pytest.raises(pd.PandaError) as e:
        pd.normalize(t, mode=mode)
    assert e.value.code == pd.ERR_DEGENERATE
    assert torch.all(t == torch.tensor(0.1, device="cuda"))
    t[rows - 1, cols - 1] = float("inf")
    with pytest.raises(pd.PandaError) as e:
        pd.normalize(t, mode=mode)
    assert e.value.code == pd.ERR_NONFINITE


# one, two and many row chunks of the column moments, and their remainders
@pytest.mark.parametrize("rows,cols", [(2, 300), (256, 33), (257, 1025), (513, 700), (20000, 5)])
def test_normalize_rowcol_chunks(torch, pd, rows, cols):
    rng = np.random.default_rng(rows + cols)
    M = f32r(rng.normal(-1.0, 3.0, size=(rows, cols)))
    t = cuda(torch, M)
    pd.normalize(t, mode=2)
    r = (M - M.mean(1, keepdims=True)) / M.std(1, keepdims=True)
    c = (M - M.mean(0, keepdims=True)) / M.std(0, keepdims=True)
    want = (r + c) / np.sqrt(2.0)
    assert np.abs(host(t) - want).max() <= 2e-7 * max(1.0, np.abs(want).max())


# ------------------------------------------------- similarity, K split by tiles --
# one tile and one K-step; one tile with a long K; tiles below, at and above
# the CU count; K not a multiple of anything
@pytest.mark.parametrize("M,K,N", [(1, 16, 1), (64, 4096, 128), (65, 4097, 129), (200, 3000, 2000),
                                   (512, 1001, 4096), (513, 999, 4097)])
def test_tanimoto_split_k(torch, pd, M, K, N):
    """|dT| <= 2 K u sum_k |x_k y_k| / sqrt(den) + 4 u |T| (FP32 accumulation
    in any order)."""
    X = f32r(I.random_dense(M + K, (M, K)))
    Y = f32r(I.random_dense(N + K, (K, N), -2.0, 2.0))
    got = host(pd.tanimoto(cuda(torch, X), cuda(torch, Y)))
    dot = X @ Y
    den = (X ** 2).sum(1)[:, None] + (Y ** 2).sum(0)[None, :] - np.abs(dot)
    want = dot / np.sqrt(den)
    bound = 2 * K * U * (np.abs(X) @ np.abs(Y)) / np.sqrt(den) + 4 * U * np.abs(want) + 1e-30
    assert np.all(np.abs(got - want) <= bound)


# rows ending in each 32-row block of a tile and either side of it; K of one
# to five 16-deep tiles (the loads run up to three ahead), either side of the
# longest unfolded sum and of a fold
@pytest.mark.parametrize("M", [1, 32, 33, 65, 97, 128, 129])
@pytest.mark.parametrize("K", [16, 32, 48, 64, 80, 1024, 1040, 2033])
def test_tanimoto_row_blocks_and_folds(torch, pd, M, K):
    """The bound of test_tanimoto_split_k."""
    X = f32r(I.random_dense(M + K, (M, K)))
    Y = f32r(I.random_dense(M * K, (K, 130), -2.0, 2.0))
    got = host(pd.tanimoto(cuda(torch, X), cuda(torch, Y)))
    dot = X @ Y
    den = (X ** 2).sum(1)[:, None] + (Y ** 2).sum(0)[None, :] - np.abs(dot)
    want = dot / np.sqrt(den)
    bound = 2 * K * U * (np.abs(X) @ np.abs(Y)) / np.sqrt(den) + 4 * U * np.abs(want) + 1e-30
    assert np.all(np.abs(got - want) <= bound)


# operands off 16-byte alignment; rows of 1024 columns and either side, chunks
# of 32 rows of Y
@pytest.mark.parametrize("M,K,N", [(5, 33, 1023), (5, 32, 1024), (64, 4, 1025), (3, 2100, 8)])
@pytest.mark.parametrize("off", [0, 1])
def test_tanimoto_packing(torch, pd, M, K, N, off):
    """The bound of test_tanimoto_split_k."""
    def put(a):
        buf = torch.zeros(a.size + off, device="cuda")
        t = buf[off:].view(a.shape)
        t.copy_(torch.from_numpy(a.astype(np.float32)))
        return t

    X = f32r(I.random_dense(M + K, (M, K)))
    Y = f32r(I.random_dense(N + K, (K, N), -2.0, 2.0))
    got = host(pd.tanimoto(put(X), put(Y)))
    dot = X @ Y
    den = (X ** 2).sum(1)[:, None] + (Y ** 2).sum(0)[None, :] - np.abs(dot)
    want = dot / np.sqrt(den)
    bound = 2 * K * U * (np.abs(X) @ np.abs(Y)) / np.sqrt(den) + 4 * U * np.abs(want) + 1e-30
    assert np.all(np.abs(got - want) <= bound)


# every tiling over networks with one live row block, a ragged last tile, and
# more TFs than an unfolded sum takes
@pytest.mark.parametrize("tiles", [0, 1, 2])
def test_batch_tiles_ragged(torch, pd, oracle, tiles):
    """One iteration against the oracle, relative to each matrix's largest entry,
    within the bound the grouped form is held to elsewhere (1e-5)."""
    shapes = [(3, 2100), (33, 2100), (161, 2100), (1100, 1150)]
    nets = [prep(oracle, 900 + i, *s) for i, s in enumerate(shapes)]
    b = pd.Batch(shapes, pd.default_options(tol=0.0))
    b.tiles = [tiles] * 4
    for i, net in enumerate(nets):
        b.load(i, *(cuda(torch, a) for a in net))
    b.iterate(1)
    for i, (W, P, C) in enumerate(nets):
        for got, want in zip(b.state(i)[:3], oracle.step(W, P, C, 1)[:3]):
            assert np.abs(host(got) - want).max() <= 1e-5 * np.abs(want).max()


# ------------------------------------ FP32 products on three bf16 planes --
def prep(oracle, seed, Ne, Na):
    W0, P0, C0 = I.priors(seed, Ne, Na, 0.1, 0.05, 40, 6)
    return tuple(f32r(oracle.normalize(M)) for M in (W0, P0, C0))


@pytest.fixture(scope="module")
def oracle():
    from oracle import oracle as O
    return O


# one K-tile of N_e and of N_a; either side of a padded row tile; K past one
# and two folds of the A product (1008 genes each); N_e past one fold
# (1024 TFs: the C update, R and W W^T fold in LDS); both layouts of C
@pytest.mark.parametrize("Ne,Na", [(3, 130), (64, 128), (65, 129), (70, 1100), (257, 2200),
                                   (1100, 260)])
@pytest.mark.parametrize("packed", [0, 1])
def test_fp32_planes_run(torch, pd, oracle, Ne, Na, packed):
    """Three iterations against the FP64 oracle: W and the off-diagonals of P
    and C to 1e-4, their diagonals to 1e-5 of their size (the plain form's
    targets); the stored state resumes bit for bit."""
    W, P, C = prep(oracle, Ne + Na, Ne, Na)
    o = pd.default_options(tol=0.0, packed_c=packed)
    g = pd.run(cuda(torch, W), cuda(torch, P), cuda(torch, C), tol=0.0, max_iter=3, opts=o)
    ref = oracle.run(W, P, C, oracle.Options(tol=0.0, max_iter=3))
    assert np.abs(host(g.W) - ref.W).max() <= 1e-4
    for got, want in ((host(g.P), ref.P), (host(g.C), ref.C)):
        d = np.diag(want)
        assert np.abs(np.diag(got) - d).max() <= 1e-5 * np.abs(d).max()
        off = ~np.eye(want.shape[0], dtype=bool)
        assert np.abs(got - want)[off].max() <= 1e-4
    # W comes back from its planes exactly: two iterations, store, load, one more
    a = pd.run(cuda(torch, W), cuda(torch, P), cuda(torch, C), tol=0.0, max_iter=2, opts=o)
    c = pd.Context(Ne, Na, o)
    c.load(a.W, a.P, a.C, t=2)
    c.iterate()
    Wb, Pb, Cb, _, _ = c.state()
    assert torch.equal(Wb, g.W) and torch.equal(Pb, g.P) and torch.equal(Cb, g.C)


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), 3.4e38])
def test_fp32_planes_extreme_entry(torch, pd, oracle, bad):
    """One extreme entry of W: the entry itself keeps its infinity, T is 0
    wherever its denominator is not positive, and no other entry is lost."""
    Ne, Na = 40, 200
    W, P, C = prep(oracle, 3, Ne, Na)
    W[4, 7] = np.float32(bad)

    def T(X, Y):
        with np.errstate(all="ignore"):
            dot = X @ Y
            den = (X ** 2).sum(1)[:, None] + (Y ** 2).sum(0)[None, :] - np.abs(dot)
            return np.where(den > 0, dot / np.sqrt(den), 0.0)

    g = pd.run(cuda(torch, W), cuda(torch, P), cuda(torch, C), tol=0.0, max_iter=1,
               opts=pd.default_options(tol=0.0))
    with np.errstate(all="ignore"):
        want = 0.9 * W + 0.05 * (T(P, W) + T(W, C))
    got = host(g.W)
    if np.isinf(bad):
        assert got[4, 7] == bad
    else:
        assert abs(got[4, 7] - 0.9 * W[4, 7]) <= 0.06 * W[4, 7]
    rest = np.ones((Ne, Na), bool)
    rest[4, :] = rest[:, 7] = False
    assert np.isfinite(got[rest]).all()
    assert np.abs(got[rest] - want[rest]).max() <= 1e-4


# --------------------------------------------------------- small networks --
# one entry a side (no spread), below, at and past one 32 x 32 tile, ragged
# in both, taller than wide, and the sizes either side of the rule that sends
# a network to the tiled kernels (N_e N_a (N_e + N_a) = 9e8, N_a = 2048)
@pytest.mark.parametrize("Ne,Na", [(1, 2), (2, 3), (31, 33), (32, 32), (33, 31), (64, 300),
                                   (150, 90), (40, 2048), (40, 2049)])
@pytest.mark.parametrize("kw", [{}, {"packed_c": 1}, {"precision": 1},
                                {"sigma_from_T": 1, "sigma_ddof": 1, "n_own": 1},
                                {"h_undamped": 1, "diag_alpha": 0, "update_last": 1}])
def test_small_kernels(torch, pd, oracle, Ne, Na, kw):
    """Four iterations one at a time against the FP64 oracle (targets of the
    plain form), a resume bit for bit, and a batch of the network with a
    smaller one beside it."""
    rng = np.random.default_rng(Ne * 3 + Na)
    W, P, C = (f32r(M) for M in (rng.normal(size=(Ne, Na)), I.random_symmetric(Ne, Ne),
                                 I.random_symmetric(Na + 1, Na)))
    ro = {k: v for k, v in kw.items() if k not in ("packed_c", "precision")}
    # the split form's own bound where the network does not take these kernels
    tol = 1e-4 if Na <= 2048 or kw.get("precision", 0) == 0 else 1e-3
    o = pd.default_options(tol=0.0, **kw)
    c = pd.Context(Ne, Na, o)
    c.load(cuda(torch, W), cuda(torch, P), cuda(torch, C))
    ref, mid = (W, P, C), None
    for t in range(1, 5):
        Wo, Po, Co, ho, _ = oracle.step(*ref, t, oracle.Options(tol=0.0, **ro))
        ref = (Wo, Po, Co)
        h, tt = c.iterate()
        assert tt == t and abs(h - ho) <= 10 * tol * ho + 1e-9
        if t == 2:
            mid = c.state()
    g = c.state()
    assert np.abs(host(g[0]) - ref[0]).max() <= tol
    for got, want in ((host(g[1]), ref[1]), (host(g[2]), ref[2])):
        d, off = np.diag(want), ~np.eye(want.shape[0], dtype=bool)
        assert np.all(np.abs(np.diag(got) - d) <= 1e-5 * np.maximum(1.0, np.abs(d)))
        assert not off.any() or np.abs(got - want)[off].max() <= tol
    r = pd.Context(Ne, Na, o)
    r.load(*mid[:3], t=2)
    for _ in range(2):
        r.iterate()
    assert all(torch.equal(x, y) for x, y in zip(r.state()[:3], g[:3]))
    if kw.get("packed_c"):
        return
    b = pd.Batch([(Ne, Na), (5, 9)], o)
    b.load(0, cuda(torch, W), cuda(torch, P), cuda(torch, C))
    b.load(1, *(cuda(torch, M) for M in (rng.normal(size=(5, 9)), I.random_symmetric(2, 5),
                                         I.random_symmetric(3, 9))))
    b.iterate(4, graph=True)
    assert np.abs(host(b.state(0)[0]) - ref[0]).max() <= tol


@pytest.mark.parametrize("precision", [0, 1])
def test_small_batch_changes_tiles(torch, pd, oracle, precision):
    """A loaded batch moved to the grouped kernels (other tiles) and back
    between iterations goes on from the same state."""
    nets = [prep(oracle, s, 40 + s, 90 + s) for s in (1, 2)]
    b = pd.Batch([n[0].shape for n in nets], pd.default_options(tol=0.0, precision=precision))
    for i, n in enumerate(nets):
        b.load(i, *(cuda(torch, M) for M in n))
    refs = [list(n) for n in nets]
    for t, tiles in enumerate(([0, 0, 0, 0], [0, 0, 1, 0], [0, 0, 1, 0], [0, 0, 0, 0]), 1):
        b.tiles = tiles
        b.iterate(1, graph=t % 2 == 0)
        for i in range(2):
            refs[i] = list(oracle.step(*refs[i], t, oracle.Options(tol=0.0))[:3])
            got = [host(x) for x in b.state(i)[:3]]
            assert np.abs(got[0] - refs[i][0]).max() <= 1e-4
            d = np.diag(refs[i][1])
            assert np.abs(np.diag(got[1]) - d).max() <= 1e-5 * np.abs(d).max()


# ---------------------------------------------------------------- load, store --
# one tile; odd rows off 16-byte alignment; rows of 1024 columns and either
# side; more than one chunk of rows; past the small kernels
@pytest.mark.parametrize("Ne,Na", [(2, 3), (33, 130), (64, 1024), (20, 1025), (130, 2300)])
@pytest.mark.parametrize("kw", [{}, {"packed_c": 1}, {"precision": 1}])
@pytest.mark.parametrize("off", [0, 1])
def test_load_store_roundtrip(torch, pd, Ne, Na, kw, off):
    """A loaded state comes back bit for bit (matrices off alignment too), the
    identity as the rounded z-score of the identity."""
    rng = np.random.default_rng(Ne * 3 + Na)

    def put(a):
        buf = torch.zeros(a.size + off, device="cuda")
        t = buf[off:].view(a.shape)
        t.copy_(torch.from_numpy(np.asarray(a, np.float32)))
        return t

    def sym(n):
        a = rng.normal(size=(n, n))
        return a + a.T

    def identity(n):
        e = np.eye(n)
        return ((e - e.mean()) / e.std()).astype(np.float32)

    W, P, C = put(rng.normal(size=(Ne, Na))), put(sym(Ne)), put(sym(Na))
    ctx = pd.Context(Ne, Na, pd.default_options(**kw))
    ctx.load(W, P, C)
    out = [put(np.zeros(t.shape)) for t in (W, P, C)]
    ctx.store(*out)
    for a, b in zip(out, (W, P, C)):
        assert torch.equal(a, b)
    ctx.load(W)
    ctx.store(*out)
    assert torch.equal(out[0], W)
    for a, n in zip(out[1:], (Ne, Na)):
        assert np.abs(host(a) - identity(n)).max() <= 2 * U * np.abs(identity(n)).max()


# ----------------------------------------------------------------- correlations --
# one tile and its edges, two tiles; rows of C on 16 bytes, off them by the
# leading dimension, and by the base
@pytest.mark.parametrize("G", [1, 3, 127, 128, 130, 259])
@pytest.mark.parametrize("pad,off", [(0, 0), (1, 0), (4, 0), (4, 1)])
def test_pearson_stores(torch, pd, G, pad, off):
    """Against numpy's corrcoef within the bound of the other sizes (1e-5);
    exactly symmetric; nothing outside the G x G result is written."""
    E = np.random.default_rng(G).normal(size=(G, 33)).astype(np.float32)
    ldc = -(-G // 4) * 4 + pad
    buf = torch.full((G * ldc + off,), 7.0, device="cuda")
    C = buf[off:].view(G, ldc)
    pd.pearson_noalloc(cuda(torch, E), C, ldc)
    got = host(C)
    assert np.abs(got[:, :G] - np.atleast_2d(np.corrcoef(E.astype(np.float64)))).max() <= 1e-5
    assert np.array_equal(got[:, :G], got[:, :G].T) and np.all(np.diag(got) == 1.0)
    assert np.all(got[:, G:] == 7.0) and np.all(host(buf[:off]) == 7.0)
