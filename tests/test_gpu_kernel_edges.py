"""Kernels at the sizes where a tile, a split or a bank can go wrong: edges,
remainders, and the smallest and largest of a rule's range."""
import numpy as np
import pytest
import torch

from paper_2603_04035_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12, 129, 5000])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_update_count_over_counter_banks(n, precision):
    """The update count (summed over the counter banks by the host) equals
    the entries of the merged lists that the initial lists did not hold, with
    fewer joined points than banks, about as many, and many more."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=n, d=20, seed=n)).cuda()
    states = []
    for iters in (0, 1):
        _, _, st, (idx, _, _) = knn.nndescent_build(X, 5, build_k=8, sample_rate=1.0, max_iters=iters, delta=0.0,
                                                    seed=3, precision=precision, return_state=True)
        states.append(idx.cpu().numpy())
    new = ~(states[1][:, :, None] == states[0][:, None, :]).any(2) & (states[1] >= 0)
    assert st["iters"] == 1 and st["updates"][0] == int(new.sum())
    assert st["emitted"][0] >= st["updates"][0] and st["pairs_joined"] > 0


def _with_shells(n, d, shells, seed):
    """A mixture plus `shells` groups of 2d + 1 integer points: a centre and
    its 2d axis neighbours at distance 1.  Every row of a group has more than
    2k equidistant nearest rows, so none is certified by the GEMM lists."""
    X = datagen.gmm_isotropic(n=n, d=d, seed=seed)
    E = np.concatenate([np.zeros((1, d)), np.eye(d), -np.eye(d)]).astype(np.float32)
    C = np.zeros((shells, d), np.float32)
    C[:, 0] = 40.0
    C[:, 1] = 8.0 * np.arange(shells)
    return np.ascontiguousarray(np.concatenate([X, (C[:, None, :] + E[None]).reshape(-1, d)]))


@pytest.mark.parametrize("shells", [1, 13, 30])
def test_fallback_rows_shared_by_workgroups(orc, shells):
    """Uncertified rows searched exhaustively: 41 rows (24 workgroups each),
    533 (one each) and 1,230 (more rows than workgroups)."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    n, d, k = 20_003, 20, 6
    X = _with_shells(n, d, shells, 4)
    idx, dist = knn.knn_exact(torch.from_numpy(X).cuda(), k)
    rows = np.concatenate([np.arange(0, n, 997), np.arange(n, len(X))])
    O, _ = orc.exact_knn(X, k, rows=rows)
    res = exact_parity(X, rows, idx.cpu().numpy()[rows], dist.cpu().numpy()[rows], O)
    assert parity_ok(res), res
    # integer distances: the order among equals is the index order
    assert np.array_equal(idx.cpu().numpy()[n], np.sort(idx.cpu().numpy()[n]))


@pytest.mark.parametrize("nq", [1, 2, 300])
def test_fallback_one_row_many_parts(orc, nq):
    """One uncertified query: as many workgroups as the lists' room allows (4
    and 8 parts) or as the references have batches (79 parts, the last of 3
    rows)."""
    import paper_2603_04035_amd as knn
    d, k = 20, 6
    X = _with_shells(20_000 - 41 + 227, d, 1, 5)     # 20,227 = 79 * 256 + 3 rows
    Q = np.ascontiguousarray(np.concatenate([X[-41:-40], X[:nq - 1]]))
    self_rows = np.concatenate([[len(X) - 41], np.arange(nq - 1)]).astype(np.int32)
    idx, dist = knn.knn_exact_query(torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda(), k,
                                    q_self=torch.from_numpy(self_rows))
    O, O2 = orc.exact_query(X, Q, k, q_self=self_rows.astype(np.int64))
    assert np.array_equal(idx.cpu().numpy()[0], O[0])
    assert np.allclose(dist.cpu().numpy(), np.sqrt(O2), rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("d,B", [(1, 1), (31, 33), (33, 32), (97, 85), (784, 171)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_gradients_at_tile_edges(orc, d, B, precision):
    """Encoder gradients where the batch is not a whole number of 32-triplet
    workgroups or 256-row chunks (3B = 3 .. 513 rows) and the inputs not one
    of 16 / 32 columns.  Bounds: FP32 sums of at most 784 + 256 terms stay
    within 1e-5 of the norm; the BF16 mode's hidden values may round the
    other way at a boundary, 1e-3 of the norm."""
    from paper_2603_04035_amd import Encoder
    X = datagen.gmm_isotropic(n=400, d=d, seed=d)
    rng = np.random.default_rng(B)
    rows = rng.integers(0, 400, size=3 * B)
    enc = Encoder(d, seed=4)
    W1, _, W2, _ = enc.get_weights()
    b1 = rng.normal(0, 0.1, size=64).astype(np.float32)
    b2 = rng.normal(0, 0.1, size=32).astype(np.float32)
    enc.set_weights(W1, b1, W2, b2)
    loss, g = enc.grads(torch.from_numpy(X).cuda(), torch.from_numpy(rows), B, precision=precision)
    g = g.cpu().numpy().astype(np.float64)
    bf = precision == "bf16"
    Zo = (orc.mlp_forward_bf16 if bf else orc.mlp_forward)(X[rows], W1, b1, W2, b2)
    lo, dZ = orc.triplet_loss(Zo, B, 1.0)
    refs = (orc.mlp_backward_bf16 if bf else orc.mlp_backward)(X[rows], W1, b1, W2, dZ)
    tol = 1e-3 if bf else 1e-5
    assert abs(loss - lo) <= (1e-4 if bf else 1e-5) * max(abs(lo), 1e-6)
    ref = np.concatenate([np.asarray(r, np.float64).ravel() for r in refs])
    scale = np.linalg.norm(ref)
    at = 0
    for r in refs:
        part = g[at:at + r.size]
        assert np.linalg.norm(part - np.asarray(r, np.float64).ravel()) <= tol * scale, (d, B, at)
        at += r.size


@pytest.mark.parametrize("d", [17, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
def test_split_gram_widths_and_types(orc, d, dt):
    """FP32 precision over row widths at the chunk edges and the input types
    (FP32: two FP16 parts per value; 16-bit: one)."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    X = torch.from_numpy(datagen.gmm_isotropic(n=1999, d=d, seed=d)).to(dt)
    idx, dist = knn.knn_exact(X.cuda(), 10)
    Xv = np.ascontiguousarray(X.float().numpy())
    O, _ = orc.exact_knn(Xv, 10)
    res = exact_parity(Xv, np.arange(1999), idx.cpu().numpy(), dist.cpu().numpy(), O)
    assert parity_ok(res), (d, dt, res)


@pytest.mark.parametrize("case", ["1e15", "1e-15", "1e-17", "outlier", "zero-rows"])
def test_split_gram_scales(orc, case):
    """FP32 precision over the range of the power-of-two scales: large and
    small data, data below the range (norms^2 under 2^-100: every row is
    searched directly), one row 10^6 times the others, and rows of zeros."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    X = datagen.gmm_isotropic(n=1500, d=40, seed=7)
    if case == "outlier":
        X[77] *= 1e6
    elif case == "zero-rows":
        X[100:104] = 0.0
    else:
        X = X * np.float32(float(case))
    X = np.ascontiguousarray(X.astype(np.float32))
    idx, dist = knn.knn_exact(torch.from_numpy(X).cuda(), 8)
    O, _ = orc.exact_knn(X, 8)
    res = exact_parity(X, np.arange(1500), idx.cpu().numpy(), dist.cpu().numpy(), O)
    assert parity_ok(res), (case, res)


@pytest.mark.parametrize("qs,rs", [(1e8, 1.0), (1e-8, 1.0), (1.0, 1e8)])
def test_split_gram_query_scale(orc, qs, rs):
    """Queries and references of very different magnitude have a scale each."""
    import paper_2603_04035_amd as knn
    R = np.ascontiguousarray(datagen.gmm_isotropic(n=1500, d=40, seed=8) * np.float32(rs))
    Q = np.ascontiguousarray(datagen.gmm_isotropic(n=130, d=40, seed=9) * np.float32(qs))
    idx, dist = knn.knn_exact_query(torch.from_numpy(Q).cuda(), torch.from_numpy(R).cuda(), 5)
    O, O2 = orc.exact_query(R, Q, 5)
    assert np.allclose(dist.cpu().numpy(), np.sqrt(O2), rtol=1e-5)


@pytest.mark.parametrize("n", [400, 513, 6200, 20_001])
@pytest.mark.parametrize("precision,d", [("fp32", 40), ("fp32", 100), ("bf16", 40), ("fp16", 100)])
def test_gated_route_equals_list_route(n, precision, d):
    """The gated route (no scratch limit) against the sorted-list route (a
    limit that fits everything) over the gate's group sizes (up to 4, up to 48
    and more tiles) and a last tile of one row: the same neighbours and
    distances, rows sorted by cluster so that a row's candidates crowd one
    split."""
    import paper_2603_04035_amd as knn
    X = datagen.gmm_isotropic(n=n, d=d, comps=12, seed=n)
    X = np.ascontiguousarray(X[np.argsort(X[:, 0] + 100 * (X @ X[:12].T).argmax(1), kind="stable")])
    Xd = torch.from_numpy(X).cuda()
    rows = torch.arange(n, dtype=torch.int32)
    a = knn.knn_exact(Xd, 14, precision=precision)
    b = knn.knn_exact_query(Xd, Xd, 14, q_self=rows, precision=precision, workspace_limit=4 << 30)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_gated_route_full_buffers(orc):
    """Buffers that overflow their 256 entries: every reference of the gate's
    sample (tiles 0, 2, 4, ... of the order below) is far from the queries and
    the near ones sit together between them, so a loose gate lets thousands
    pass and the rows' best 32 are kept again and again."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    rng = np.random.default_rng(3)
    n, d = 40_000, 24
    X = (rng.normal(size=(n, d)) + 30.0).astype(np.float32)
    near = rng.normal(size=(6000, d)).astype(np.float32)
    X[17_000:23_000] = near                       # 47 tiles in a row hold the queries' neighbours
    Q = np.ascontiguousarray(near[:257])
    idx, dist = knn.knn_exact_query(torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda(), 10,
                                    q_self=torch.arange(17_000, 17_257, dtype=torch.int32))
    rows = np.arange(17_000, 17_257)
    O, _ = orc.exact_knn(X, 10, rows=rows)
    res = exact_parity(X, rows, idx.cpu().numpy(), dist.cpu().numpy(), O)
    assert parity_ok(res), res


@pytest.mark.parametrize("n,d", [(2, 3), (63, 50), (65, 31), (300, 33), (500, 784), (1000, 64)])
def test_small_search(orc, n, d):
    """The one-launch search at its edges: fewer references than a batch of
    64, one more, chunks of 32 coordinates and their remainders."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    X = datagen.gmm_isotropic(n=n, d=d, comps=3, seed=n + d)
    k = min(n - 1, 32)
    idx, dist = knn.knn_exact(torch.from_numpy(X).cuda(), k)
    O, _ = orc.exact_knn(X, k)
    res = exact_parity(X, np.arange(n), idx.cpu().numpy(), dist.cpu().numpy(), O)
    assert parity_ok(res), res
    Q = np.ascontiguousarray(X[:min(n, 5)] + np.float32(0.25))
    idx, dist = knn.knn_exact_query(torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda(), k)
    O, O2 = orc.exact_query(X, Q, k)
    assert np.allclose(dist.cpu().numpy(), np.sqrt(O2), rtol=1e-5)


def _spectrum(n, d, lam, seed):
    rng = np.random.default_rng(seed)
    G = rng.normal(size=(n, d))
    G -= G.mean(axis=0)
    U, _ = np.linalg.qr(G)
    Q, _ = np.linalg.qr(rng.normal(size=(d, d)))
    return np.ascontiguousarray((1.5 + (U * np.sqrt((n - 1) * np.asarray(lam))) @ Q.T).astype(np.float32))


@pytest.mark.parametrize("name", ["slow", "steep", "cliff", "odd"])
def test_pca_filter_spectra(orc, name):
    """The filtered iteration on spectra that drive its rules: a slow decay
    (many products), seven decades (one product per round), a cliff inside
    the block (dependent columns), and an odd block width (m = 21: the
    eigensolver's bye).  Bounds as the other PCA tests: eigenvalues 1e-10,
    vectors 1e-8 (gaps above 1e-3)."""
    import paper_2603_04035_amd as knn
    d, p, lam = {"slow": (90, 12, np.arange(1, 91) ** -0.7),
                 "steep": (90, 8, np.geomspace(1.0, 1e-7, 90)),
                 "cliff": (90, 6, np.concatenate([np.geomspace(1.0, 0.5, 6), 1e-4 * np.geomspace(1, 0.5, 84)])),
                 "odd": (60, 5, np.arange(1, 61) ** -1.5)}[name]
    X = _spectrum(4000, d, lam, 11)
    Z, V, w, mu = (t.cpu().numpy() for t in knn.pca(torch.from_numpy(X).cuda(), p))
    oZ, oV, ow, omu = orc.pca(X, p)
    np.testing.assert_allclose(w, ow, rtol=1e-10)
    assert np.abs(V - oV).max() <= 1e-8
    assert np.abs(V.T @ V - np.eye(p)).max() <= 1e-12


@pytest.mark.parametrize("X", ["rank", "rounded", "rows", "zero"])
def test_pca_refuses_low_rank(X):
    """Rank below the subspace width (m = 19 and 18) stays refused."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(1)
    X = {"rank": rng.integers(-3, 4, size=(2000, 5)).astype(float) @ rng.integers(-2, 3, size=(5, 100)).astype(float),
         "rounded": rng.normal(size=(2000, 5)) @ rng.normal(size=(5, 100)) + 30.0,
         "rows": rng.normal(size=(15, 100)), "zero": np.zeros((100, 50))}[X]
    with pytest.raises(knn.KnnError):
        knn.pca(torch.from_numpy(np.ascontiguousarray(X.astype(np.float32))).cuda(), 3 if X.shape[1] == 100 else 2)


@pytest.mark.parametrize("d,e", [(17, 2), (33, 17), (64, 40), (65, 3), (130, 129)])
@pytest.mark.parametrize("k", [8, 9, 16])
def test_rank_pass_widths(orc, d, e, k):
    """The rank pass over its probe widths (8, 12, 16) and row widths (one
    to five chunks of 32, with and without resident query rows), with (X) and
    without (Y above 16 dimensions) the neighbour lists; one tile and a row
    past four."""
    X = datagen.gmm_isotropic(n=513, d=d, comps=4, seed=d)
    rng = np.random.default_rng(e)
    Y = (X @ rng.normal(size=(d, e)) + rng.normal(scale=0.5, size=(513, e))).astype(np.float32)
    import paper_2603_04035_amd as knn
    _, (h, t, c) = knn.quality(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k, per_row=True)
    oh, ot, oc = orc.quality_rows(X, Y, k, canonical=True)
    assert np.array_equal(h.cpu().numpy(), oh) and np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(c.cpu().numpy(), oc)


@pytest.mark.parametrize("n", [1536, 1537, 6143, 6144, 8192, 8193, 262_144, 262_145])
@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("kind", ["normal", "copies", "line", "inf-nan", "huge", "half"])
def test_pruned_search_equals_all_pairs(n, d, kind):
    """One to three coordinates: the search pruned by boxes gives the bits of
    the one over all pairs (taken under a workspace limit), as a self search
    and for queries; last tiles and groups whole and in part, both grid
    resolutions, ties, copies, distances that overflow or are NaN."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "copies":
        X = np.round(X)
        X[:200] = X[0]
    if kind == "line":
        X[:, 0] = 1e4
    if kind == "inf-nan":
        X[[3, n // 2], 0] = np.inf, np.nan
        X[n - 1, d - 1] = -np.inf
    if kind == "huge":
        X *= 1.5e19
    X = torch.from_numpy(X).cuda()
    X = X.half() if kind == "half" else X
    rows = torch.unique(torch.cat([torch.arange(0, n, max(1, n // 300)), torch.tensor([1, 3, n // 2, n - 1])])).cuda()
    Q, own = X[rows].contiguous(), rows.to(torch.int32)
    for k in (1, 32):
        ref_i, ref_d = knn.knn_exact_query(Q, X, k, q_self=own, workspace_limit=1 << 30)[:2]
        for i, dist in (knn.knn_exact(X, k)[:2], knn.knn_exact_query(Q, X, k, q_self=own)[:2]):
            if len(i) == n:
                i, dist = i[rows], dist[rows]
            assert torch.equal(i, ref_i) and torch.equal(dist, ref_d)
    ref_i, ref_d = knn.knn_exact_query(Q + 0.25, X, 10, workspace_limit=1 << 30)[:2]
    i, dist = knn.knn_exact_query(Q + 0.25, X, 10)[:2]
    assert torch.equal(i, ref_i) and torch.equal(dist, ref_d)


@pytest.mark.parametrize("n,d", [(2, 1), (64, 2), (1536, 3), (1537, 4), (2560, 16), (2561, 8)])
def test_small_search_few_coordinates(n, d):
    """Up to 1536 (d <= 3) and 2560 references the one-launch search gives the
    bits of the direct one."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(np.random.default_rng(n).integers(-5, 6, (n, d)).astype(np.float32) / 3).cuda()
    k = min(n - 1, 12)
    own = torch.arange(n, dtype=torch.int32).cuda()
    ref_i, ref_d = knn.knn_exact_query(X, X, k, q_self=own, workspace_limit=1 << 30)[:2]
    i, dist = knn.knn_exact(X, k)[:2]
    assert torch.equal(i, ref_i) and torch.equal(dist, ref_d)


@pytest.mark.parametrize("m", [1, 5, 64, 1023, 1024, 1025, 131_072, 131_073, 135_168, 135_169])
def test_union_order_at_sort_tiles(m):
    """Edges sorted by target at the edges of the sort's tiles (1,024 pairs up
    to 131,072, 4,096 above), sources in order within a target: with one
    neighbour per row, every row of the union holds its neighbour and the
    rows that point at it, ascending."""
    import paper_2603_04035_amd as knn
    n = max(2, m)
    rng = np.random.default_rng(n)
    to = (np.arange(n) + rng.integers(1, n, n)) % n   # never the row itself
    to[: n // 3] = np.where(np.arange(n // 3) == n // 2, to[: n // 3], n // 2)   # a hub
    idx = torch.from_numpy(to.astype(np.int32)[:, None]).cuda()
    dist = torch.ones((n, 1), device="cuda")
    _, _, _, ptr, col, _ = knn.fuzzy_graph(idx, dist)
    i = np.arange(n, dtype=np.int64)
    want = np.unique(np.concatenate([i * n + to, to * n + i]))
    got = np.repeat(i, np.diff(ptr.cpu().numpy())) * n + col.cpu().numpy()[: int(ptr[-1])]
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n", [34, 255, 256, 257, 1039])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 31, 32])
def test_fuzzy_rows_and_unions_at_group_edges(orc, n, k):
    """Rows in groups of 16 and of 32 lanes, whole and part workgroups: random
    neighbours (hubs among them, so that segments span the waves' chunks),
    distances over ten orders of magnitude and with ties, against the oracle
    within the bars of the fuzzy tests."""
    from tests.test_gpu_fuzzy import _check
    rng = np.random.default_rng(100 * n + k)
    p = np.where(np.arange(n) < 4, 20.0, 1.0)
    G = np.empty((n, k), np.int32)
    for i in range(n):
        q = p.copy()
        q[i] = 0.0
        G[i] = rng.choice(n, size=k, replace=False, p=q / q.sum())
    D = rng.uniform(0.5, 2.0, size=(n, k)).astype(np.float32) * 10.0 ** rng.integers(-5, 6, size=(n, 1))
    D[::7] = np.round(D[::7])
    D = np.sort(D, axis=1).astype(np.float32)
    _check(orc, torch.from_numpy(G).cuda(), torch.from_numpy(D).cuda())


@pytest.mark.parametrize("precision,limit", [("fp32", 1_468_928), ("bf16", 1_667_072)])
def test_nnd_workspace_limit_unchanged(precision, limit):
    """The least accepted limit of a 1,500 x 20 build does not move with the
    sizes of counters and sort tiles."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=1500, d=20, seed=1)).cuda()
    knn.nndescent_build(X, 5, build_k=8, max_iters=1, precision=precision, workspace_limit_bytes=limit)
    with pytest.raises(knn.KnnError) as e:
        knn.nndescent_build(X, 5, build_k=8, max_iters=1, precision=precision, workspace_limit_bytes=limit - 1)
    assert e.value.status == -2


@pytest.mark.parametrize("n", [40, 600, 5000, 40_001])
@pytest.mark.parametrize("precision,d,wide", [("fp32", 32, 33), ("fp32", 20, 400), ("fp32", 200, 376), ("fp32", 370, 385),
                                              ("bf16", 64, 65), ("fp16", 50, 300)])
@pytest.mark.parametrize("K,rho", [(8, 0.5), (31, 1.0)])
def test_join_forms_agree(n, precision, d, wide, K, rho):
    """Rows padded with zero columns to a width of another form of the join (4
    pieces of 32 bytes and 5, 47 and 48 of them, with new lists within and
    beyond one block; 40,001 points: shared out in the widest form) give the
    same lists bit for bit: zeros change no sum."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=n, d=d, seed=d)).cuda()
    W = torch.cat([X, torch.zeros((n, wide - d), device="cuda")], 1).contiguous()
    args = dict(build_k=K, sample_rate=rho, max_iters=3, delta=0.0, seed=5, precision=precision)
    a, b = knn.nndescent_build(X, 7, **args)[:2], knn.nndescent_build(W, 7, **args)[:2]
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("p", [1, 15, 16, 17, 24, 32, 39, 40, 64])
def test_pca_factor_block_edges(orc, p):
    """Subspaces of 17, 31, 32, 34, 48, 64, 78 and 80 columns: the factor's blocks
    of 16 whole and in part.  Bounds as the other PCA tests."""
    import paper_2603_04035_amd as knn
    X = _spectrum(3000, 100, np.arange(1, 101) ** -0.7, 5)
    Z, V, w, mu = (t.cpu().numpy() for t in knn.pca(torch.from_numpy(X).cuda(), p))
    oZ, oV, ow, omu = orc.pca(X, p)
    np.testing.assert_allclose(w, ow, rtol=1e-10)
    assert np.abs(V - oV).max() <= 1e-8
    assert np.abs(V.T @ V - np.eye(p)).max() <= 1e-12


@pytest.mark.parametrize("nq", [1, 3, 255, 256, 257])
@pytest.mark.parametrize("n,d", [(511, 40), (512, 40), (513, 5), (1000, 33), (4096, 64)])
def test_small_search_few_queries(nq, n, d):
    """Up to 256 queries in 512 references and more: four waves per query give
    the bits of the list route (a workspace limit, on a set that is not small: the same
    references with 5,000 far copies appended)."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(nq + n)
    X = torch.from_numpy(rng.integers(-9, 10, (n, d)).astype(np.float32) / 4).cuda()
    Q = torch.from_numpy(rng.integers(-9, 10, (nq, d)).astype(np.float32) / 4).cuda()
    far = torch.cat([X, X.new_full((5000, d), 100.0)]).contiguous()
    k = 20
    i, dist = knn.knn_exact_query(Q, X, k)[:2]
    ref_i, ref_d = knn.knn_exact_query(Q, far, k, workspace_limit=1 << 30)[:2]
    assert torch.equal(i, ref_i) and torch.equal(dist, ref_d)


@pytest.mark.parametrize("n", [60, 255, 256, 257, 1029])
@pytest.mark.parametrize("e", [1, 2, 3, 7])
@pytest.mark.parametrize("k", [8, 12, 13])
def test_direct_ranks_with_ties(orc, n, e, k):
    """Ranks in a low-dimensional space, probe widths 8, 12 and 16: lattice
    rows, so that references tie with probes before, in and behind the probes'
    groups of 8; whole and part tiles of 256; equal to the oracle's terms."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(n + e)
    X = rng.integers(0, 4, (n, e + 1)).astype(np.float32)
    Y = rng.integers(0, 4, (n, e)).astype(np.float32)
    _, (h, t, c) = knn.quality(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k, per_row=True)
    oh, ot, oc = orc.quality_rows(X, Y, k, canonical=True)
    assert np.array_equal(h.cpu().numpy(), oh) and np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(c.cpu().numpy(), oc)


@pytest.mark.parametrize("n", [40, 128, 129, 400, 512])
@pytest.mark.parametrize("precision,d", [("bf16", 200), ("fp16", 256), ("bf16", 257), ("fp16", 700)])
def test_gated_route_few_references(n, precision, d):
    """Up to four tiles of references, rows where the gate is taken and where it
    is not: the bits of the list route (a limit that fits everything)."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=n, d=d, comps=3, seed=n)).cuda()
    Q = torch.from_numpy(datagen.gmm_isotropic(n=1500, d=d, comps=3, seed=n)).cuda()
    own = torch.arange(n, dtype=torch.int32).cuda()
    for q, s in ((X, own), (Q, None)):
        a = knn.knn_exact_query(q, X, 12, q_self=s, precision=precision)
        b = knn.knn_exact_query(q, X, 12, q_self=s, precision=precision, workspace_limit=4 << 30)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def _with_room(X):
    """X's rows at the front of a buffer whose other rows are copies of row 0:
    a row past the end would be at distance 0 of row 0."""
    buf = torch.from_numpy(X[:1].repeat(len(X) + 256, 0))
    buf[: len(X)] = torch.from_numpy(X)
    return buf.cuda()[: len(X)]


@pytest.mark.parametrize("n", [2, 3, 5, 12, 16, 20, 31, 32, 33])
@pytest.mark.parametrize("precision,d", [("fp32", 20), ("bf16", 20), ("fp16", 50), ("bf16", 100), ("fp16", 300)])
def test_fewer_references_than_rerank_width(orc, n, precision, d):
    """Every other row is a neighbour or a candidate (k = n - 1, and 15 with a
    re-rank width of 30): all are found, in the canonical order, and nothing past
    the end of the references is."""
    import paper_2603_04035_amd as knn
    from oracle.compare import exact_parity, parity_ok
    X = datagen.gmm_isotropic(n=n, d=d, comps=3, seed=n + d)
    Xd = _with_room(X)
    own = torch.arange(n, dtype=torch.int32).cuda()
    for k in {min(n - 1, 32), min(n - 1, 15)}:
        idx, dist = knn.knn_exact(Xd, k, precision=precision)[:2]
        ref = knn.knn_exact_query(Xd, Xd, k, q_self=own, precision=precision, workspace_limit=1 << 30)
        assert int(idx.min()) >= 0 and int(idx.max()) < n
        assert torch.equal(idx, ref[0]) and torch.equal(dist, ref[1])
        O, _ = orc.exact_knn(X, k)
        res = exact_parity(X, np.arange(n), idx.cpu().numpy(), dist.cpu().numpy(), O)
        assert parity_ok(res), (k, res)


@pytest.mark.parametrize("nr", [20, 31])
def test_many_queries_in_few_references(orc, nr):
    """FP32 queries past the one-launch search's work, in fewer references
    than the re-rank width."""
    import paper_2603_04035_amd as knn
    nq, d, k = 40_001, 700, 16
    R = datagen.gmm_isotropic(n=nr, d=d, comps=3, seed=nr)
    Q = datagen.gmm_isotropic(n=nq, d=d, comps=3, seed=5)
    assert nq * nr * (6.0 * d + 150.0) > 3e9
    idx, dist = knn.knn_exact_query(torch.from_numpy(Q).cuda(), _with_room(R), k)[:2]
    assert int(idx.min()) >= 0 and int(idx.max()) < nr
    rows = np.arange(0, nq, 397)
    O, O2 = orc.exact_query(R, np.ascontiguousarray(Q[rows]), k)
    assert np.allclose(dist.cpu().numpy()[rows], np.sqrt(O2), rtol=1e-5)


@pytest.mark.parametrize("n,k", [(4, 2), (12, 7), (20, 12), (26, 16), (32, 16)])
def test_quality_few_rows(orc, n, k):
    """The rank pass's neighbour lists where a row has fewer others than the
    lists' re-rank width, 2 k."""
    import paper_2603_04035_amd as knn
    X = datagen.gmm_isotropic(n=n, d=20, comps=3, seed=n)
    Y = np.ascontiguousarray(np.random.default_rng(n).normal(size=(n, 2)).astype(np.float32))
    _, (h, t, c) = knn.quality(_with_room(X), torch.from_numpy(Y).cuda(), k, per_row=True)
    oh, ot, oc = orc.quality_rows(X, Y, k, canonical=True)
    assert np.array_equal(h.cpu().numpy(), oh) and np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(c.cpu().numpy(), oc)


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k,rerank", [(16, 0), (31, 0), (32, 0), (20, 20), (19, 20)])
def test_compacted_buffers_leave_self_out(precision, k, rerank):
    """Rows along a curve, neighbours next to each other: hundreds of
    references pass a row's gate and its buffer is cut back again and again.  The
    row's own index, nearest of all, is not one of those kept: the bits of the
    list route (a limit that fits everything), as a self search and as queries."""
    import paper_2603_04035_amd as knn
    n, d = 5000, 50
    rng = np.random.default_rng(2)
    t = np.linspace(0.0, 1.0, n)[:, None]
    X = np.sin(t * rng.uniform(2.0, 9.0, (1, d)) + rng.uniform(0.0, 6.0, (1, d)))
    X = torch.from_numpy((20 * X + 0.02 * rng.standard_normal((n, d))).astype(np.float32)).cuda()
    own = torch.arange(n, dtype=torch.int32).cuda()
    args = dict(precision=precision, rerank_k=rerank)
    ref = knn.knn_exact_query(X, X, k, q_self=own, workspace_limit=4 << 30, **args)
    for got in (knn.knn_exact(X, k, **args), knn.knn_exact_query(X, X, k, q_self=own, **args)):
        assert int(got[0].min()) >= 0
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


@pytest.mark.parametrize("case", ["1e4", "1e6", "1e7", "1e9", "spread", "small"])
@pytest.mark.parametrize("d,e", [(64, 2), (20, 33), (300, 40)])
def test_ranks_of_rows_of_unlike_norms(orc, case, d, e):
    """The rank pass where the rows' norms differ widely (one row enlarged;
    norms over twelve decades; every row below the scales' range), in X and in
    an embedding above 16 dimensions: equal to the oracle's integers."""
    import paper_2603_04035_amd as knn
    n, k = 600, 10
    rng = np.random.default_rng(d)
    X = rng.normal(size=(n, d)).astype(np.float32)
    Y = (X @ rng.normal(size=(d, e)) + rng.normal(scale=0.5, size=(n, e))).astype(np.float32)
    for A in (X, Y):
        if case == "spread":
            A *= (10.0 ** rng.uniform(-6, 6, size=(n, 1))).astype(np.float32)
        elif case == "small":
            A *= np.float32(1e-17)
        else:
            A[77] *= np.float32(float(case))
    _, (h, t, c) = knn.quality(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k, per_row=True)
    oh, ot, oc = orc.quality_rows(X, Y, k, canonical=True)
    assert np.array_equal(h.cpu().numpy(), oh) and np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(c.cpu().numpy(), oc)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [40, 200])
@pytest.mark.parametrize("far", [1e3, 1e5, 1e7, 1e10])
def test_one_query_far_outside(orc, dt, d, far):
    """One query of a norm far above the others' and the references': the
    others' neighbours are found as without it (FP32 precision)."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(d)
    R = torch.from_numpy(rng.normal(size=(5000, d)).astype(np.float32)).to(dt)
    Q = torch.from_numpy(rng.normal(size=(300, d)).astype(np.float32))
    Q[123] *= far
    Q = Q.to(dt)
    k = 10
    idx, dist = knn.knn_exact_query(Q.cuda(), R.cuda(), k)[:2]
    Qf, Rf = (np.ascontiguousarray(a.float().numpy()) for a in (Q, R))
    O, O2 = orc.exact_query(Rf, Qf, k)
    G = idx.cpu().numpy()
    D = np.sqrt(((Qf.astype(np.float64)[:, None, :] - Rf.astype(np.float64)[G]) ** 2).sum(2))
    assert np.allclose(D, np.sqrt(O2), rtol=2e-6) and np.allclose(dist.cpu().numpy(), D, rtol=2e-6)


@pytest.mark.parametrize("case", ["offset", "spread", "few"])
@pytest.mark.parametrize("d,e", [(64, 2), (20, 33)])
def test_ranks_of_rows_whose_norms_overflow(orc, case, d, e):
    """Finite rows with squared norms past FP32's range: far from the origin
    with ordinary distances, distances that overflow too, and a few such rows
    among ordinary ones (more than one and fewer than a tile past the last
    whole one).  Equal to the oracle's integers."""
    import paper_2603_04035_amd as knn
    n, k = 300, 10
    rng = np.random.default_rng(d)
    X = rng.normal(size=(n, d)).astype(np.float32)
    Y = (X @ rng.normal(size=(d, e)) + rng.normal(scale=0.5, size=(n, e))).astype(np.float32)
    for A in (X, Y):
        if case == "offset":
            A *= np.float32(1e16)
            A += np.float32(1e19)
        elif case == "spread":
            A *= np.float32(1.5e19)
        else:
            A[::50] *= np.float32(1e20)
    _, (h, t, c) = knn.quality(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), k, per_row=True)
    with np.errstate(over="ignore"):
        oh, ot, oc = orc.quality_rows(X, Y, k, canonical=True)
    assert np.array_equal(h.cpu().numpy(), oh) and np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(c.cpu().numpy(), oc)


@pytest.mark.parametrize("lead", [2.0, 64.0, 4096.0])
def test_pca_vectors_beside_a_leading_eigenvalue(lead):
    """The eigensolver alone (the block is all of R^16) on Hadamard columns, whose
    sums are exact: two of variance near 1 with a covariance of 2^-22 and one
    `lead` times as long.  The covariance is nothing against the whole norm, but
    turns the two vectors by 1.5e-5.  Bound: 100 roundings."""
    import paper_2603_04035_amd as knn
    n, d, p = 64, 16, 4
    H = np.ones((1, 1))
    while len(H) < n:
        H = np.block([[H, H], [H, -H]])
    X = H[:, 1:d + 1] * np.concatenate([[lead, 1.0078125, 1.0], 2.0 ** -np.arange(1, d - 2)])
    X[:, 2] += 2.0 ** -22 * H[:, 2]
    assert np.array_equal(X, X.astype(np.float32))
    B = X[:, 1:3].T @ X[:, 1:3]
    ref = np.linalg.eigh(B)[1][:, ::-1]
    ref = ref * np.sign(ref[np.abs(ref).argmax(0), np.arange(2)])
    V = knn.pca(torch.from_numpy(X.astype(np.float32)).cuda(), p)[1].cpu().numpy()
    print(lead, np.abs(V[1:3, 1:3] - ref).max(), ref[0, 1])
    assert np.abs(V[1:3, 1:3] - ref).max() <= 1e-14


@pytest.mark.parametrize("a,lead,iters", [(0.1, 1e5, 0), (0.2, 1e5, 0), (0.3, 1e5, 0), (0.1, 1.0, 0), (0.2, 1e5, 40),
                                          (0.1, 1.0, 10), ("drop", 1.0, 6), ("drop", 1e5, 0)])
def test_pca_at_least_the_power_iterations(a, lead, iters):
    """Spectra on which the filter is slow: a flat tail, alone and under one
    eigenvalue 10^5 times as large (one product per round), and a drop right
    behind the block, below which the filter is flat.  Bound: twice the error
    of `iters` (0: 200) plain iterations of the same width, or 1e-9
    (rounding against the leading eigenvalue)."""
    import paper_2603_04035_amd as knn
    d, p, m = 300, 50, 80
    lam = np.concatenate([np.linspace(1.1, 1.0, 80), np.linspace(0.1, 0.05, d - 80)]) if a == "drop" else \
        np.arange(1, d + 1) ** -a
    lam[0] *= lead
    X = _spectrum(3000, d, lam, 3)
    Xc = X.astype(np.float64)
    Xc -= Xc.mean(0)
    C = Xc.T @ Xc / (len(X) - 1)

    def signed(U):
        return U * np.sign(U[np.abs(U).argmax(0), np.arange(U.shape[1])])
    ref = signed(np.linalg.eigh(C)[1][:, ::-1][:, :p])
    V = np.random.default_rng(0).normal(size=(d, m))
    for _ in range(iters or 200):
        V = np.linalg.qr(C @ V)[0]
    plain = signed(V @ np.linalg.eigh(V.T @ C @ V)[1][:, ::-1][:, :p])
    got = knn.pca(torch.from_numpy(X).cuda(), p, iters=iters)[1].cpu().numpy()
    print(np.abs(got - ref).max(), np.abs(plain - ref).max())
    assert np.abs(got - ref).max() <= max(2 * np.abs(plain - ref).max(), 1e-9)


@pytest.mark.parametrize("n", [12, 271, 272, 1024, 1025, 5000, 131_072, 131_073])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_build_within_its_least_limit(n, precision):
    """The least workspace limit a build accepts holds all it takes (counters
    and sort counts lie in scratch that is free by then): the same lists and
    counts as without a limit, with a bank of counters of their own (fewer than
    272 rows) and 128 banks, and at the edges of the sort's tiles."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=n, d=12, seed=n)).cuda()
    args = dict(build_k=8, max_iters=3, delta=0.0, precision=precision, seed=3)
    lo, hi = 0, 4000 * n + (1 << 20)   # refused, accepted
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            knn.nndescent_build(X, 5, workspace_limit_bytes=mid, **args)
            hi = mid
        except knn.KnnError as e:
            assert e.status == -2
            lo = mid
    a = knn.nndescent_build(X, 5, workspace_limit_bytes=hi, **args)
    b = knn.nndescent_build(X, 5, **args)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    for key in ("updates", "pairs_joined", "list_dropped"):   # offers race for slots
        assert np.array_equal(a[2][key], b[2][key]), key


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("nq", [1, 2, 4, 5, 16])
@pytest.mark.parametrize("nr,d", [(600, 50), (1024, 200), (2000, 300), (4096, 64), (4097, 64), (9000, 40)])
def test_few_queries_routes_agree(precision, nq, nr, d):
    """Few queries on both sides of the rule for lists (at most four, at most
    4,096 pairs), and the gated route's splits with one block of queries:
    the bits of the list route."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=nr, d=d, comps=5, seed=nr)).cuda()
    Q = torch.from_numpy(datagen.gmm_isotropic(n=nq, d=d, comps=5, seed=nr)).cuda()
    a = knn.knn_exact_query(Q, X, 12, precision=precision)
    b = knn.knn_exact_query(Q, X, 12, precision=precision, workspace_limit=4 << 30)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("nq,nr,d", [(32_000, 92, 2), (32_000, 93, 2), (3333, 1436, 3), (3334, 1436, 3), (4000, 2560, 9),
                                     (4192, 2560, 9), (4193, 2560, 9)])
def test_many_queries_few_coordinates(nq, nr, d):
    """Both sides of the one-launch search's bounds on queries x references (up
    to 3 and up to 16 coordinates): the bits of the direct search."""
    import paper_2603_04035_amd as knn
    rng = np.random.default_rng(nq)
    X = torch.from_numpy(rng.integers(-9, 10, (nr, d)).astype(np.float32) / 4).cuda()
    Q = torch.from_numpy(rng.integers(-9, 10, (nq, d)).astype(np.float32) / 4).cuda()
    i, dist = knn.knn_exact_query(Q, X, 10)[:2]
    ref_i, ref_d = knn.knn_exact_query(Q, X, 10, workspace_limit=1 << 30)[:2]
    assert torch.equal(i, ref_i) and torch.equal(dist, ref_d)


def test_device_nearly_full(orc):
    """600 MB of device memory left: the gated search's buffers (1.2 GB for
    65,600 rows) give way to lists, and the rank pass to smaller launches; the
    results are the usual ones.  In a process of its own, whose scratch arena is
    empty."""
    import subprocess
    import sys
    code = """
import numpy as np, torch
import paper_2603_04035_amd as knn
from paper_2603_04035_amd import datagen
X = torch.from_numpy(datagen.gmm_isotropic(n=65_600, d=20, seed=3)).cuda()
Y = X[:, :2].contiguous()
hog = torch.empty(torch.cuda.mem_get_info()[0] - (600 << 20), dtype=torch.uint8, device="cuda")
low = knn.knn_exact(X, 10), knn.quality(X, Y, 10)
del hog
torch.cuda.empty_cache()
full = knn.knn_exact(X, 10), knn.quality(X, Y, 10)
assert torch.equal(low[0][0], full[0][0]) and torch.equal(low[0][1], full[0][1])
assert low[1] == full[1], (low[1], full[1])
print("same")
"""
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert out.stdout.strip().endswith("same"), out.stderr[-800:]
