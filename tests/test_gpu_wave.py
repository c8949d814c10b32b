"""GPU parity of the wave kernel (descents side by side, expansions one query per wavefront) at
the edges of its layout: queries per wavefront, lanes per query, positions of N."""
import numpy as np
import pytest

from tests._compare import compare_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    oracle.build(force=False)
    from paper_2605_02224_amd import api as A
    from paper_2605_02224_amd import workloads as W
    c = W.random_cloud(4000, seed=5, shape="torus")
    return torch, oracle, A, W, c.by_rank, A.Cloud.build(c.by_rank).upload()


def _rows(torch, cl, Q, k, m=None):
    idx, dist = cl.knn(torch.from_numpy(Q).cuda(), k, m)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), dist.cpu().numpy()


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("nq", [1, 3, 5, 8195])
def test_rows_at_layout_edges(env, k, nq):
    """Ranks equal the FP64 brute force's (near-ties excused), distances its float32."""
    torch, oracle, A, W, P, cl = env
    lo, hi = W.bbox_expanded(P, 1.1)
    Q = W.uniform_in_box(np.random.default_rng(10 * k + nq), nq, lo, hi)
    for m in (None, k, 500):
        idx, dist = _rows(torch, cl, Q, k, m)
        ri, _, rD = oracle.knn_bruteforce(P, Q, k + 1, m)
        assert compare_rows(idx, dist, ri[:, :k], rD[:, :k], rD[:, k], P=P, Q=Q, m=m) <= 2


@pytest.mark.parametrize("k", [8, 16, 32, 64])
def test_equal_distances(env, k):
    """A lattice: whole shells of sites at one distance, ranked by age, exactly."""
    torch, oracle, A, W, _, _ = env
    rng = np.random.default_rng(k)
    g = np.stack(np.meshgrid(*[np.arange(12)] * 3, indexing="ij"), -1).reshape(-1, 3)
    P = g[rng.permutation(len(g))].astype(np.float32)
    cl = A.Cloud.build(P).upload()
    Q = np.concatenate([P[:300], P[:300] + np.float32(0.5)])
    idx, _ = _rows(torch, cl, Q, k)
    D = ((Q[:, None, :].astype(np.float64) - P[None].astype(np.float64)) ** 2).sum(-1)
    assert np.array_equal(idx, np.argsort(D, axis=1, kind="stable")[:, :k])


def test_distances_not_finite(env):
    """NaN and infinite coordinates, and distances past the float32 range: the same rows as
    the row kernel's order (D, age) gives; other queries of the wavefront are not disturbed."""
    torch, oracle, A, W, P, cl = env
    lo, hi = W.bbox_expanded(P, 1.1)
    Q = W.uniform_in_box(np.random.default_rng(1), 64, lo, hi)
    want = _rows(torch, cl, Q, 16)[0]
    B = Q.copy()
    B[3] = np.nan
    B[9, 0] = np.inf
    B[17, 1] = 1e30
    idx, dist = _rows(torch, cl, B, 16)
    keep = [i for i in range(64) if i not in (3, 9, 17)]
    assert np.array_equal(idx[keep], want[keep])
    assert idx[9].tolist() == list(range(16)) and np.isinf(dist[9]).all()
    D = ((B[17].astype(np.float64) - P.astype(np.float64)) ** 2).sum(-1)
    assert np.array_equal(idx[17], np.argsort(D, kind="stable")[:16])


def _chunks(torch, q, f, size=50000):
    parts = [f(q[i:i + size].contiguous()) for i in range(0, q.shape[0], size)]
    torch.cuda.synchronize()
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])


def _lattice(A, side, seed):
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)
    P = g[np.random.default_rng(seed).permutation(len(g))].astype(np.float32)
    return P, A.Cloud.build(P).upload()


@pytest.mark.parametrize("k", [9, 12, 16])
@pytest.mark.parametrize("shape", ["torus", "lattice"])
def test_gathered_rows(env, k, shape):
    """Launches and batches large enough that rows gather their candidates (k > 8) against the
    same queries in small launches: the same ranks and distances, NaN and infinities included."""
    torch, oracle, A, W, P, cl = env
    if shape == "lattice":
        P, cl = _lattice(A, 15, k)
    rng = np.random.default_rng(k)
    lo, hi = W.bbox_expanded(P, 1.1)
    Q = W.uniform_in_box(rng, 196608, lo, hi)
    if shape == "lattice":
        Q = np.round(2 * Q).astype(np.float32) / 2
    Q[5, 0], Q[77, 2] = np.inf, 1e30
    q = torch.from_numpy(Q).cuda()
    for m in (None, 300):
        idx, dist = cl.knn(q, k, m)
        ri, rd = _chunks(torch, q, lambda c: cl.knn(c, k, m))
        assert torch.equal(idx, ri) and torch.equal(dist, rd)
    items = A.alloc_outputs([(cl, q, k, None), (cl, q[:100].contiguous(), k, None)])
    plan = A.BatchPlan(len(items), sum(it[1].shape[0] for it in items))
    plan.run(items)
    torch.cuda.synchronize()
    ri, rd = _chunks(torch, q, lambda c: cl.knn(c, k))
    assert torch.equal(items[0][4], ri) and torch.equal(items[0][5], rd)
    assert torch.equal(items[1][4], ri[:100])
    plan.close()


@pytest.mark.parametrize("kmax", [2, 16, 17, 32, 64])
@pytest.mark.parametrize("shape", ["torus", "lattice"])
def test_scanned_lists(env, kmax, shape):
    """Large launches that scan lists by rows (a k and prefix per query; prefixes with long
    rows) against the same queries in small launches."""
    torch, oracle, A, W, P, cl = env
    if shape == "lattice":
        P, cl = _lattice(A, 15, kmax)
    rng = np.random.default_rng(kmax)
    lo, hi = W.bbox_expanded(P, 1.1)
    Q = W.uniform_in_box(rng, 65537, lo, hi)
    if shape == "lattice":
        Q = np.round(2 * Q).astype(np.float32) / 2
    Q[5, 0], Q[77, 2] = np.inf, 1e30
    q = torch.from_numpy(Q).cuda()
    kq = torch.from_numpy(rng.integers(1, kmax + 1, len(Q)).astype(np.int32)).cuda()
    kq[:200] = kmax
    mq = torch.from_numpy(np.exp(rng.uniform(0, np.log(len(P)), len(Q))).astype(np.int32)).cuda()
    mq = mq.clamp(1, len(P))
    got = cl.knn_var(q, kq, mq)
    parts = []
    for i in range(0, len(Q), 16000):
        parts.append(cl.knn_var(q[i:i + 16000].contiguous(), kq[i:i + 16000].contiguous(),
                                mq[i:i + 16000].contiguous()))
    torch.cuda.synchronize()
    assert torch.equal(got[0], torch.cat([p[0] for p in parts]))
    assert torch.equal(got[1], torch.cat([p[1] for p in parts]))
    for m in (1, kmax, 600):
        idx, dist = cl.knn(q, kmax, m)
        ri, rd = _chunks(torch, q, lambda c: cl.knn(c, kmax, m), 16000)
        assert torch.equal(idx, ri) and torch.equal(dist, rd)


@pytest.mark.parametrize("n", [1, 2, 4, 5, 17, 300, 4097])
def test_arena_gathered_on_device(env, n):
    """The records an upload gathers on the device against the image packed on the host
    (compact), and both against the brute force."""
    torch, oracle, A, W, _, _ = env
    rng = np.random.default_rng(n)
    P = rng.standard_normal((n, 3)).astype(np.float32)
    cl = A.Cloud.build(P).upload()
    Q = rng.standard_normal((130, 3)).astype(np.float32)
    a = _rows(torch, cl, Q, 8)
    cl.compact()
    b = _rows(torch, cl, Q, 8)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    D = ((Q[:, None, :].astype(np.float64) - P[None].astype(np.float64)) ** 2).sum(-1)
    k = min(8, n)
    assert np.array_equal(a[0][:, :k], np.argsort(D, axis=1, kind="stable")[:, :k])
    assert (a[0][:, k:] == -1).all()


@pytest.mark.parametrize("nq", [1, 5, 203])
def test_batch_classes_by_rows_and_waves(env, nq):
    """One plan, run with whole clouds (classes of k > 16 by waves), prefixes (by rows), both in
    one class, and whole clouds again (the same graph): always the plain launch's rows."""
    torch, oracle, A, W, P, cl = env
    rng = np.random.default_rng(nq)
    lo, hi = W.bbox_expanded(P, 1.1)
    plan = A.BatchPlan(8, 8 * 203)
    for ms in ((None,) * 5, (900,) * 5, (None, 900, None, 900, None), (None,) * 5):
        reqs = [(cl, torch.from_numpy(W.uniform_in_box(rng, nq + i, lo, hi)).cuda(), k, m)
                for i, (k, m) in enumerate(zip((10, 17, 32, 33, 64), ms))]
        items = A.alloc_outputs([r[:3] + (cl.n if r[3] is None else r[3],) for r in reqs])
        plan.run(items)
        torch.cuda.synchronize()
        for (_, q, k, m), it in zip(reqs, items):
            ri, rd = cl.knn(q, k, m)
            torch.cuda.synchronize()
            assert torch.equal(it[4], ri) and torch.equal(it[5], rd)
    plan.close()


def _exact_rows(P, Q, k, m, live=None):
    """Ranks of the k nearest of the first m points by (D, age), float64."""
    d = Q[:, None, :].astype(np.float64) - P[None, :m].astype(np.float64)
    D = d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1] + d[..., 2] * d[..., 2]
    if live is not None:
        D[:, ~live[:m]] = np.inf
    return np.argsort(D, axis=1, kind="stable")[:, :k]


@pytest.mark.parametrize("jitter", [0.0, 1e-5])
@pytest.mark.parametrize("sites", [64, 65, 66, 68, 72, 80])
def test_last_position_fills_within_an_insertion(env, sites, jitter):
    """Little more than 64 sites, whole shells of them at one distance or nearly so: the 64th
    position fills among a few new keys.  Whole clouds and prefixes, the plain and the batched
    call, pending deletions that widen the walk to 64; by (D, age) in float64, exactly."""
    torch, oracle, A, W, _, _ = env
    rng = np.random.default_rng(1000 * sites + (jitter > 0))
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    Q = (rng.integers(-1, 12, (1500, 3)) / 2).astype(np.float32)
    q = torch.from_numpy(Q).cuda()
    for n in (sites, 216):
        P = g[rng.permutation(216)[:n]].astype(np.float32)
        P = (P + jitter * rng.standard_normal(P.shape)).astype(np.float32)
        cl = A.Cloud.build(P).upload()
        items = []
        for k in (60, 62, 63, 64):
            idx, _ = _rows(torch, cl, Q, k, sites)
            assert np.array_equal(idx, _exact_rows(P, Q, k, sites)), (n, k)
            items.append((cl, q, k, sites))
        items = A.alloc_outputs(items)
        plan = A.BatchPlan(len(items), len(items) * len(Q))
        plan.run(items)
        torch.cuda.synchronize()
        for it in items:
            assert np.array_equal(it[4].cpu().numpy(), _exact_rows(P, Q, it[2], sites)), (n, it[2])
        plan.close()
        gone = rng.choice(np.arange(1, sites), 15, replace=False).astype(np.int32)
        live = np.ones(n, bool)
        live[gone] = False
        cl.delete_lazy(gone)
        k = min(48, sites - 16)
        idx, _ = _rows(torch, cl, Q, k, sites)
        assert np.array_equal(idx, _exact_rows(P, Q, k, sites, live)), (n, "pending")


@pytest.fixture(scope="module")
def hubs(env):
    """Clouds with lists that are a good part of them: a sphere around its centre, the oldest
    point; a sheet and a few points far off it."""
    torch, oracle, A, W, _, _ = env
    rng = np.random.default_rng(7)
    s = rng.standard_normal((9000, 3))
    s *= (1 + 1e-3 * rng.standard_normal((9000, 1))) / np.linalg.norm(s, axis=1, keepdims=True)
    s[0] = 0
    xy = rng.random((8980, 2))
    out = np.r_[np.c_[xy, 0.1 * np.sin(9 * xy[:, 0])], 10 * rng.random((20, 3))][rng.permutation(9000)]
    clouds = {}
    for name, P in (("centre", s), ("outliers", out)):
        P = P.astype(np.float32)
        cl = A.Cloud.build(P).upload()
        off, _ = cl.successors()
        assert (off[1:] - off[:-1]).max() > (4096 if name == "centre" else 1024)
        clouds[name] = (P, cl)
    return clouds


@pytest.mark.parametrize("nq", [300, 9000, 70001])
@pytest.mark.parametrize("name", ["centre", "outliers"])
def test_long_lists(env, hubs, name, nq):
    """Lists of thousands of entries, read 64 at a time to their end or the prefix's: ranks equal
    the FP64 brute force's (near-ties excused)."""
    torch, oracle, A, W, _, _ = env
    P, cl = hubs[name]
    rng = np.random.default_rng(nq)
    Q = W.uniform_in_box(rng, nq, *W.bbox_expanded(P, 1.1))
    pick = np.sort(rng.choice(nq, 300, replace=False))
    for m in (9000, 2500):
        ri, _, rD = oracle.knn_bruteforce(P, Q[pick], 65, m)
        for k in (1, 8, 20, 32, 64):
            idx, dist = _rows(torch, cl, Q, k, m)
            assert compare_rows(idx[pick], dist[pick], ri[:, :k], rD[:, :k], rD[:, k], P=P, Q=Q[pick],
                                m=m) <= 2, (k, m)
    q = torch.from_numpy(Q).cuda()
    for kmax in (4, 32):
        kq = rng.integers(1, kmax + 1, nq).astype(np.int32)
        mq = rng.integers(1, 9001, nq).astype(np.int32)
        idx, dist, off = cl.knn_var(q, torch.from_numpy(kq).cuda(), torch.from_numpy(mq).cuda())
        torch.cuda.synchronize()
        idx, dist, off = idx.cpu().numpy(), dist.cpu().numpy(), off.cpu().numpy()
        ex = 0
        for i in pick[:60]:
            ri, _, rD = oracle.knn_bruteforce(P, Q[i:i + 1], int(kq[i]), int(mq[i]))
            ex += compare_rows(idx[None, off[i]:off[i + 1]], dist[None, off[i]:off[i + 1]], ri, rD, P=P,
                               Q=Q[i:i + 1], m=int(mq[i]))
        assert ex <= 2
    items = A.alloc_outputs([(cl, q[:2000].contiguous(), k, None) for k in (8, 20, 40, 64)])
    plan = A.BatchPlan(4, 8000)
    plan.run(items)
    torch.cuda.synchronize()
    for it in items:
        ri, rd = cl.knn(it[1], it[2])
        torch.cuda.synchronize()
        assert torch.equal(it[4], ri) and torch.equal(it[5], rd)
    plan.close()


@pytest.mark.parametrize("k", [33, 48, 63, 64])
def test_keys_that_agree(env, k):
    """Queries near the middle of a shell: the distances of all sites agree in the upper bits of
    their keys, so which of them are the k nearest is decided by the exact ones alone."""
    torch, oracle, A, W, _, _ = env
    rng = np.random.default_rng(k)
    for spread in (0.0, 1e-7, 1e-4):
        P = rng.standard_normal((600, 3))
        P *= (1 + spread * rng.standard_normal((600, 1))) / np.linalg.norm(P, axis=1, keepdims=True)
        P = P.astype(np.float32)
        cl = A.Cloud.build(P).upload()
        Q = (1e-7 * rng.standard_normal((200, 3))).astype(np.float32)
        Q[:60] = 0
        Q[60:90] *= 1e9
        for m in (600, 66, 200):
            idx, dist = _rows(torch, cl, Q, k, m)
            ri, _, rD = oracle.knn_bruteforce(P, Q, k + 1, m)
            # (near-ties, which are all of the sites here, may stand for each other; the rest of
            # the rule holds: true distances, ordered by (D, age), no rank twice)
            compare_rows(idx, dist, ri[:, :k], rD[:, :k], rD[:, k], P=P, Q=Q, m=m)


@pytest.mark.parametrize("n", [3, 300, 5000, 90000])
def test_upload_takes_the_arena_alone(env, n):
    """An upload needs no device memory beside what the cloud then holds: the stream-ordered pool's
    high mark does not move."""
    import ctypes
    torch, oracle, A, W, _, _ = env
    hip = A._lib.lib()   # (symbols of the HIP runtime it is linked with)
    pool, v = ctypes.c_void_p(), ctypes.c_uint64(0)
    high = 8             # hipMemPoolAttrUsedMemHigh
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    P = np.random.default_rng(n).standard_normal((n, 3)).astype(np.float32)
    cl = A.Cloud.build(P, device=n > 3000)
    torch.cuda.synchronize()

    def mark():
        assert hip.hipMemPoolGetAttribute(pool, high, ctypes.byref(v)) == 0
        return v.value
    assert hip.hipMemPoolSetAttribute(pool, high, ctypes.byref(ctypes.c_uint64(0))) == 0
    before = mark()
    cl.upload()
    torch.cuda.synchronize()
    assert mark() == before
    Q = P[:40]
    idx, _ = _rows(torch, cl, Q, 1)
    assert (idx[:, 0] == np.arange(len(Q))).all()


# Launches of every kernel the rule can choose, above its thresholds: (queries, k, prefix; "var": a k
# and prefix per query up to these), for a cloud of 4000 points
ROUTES = {
    "gathered_k9": (196608, 9, None), "gathered_k16": (196609, 16, None),
    "gathered_prefix": (196608, 12, 700), "rows_k2": (65537, 2, None), "rows_k8": (70001, 8, None),
    "rows_k16": (70003, 16, None), "rows_prefix_k3": (6001, 3, 1700), "rows_prefix_k8": (8191, 8, 120),
    "rows_prefix_k17": (20001, 17, 1500), "rows_prefix_k33": (20002, 33, 1500),
    "rows_prefix_k64": (20003, 64, 1500), "rows_one_site_more": (20001, 64, 65),
    "rows_as_many": (20001, 32, 32), "waves_k20": (70001, 20, None), "waves_k64": (131073, 64, None),
    "waves_one_site_more": (3001, 64, 65), "waves_k1": (70001, 1, None), "scan_k33": (65537, 33, 1500),
    "scan_k64": (65538, 64, 66), "scan_k20": (262144, 20, 900), "scan_one_site_more": (262145, 32, 33),
    "var_waves": (70001, 32, "var"), "var_scan_32": (98305, 32, "var"), "var_scan_64": (70002, 64, "var"),
    "var_rows": (131073, 16, "var"), "var_rows_k4": (262145, 4, "var"),
}


@pytest.mark.parametrize("shape", ["torus", "lattice"])
@pytest.mark.parametrize("route", list(ROUTES))
def test_routes_against_brute_force(env, route, shape):
    """Sampled rows of large launches: ranks equal the FP64 brute force's; on the lattice, where whole
    shells tie, by (D, age) exactly."""
    torch, oracle, A, W, P, cl = env
    if shape == "lattice":
        P, cl = _lattice(A, 16, 3)
    n = len(P)
    nq, k, m = ROUTES[route]
    rng = np.random.default_rng(nq + k)
    Q = W.uniform_in_box(rng, nq, *W.bbox_expanded(P, 1.1))
    if shape == "lattice":
        Q = (np.round(2 * Q) / 2).astype(np.float32)
    q = torch.from_numpy(Q).cuda()
    pick = np.sort(rng.choice(nq, 400, replace=False))
    if m == "var":
        kq = rng.integers(1, k + 1, nq).astype(np.int32)
        kq[0] = k
        mq = np.exp(rng.uniform(0, np.log(n), nq)).astype(np.int32).clip(1, n)
        mq[rng.random(nq) < 0.3] = n
        idx, dist, off = cl.knn_var(q, torch.from_numpy(kq).cuda(), torch.from_numpy(mq).cuda())
        torch.cuda.synchronize()
        off = off.cpu().numpy()
        rows = [(i, int(kq[i]), int(mq[i])) for i in pick]
        idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
        got = [(idx[off[i]:off[i] + kk], dist[off[i]:off[i] + kk]) for i, kk, _ in rows]
    else:
        idx, dist = _rows(torch, cl, Q, k, m)
        rows = [(i, k, m or n) for i in pick]
        got = [(idx[i], dist[i]) for i in pick]
    ex = 0
    for (i, kk, mm), (gi, gd) in zip(rows, got):
        D = ((Q[i].astype(np.float64) - P[:mm].astype(np.float64)) ** 2)
        D = D[:, 0] + D[:, 1] + D[:, 2]
        order = np.argsort(D, kind="stable")[:kk]
        ri = np.full(kk, -1)
        ri[:len(order)] = order
        rD = np.full(kk, np.inf)
        rD[:len(order)] = D[order]
        if shape == "lattice":
            assert np.array_equal(gi, ri), (i, kk, mm)
        else:
            ex += compare_rows(gi[None], gd[None], ri[None], rD[None], P=P, Q=Q[i:i + 1], m=mm)
    assert ex <= 2


@pytest.mark.parametrize("nq,k,m", [(20001, 8, 2500), (20002, 30, 2500), (20003, 47, 2500),
                                    (70001, 16, None), (262144, 12, 2500), (3001, 40, None)])
def test_pending_deletions_on_every_route(env, nq, k, m):
    """Rows filtered by pending deletions, by the row, wave and scan kernels (k + 16 neighbours
    walked for), and per query; against the brute force over what is left."""
    torch, oracle, A, W, P, _ = env
    n = len(P)
    cl = A.Cloud.build(P).upload()
    rng = np.random.default_rng(nq)
    gone = rng.choice(np.arange(1, n), 40, replace=False).astype(np.int32)
    cl.delete_lazy(gone)
    live = np.ones(n, np.uint8)
    live[gone] = 0
    Q = W.uniform_in_box(rng, nq, *W.bbox_expanded(P, 1.1))
    pick = np.sort(rng.choice(nq, 500, replace=False))
    idx, dist = _rows(torch, cl, Q, k, m)
    assert cl.pending_deletes == len(gone)
    ri, _, rD = oracle.knn_bruteforce(P, Q[pick], k, m, live=live)
    assert compare_rows(idx[pick], dist[pick], ri, rD, P=P, Q=Q[pick], m=m, live=live) <= 2
    kq = rng.integers(1, k + 1, nq).astype(np.int32)
    mq = rng.integers(1, n + 1, nq).astype(np.int32)
    idx, dist, off = cl.knn_var(torch.from_numpy(Q).cuda(), torch.from_numpy(kq).cuda(),
                                torch.from_numpy(mq).cuda())
    torch.cuda.synchronize()
    idx, dist, off = idx.cpu().numpy(), dist.cpu().numpy(), off.cpu().numpy()
    ex = 0
    for i in pick[:80]:
        ri, _, rD = oracle.knn_bruteforce(P, Q[i:i + 1], int(kq[i]), int(mq[i]), live=live)
        ex += compare_rows(idx[None, off[i]:off[i + 1]], dist[None, off[i]:off[i + 1]], ri, rD, P=P,
                           Q=Q[i:i + 1], m=int(mq[i]), live=live)
    assert ex <= 2


def test_not_a_number_by_every_kernel(env):
    """NaN queries, nearer to nothing, get at most the site that their descent starts from (the rows
    may drop it, which order it behind nothing), and leave the other queries of their wavefront
    alone."""
    torch, oracle, A, W, P, cl = env
    for nq, k, m in ((64, 1, None), (64, 16, None), (70001, 1, None), (70001, 8, None), (70001, 20, None),
                     (196608, 12, None), (65537, 40, 1500), (20001, 20, 1500)):
        Q = W.uniform_in_box(np.random.default_rng(nq + k), nq, *W.bbox_expanded(P, 1.1))
        want, _ = _rows(torch, cl, Q, k, m)
        at = np.arange(5, nq, 97)
        B = Q.copy()
        B[at, at % 3] = np.nan
        idx, dist = _rows(torch, cl, B, k, m)
        assert np.isin(idx[at], (0, -1)).all() and ((idx[at] == 0).sum(1) <= 1).all(), (nq, k)
        assert np.isnan(dist[at][idx[at] == 0]).all() and np.isinf(dist[at][idx[at] == -1]).all(), (nq, k)
        keep = np.ones(nq, bool)
        keep[at] = False
        assert np.array_equal(idx[keep], want[keep]), (nq, k)
