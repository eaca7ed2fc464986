"""GPU parity of contraction steps (every node aggregating its peers at once).

Nodes hear random peer lists (some including themselves, in random order).
For each node whose decisions are all pinned (the pinning checks of
tests/parity.py on the node's own sub-matrix of distances and bounds), the
selected rows must equal the oracle's; every output row must match the
oracle's within max(1e-5 |oracle|, 1e-6) (Krum, Median and Average bit for
bit: a copy, an input value, and the same fp64 sum in the same order). With
every node hearing all n nodes in order, each row equals the plain rule call
bit for bit. Both distance engines are covered (n <= 20 direct, larger Gram).
"""
import numpy as np
import pytest
import torch

import oracle
import parity
import paper_2010_05888_amd as gf

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _library():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    gf.load()
    gf.set_direct_max_n(20)


def _inputs(n, d, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n, d)) * (1.0 + rng.permutation(n)[:, None] / n)).astype(np.float32)
    x[: max(1, n // 8)] *= 10.0
    return rng, x


def _pinned_nodes(rule, x, peers, f, m, B):
    ok = []
    D = oracle.pairwise_sqdist(x)
    for v in range(x.shape[0]):
        p = list(peers[v])
        xs = np.ascontiguousarray(x[p])
        Ds, Bs = D[np.ix_(p, p)], B[np.ix_(p, p)]
        same = parity.identical_rows(Ds)
        if rule in ("krum", "multikrum"):
            mm = 1 if rule == "krum" else m
            _, _, sc = oracle.multikrum(xs, f, mm, return_scores=True)
            ok.append(parity.krum_pinned(sc, Ds, Bs, f, mm, same)[0])
        elif rule in ("bulyan", "multikrum_iterated"):
            res = (oracle.bulyan(xs, f, return_rounds=True) if rule == "bulyan"
                   else oracle.multikrum_iterated(xs, f, m, return_rounds=True))
            ok.append(parity.bulyan_pinned(res[2], res[3], Ds, Bs, len(p), f, same)[0])
        elif rule == "mda":
            _, sel = oracle.mda(xs, f)
            ok.append(parity.mda_pinned(Ds, Bs, len(p), f, sel)[0])
        else:
            ok.append(True)
    return ok


CASES = [("average", 0, None), ("median", 3, None), ("krum", 2, None), ("multikrum", 2, 5),
         ("multikrum_iterated", 2, 5), ("bulyan", 2, None), ("mda", 2, None)]


@pytest.mark.parametrize("n,q,d", [(12, 11, 5003), (20, 15, 4097), (40, 23, 3001)])
@pytest.mark.parametrize("rule,f,m", CASES)
def test_step_matches_the_oracle(rule, f, m, n, q, d):
    rng, x = _inputs(n, d, 1000 * n + q)
    peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
    xt = torch.from_numpy(x).to(DEV)
    pt = torch.from_numpy(peers).to(DEV)
    y = gf.contract_step(rule, xt, pt, f, m).cpu().numpy()
    want, want_sel = oracle.contract_step(rule, x, peers, f, m)
    eng = gf.distance_engine(n, d)
    ref = parity.checked_reference(x, gf.gram_reference(xt)) if eng == "gram" else None
    B = parity.dist_bounds(oracle.pairwise_sqdist(x), eng, ref, x)
    pinned = _pinned_nodes(rule, x, peers, f, m, B)
    assert sum(pinned) >= n // 2, "too few pinned nodes to test"
    for v in range(n):
        if not pinned[v]:
            continue
        if rule in ("krum", "median", "average"):
            assert np.array_equal(y[v], want[v]), (rule, v)
        else:
            ok, at, err = parity.agg_close(y[v], want[v])
            assert ok, (rule, v, at, err)


@pytest.mark.parametrize("rule,f", [("multikrum", 2), ("bulyan", 2), ("median", 3), ("krum", 1),
                                    ("multikrum_iterated", 2), ("average", 0), ("mda", 2)])
@pytest.mark.parametrize("n", [11, 33])
def test_all_peers_in_order_equal_the_plain_rule(rule, f, n):
    if rule == "bulyan" and n < 4 * f + 3:
        pytest.skip("below Bulyan's requirement")
    _, x = _inputs(n, 7001, n)
    xt = torch.from_numpy(x).to(DEV)
    peers = torch.arange(n, dtype=torch.int32, device=DEV).repeat(n, 1)
    y = gf.contract_step(rule, xt, peers, f)
    if rule == "average":
        want = gf.average(xt)
    else:
        want = gf.gar(rule, xt, f)[0]
    assert all(torch.equal(y[v], want) for v in range(n))


def test_mda_with_64_peers():
    # 64 peers per node: the subset search's dynamic LDS (D, prefix maxima and
    # indices) exceeds 64 KB and is requested from the runtime
    n, f = 64, 2
    _, x = _inputs(n, 3001, 64)
    xt = torch.from_numpy(x).to(DEV)
    peers = torch.arange(n, dtype=torch.int32, device=DEV).repeat(n, 1)
    y = gf.contract_step("mda", xt, peers, f)
    want = gf.gar("mda", xt, f)[0]
    assert all(torch.equal(y[v], want) for v in range(n))


def test_several_steps():
    n, q, d, f = 16, 9, 2049, 2
    rng, x = _inputs(n, d, 5)
    peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
    xt = torch.from_numpy(x).to(DEV)
    pt = torch.from_numpy(peers).to(DEV)
    got = gf.contract("median", xt, pt, f, 3).cpu().numpy()
    want = x
    for _ in range(3):
        want, _ = oracle.contract_step("median", want, peers, f)
    assert np.array_equal(got, want)
    spread = lambda a: (a.max(0) - a.min(0)).max()
    assert spread(got) <= spread(x)


def test_invalid_arguments_are_rejected():
    x = torch.zeros((6, 10), dtype=torch.float32, device=DEV)
    p = torch.zeros((6, 7), dtype=torch.int32, device=DEV)
    with pytest.raises(gf.GarfieldError) as e:
        gf.contract_step("median", x, p, 0)  # q > n
    assert e.value.code == gf.EINVAL
    p = torch.arange(5, dtype=torch.int32, device=DEV).repeat(6, 1)
    with pytest.raises(gf.GarfieldError) as e:
        gf.contract_step("dist", x, p, 1)
    assert e.value.code == gf.EINVAL
    with pytest.raises(gf.GarfieldError) as e:
        gf.contract_step("krum", x, p, 2)  # q = 5 < 2f+3
    assert e.value.code == gf.EREQ
    x = torch.zeros((30, 10), dtype=torch.float32, device=DEV)
    p = torch.arange(30, dtype=torch.int32, device=DEV).repeat(30, 1)
    with pytest.raises(gf.GarfieldError) as e:
        gf.contract_step("mda", x, p, 8)  # C(30, 8) subsets per node, above the per-node cap
    assert e.value.code == gf.ETOOBIG


def test_mda_small_integer_ties():
    # exact distances: many equal diameters, the first subset of positions wins
    rng = np.random.default_rng(9)
    for trial in range(10):
        n = int(rng.integers(5, 16))
        q = int(rng.integers(3, n + 1))
        f = int(rng.integers(0, (q - 1) // 2 + 1))
        x = rng.integers(-2, 3, size=(n, 33)).astype(np.float32)
        peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
        y = gf.contract_step("mda", torch.from_numpy(x).to(DEV), torch.from_numpy(peers).to(DEV), f)
        want, want_sel = oracle.contract_step("mda", x, peers, f)
        got = y.cpu().numpy()
        for v in range(n):  # exact sums of small integers: equal iff the same rows were taken
            assert np.array_equal(got[v], want[v]), (trial, n, q, f, v, want_sel[v])


def _shared(n, absent):
    """Coordinates from which on the median shares a coordinate's rows between
    the nodes."""
    if 11 * absent >= 3 * n and n < 21:
        return 1 << (22 if n < 16 else 21)
    return 3 << 17 if n < 14 else 1 << 18


# the forms that share a coordinate's rows between the nodes, at the smallest
# lengths that take them: n at both sides of their limit of 32 rows, every count
# of absent rows up to and past 6, whole and ragged tiles of 512 coordinates
@pytest.mark.parametrize("n,absent,extra", [(1, 0, 1), (3, 0, 0), (4, 1, 1), (8, 2, 511),
                                            (10, 3, 510), (13, 4, 2), (20, 5, 513), (19, 6, 2),
                                            (18, 6, 3), (32, 6, 1025), (32, 7, 188), (32, 0, 511),
                                            (33, 3, 188)])
def test_shared_rows(n, absent, extra):
    d = _shared(n, absent) + extra
    q = n - absent
    rng = np.random.default_rng(7 * n + absent)
    g = torch.Generator(device=DEV).manual_seed(7 * n + absent)
    xt = torch.randn((n, d), device=DEV, generator=g)
    xt *= torch.from_numpy(1.0 + rng.permutation(n) / n).to(DEV).float()[:, None]
    xt[: max(1, n // 8)] *= 10.0
    peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
    if q > 1:
        peers[0, q - 1] = peers[0, 0]  # a list that repeats a row: the general form
    pt = torch.from_numpy(peers).to(DEV)
    got = gf.contract_step("median", xt, pt, 0)
    for v in range(n):
        srt = xt[pt[v].long()].sort(0).values.double()
        want = ((srt[(q - 1) // 2] + srt[q // 2]) / 2).float()
        assert torch.equal(got[v], want), v
    if q < 3:
        return
    # Multi-Krum of all q rows: the selection is the list, in ascending order
    # (a list that repeats a row has no such selection)
    if n > 18:
        xt = torch.cat([xt, xt.flip(1)], 1)  # where the mean shares too
    got = gf.contract_step("multikrum", xt, pt, 0, q)
    for v in range(1, n):
        acc = torch.zeros(xt.shape[1], dtype=torch.float64, device=DEV)
        for r in np.sort(peers[v]):
            acc += xt[int(r)].double()
        assert torch.equal(got[v], (acc / q).float()), v


@pytest.mark.parametrize("q,f,search", [(10, 4, "peer_mda"), (11, 4, "peer_mda"),
                                        (11, 5, "peer_mda"), (12, 4, "peer_mda"),
                                        (13, 3, "peer_cover"), (12, 5, "peer_cover"),
                                        (23, 2, "peer_mda"), (24, 2, "peer_cover")])
def test_mda_search_of_a_node(q, f, search):
    """One or two subsets a thread, or covers: the search each size takes, and the
    first subset of least diameter among small-integer ties from either."""
    n = q + 1
    rng = np.random.default_rng(100 * q + f)
    x = rng.integers(-2, 3, size=(n, 33)).astype(np.float32)
    peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
    xt, pt = torch.from_numpy(x).to(DEV), torch.from_numpy(peers).to(DEV)
    gf.set_kernel_timing(True)
    y = gf.contract_step("mda", xt, pt, f)
    names = set(gf.kernel_timing())
    gf.set_kernel_timing(False)
    assert {"peer_mda", "peer_cover"} & names == {search}
    want, _ = oracle.contract_step("mda", x, peers, f)
    assert np.array_equal(y.cpu().numpy(), want)


def test_shared_mean_leaves_out_what_is_not_finite():
    n, q, d = 12, 9, 1 << 19
    rng, x = _inputs(n, d, 3)
    x[11, 700] = np.inf
    x[10, 40] = np.nan
    peers = np.tile(np.arange(q, dtype=np.int32), (n, 1))  # nobody hears rows 9 to 11
    y = gf.contract_step("multikrum", torch.from_numpy(x).to(DEV), torch.from_numpy(peers).to(DEV),
                         0, q).cpu().numpy()
    acc = np.zeros(d)
    for r in range(q):
        acc += x[r].astype(np.float64)
    assert np.array_equal(y, np.tile((acc / q).astype(np.float32), (n, 1)))


@pytest.mark.parametrize("n,absent", [(5, 1), (9, 2), (12, 3), (20, 3), (20, 5)])
def test_shared_median_leaves_out_what_is_nan(n, absent):
    """NaN and infinities in rows that a node does not hear leave its median as
    it is, for odd and even counts of rows and whole and ragged tiles."""
    q, d = n - absent, _shared(n, absent) + 3
    rng, x = _inputs(n, d, 31 * n + absent)
    at = rng.random(d)
    x[n - 1, at < 0.5] = np.nan  # nobody hears the last rows
    x[n - absent, at > 0.7] = -np.inf
    peers = np.stack([rng.permutation(q) for _ in range(n)]).astype(np.int32)
    got = gf.contract_step("median", torch.from_numpy(x).to(DEV), torch.from_numpy(peers).to(DEV),
                           0).cpu().numpy()
    srt = np.sort(x[:q].astype(np.float64), axis=0)
    want = ((srt[(q - 1) // 2] + srt[q // 2]) / 2).astype(np.float32)
    assert np.array_equal(got, np.tile(want, (n, 1)))


@pytest.mark.parametrize("n,absent", [(4, 1), (9, 2), (12, 3), (20, 3), (22, 6), (8, 0)])
def test_medians_keep_the_sign_of_a_zero(n, absent):
    """Rows with zeros of both signs, -0 before +0: the same bits from the form
    that shares a coordinate's rows and, on the first coordinates alone, from
    each node's own network."""
    q, d = n - absent, _shared(n, absent) + 5
    rng = np.random.default_rng(n)
    x = rng.choice(np.array([-1.5, -0.0, 0.0, 0.0, 2.0], np.float32), (n, d))
    peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
    pt = torch.from_numpy(peers).to(DEV)
    got = gf.contract_step("median", torch.from_numpy(x).to(DEV), pt, 0).cpu().numpy()
    own = gf.contract_step("median", torch.from_numpy(x[:, :4099].copy()).to(DEV), pt, 0)
    bits = x.view(np.int32)
    keys = np.sort((bits ^ ((bits >> 31) & 0x7fffffff))[peers], axis=1)
    srt = (keys ^ ((keys >> 31) & 0x7fffffff)).view(np.float32).astype(np.float64)
    lo, hi = srt[:, (q - 1) // 2], srt[:, q // 2]
    want = (lo if q % 2 else (lo + hi) * 0.5).astype(np.float32).view(np.int32)
    assert np.array_equal(got.view(np.int32), want)
    assert np.array_equal(own.cpu().numpy().view(np.int32), want[:, :4099])


def test_mda_searches_agree():
    """Nodes of few subsets are enumerated, the others searched through covers:
    the same first subset of least diameter, ties (small integers) included."""
    rng = np.random.default_rng(4)
    for n, q, f in [(11, 10, 3), (14, 11, 4), (22, 22, 2), (22, 23 - 1, 3), (26, 24, 5)]:
        x = rng.integers(-2, 3, size=(n, 65)).astype(np.float32)
        peers = np.stack([rng.permutation(n)[:q] for _ in range(n)]).astype(np.int32)
        got = gf.contract_step("mda", torch.from_numpy(x).to(DEV), torch.from_numpy(peers).to(DEV),
                               f).cpu().numpy()
        want, _ = oracle.contract_step("mda", x, peers, f)
        assert np.array_equal(got, want), (n, q, f)
