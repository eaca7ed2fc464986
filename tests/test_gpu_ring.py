"""The direct engine's ring form (long inputs of up to 20 rows) and the mean it
writes on a guessed selection, at the smallest lengths that take it: whole and
ragged last stages, every split of the pairs over wave groups, and the three
ways a guess can end (right, the samples disagree, all of them wrong)."""
import itertools

import pytest
import torch

import paper_2010_05888_amd as gf

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _least(n):
    return 1 << (21 if n >= 16 else 23)


def _rows(n, d, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn((n, d), device=DEV, generator=g)


def _dist64(x):
    n, d = x.shape
    D = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    for a in range(0, d, 1 << 20):
        c = x[:, a:a + (1 << 20)].double()
        for i in range(n):
            D[i] += (c - c[i]).square_().sum(1)
    return D


def _kernels(call):
    gf.set_kernel_timing(True)
    out = call()
    torch.cuda.synchronize()
    names = set(gf.kernel_timing())
    gf.set_kernel_timing(False)
    return out, names


# every group count and pair split, stages of 1,024 and 512 coordinates; the
# last stage empty, of one coordinate, and one coordinate short of whole
@pytest.mark.parametrize("n,extra", [(2, 0), (8, 1), (9, 1023), (10, 0), (11, 511), (12, 1),
                                     (13, 0), (14, 511), (15, 1), (16, 0), (17, 1), (18, 511),
                                     (19, 0), (20, 1)])
def test_distances(n, extra):
    d = _least(n) + extra
    x = _rows(n, d, 100 * n + extra)
    x[n - 1] = x[0]  # equal rows, in different groups
    D, names = _kernels(lambda: gf.pairwise_sqdist(x))
    assert "dist_ring" in names
    W = _dist64(x)
    # a rounded difference and at most 16 fp32 multiply-adds per lane and run,
    # fp64 beyond: 18 * 2^-24 of a sum of positive terms
    assert bool(((D - W).abs() <= 18 * 2.0 ** -24 * W).all())
    assert torch.equal(D, D.T) and D[0, n - 1].item() == 0.0
    others = list(range(1, n - 1))
    assert torch.equal(D[0, others], D[n - 1, others])
    # whichever groups the pairs fall in, their sums are formed alike
    perm = torch.randperm(n, generator=torch.Generator().manual_seed(n)).to(DEV)
    assert torch.equal(gf.pairwise_sqdist(x[perm].contiguous()), D[perm][:, perm])


def _krum(D, f, m):
    n = len(D)
    scores = sorted((sum(sorted(D[i][j] for j in range(n) if j != i)[:n - f - 2]), i)
                    for i in range(n))
    return sorted(i for _, i in scores[:m])


def _mda(D, f):
    n = len(D)
    return list(min(itertools.combinations(range(n), n - f),
                    key=lambda s: max(D[i][j] for i in s for j in s)))


def _mean64(x, rows):
    acc = torch.zeros(x.shape[1], dtype=torch.float64, device=DEV)
    for r in rows:
        acc += x[r].double()
    return (acc / len(rows)).float()


def _samples(x, f, m):
    """Multi-Krum's selection on each of the guess's eight samples, and the least
    gap between the scores of its last row in and its first row out."""
    n, d = x.shape
    picks, gap = [], 1.0
    for r in range(8):
        a = r * (d // 8)
        D = _dist64(x[:, a:a + 1024]).tolist()
        s = sorted((sum(sorted(D[i][j] for j in range(n) if j != i)[:n - f - 2]), i)
                   for i in range(n))
        picks.append(sorted(i for _, i in s[:m]))
        if m < n:
            gap = min(gap, s[m][0] / s[m - 1][0] - 1.0)
    return picks, gap


# m beside the default: with n <= 12 and 2m > n + 4 a disagreement leaves the
# column sums, otherwise nothing; a guess of every row is always right
@pytest.mark.parametrize("rule,n,f,m,extra,ends", [
    (*case, ends) for case in [
        ("multikrum", 3, 0, 3, 0), ("multikrum", 7, 1, 6, 1023), ("multikrum", 11, 2, 9, 511),
        ("multikrum", 11, 2, 7, 1), ("multikrum", 12, 2, 10, 0), ("mda", 10, 3, 7, 1),
        ("multikrum", 13, 2, 11, 511), ("mda", 16, 2, 14, 0), ("multikrum", 18, 4, 14, 1),
        ("multikrum", 20, 4, 16, 511)]
    for ends in ["right", "disagree", "wrong"] if case[3] < case[1] or ends == "right"])
def test_mean_on_a_guess(rule, n, f, m, extra, ends):
    d = (1 << (23 if n >= 11 or m == n or 2 * m > n + 4 else 24)) + extra
    x = _rows(n, d, 7 * n + m)
    out_rows = list(range(1, 1 + n - m))  # to be left out
    if ends != "disagree":
        for r in out_rows:
            x[r] *= 30.0 + r
    else:
        # values 2^30 apart in some coordinates: their column sums are not exact
        for r in range(n):
            x[r, 1001 * r::1001 * n] *= 2.0 ** 30
    if ends == "wrong":
        # every sample (1,024 coordinates from r * (d // 8) on) shows others
        for r in range(8):
            a = r * (d // 8)
            w = x[:, a:a + 1024]
            w[out_rows] /= torch.tensor([30.0 + q for q in out_rows], device=DEV)[:, None]
            w[[n - 1 - i for i in range(len(out_rows))]] *= 100.0
    kw = {} if rule == "mda" else {"m": m}
    (out, sel), names = _kernels(lambda: getattr(gf, rule)(x, f, **kw))
    assert {"guess", "dist_ring_mean", "mean_after"} <= names
    D = _dist64(x).tolist()
    want = _mda(D, f) if rule == "mda" else _krum(D, f, m)
    assert sel.tolist() == want
    if ends != "disagree":
        assert want == [i for i in range(n) if i not in out_rows]
    assert torch.equal(out, _mean64(x, want))  # bit for bit: the same fp64 sum, rounded once
    # the call did end that way: the kernel's fp32 sums of 1,024 squares (4 in a
    # lane, then a tree) are within 16 * 2^-24, the scores' gap is wider than twice that
    picks, gap = _samples(x, f, m)
    assert gap > 2e-6
    assert gf.guessed_selections(x, f, m) == picks
    if ends == "disagree":
        assert any(p != picks[0] for p in picks)
    else:
        assert all(p == picks[0] for p in picks)
        assert (picks[0] == want) == (ends == "right")


def test_column_sums_without_a_guess():
    """The iterated rule's selection is never guessed; with n <= 12 its mean
    takes the column sums, the selected rows' sum where those are not exact."""
    n, f, m, d = 11, 2, 9, (1 << 23) + 257
    x = _rows(n, d, 5)
    x[3] *= 2.0
    x[4, ::1001] *= 2.0 ** 30
    (out, sel), names = _kernels(lambda: gf.multikrum_iterated(x, f, m))
    assert {"dist_ring_mean", "mean_complement"} <= names and "guess" not in names
    assert torch.equal(out, _mean64(x, sel.tolist()))


@pytest.mark.parametrize("n,f,d", [(5, 1, (1 << 23) + 1), (7, 1, (1 << 23) + 1),
                                   (8, 1, (1 << 24) - 3), (16, 2, (1 << 21) + 3)])
def test_every_call_sees_the_same_distances(n, f, d):
    """Two outliers, one the other's mirror image among rows that are their own:
    their scores are equal but for the order of the sums, so the rounding of the
    distances decides which one is left out, and every call decides alike."""
    for seed in range(6):
        half = _rows(n, (d + 1) // 2, 100 * n + seed)
        x = torch.cat([half, half[:, :d // 2].flip(1)], 1)
        x[n - 2] = 3.0 * _rows(1, d, 7 * n + seed)[0]
        x[n - 1] = x[n - 2].flip(0)
        m = n - f
        _, sel = gf.multikrum(x, f, m)
        assert torch.equal(gf.multikrum(x, f, m, aggregate=False)[1], sel)
        out, fixed = torch.empty(d, device=DEV), torch.empty_like(sel)
        s = torch.cuda.current_stream().cuda_stream
        assert gf.load().garfield_multikrum_noalloc(
            x.data_ptr(), n, f, d, m, out.data_ptr(), fixed.data_ptr(), s) == gf.OK
        assert torch.equal(fixed, sel)
        if f > 1:
            continue
        # the scores, as garfield_pairwise_sqdist's distances give them (the k
        # smallest of a row added as a balanced tree)
        D = gf.pairwise_sqdist(x).tolist()
        scores = []
        for i in range(n):
            s = sorted(D[i][j] for j in range(n) if j != i)[:n - f - 2]
            s += [0.0] * (16 - len(s))
            while len(s) > 1:
                s = [a + b for a, b in zip(s[::2], s[1::2])]
            scores.append((s[0], i))
        assert sel.tolist() == sorted(i for _, i in sorted(scores)[:m])


def test_out_inside_the_input_is_not_guessed():
    """A caller that lets the aggregate overwrite one of its rows gets the mean
    of the rows as they were, also where samples would mislead a guess."""
    import ctypes
    n, f, d = 11, 2, 1 << 23
    x = _rows(n, d, 9)
    x[5] *= 40.0
    x[6] *= 50.0
    want = _mean64(x, [i for i in range(n) if i not in (5, 6)])
    sel = torch.empty(n - f, dtype=torch.int32, device=DEV)
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = [ctypes.c_void_p(t.data_ptr()) for t in (x, x[2], sel)]
    code, names = _kernels(lambda: gf.load().garfield_multikrum(p[0], n, f, d, 0, p[1], p[2], s))
    assert code == gf.OK and "guess" not in names
    assert torch.equal(x[2], want)
