"""The work that a program using this framework has it do, as cases to be timed.

Every case goes through the package's public entry points on inputs that are
already on the GPU, drawn from a seed by the package's own generator
(``synth``): an aggregating server or peer holds its n gradient vectors and
applies one rule per training step. ``listed()`` holds the sizes of the
benchmark and of the paper's micro-benchmark; ``draw()`` gives more of the same
ranges, with odd lengths and with fewer attackers than the rule tolerates.
``exact()`` is the same computation in plain torch, in 64 bits.
"""
import itertools
import math
import random

import torch

import paper_2010_05888_amd as gf
from paper_2010_05888_amd import synth

VGG16, RESNET50, RESNET18 = 138_357_544, 25_557_032, 11_173_962

# honest rows are N(mean, noise^2) around a shared N(0, sigma_mean^2) vector
SCALES = {"scaled_mean_-10": (1.0, 0.1), "iid": (0.0, 1.0)}


def listed():
    def case(name, kind, rule, n, f, d, attack, byz, m=0, **more):
        return dict(name=name, kind=kind, rule=rule, n=n, f=f, m=m, d=d, attack=attack, byz=byz,
                    **more)

    return [
        # the smallest model: Krum, and the median beside it, bound by latency
        case("krum_and_median_n7_d1e5", "krum+median", "krum", 7, 1, 100_000,
             "scaled_mean_-10", 1),
        # the micro-benchmark's sweep over d at n = 17, in the middle: few launches, little data
        case("multikrum_n17_d1e6", "rule", "multikrum", 17, 3, 1_000_000, "iid", 0, 14),
        # ordinary training steps of ResNet-18 and ResNet-50 gradients; in the first every
        # other row is only 8-byte aligned
        case("multikrum_n11_resnet18", "rule", "multikrum", 11, 2, RESNET18, "gaussian_1", 2, 9),
        case("mda_n10_resnet50", "rule", "mda", 10, 3, RESNET50, "offset_5x_spread", 3),
        case("bulyan_n19_resnet50", "rule", "bulyan", 19, 4, RESNET50,
             "little_is_enough_1.5", 4),
        # the micro-benchmark's sweep over n at d = 10^7, large n: MDA's search, Bulyan's rounds
        case("mda_n39_d1e7", "rule", "mda", 39, 9, 10_000_000, "iid", 0),
        case("bulyan_n63_d1e7", "rule", "bulyan", 63, 15, 10_000_000, "iid", 0),
        # the largest: the median of Multi-Krum's selection over 64 VGG-16 gradients
        case("multikrum_median_n64_vgg16", "rule", "multikrum-median", 64, 15, VGG16,
             "scaled_mean_-4+gaussian_1", 15, 49),
        # per-layer gradients of 11 workers where they lie (161 tensors, ragged)
        case("layers_multikrum_n11", "layers", "multikrum", 11, 2, RESNET18, "gaussian_1", 2, 9,
             layers=161),
        # decentralized learning: every node aggregates 17 of the 20 nodes' vectors
        case("contract_multikrum_n20", "contract", "multikrum", 20, 3, RESNET18, "gaussian_1", 3,
             14, q=17),
        case("contract_median_n20", "contract", "median", 20, 3, RESNET18, "gaussian_1", 3, q=17),
        # a Byzantine experiment's own rows, and the variance condition of the honest ones
        case("little_is_enough_variance_n19", "byzantine", "little", 19, 4, RESNET50, "iid", 0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["krum+median", "rule", "rule", "rule", "rule", "layers", "contract",
                       "byzantine"])
    attack = rng.choice(["iid", "gaussian_1", "little_is_enough_1.5", "scaled_mean_-10",
                         "offset_5x_spread"])
    c = dict(kind=kind, attack=attack, m=0)
    if kind == "krum+median":
        c.update(rule="krum", n=rng.randint(5, 12), d=_log(rng, 10_000, 1_000_000))
    elif kind == "rule":
        c["rule"] = rng.choice(["multikrum", "multikrum", "multikrum_iterated", "bulyan", "mda",
                                "median", "average", "multikrum-median"])
        c.update(n=_log(rng, 7, 39 if c["rule"] == "mda" else 64), d=_log(rng, 30_000, 30_000_000))
    elif kind == "layers":
        c.update(rule=rng.choice(["multikrum", "bulyan", "median"]), n=_log(rng, 7, 40),
                 d=_log(rng, 1_000_000, RESNET50), layers=_log(rng, 8, 200))
    elif kind == "contract":
        c.update(rule=rng.choice(["multikrum", "median", "bulyan", "mda", "average"]),
                 n=rng.randint(9, 24), d=_log(rng, 100_000, RESNET18))
        c["q"] = max(7, c["n"] - rng.randint(0, 5))
    else:
        c.update(rule=rng.choice(["little", "empire", "reverse"]), n=_log(rng, 7, 40),
                 d=_log(rng, 100_000, RESNET50))
    voters = c.get("q", c["n"])
    c["f"] = (voters - 3) // 4 or 1
    if c["rule"].startswith("multikrum") and rng.random() < 0.5:
        c["m"] = rng.randint(2, voters - c["f"])
    c["byz"] = 0 if attack == "iid" else rng.randint(1, c["f"])
    return c


def _layers(case):
    """Lengths of the layers: spread over their logarithm, their sum d."""
    k, d = case["layers"], case["d"]
    r = random.Random(k * 1_000_003 + d)
    w = [math.exp(r.uniform(math.log(64), math.log(2_400_000))) for _ in range(k)]
    cuts = [int(d * s / sum(w)) for s in itertools.accumulate(w)]
    cuts[-1] = d
    return [b - a for a, b in zip([0] + cuts[:-1], cuts)]


def _input(case, seed):
    sigma_mean, sigma_noise = SCALES.get(case["attack"], (0.01, 0.01))
    w = synth.Workload(0, "", (case["rule"],), case["n"], case["f"], case["d"], case["m"] or None,
                       seed, "gaussian_1" if case["attack"] == "iid" else case["attack"],
                       sigma_mean, sigma_noise, case["byz"])
    return synth.generate(w, "cuda", seed=seed).x


def _peers(case, seed):
    """Every node hears from itself and q - 1 others, in an order of its own."""
    r = random.Random(seed)
    rows = []
    for v in range(case["n"]):
        peers = [v] + r.sample([u for u in range(case["n"]) if u != v], case["q"] - 1)
        r.shuffle(peers)
        rows.append(peers)
    return torch.tensor(rows, dtype=torch.int32)


def prepare(case, seed):
    x = _input(case, seed)
    s = {"case": case, "x": x}
    if case["kind"] == "layers":
        lens = _layers(case)
        s["table"] = gf.SegmentTable([list(torch.split(row, lens)) for row in x])
        s["session"] = gf.Segmented(case["rule"], case["n"], case["f"], case["m"] or None)
        s["out"] = torch.empty(case["d"], device="cuda")
        s["outs"] = list(torch.split(s["out"], lens))
    elif case["kind"] == "contract":
        s["peers"] = _peers(case, seed).cuda()
        s["y"] = torch.empty_like(x)
    elif case["kind"] == "byzantine":
        s["grad"] = x[: case["n"] - case["f"]].mean(0)
    return s


PARAM = {"little": 1.5, "empire": 0.1, "reverse": -100.0}


def run(s):
    case, x = s["case"], s["x"]
    kind, rule, f, m = case["kind"], case["rule"], case["f"], case["m"] or None
    if kind == "krum+median":
        out, sel = gf.gar("krum", x, f)
        return [out, sel, gf.gar("median", x, f)[0]]
    if kind == "rule":
        out, sel = gf.gar(rule, x, f, **({"m": m} if rule.startswith("multikrum") else {}))
        return [out] if sel is None else [out, sel]
    if kind == "layers":
        seg = s["session"]
        seg.reset()
        seg.accumulate_table(s["table"])
        sel = seg.select()
        seg.aggregate_table(s["table"], s["outs"])
        return [s["out"]] if sel is None else [s["out"], sel]
    if kind == "contract":
        return [gf.contract_step(rule, x, s["peers"], f, m, out=s["y"])]
    h = case["n"] - f
    gf.attack(rule, x[:h], f, PARAM[rule], out=x[h:])
    return [x[h:], gf.variance_stats(x[:h], s["grad"])]


def _pairs(case):
    """Pairs of rows whose distances the pass needs (3 operations a coordinate each)."""
    if case["rule"] in ("median", "average"):
        return 0
    h = case["n"] - (case["f"] if case["kind"] == "byzantine" else 0)
    return h * (h - 1) // 2


def work(case):
    n, d, f = case["n"], case["d"], case["f"]
    rows_in, rows_out = n, 1
    if case["kind"] == "krum+median":
        rows_out = 2
    elif case["kind"] == "contract":
        rows_out = n
    elif case["kind"] == "byzantine":
        rows_in, rows_out = n - f + 1, f
    return {"bytes": 4 * d * (rows_in + rows_out), "flops": d * (3 * _pairs(case) + n)}


def tolerance(case):
    # one rounding to 32 bits of a 64-bit value: 2.5e-8 measured against exact(), four times that;
    # the statistics (32-bit partial sums of 16 squares, added in 64 bits) are nearer
    return {"rel": 1e-7, "max": 5e-7}


# ---------------------------------------------------------------------------
# The rules in 64 bits, as Section 3.1 of the paper defines them.
CHUNK = 1 << 20


def _distances(x):
    n, d = x.shape
    dist = torch.zeros((n, n), dtype=torch.float64, device=x.device)
    for a in range(0, d, CHUNK):
        c = x[:, a:a + CHUNK].double()
        for i in range(n - 1):
            dist[i, i + 1:] += (c[i + 1:] - c[i]).square_().sum(1)
    return (dist + dist.T).tolist()


def _scores(dist, left, f):
    k = max(len(left) - f - 2, 0)
    return sorted((math.fsum(sorted(dist[i][j] for j in left if j != i)[:k]), i) for i in left)


def _rounds(dist, n, f, rounds):
    left = list(range(n))
    for _ in range(rounds):
        left.remove(_scores(dist, left, f)[0][1])
    return sorted(set(range(n)) - set(left))


def _covered(adj, k):
    """Whether k vertices touch every edge of the graph (a dict of neighbour sets)."""
    v = max(adj, key=lambda u: len(adj[u]), default=None)
    if v is None or not adj[v]:
        return True
    if k <= 0 or sum(len(e) for e in adj.values()) > 2 * k * len(adj[v]):
        return False

    def without(gone):
        return {u: e - gone for u, e in adj.items() if u not in gone}

    return _covered(without({v}), k - 1) or \
        (len(adj[v]) <= k and _covered(without(adj[v]), k - len(adj[v])))


def _mda(dist, n, f):
    def fits(within, start):
        rest = [u for u in range(n) if u >= start and all(dist[u][w] <= limit for w in within)]
        need = n - f - len(within)
        adj = {u: {w for w in rest if dist[u][w] > limit} for u in rest}
        return len(rest) >= need and _covered(adj, len(rest) - need)

    values = sorted({dist[i][j] for i in range(n) for j in range(i)} | {0.0})
    lo, hi = 0, len(values) - 1
    while lo < hi:
        limit = values[(lo + hi) // 2]
        lo, hi = (lo, (lo + hi) // 2) if fits([], 0) else ((lo + hi) // 2 + 1, hi)
    limit, within = values[lo], []
    for v in range(n):
        if len(within) < n - f and all(dist[v][w] <= limit for w in within) \
                and fits(within + [v], v + 1):
            within.append(v)
    return within


def _select(rule, dist, n, f, m):
    m = m or n - f
    if rule == "krum":
        m = 1
    if rule in ("krum", "multikrum", "multikrum-median"):
        return sorted(i for _, i in _scores(dist, list(range(n)), f)[:m])
    if rule == "multikrum_iterated":
        return _rounds(dist, n, f, m)
    if rule == "bulyan":
        return _rounds(dist, n, f, n - 2 * f)
    return _mda(dist, n, f)


def _combine(rule, rows, f, out):
    """The rule's aggregate of the selected rows, into out (float64)."""
    for a in range(0, rows[0].numel(), CHUNK):
        c = torch.stack([r[a:a + CHUNK] for r in rows])
        if rule in ("median", "multikrum-median", "bulyan"):
            c = c.T.contiguous().sort(1).values.double()
            k = c.shape[1]
            mid = (c[:, (k - 1) // 2] + c[:, k // 2]) / 2
            if rule == "bulyan":
                near = (c - mid[:, None]).abs().sort(dim=1, stable=True).indices[:, :k - 2 * f]
                mid = c.gather(1, near).mean(1)
            out[a:a + CHUNK] = mid
        else:
            out[a:a + CHUNK] = c.double().mean(0)
    return out


def exact(case, seed):
    kind, rule, n, f, d, m = (case[k] for k in ("kind", "rule", "n", "f", "d", "m"))
    x = _input(case, seed)

    def empty(*shape):
        return torch.empty(shape, dtype=torch.float64, device="cuda")

    if kind == "byzantine":
        h = n - f
        rows, grad = empty(f, d), x[:h].mean(0).double()
        for a in range(0, d, CHUNK):
            c = x[:h, a:a + CHUNK].double()
            if rule == "reverse":
                rows[:, a:a + CHUNK] = PARAM[rule] * c[[b % h for b in range(f)]]
            elif rule == "little":
                rows[:, a:a + CHUNK] = c.mean(0) - PARAM[rule] * c.std(0, unbiased=False)
            else:
                rows[:, a:a + CHUNK] = -PARAM[rule] * c.mean(0)
        dist = _distances(x[:h])
        var = math.fsum(dist[i][j] for i in range(h) for j in range(i)) / (h * (h - 1))
        return [rows, torch.tensor([var, float(grad.square().sum())], dtype=torch.float64)]
    dist = None if rule in ("median", "average") else _distances(x)
    if kind == "contract":
        y = empty(n, d)
        for v, peers in enumerate(_peers(case, seed).tolist()):
            if dist is None:
                rows = peers
            else:
                sub = [[dist[a][b] for b in peers] for a in peers]
                rows = [peers[i] for i in _select(rule, sub, len(peers), f, m)]
            _combine(rule, [x[r] for r in rows], f, y[v])
        return [y]
    rows = list(range(n)) if dist is None else _select(rule, dist, n, f, m)
    out = _combine(rule, [x[r] for r in rows], f, empty(d))
    if kind == "krum+median":
        return [out, torch.tensor(rows), _combine("median", list(x), f, empty(d))]
    return [out] if dist is None else [out, torch.tensor(rows)]
