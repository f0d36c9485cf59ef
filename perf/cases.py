"""The work that users of this package have it do, as cases that can be timed.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (catalogues on the GPU, a plan, a batch, a model), `run` makes one
pass through the public entry points, `work` says what a pass cannot do
without, and `exact` evaluates the same definitions in 64 bits with plain
torch.  `listed` names the cases, `draw` gives more of the same ranges.

Paths:
  box     auto counts of a periodic simulation box, line of sight z
  survey  an open survey shell: data x randoms, or data and randoms to an
          estimate of the correlation function
  mocks   the counts of many catalogues, or of a list of catalogue pairs, in
          one batch
  squared the histogram update on given squared separations
  tri     triangle counts
  sky     angular counts of sky positions
  model   the work-item cost model: predictions, and gradients of its loss
"""
import math

import numpy as np
import torch

from paper_2301_12557_amd import fcfc, synth

DEV = "cuda"
SHELL_VOLUME = math.radians(60.0) * 2 * math.sin(math.radians(15.0)) * (2000.0 ** 3 - 1000.0 ** 3) / 3
SURVEY_LO, SURVEY_HI = (450.0, -1.0, -520.0), (2000.0, 1740.0, 520.0)
EXACT_PAIRS = 2.5e10   # pair separations evaluated one by one in a few seconds


def listed():
    return [
        # One call on a small uniform box: a test, a quick look, an inner loop; launches and latency.
        dict(name="box_s_20k", path="box", n=20_000, L=1000.0, kind="s", n1=40, n2=1, smax=200.0, spacing="lin",
             weighted=False, lognormal=False, onecall=True),
        # One simulation mock, the plan kept from mock to mock: (s, mu) for multipoles.
        dict(name="box_smu_mock", path="box", n=200_003, L=1000.0, kind="smu", n1=40, n2=100, smax=200.0,
             spacing="lin", weighted=False, lognormal=True, onecall=False),
        # A simulation box with per-galaxy weights: the benchmark's default step.
        dict(name="box_smu_weighted_1m", path="box", n=1_000_000, L=2000.0, kind="smu", n1=40, n2=100, smax=200.0,
             spacing="lin", weighted=True, lognormal=True, onecall=False),
        # A large sparse-pair box: many points, few neighbours each, logarithmic bins.
        dict(name="box_s_log_10m", path="box", n=10_000_000, L=3000.0, kind="s", n1=50, n2=1, smax=50.0,
             spacing="log", weighted=False, lognormal=True, onecall=False),
        # The weighted DR count of a survey, (s_perp, pi) with the mid-point line of sight: the longest calls.
        dict(name="survey_dr_spi", path="survey", nd=200_003, nr=4_000_037, kind="spi", n1=40, n2=40, smax=200.0,
             weighted=True, counts="dr", leaf=0),
        # The same kind of count through the k-d tree, unweighted and smaller.
        dict(name="survey_dr_tree", path="survey", nd=50_021, nr=1_000_003, kind="spi", n1=40, n2=40, smax=200.0,
             weighted=False, counts="dr", leaf=128),
        # A small survey from catalogues to multipoles: DD, DR, RR, the estimator, its multipoles.
        dict(name="survey_ls_smu", path="survey", nd=20_011, nr=200_017, kind="smu", n1=40, n2=100, smax=200.0,
             weighted=False, counts="ls", leaf=0),
        # Many mocks in one batch, replayed: covariance matrices.
        dict(name="mocks_smu_16", path="mocks", ncat=16, nmin=100_000, nmax=500_000, pairs=False, kind="smu", n1=40,
             n2=100, smax=200.0, weighted=False),
        # The histogram update alone, on separations that another code has formed.
        dict(name="squared_200lin", path="squared", n=1_600_000_003, n1=200, smax=200.0, spacing="lin"),
        # Triangles of a periodic box, unweighted.
        dict(name="tri_1m", path="tri", n=1_000_003, L=1000.0, n1=15, smax=30.0, weighted=False, periodic=True,
             lognormal=False),
        # Angular counts of one patch, from right ascension and declination.
        dict(name="sky_100k", path="sky", n=100_003, n1=20, tmax=5.0),
        # The cost model on the work items of one count: forward, and forward with backward.
        dict(name="model_500k", path="model", m=500_009),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["box", "box", "box", "survey", "survey", "mocks", "squared", "tri", "sky", "model"])
    if path == "box":
        kind = rng.choice(["s", "smu", "spi"])
        smax = rng.choice([50.0, 100.0, 150.0, 200.0])
        L = rng.choice([1000.0, 2000.0, 3000.0])
        n = _log_int(rng, 2_000, 10_000_000)
        c = dict(path="box", n=n, L=L, kind=kind, n1=rng.randint(10, 50),
                 n2=1 if kind == "s" else rng.randint(10, 100 if kind == "smu" else 40), smax=smax,
                 spacing=rng.choice(["lin", "log"]) if kind == "s" else "lin", weighted=rng.random() < 0.4,
                 lognormal=rng.random() < 0.6, onecall=rng.random() < 0.3)
        most = 1.5e9
        pairs = _box_pairs(c)
        if pairs > most:
            c["n"] = max(2_000, int(n * math.sqrt(most / pairs)))
        return c
    if path == "survey":
        nd = _log_int(rng, 3_000, 100_000)
        kind = rng.choice(["smu", "spi"])
        counts = rng.choice(["dr", "ls"]) if kind == "smu" else "dr"
        nr = int(nd * rng.uniform(8, 20))
        if counts == "ls":
            nd, nr = min(nd, 30_000), min(nr, 300_000)
        return dict(path="survey", nd=nd, nr=nr, kind=kind, n1=rng.randint(10, 40), n2=rng.randint(10, 40),
                    smax=rng.choice([60.0, 100.0, 150.0, 200.0]), weighted=counts == "dr" and rng.random() < 0.6,
                    counts=counts, leaf=rng.choice([0, 0, 64, 128]) if counts == "dr" else 0)
    if path == "mocks":
        pairs = rng.random() < 0.4
        kind = rng.choice(["s", "smu"])
        return dict(path="mocks", ncat=rng.randint(2, 4) if pairs else rng.randint(2, 16), nmin=_log_int(rng, 5_000, 60_000),
                    nmax=_log_int(rng, 60_000, 300_000), pairs=pairs, kind=kind, n1=rng.randint(10, 40),
                    n2=1 if kind == "s" else rng.randint(10, 100), smax=rng.choice([50.0, 100.0, 150.0]),
                    weighted=rng.random() < 0.4)
    if path == "squared":
        return dict(path="squared", n=_log_int(rng, 10_000, 1_600_000_000), n1=rng.randint(10, 400),
                    smax=rng.choice([50.0, 150.0, 200.0]), spacing=rng.choice(["lin", "log"]))
    if path == "tri":
        return dict(path="tri", n=_log_int(rng, 5_000, 1_000_000), L=1000.0, n1=rng.randint(5, 20),
                    smax=rng.choice([10.0, 20.0, 30.0]), weighted=rng.random() < 0.3, periodic=rng.random() < 0.6,
                    lognormal=rng.random() < 0.4)
    if path == "sky":
        return dict(path="sky", n=_log_int(rng, 3_000, 300_000), n1=rng.randint(10, 40), tmax=rng.choice([4.0, 5.0, 8.0, 10.0]))
    return dict(path="model", m=_log_int(rng, 10_000, 1_000_000))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + 7919 * (k + 1)) & 0x7FFFFFFFFFFFFFFF)
    return g


def _uniform(shape, lo, hi, seed, k):
    return torch.rand(shape, generator=_gen(seed, k), device=DEV, dtype=torch.float64) * (hi - lo) + lo


def _box_points(n, L, lognormal, seed, k=0):
    if lognormal:
        ngrid = 128 if n < 500_000 else 256
        return synth.lognormal_box_torch(n, L, int(seed) * 64 + k + 1, device=DEV, ngrid=ngrid)
    return _uniform((n, 3), 0.0, L, seed, k).clamp_(max=float(np.nextafter(L, 0.0))).contiguous()


def _shell_points(n, seed, k):
    """synth.survey_shell's distribution, drawn on the GPU."""
    u = _uniform((n, 3), 0.0, 1.0, seed, k)
    r = (1000.0 ** 3 + u[:, 0] * (2000.0 ** 3 - 1000.0 ** 3)) ** (1.0 / 3.0)
    ra = math.radians(60.0) * u[:, 1]
    s = math.sin(math.radians(15.0)) * (2 * u[:, 2] - 1)
    c = torch.sqrt(1 - s * s)
    return torch.stack([r * c * torch.cos(ra), r * c * torch.sin(ra), r * s], 1).contiguous()


def _edges(c):
    e1 = synth.log_edges(c["smax"] / 500.0, c["smax"], c["n1"]) if c.get("spacing") == "log" else \
        synth.linear_edges(0, c["smax"], c["n1"])
    kind = c.get("kind", "s")
    e2 = None if kind == "s" else synth.mu_edges(c["n2"]) if kind == "smu" else synth.linear_edges(0, c["smax"], c["n2"])
    return e1, e2


def _mock_sizes(c):
    m = c["ncat"]
    return [int(c["nmin"] + (c["nmax"] - c["nmin"]) * ((7 * i + 3) % m + 0.5) / m) for i in range(m)]


def _mock_pairs(c):
    m = c["ncat"]
    return [(a, b) for a in range(m) for b in range(a, m)] if c["pairs"] else [(a, a) for a in range(m)]


def _inputs(c, seed):
    """The arrays of a case, from the seed alone."""
    path = c["path"]
    s = dict(case=c)
    if path == "box":
        s["x"] = _box_points(c["n"], c["L"], c["lognormal"], seed)
        s["w"] = _uniform(c["n"], 0.5, 1.5, seed, 1) if c["weighted"] else None
    elif path == "survey":
        s["d"], s["r"] = _shell_points(c["nd"], seed, 0), _shell_points(c["nr"], seed, 1)
        s["wd"] = _uniform(c["nd"], 0.5, 2.0, seed, 2) if c["weighted"] else None
        s["wr"] = _uniform(c["nr"], 0.5, 2.0, seed, 3) if c["weighted"] else None
    elif path == "mocks":
        s["x"] = [_box_points(n, 1000.0, True, seed, k) for k, n in enumerate(_mock_sizes(c))]
        s["w"] = [_uniform(len(x), 0.5, 1.5, seed, 100 + k) if c["weighted"] else None for k, x in enumerate(s["x"])]
    elif path == "squared":
        s["s2"] = synth.s2_samples_torch(c["n"], c["smax"], int(seed) + 1, device=DEV)
    elif path == "tri":
        s["x"] = _box_points(c["n"], c["L"], c["lognormal"], seed)
        s["w"] = _uniform(c["n"], 0.5, 1.5, seed, 1) if c["weighted"] else None
    elif path == "sky":
        s["ra"] = _uniform(c["n"], 0.0, 60.0, seed, 0)
        s["dec"] = torch.rad2deg(torch.asin(_uniform(c["n"], -math.sin(math.radians(15)), math.sin(math.radians(15)), seed, 1)))
    else:
        m = c["m"]
        a = torch.floor(_uniform(m, 1.0, 129.0, seed, 0))
        b = torch.floor(torch.exp2(_uniform(m, 0.0, 14.0, seed, 1)))
        t = _uniform(m, 0.0, 3.0, seed, 2)
        k = torch.floor(_uniform(m, 1.0, 6.0, seed, 3))
        noise = torch.randn(m, generator=_gen(seed, 4), device=DEV, dtype=torch.float64)
        s["feat"] = torch.stack([torch.log2(1 + a), torch.log2(1 + b), t, k], 1).float().contiguous()
        s["target"] = (torch.log2(1 + 20 + 0.002 * a * b) + 0.2 * noise).float()
        s["params"], s["norm"] = _model_params(seed), _model_norm(s["feat"], s["target"])
    return s


def _model_params(seed):
    """He-uniform weights, small biases, packed W1 b1 W2 b2 W3 b3 W4 b4."""
    rng = np.random.default_rng(int(seed) + 11)
    parts = []
    for rows, cols in ((64, 4), (64, 64), (64, 64), (1, 64)):
        lim = math.sqrt(6.0 / cols)
        parts += [rng.uniform(-lim, lim, rows * cols), rng.uniform(-0.05, 0.05, rows)]
    return np.concatenate(parts).astype(np.float32)


def _model_norm(feat, target):
    f, t = feat.double(), target.double()
    v = torch.cat([f.mean(0), f.std(0, unbiased=False), t.mean().view(1), t.std(unbiased=False).view(1)])
    return v.float().cpu().numpy()


def prepare(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    path = c["path"]
    e1, e2 = _edges(c) if path in ("box", "survey", "mocks", "squared", "tri") else (None, None)
    if path == "box" and not c["onecall"]:
        s["plan"] = fcfc.Plan(c["kind"], e1, e2, box=c["L"], n_hint=c["n"])
    elif path == "survey":
        tune = dict(tree_leaf=c["leaf"]) if c["leaf"] else {}
        s["plan"] = fcfc.Plan(c["kind"], e1, e2, los="mid", n_hint=c["nr"], **tune)
        s["plan"].set_bounds(SURVEY_LO, SURVEY_HI)
    elif path == "mocks":
        plan = fcfc.Plan(c["kind"], e1, e2, box=1000.0, n_hint=int(np.mean(_mock_sizes(c))))
        pairs = _mock_pairs(c)
        s["batch"] = fcfc.Batch(plan, list(zip(s["x"], s["w"])), pairs=pairs if c["pairs"] else None)
        nb = len(pairs) * c["n1"] * c["n2"]
        s["out"] = torch.empty(nb, dtype=torch.int64, device=DEV)
        s["wout"] = torch.empty(nb, dtype=torch.float64, device=DEV) if c["weighted"] else None
    elif path == "squared":
        s["plan"] = fcfc.Plan("s", e1)
    elif path == "tri":
        s["plan"] = fcfc.Plan("s", e1, box=c["L"] if c["periodic"] else 0.0, n_hint=c["n"])
        if not c["periodic"]:
            s["plan"].set_bounds((0.0,) * 3, (c["L"],) * 3)
    elif path == "model":
        s["model"] = fcfc.Model(seed=0)
        s["model"].set(s["params"], s["norm"])
    s["edges"] = (e1, e2)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    return _RUN[s["case"]["path"]](s)


def _run_box(s):
    c = s["case"]
    e1, e2 = s["edges"]
    if c["onecall"]:
        return fcfc.count_pairs(s["x"], kind=c["kind"], edges1=e1, edges2=e2, box=c["L"], w1=s["w"])
    cells = s["plan"].build_cells(s["x"], s["w"])
    out = s["plan"].count(cells, weighted=c["weighted"])
    cells.close()
    return out


def _run_survey(s):
    c, plan = s["case"], s["plan"]
    cd = plan.build_cells(s["d"], s["wd"])
    cr = plan.build_cells(s["r"], s["wr"])
    if c["counts"] == "dr":
        out = plan.count(cd, cr, weighted=c["weighted"])
    else:
        dd, dr, rr = plan.count(cd)[0], plan.count(cd, cr)[0], plan.count(cr)[0]
        xi = fcfc.landy_szalay(dd, dr, rr, c["nd"], c["nr"])
        out = (dd, dr, rr, xi, fcfc.multipoles(xi, s["edges"][1], (0, 2, 4)))
    cd.close()
    cr.close()
    return out


def _run_mocks(s):
    s["batch"].run(s["out"], s["wout"])
    return s["out"], s["wout"]


def _run_squared(s):
    return s["plan"].bin_squared(s["s2"])


def _run_tri(s):
    c = s["case"]
    cells = s["plan"].build_cells(s["x"], s["w"])
    out = s["plan"].count_triplets(cells, weighted=c["weighted"])
    cells.close()
    return out


def _run_sky(s):
    u = fcfc.radec_to_unit(s["ra"], s["dec"])
    theta = synth.linear_edges(0, s["case"]["tmax"], s["case"]["n1"])
    counts, _, _ = fcfc.angular_count(u, theta_deg=theta)
    return u, counts


def _run_model(s):
    pred = s["model"].predict(s["feat"])
    grad, loss = s["model"].grad(s["feat"], s["target"])
    return pred, grad, loss


_RUN = dict(box=_run_box, survey=_run_survey, mocks=_run_mocks, squared=_run_squared, tri=_run_tri, sky=_run_sky,
            model=_run_model)


# ---------------------------------------------------------------------------
# What a pass cannot do without: catalogues read and histograms written once,
# and 8 floating-point operations for the squared separation of each pair
# that is counted (of the unclustered density; clustering adds to it).
# ---------------------------------------------------------------------------

def _reach(c):
    """Volume around a point in which its counted pairs lie."""
    return math.pi * c["smax"] ** 2 * 2 * c["smax"] if c["kind"] == "spi" else 4 / 3 * math.pi * c["smax"] ** 3


def _box_pairs(c):
    return 0.5 * c["n"] ** 2 * _reach(c) / c["L"] ** 3


def work(case):
    c = case
    path = c["path"]
    if path == "box":
        per = 32 if c["weighted"] else 24
        return dict(bytes=per * c["n"] + 16 * c["n1"] * c["n2"], flops=8 * _box_pairs(c))
    if path == "survey":
        per = 32 if c["weighted"] else 24
        pairs = c["nd"] * c["nr"]
        if c["counts"] == "ls":
            pairs += 0.5 * c["nd"] ** 2 + 0.5 * c["nr"] ** 2
        return dict(bytes=per * (c["nd"] + c["nr"]) + 48 * c["n1"] * c["n2"], flops=8 * pairs * _reach(c) / SHELL_VOLUME)
    if path == "mocks":
        n = _mock_sizes(c)
        pairs = sum(0.5 * n[a] ** 2 if a == b else n[a] * n[b] for a, b in _mock_pairs(c))
        per = 32 if c["weighted"] else 24
        return dict(bytes=per * sum(n) + 16 * len(_mock_pairs(c)) * c["n1"] * c["n2"], flops=8 * pairs * _reach(c) / 1e9)
    if path == "squared":
        return dict(bytes=8 * c["n"] + 8 * c["n1"], flops=2 * c["n"])
    if path == "tri":
        # neighbours after a point in a fixed order, and the third side of every pair of them
        m = 0.5 * c["n"] * 4 / 3 * math.pi * c["smax"] ** 3 / c["L"] ** 3
        per = 32 if c["weighted"] else 24
        return dict(bytes=per * c["n"] + 16 * c["n1"] ** 3, flops=8 * c["n"] * (m + 0.5 * m * m))
    if path == "sky":
        area = 2 * math.radians(60.0) * math.sin(math.radians(15.0))
        cap = 2 * math.pi * (1 - math.cos(math.radians(c["tmax"])))
        return dict(bytes=40 * c["n"] + 8 * c["n1"], flops=8 * 0.5 * c["n"] ** 2 * cap / area)
    fma = 4 * 64 + 2 * 64 * 64 + 64
    return dict(bytes=2 * 20 * c["m"] + 4 * 8705, flops=2 * fma * c["m"] * 4)


# ---------------------------------------------------------------------------
# The same in 64 bits with plain torch
# ---------------------------------------------------------------------------

def exact(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    path = c["path"]
    if path == "box":
        if 0.5 * c["n"] ** 2 > EXACT_PAIRS:
            return None
        return _exact_count(c, s["x"], None, s["w"], None, c["L"], "z")
    if path == "survey":
        if c["nd"] * c["nr"] + (0.5 * c["nr"] ** 2 if c["counts"] == "ls" else 0) > EXACT_PAIRS:
            return None
        if c["counts"] == "dr":
            return _exact_count(c, s["d"], s["r"], s["wd"], s["wr"], 0.0, "mid")
        dd, dr, rr = (_exact_count(c, a, b, None, None, 0.0, "mid")[0]
                      for a, b in ((s["d"], None), (s["d"], s["r"]), (s["r"], None)))
        nd, nr = c["nd"], c["nr"]
        fr = rr.double() / (0.5 * nr * (nr - 1))
        xi = (dd.double() / (0.5 * nd * (nd - 1)) - 2 * dr.double() / (nd * nr) + fr) / fr
        return dd, dr, rr, xi, _exact_multipoles(xi)
    if path == "mocks":
        if sum(len(s["x"][a]) * len(s["x"][b]) for a, b in _mock_pairs(c)) > EXACT_PAIRS:
            return None
        got = [_exact_count(c, s["x"][a], None if a == b else s["x"][b], s["w"][a], s["w"][b], 1000.0, "z")
               for a, b in _mock_pairs(c)]
        return torch.cat([g[0].view(-1) for g in got]), (torch.cat([g[1].view(-1) for g in got]) if c["weighted"] else None)
    if path == "squared":
        e = _edges(c)[0]
        E = torch.from_numpy(e * e).to(DEV)
        h = torch.zeros(c["n1"] + 2, dtype=torch.int64, device=DEV)
        for lo in range(0, c["n"], 1 << 27):
            h += torch.bincount(torch.bucketize(s["s2"][lo:lo + (1 << 27)], E, right=True), minlength=c["n1"] + 2)
        return h[1:-1].clone()
    if path == "sky":
        a, d = torch.deg2rad(s["ra"]), torch.deg2rad(s["dec"])
        u = torch.stack([torch.cos(d) * torch.cos(a), torch.cos(d) * torch.sin(a), torch.sin(d)], 1)
        if 0.5 * c["n"] ** 2 > EXACT_PAIRS:
            return u, None
        chord = 2 * np.sin(np.deg2rad(synth.linear_edges(0, c["tmax"], c["n1"])) / 2)
        cc = dict(kind="s", n1=c["n1"], n2=1, smax=float(chord[-1]), weighted=False)
        return u, _exact_count(cc, u, None, None, None, 0.0, "z", chord)[0]
    if path == "model":
        return _exact_model(s)
    return None


def _exact_count(c, x1, x2, w1, w2, L, los, e1=None):
    """Every pair, one by one: counts, and weighted counts if the case has them."""
    auto = x2 is None
    if auto:
        x2, w2 = x1, w1
    f1, e2 = _edges(c) if e1 is None else (e1, None)
    E1 = torch.from_numpy(np.asarray(f1) * np.asarray(f1)).to(DEV)
    n1, n2, kind = c["n1"], c["n2"], c["kind"]
    E2 = torch.from_numpy(e2 * e2).to(DEV) if kind == "spi" else None
    top = float(E1[-1]) if kind != "spi" else float(E1[-1] + E2[-1]) * (1 + 1e-9)
    cnt = torch.zeros(n1 * n2, dtype=torch.int64, device=DEV)
    wc = torch.zeros(n1 * n2, dtype=torch.float64, device=DEV)
    b = [x2[:, k].contiguous() for k in range(3)]
    rows = max(1, (1 << 25) // len(x2))
    for lo in range(0, len(x1), rows):
        c0 = lo if auto else 0
        a = x1[lo:lo + rows]
        d = []
        for k in range(3):
            v = a[:, k, None] - b[k][None, c0:]
            if L:
                v = torch.where(v > L / 2, v - L, torch.where(v < -L / 2, v + L, v))
            d.append(v)
        d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        m = d2 < top
        if auto:
            m &= torch.arange(len(x2) - c0, device=DEV)[None, :] > torch.arange(len(a), device=DEV)[:, None]
        i, j = torch.nonzero(m, as_tuple=True)
        d2 = d2[i, j]
        if kind == "s":
            first, second = d2, None
        else:
            if los == "z":
                p2 = d[2][i, j] ** 2
                t2 = d[0][i, j] ** 2 + d[1][i, j] ** 2 if kind == "spi" else None
            else:
                p, q = x1[lo + i], x2[c0 + j]
                l = p + q
                v = p - q
                dot = (v[:, 0] * l[:, 0] + v[:, 1] * l[:, 1]) + v[:, 2] * l[:, 2]
                ll = (l[:, 0] * l[:, 0] + l[:, 1] * l[:, 1]) + l[:, 2] * l[:, 2]
                p2 = torch.where(ll > 0, dot * dot / ll, torch.zeros_like(ll))
                t2 = (d2 - p2).clamp_min(0.0)
            first, second = (t2, p2) if kind == "spi" else (d2, p2)
        k1 = torch.bucketize(first, E1, right=True) - 1
        ok = (k1 >= 0) & (k1 < n1)
        k = k1
        if kind == "smu":
            k2 = (n2 * torch.sqrt(second / d2.clamp_min(1e-300))).floor().clamp(0, n2 - 1)
            k2 = torch.where((k2 / n2) ** 2 * d2 > second, k2 - 1, k2)
            up = (k2 + 1) / n2
            k2 = torch.where((k2 + 1 < n2) & (up * up * d2 <= second) & (d2 > 0), k2 + 1, k2).long()
            k = k1 * n2 + k2
        elif kind == "spi":
            k2 = torch.bucketize(second, E2, right=True) - 1
            ok &= (k2 >= 0) & (k2 < n2)
            k = k1 * n2 + k2
        cnt += torch.bincount(k[ok], minlength=n1 * n2)
        if c["weighted"]:
            wc += torch.bincount(k[ok], weights=(w1[lo + i] * w2[c0 + j])[ok], minlength=n1 * n2)
    shape = (n1,) if kind == "s" else (n1, n2)
    return cnt.view(shape), (wc.view(shape) if c["weighted"] else None)


def _exact_multipoles(xi):
    mu = torch.arange(xi.shape[1] + 1, device=DEV, dtype=torch.float64) / xi.shape[1]
    anti = [mu, (mu ** 3 - mu) / 2, (7 * mu ** 5 - 10 * mu ** 3 + 3 * mu) / 8]
    return torch.stack([(2 * l + 1) * (xi * (a[1:] - a[:-1])).sum(1) for l, a in zip((0, 2, 4), anti)])


def _exact_model(s):
    p = torch.from_numpy(s["params"]).double().to(DEV).requires_grad_(True)
    nm = torch.from_numpy(s["norm"]).double().to(DEV)
    h = (s["feat"].double() - nm[:4]) / nm[4:8]
    at = 0
    for rows, cols in ((64, 4), (64, 64), (64, 64), (1, 64)):
        w, b = p[at:at + rows * cols].view(rows, cols), p[at + rows * cols:at + rows * cols + rows]
        at += rows * cols + rows
        h = h @ w.t().contiguous() + b
        if rows > 1:
            h = torch.relu(h)
    y = h.view(-1)
    loss = 0.5 * ((y - (s["target"].double() - nm[8]) / nm[9]) ** 2).sum()
    g, = torch.autograd.grad(loss, p)
    return (y * nm[9] + nm[8]).detach(), g.cpu().numpy(), float(loss)
