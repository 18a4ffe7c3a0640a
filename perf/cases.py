"""The work a user of this framework has it do, as cases that can be timed.

A case is one pass through the public entry points of the Python binding: one
integral (`integrate_request`, `integrate_noalloc`), a batch
(`integrate_batch`), a burst of requests to the serving lanes (`submit` /
`poll`), or one integral of a user's own function (`register_integrand`).
Every request takes its RNG key from the seed, and the Genz families and the
monomial their coefficients too.

`exact` forms the same estimate (the same random words, the same tree rules)
in float64 with plain torch operations, for cases that are small enough.
"""
import math

import numpy as np
import torch

from paper_1902_07916_amd import Integrator, register_integrand, request_from_dict, workloads

# Device memory of the one library context a program holds: a quarter serves
# the synchronous calls, the rest the serving lanes.
ARENA_BYTES = 32 << 30

FAMILIES = {"gauss": workloads.GAUSS, "sin_sum": workloads.SIN_SUM, "genz_osc": workloads.GENZ_OSC,
            "genz_ppeak": workloads.GENZ_PPEAK, "genz_cpeak": workloads.GENZ_CPEAK,
            "genz_gauss": workloads.GENZ_GAUSS, "monomial": workloads.MONOMIAL}

# A user's own functions: a Gaussian of width p[0] around p[1], and a damped
# wave of phase p[0] and frequency p[1].
BODIES = {
    "user_gauss": "real q = 0; for (int i = 0; i < D; ++i) { real d = x[i] - (real)p[1]; q += d * d; } "
                  "return exp(-q / (real)(2 * p[0] * p[0]));",
    "user_wave": "real t = 0; for (int i = 0; i < D; ++i) t += x[i]; "
                 "return exp(-t) * cos((real)p[0] + (real)p[1] * t);",
}


def listed():
    return [
        # the smallest call a program makes: a 3-D peak, 64 cubes, on the
        # static scratch (a tight loop that must not allocate)
        dict(name="noalloc_3d_fp64", kind="noalloc", f="genz_gauss", dim=3, lower=0.0, upper=1.0, divisions=4,
             samples=1000, trials=3, depth=2, sigma=1.0, eval="fp64"),
        # the 4-D Gaussian workload: a small integral alone, plain FP64
        dict(name="gauss4d_fp64", kind="one", f="gauss", width=0.2, dim=4, lower=-1.0, upper=1.0, divisions=4,
             samples=4096, trials=5, depth=1, sigma=1.0, eval="fp64"),
        # a client of the serving lanes with 32 requests in flight
        dict(name="serve_burst32_fp32", kind="serve", n=32, samples=4096, trials=3, depth=4, sigma=5.0, cap=1 << 18,
             roots=4096, eval="fp32"),
        # many small integrals together, few points in each cube
        dict(name="batch128_n256_fp64", kind="batch", n=128, samples=256, trials=3, depth=2, sigma=5.0, cap=1 << 16,
             roots=60_000, eval="fp64"),
        # a share of the 4096-integral Genz batch, under the serving mix's
        # level cap
        dict(name="batch64_n4096_fp32", kind="batch", n=64, samples=4096, trials=3, depth=2, sigma=5.0, cap=1 << 18,
             roots=100_000, eval="fp32"),
        # the benchmark's integral (f1 of the paper) with one refinement, in
        # both evaluation modes
        dict(name="sin6d_fp32", kind="one", f="sin_sum", dim=6, lower=0.0, upper=10.0, divisions=6, samples=16384,
             trials=5, depth=1, sigma=1.0, eval="fp32"),
        dict(name="sin6d_fp64", kind="one", f="sin_sum", dim=6, lower=0.0, upper=10.0, divisions=6, samples=16384,
             trials=5, depth=1, sigma=1.0, eval="fp64"),
        # the narrow 9-D Gaussian: a very uneven tree, long cubes
        dict(name="gauss9d_fp32", kind="one", f="gauss", width=0.02, dim=9, lower=0.0, upper=1.0, divisions=3,
             samples=65536, trials=5, depth=3, sigma=0.5, eval="fp32"),
        # the paper's f2 at its point count (3^9, odd), split into d parts per
        # axis as the paper counts
        dict(name="paper_f2_split3_fp64", kind="one", f="gauss", width=0.01, dim=9, lower=-1.0, upper=1.0,
             divisions=3, samples=19683, trials=5, depth=3, sigma=5.0, split=3, eval="fp64"),
        # a ragged point count and per-parent thresholds
        dict(name="ppeak5d_ragged_fp64", kind="one", f="genz_ppeak", dim=5, lower=0.0, upper=1.0, divisions=5,
             samples=3001, trials=4, depth=2, sigma=1.0, scope=1, eval="fp64"),
        # a user's function over 7^6 cubes, FP32
        dict(name="user_gauss6d_fp32", kind="user", f="user_gauss", dim=6, lower=0.0, upper=1.0, divisions=7,
             samples=4096, trials=3, depth=0, sigma=1.0, eval="fp32"),
        # a user's function with a refined tree and an odd point count, FP64
        dict(name="user_wave4d_fp64", kind="user", f="user_wave", dim=4, lower=0.0, upper=2.0, divisions=6,
             samples=2501, trials=4, depth=2, sigma=0.5, eval="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    ev = rng.choice(["fp32", "fp64"])
    kind = rng.choice(["one"] * 5 + ["noalloc", "batch", "batch", "serve", "user", "user"])
    if kind == "batch":
        samples, trials = _log_int(rng, 64, 4096), rng.randint(2, 5)
        n = _log_int(rng, 2, min(128, 1e6 / (samples * trials)))  # a quarter of the largest listed batch's points
        return dict(kind=kind, n=n, samples=samples, trials=trials, depth=rng.randint(0, 2),
                    sigma=rng.choice([3.0, 5.0]), cap=1 << 16, roots=_log_int(rng, 100, 6e4), eval=ev)
    if kind == "serve":
        return dict(kind=kind, n=_log_int(rng, 1, 48), samples=_log_int(rng, 500, 4096), trials=3,
                    depth=rng.randint(1, 4), sigma=rng.choice([3.0, 5.0]), cap=1 << 17, roots=_log_int(rng, 100, 4096),
                    eval="fp32")
    small = kind == "noalloc"
    dim = rng.randint(1, 6 if small else 16)
    roots = _log_int(rng, 1, 500 if small else 50_000)
    c = dict(kind=kind, dim=dim, lower=0.0, upper=1.0, divisions=max(2, int(roots ** (1.0 / dim) + 1e-9)),
             samples=_log_int(rng, 64, 4096 if small else 131072), trials=rng.randint(2, 8), depth=rng.randint(0, 3),
             sigma=rng.choice([0.5, 1.0, 3.0, 5.0]), eval=ev)
    if kind == "user":
        c["f"] = rng.choice(sorted(BODIES))
    else:
        c["f"] = rng.choice(sorted(FAMILIES))
        if c["f"] == "gauss":
            c["width"] = round(rng.uniform(0.05, 0.5), 3)
        if c["f"] == "sin_sum":
            c["upper"] = rng.choice([1.0, 10.0])
    if rng.random() < 0.25 and 3 ** dim <= 20000:
        c["split"] = 3
    if rng.random() < 0.2:
        c["scope"] = 1
    # at most about 5e9 six-dimensional points at the roots, and again at
    # each refined level
    per_cube = c["trials"] * dim / 6.0
    cubes = c["divisions"] ** dim
    c["samples"] = max(1, min(c["samples"], int(5e9 / (cubes * per_cube))))
    c["cap"] = max(cubes, 1000 if small else min(1 << 21, int(5e9 / (c["samples"] * per_cube))))
    return c


# ---------------------------------------------------------------------------
def _requests(case, seed):
    """The case's integrals as workload dicts; keys and coefficients from the seed."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":
        return workloads.genz_batch(n=case["n"], seed=seed, samples=case["samples"], trials=case["trials"],
                                    max_depth=case["depth"], sigma_mult=case["sigma"], eval=case["eval"],
                                    max_cubes_per_level=case["cap"], max_root_cubes=case["roots"])
    if case["kind"] == "serve":
        stream = workloads.serving_stream(rate=200.0, duration=1.0 + case["n"] / 100.0, seed=seed,
                                          samples=case["samples"], trials=case["trials"], max_depth=case["depth"],
                                          sigma_mult=case["sigma"], eval=case["eval"], max_root_cubes=case["roots"],
                                          max_cubes_per_level=case["cap"])
        return [w for _, w in stream[:case["n"]]]
    D, f = case["dim"], case["f"]
    if f == "gauss":
        centre = 0.5 * (case["lower"] + case["upper"])
        params = [case["width"], (math.sqrt(2 * math.pi) * case["width"]) ** -D] + [centre] * D
    elif f == "sin_sum":
        params = []
    elif f == "genz_osc":
        params = rng.uniform(0.0, 1.0, 1).tolist() + rng.uniform(0.5, 5.0, D).tolist()
    elif f == "genz_cpeak":
        params = rng.uniform(0.5, 5.0, D).tolist()
    elif f in ("genz_ppeak", "genz_gauss"):
        params = rng.uniform(0.5, 5.0, D).tolist() + rng.uniform(0.0, 1.0, D).tolist()
    elif f == "monomial":
        params = [float(v) for v in rng.integers(0, 5, D)]
    elif f == "user_gauss":
        params = [float(rng.uniform(0.1, 0.4)), float(rng.uniform(0.3, 0.7))]
    else:
        params = [float(rng.uniform(0.0, 6.0)), float(rng.uniform(1.0, 8.0))]
    return [dict(integrand=FAMILIES.get(f, -1), params=params, lower=[case["lower"]] * D, upper=[case["upper"]] * D,
                 divisions=case["divisions"], samples=case["samples"], trials=case["trials"], max_depth=case["depth"],
                 sigma_mult=case["sigma"], seed=int(rng.integers(1, 1 << 62)), eval=case["eval"],
                 split=case.get("split", 0), scope=case.get("scope", 0), max_cubes_per_level=case.get("cap", 0))]


_context = []
_user_ids = {}


def _integrator():
    """The library holds one context per process; a program opens it once."""
    if not _context:
        _context.append(Integrator(arena_bytes=ARENA_BYTES, serve=True))
    return _context[0]


def prepare(case, seed):
    zi = _integrator()
    ws = _requests(case, seed)
    if case["kind"] == "user":
        if case["f"] not in _user_ids:
            _user_ids[case["f"]] = register_integrand(BODIES[case["f"]], 2)
        ws[0]["integrand"] = _user_ids[case["f"]]
    return dict(kind=case["kind"], zi=zi, reqs=[request_from_dict(w) for w in ws])


def _values(r):
    return dict(integral=np.float64(r.integral), std=np.float64(r.std), stderr=np.float64(r.stderr),
                thr=np.array(r.thr_per_level), counts=[r.n_samples, r.n_cubes, r.flags, r.status],
                cubes=np.array(r.cubes_per_level + r.selected_per_level))


def _table(rs):
    """A batch's values as arrays, levels padded to the longest tree."""
    levels = max(r.levels_run for r in rs)
    thr = np.full((len(rs), levels), np.nan)
    cubes = np.zeros((len(rs), levels, 2), dtype=np.int64)
    for i, r in enumerate(rs):
        thr[i, :r.levels_run] = r.thr_per_level
        cubes[i, :r.levels_run, 0] = r.cubes_per_level
        cubes[i, :r.levels_run, 1] = r.selected_per_level
    return dict(integral=np.array([r.integral for r in rs]), std=np.array([r.std for r in rs]),
                stderr=np.array([r.stderr for r in rs]), thr=thr, cubes=cubes,
                counts=np.array([[r.n_samples, r.n_cubes, r.flags, r.status] for r in rs], dtype=np.int64))


def run(state):
    zi, reqs, kind = state["zi"], state["reqs"], state["kind"]
    if kind == "noalloc":
        return _values(zi.integrate_noalloc(reqs[0]))
    if kind == "batch":
        return _table(zi.integrate_batch(reqs))
    if kind == "serve":
        tickets = [zi.submit(r) for r in reqs]
        return _table([zi.poll(t, wait=True) for t in tickets])
    return _values(zi.integrate_request(reqs[0]))


def work(case):
    """Operations of the points of the root cubes (the refined levels depend
    on the draw and are not counted): per point D/4 Philox4x32-10 blocks of 40
    integer products and three-input XORs, two operations to place each
    coordinate, two to four per coordinate and a transcendental for the
    integrand, and the sum.  Nothing but the requests and the results has to
    be read or written."""
    flops = 0.0
    ws = _requests(case, 1)
    for w in ws:
        D = len(w["lower"])
        flops += float(w["divisions"]) ** D * w["trials"] * w["samples"] * (10.0 * D + 5.0 * D + 12.0)
    return dict(bytes=1400.0 * len(ws), flops=flops)


# ---------------------------------------------------------------------------
# The estimate in float64, with plain torch operations.

_M32 = 0xFFFFFFFF
_BLOCKS = 1 << 24     # Philox blocks formed at a time
_MAX_BLOCKS = 6e9     # of one case


def _philox(c0, c1, c2, c3, seed):
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64
        c0, c1, c2, c3 = ((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _f(w, name, x):
    D, p = x.shape[-1], w["params"]
    t = lambda v: torch.tensor(v, dtype=torch.float64, device=x.device)  # noqa: E731
    if name == "gauss":
        return p[1] * torch.exp(-((x - t(p[2:])) ** 2).sum(-1) / (2 * p[0] ** 2))
    if name == "sin_sum":
        return torch.sin(x.sum(-1))
    if name == "genz_osc":
        return torch.cos(2 * math.pi * p[0] + (x * t(p[1:])).sum(-1))
    if name == "genz_ppeak":
        return 1 / (t(p[:D]) ** -2 + (x - t(p[D:])) ** 2).prod(-1)
    if name == "genz_cpeak":
        return (1 + (x * t(p)).sum(-1)) ** -(D + 1)
    if name == "genz_gauss":
        return torch.exp(-((t(p[:D]) * (x - t(p[D:]))) ** 2).sum(-1))
    if name == "monomial":
        return (x ** t(p)).prod(-1)
    if name == "user_gauss":
        return torch.exp(-((x - p[1]) ** 2).sum(-1) / (2 * p[0] ** 2))
    s = x.sum(-1)
    return torch.exp(-s) * torch.cos(p[0] + p[1] * s)


def _std(v, dim):
    """Population standard deviation, deviations scaled to order one."""
    d = v - v.mean(dim, keepdim=True)
    top = d.abs().amax(dim, keepdim=True)
    return (top * ((d / torch.where(top > 0, top, 1.0)) ** 2).mean(dim, keepdim=True).sqrt()).squeeze(dim)


def _cells(w, level, uid):
    """Lattice cell of each cube on the level's grid, and the cells per axis."""
    D, d, b = len(w["lower"]), w["divisions"], w.get("split", 0) or 2
    K = torch.zeros(len(uid), D, dtype=torch.int64, device=uid.device)
    rest, mult = uid.clone(), 1
    for _ in range(level):
        c, rest = rest % b ** D, rest // b ** D
        for i in range(D - 1, -1, -1):
            K[:, i] += (c % b) * mult
            c = c // b
        mult *= b
    for i in range(D - 1, -1, -1):
        K[:, i] += (rest % d) * mult
        rest = rest // d
    return K, mult


def _estimates(w, name, level, uid):
    """m and s of each cube: mean and population std of its trials."""
    dev, D, T, N = uid.device, len(w["lower"]), w["trials"], w["samples"]
    K, parts = _cells(w, level, uid)
    lower = torch.tensor(w["lower"], dtype=torch.float64, device=dev)
    h = (torch.tensor(w["upper"], dtype=torch.float64, device=dev) - lower) / w["divisions"] / parts
    volume = float(h.prod())
    blocks = -(-N * D // 4)
    at_once = max(1, _BLOCKS // (blocks * T))
    I = torch.empty(len(uid), T, dtype=torch.float64, device=dev)
    k = torch.arange(blocks, device=dev)
    t = torch.arange(T, device=dev).view(1, T, 1)
    for a in range(0, len(uid), at_once):
        u = uid[a:a + at_once].view(-1, 1, 1)
        shape = (len(u), T, blocks)
        words = _philox(k.expand(shape), (t | (level << 8)).expand(shape), (u & _M32).expand(shape),
                        ((u >> 32) & _M32).expand(shape), w["seed"])
        n = torch.stack(words, -1).view(len(u), T, -1)[:, :, :N * D].reshape(len(u), T, N, D)
        x = lower + h * (K[a:a + at_once].view(-1, 1, 1, D) + (2 * (n >> 9) + 1).double() * 2.0 ** -24)
        I[a:a + at_once] = volume * _f(w, name, x).mean(-1)
    return I.mean(1), _std(I, 1)


def _tree(w, name, left):
    """The whole search of one integral; None if it takes over `left` blocks
    or ids above 63 bits."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    D, T, b = len(w["lower"]), w["trials"], w.get("split", 0) or 2
    kids = b ** D
    if w["divisions"] ** D * kids ** w["max_depth"] >= 1 << 63:
        return None
    cap = w.get("max_cubes_per_level", 0) or 1 << 24
    uid = torch.arange(w["divisions"] ** D, device=dev)
    M, V, thrs, used = 0.0, 0.0, [], 0.0
    for level in range(w["max_depth"] + 1):
        used += len(uid) * T * -(-w["samples"] * D // 4)
        if used > left:
            return None
        m, s = _estimates(w, name, level, uid)
        if level == w["max_depth"]:
            sel = torch.zeros_like(s, dtype=torch.bool)
            thrs.append(math.nan)
        elif w.get("scope", 0) == 1 and level > 0 and len(uid) > kids:
            g = s.view(-1, kids)
            sel = (g > (g.mean(1) + w["sigma_mult"] * _std(g, 1))[:, None]).view(-1)
            thrs.append(math.nan)
        else:
            thrs.append(float(s.mean() + w["sigma_mult"] * _std(s, 0)))
            sel = s > thrs[-1]
        n = int(sel.sum())
        every = (M + float(m.sum()), V + float((s ** 2).sum()))
        met = w.get("rtol", 0.0) > 0 and math.sqrt(every[1] / (T - 1)) <= w["rtol"] * abs(every[0])
        if n == 0 or met or n * kids > cap:
            M, V = every
            break
        M, V = M + float(m[~sel].sum()), V + float((s[~sel] ** 2).sum())
        uid = (uid[sel][:, None] * kids + torch.arange(kids, device=dev)).view(-1)
    return M, math.sqrt(V), math.sqrt(V / (T - 1)), thrs, used


def exact(case, seed):
    """What `run` returns for these inputs, in float64; None where the points
    are too many.  The whole-numbered outputs have no value here."""
    out, left = [], _MAX_BLOCKS
    for w in _requests(case, seed):
        name = case.get("f") or next(k for k, v in FAMILIES.items() if v == w["integrand"])
        r = _tree(w, name, left)
        if r is None:
            return None
        left -= r[4]
        out.append(r)
    if case["kind"] not in ("batch", "serve"):
        M, std, err, thrs, _ = out[0]
        return dict(integral=np.float64(M), std=np.float64(std), stderr=np.float64(err), thr=np.array(thrs),
                    counts=[None] * 4, cubes=None)
    thr = np.full((len(out), max(len(r[3]) for r in out)), np.nan)
    for i, r in enumerate(out):
        thr[i, :len(r[3])] = r[3]
    return dict(integral=np.array([r[0] for r in out]), std=np.array([r[1] for r in out]),
                stderr=np.array([r[2] for r in out]), thr=thr, cubes=None, counts=None)
