"""The work that users of this package have it do, as a list of cases and the ranges around them.

Seven kinds of call, each through the package's public entry points:

  sketch   SA = S A alone (Lemma 3), every family, either precision
  solve    a whole ridge solve: sketch, (optionally the statistical dimension
           estimate that sets the momentum,) M-IHS with CG or AAb_Solver inner
  dual     an under-determined problem: sketch of A^T, Dual M-IHS
  pd       a square-like problem: two-stage sketch, Primal-Dual M-IHS
  diff     the differentiable ridge layer: sketch, forward and backward
  batched  many problems with a lambda path each: the sketches, one launch

Matrices follow the package's workload recipe: A = G diag(sigma) Q with
sigma_i = exp(-rate i / d) or i^-rate, Q orthogonal, b = A x0 + 1% noise, and
lambda set from a nominal statistical dimension sd.  Q is a product of four
random Householder reflections (dense, cheap to apply at every size).
Everything is drawn on the GPU from the seed alone.
"""
import math

import numpy as np
import torch

import paper_1912_03514_amd as mihs

DEV = "cuda:0"
ROWS = 1 << 26  # entries of A drawn at a time


def listed():
    return [
        # the smallest calls: one short sketch of a matrix with odd sizes, all launches
        dict(name="sketch_gauss_1500x61", kind="sketch", sketch="gaussian", n=1500, d=61, m=200,
             m2=0, a="f64", precision="plain", decay="exp", rate=6.0),
        # a small least-squares fit solved to a tight inner tolerance: latency of the CG
        dict(name="small_gauss_4096x256", kind="solve", sketch="gaussian", n=4096, d=256, m=256,
             m2=0, a="f64", precision="plain", decay="exp", rate=6.0, sd=64.0, eps_sub=1e-8,
             tol=5e-11, inner="cg", estimate=False, sync=True),
        # an FP64 Gaussian sketch of an ordinary, ragged matrix
        dict(name="sketch_gauss_30011x700", kind="sketch", sketch="gaussian", n=30011, d=700,
             m=1400, m2=0, a="f64", precision="plain", decay="exp", rate=6.0),
        # an FP32 matrix sketched by SRHT to more than 2048 rows
        dict(name="sketch_srht_2p17x1500", kind="sketch", sketch="srht", n=1 << 17, d=1500,
             m=3000, m2=0, a="f32", precision="mixed", decay="exp", rate=8.0),
        # CountSketch of a tall FP32 matrix whose row count is no power of two
        dict(name="sketch_count_500009x1000", kind="sketch", sketch="countsketch", n=500009,
             d=1000, m=4000, m2=0, a="f32", precision="mixed", decay="exp", rate=8.0),
        # nothing known beforehand: sketch below d rows, estimate sd, set the momentum, solve
        # with the paper's AAb_Solver streaming SA
        dict(name="estimate_aab_300000x1536", kind="solve", sketch="count_gauss", n=300000,
             d=1536, m=6000, m2=1000, a="f64", precision="plain", decay="exp", rate=8.0,
             sd=250.0, eps_sub=0.1, tol=1e-11, inner="aab", estimate=True, sync=False),
        # the headline workload of bench.py
        dict(name="srht_2p18x2048", kind="solve", sketch="srht", n=1 << 18, d=2048, m=2048, m2=0,
             a="f64", precision="mixed", decay="exp", rate=8.0, sd=512.0, eps_sub=0.1, tol=1e-10,
             inner="cg", estimate=False, sync=False),
        # the largest: a wide, ill-conditioned FP32 problem, thousands of inner CG steps
        dict(name="count_2p20x4096", kind="solve", sketch="count_gauss", n=1 << 20, d=4096,
             m=8192, m2=4096, a="f32", precision="mixed", decay="poly", rate=1.5, sd=1024.0,
             eps_sub=1e-2, tol=2e-12, inner="cg", estimate=False, sync=False),
        # under-determined, the shape of the paper's Figure 4
        dict(name="dual_4096x2p16", kind="dual", sketch="srht", n=4096, d=1 << 16, m=4096,
             m2=0, a="f64", precision="mixed", decay="exp", rate=8.0, sd=462.0, eps_sub=0.1,
             tol=5e-11),
        # square-like, shaped like the paper's Figure 5
        dict(name="pd_16384x4096", kind="pd", sketch="srht", n=1 << 14, d=4096, m=2048, m2=2048,
             a="f64", precision="plain", decay="exp", rate=8.0, sd=256.0, eps_sub=0.1, tol=5e-11,
             inner="aab"),
        # the ridge layer of a network: 64 right-hand sides, forward and backward
        dict(name="diff_2p18x1024", kind="diff", sketch="srht", n=1 << 18, d=1024, m=1024, m2=0,
             a="f32", precision="plain", decay="exp", rate=8.0, sd=256.0, nrhs=64, eps_sub=1e-2,
             tol=1e-12),
        # lambda paths of many regressions of mixed sizes in one launch
        dict(name="batched_40_paths", kind="batched", sketch="gaussian", nprob=40, nlam=16,
             nmin=4096, nmax=65536, dmin=64, dmax=512, precision="mixed", rate=6.0, eps_sub=0.1,
             tol=3e-12),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _pow2(rng, lo, hi):
    return 1 << rng.randint(lo, hi)


def draw(rng):
    """One more case of the same ranges: the seven kinds, sizes over the logarithm."""
    kind = rng.choice(["sketch", "sketch", "solve", "solve", "dual", "pd", "diff", "batched"])
    if kind == "sketch":
        sketch = rng.choice(["gaussian", "srht", "countsketch", "count_gauss"])
        d = int(_log(rng, 20, 4096))
        n = int(_log(rng, 1000, (1 << 16) if sketch == "gaussian" else (1 << 28) / d))
        n = 1 << max(6, int(math.log2(n))) if sketch == "srht" else max(n, 64)
        m = max(16, min(int(_log(rng, 0.5, 4.0) * d), 8192, n))
        m2 = max(16, m // 2) if sketch == "count_gauss" else 0
        return dict(kind=kind, sketch=sketch, n=n, d=d, m=m, m2=m2, a=rng.choice(["f64", "f32"]),
                    precision=rng.choice(["plain", "mixed"]), decay="exp", rate=6.0)
    if kind == "solve":
        d = int(_log(rng, 64, 4096))
        sd = float(int(d / rng.uniform(3.5, 12.0)))
        sketch = rng.choice(["gaussian", "srht", "count_gauss"])
        top = (1 << 16) if sketch == "gaussian" else min(1 << 20, (1 << 29) // d)
        n = int(_log(rng, max(4 * d, 2000), max(top, 5 * d)))
        n = 1 << int(math.log2(n)) if sketch == "srht" else n
        # rows of the sketch the solver sees: from 3.5 sd to a little over d
        rows = max(64, int(rng.choice([3.5 * sd, 4.5 * sd, d, 1.2 * d])))
        m, m2 = (2 * rows, rows) if sketch == "count_gauss" else (rows, 0)
        if sketch == "count_gauss" and m > n // 2:
            sketch, m, m2 = "gaussian", rows, 0
        return dict(kind=kind, sketch=sketch, n=n, d=d, m=m, m2=m2, a=rng.choice(["f64", "f32"]),
                    precision=rng.choice(["plain", "mixed"]), decay="exp",
                    rate=round(rng.uniform(4.0, 8.0), 2), sd=sd, eps_sub=0.1, tol=1e-11,
                    inner=rng.choice(["cg", "cg", "aab"]), estimate=rng.random() < 0.3,
                    sync=rng.random() < 0.5)
    if kind == "dual":
        n = int(_log(rng, 300, 4096))
        d = _pow2(rng, max(13, int(math.log2(n)) + 2), 16)
        return dict(kind=kind, sketch=rng.choice(["srht", "countsketch"]), n=n, d=d,
                    m=int(rng.choice([0.6, 1.0]) * n), m2=0, a=rng.choice(["f64", "f32"]),
                    precision=rng.choice(["plain", "mixed"]), decay="exp", rate=8.0,
                    sd=float(n // 10), eps_sub=0.1, tol=1e-11)
    if kind == "pd":
        d = int(_log(rng, 500, 4096))
        n = int(_log(rng, 1.5 * d, 5 * d))
        sd = float(d // 16)
        m = int(8 * sd)
        return dict(kind=kind, sketch="gaussian", n=n, d=d, m=m, m2=m, a=rng.choice(["f64", "f32"]),
                    precision=rng.choice(["plain", "mixed"]), decay="exp", rate=8.0, sd=sd,
                    eps_sub=0.1, tol=1e-11, inner=rng.choice(["aab", "cg"]))
    if kind == "diff":
        d = int(_log(rng, 60, 1024))
        n = _pow2(rng, 13, 18)
        return dict(kind=kind, sketch="srht", n=n, d=d, m=d, m2=0, a=rng.choice(["f64", "f32"]),
                    precision="plain", decay="exp", rate=8.0, sd=float(max(4, d // 4)),
                    nrhs=rng.randint(1, 64), eps_sub=1e-2, tol=1e-12)
    dmax = int(_log(rng, 80, 512))
    nmax = int(_log(rng, 6000, 65536))
    return dict(kind=kind, sketch="gaussian", nprob=rng.randint(2, 40), nlam=16, nmin=4096,
                nmax=nmax, dmin=64, dmax=dmax, precision=rng.choice(["plain", "mixed"]), rate=6.0,
                eps_sub=0.1, tol=3e-12)


# ---- inputs ----------------------------------------------------------------------

def _sigma(decay, rate, d):
    i = np.arange(1, d + 1, dtype=np.float64)
    return np.exp(-rate * i / d) if decay == "exp" else i ** -rate


def _sd_of(sigma, lam):
    s2 = sigma * sigma
    return float(np.sum(s2 / (s2 + lam)))


def _lambda(sigma, sd):
    lo, hi = 1e-30, 1e10
    for _ in range(120):
        mid = math.sqrt(lo * hi)
        lo, hi = (mid, hi) if _sd_of(sigma, mid) > sd else (lo, mid)
    return math.sqrt(lo * hi)


def _matrix(g, n, d, sigma, dtype, padded):
    """n x d of the recipe; `padded`: rows that start on 16-byte boundaries, as a program lays out
    a matrix that it solves with more than once."""
    per = 16 // (8 if dtype == torch.float64 else 4)
    ld = (d + per - 1) // per * per if padded else d
    A = (torch.zeros if ld > d else torch.empty)((n, ld), dtype=dtype, device=DEV)[:, :d]
    sig = torch.as_tensor(sigma, device=DEV) / math.sqrt(n)
    refl = torch.randn(4, d, generator=g, dtype=torch.float64, device=DEV)
    refl /= refl.norm(dim=1, keepdim=True)
    rows = max(1, ROWS // d)
    for r0 in range(0, n, rows):
        G = torch.randn(min(rows, n - r0), d, generator=g, dtype=torch.float64, device=DEV)
        G *= sig
        for v in refl:
            G.addr_(G @ v, v, alpha=-2.0)
        A[r0:r0 + rows] = G.to(dtype)
    return A


def _apply(A, x):
    """A x in FP64, in row chunks."""
    rows = max(1, (1 << 27) // A.shape[1])
    return torch.cat([A[r:r + rows].double() @ x for r in range(0, A.shape[0], rows)])


def _adjoint(A, y):
    rows = max(1, (1 << 27) // A.shape[1])
    out = 0.0
    for r in range(0, A.shape[0], rows):
        out = out + A[r:r + rows].double().T.contiguous() @ y[r:r + rows]
    return out


def _noisy(g, y):
    e = torch.randn(y.shape, generator=g, dtype=torch.float64, device=DEV)
    return (y + 1e-2 * e * (y.norm() / math.sqrt(y.numel()))).contiguous()


def _dtype(case):
    return torch.float64 if case["a"] == "f64" else torch.float32


def _inputs(case, seed):
    """What the problem is: the matrix, the right-hand side, lambda and the sketch's seed."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    s = {"seed": (seed * 2654435761 + 7) & 0x7FFFFFFF}
    if kind == "batched":
        rng = np.random.default_rng(seed)
        s["probs"] = []
        # the sizes belong to the case, the values to the seed
        sizes = np.random.default_rng(case["nprob"])
        for _ in range(case["nprob"]):
            n = int(sizes.integers(case["nmin"], case["nmax"] + 1))
            d = int(sizes.integers(case["dmin"], case["dmax"] + 1))
            sigma = _sigma("exp", case["rate"], d)
            A = _matrix(g, n, d, sigma, torch.float64, True)
            x0 = torch.randn(d, generator=g, dtype=torch.float64, device=DEV) / math.sqrt(d)
            lams = sigma[0] ** 2 * np.logspace(-6.0, -1.0, case["nlam"])
            sds = np.array([_sd_of(sigma, float(v)) for v in lams])
            m = int(math.ceil(4.0 * sds[0]))
            beta = np.minimum(sds / m, 0.95)
            s["probs"].append(dict(A=A, b=_noisy(g, _apply(A, x0)), lams=lams, m=m, beta=beta,
                                   seed=int(rng.integers(1 << 31))))
        return s
    n, d = case["n"], case["d"]
    rows, cols = (d, n) if kind == "dual" else (n, d)
    sigma = _sigma(case["decay"], case["rate"], cols)
    s["A"] = A = _matrix(g, rows, cols, sigma, _dtype(case), kind != "sketch")
    if kind == "sketch":
        return s
    s["lam"] = _lambda(sigma, case["sd"])
    if kind == "dual":  # A is A^T here: d x n
        x0 = torch.randn(d, generator=g, dtype=torch.float64, device=DEV) / math.sqrt(d)
        s["b"] = _noisy(g, _adjoint(A, x0))
        return s
    if kind == "diff":
        x0 = torch.randn(d, case["nrhs"], generator=g, dtype=torch.float64, device=DEV)
        s["b"] = _noisy(g, _apply(A, x0 / math.sqrt(d)))
        s["gbar"] = torch.randn(d, case["nrhs"], generator=g, dtype=torch.float64, device=DEV)
        return s
    x0 = torch.randn(d, generator=g, dtype=torch.float64, device=DEV) / math.sqrt(d)
    s["b"] = _noisy(g, _apply(A, x0))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind, prec = case["kind"], case.get("precision")
    if kind == "solve":
        rows = case["m2"] or case["m"]
        s["alpha"], s["beta"] = mihs.momentum(case["sd"], rows)
        s["ws"] = mihs.SolveWorkspace(case["n"], case["d"], rows, prec, torch.device(DEV))
    elif kind == "dual":
        s["alpha"], s["beta"] = mihs.momentum(case["sd"], case["m"])
    elif kind == "pd":
        s["mom"] = (*mihs.momentum(case["sd"], case["m"]), *mihs.momentum(case["sd"], case["m2"]))
    elif kind == "diff":
        s["alpha"], s["beta"] = mihs.momentum(case["sd"], case["m"])
        s["loglam"] = torch.tensor(math.log(s["lam"]), dtype=torch.float64, device=DEV,
                                   requires_grad=True)
        s["b"].requires_grad_(True)
    elif kind == "batched":
        dt, per = (torch.float32, 4) if prec == "mixed" else (torch.float64, 2)
        need = 0
        for p in s["probs"]:
            n, d = p["A"].shape
            ld = (d + per - 1) // per * per
            p["SA"] = torch.zeros((p["m"], ld), dtype=dt, device=DEV)[:, :d]
            need = max(need, mihs.sketch_workspace_bytes(n, d, p["m"], "gaussian", prec))
        s["sketch_ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        beta = np.stack([p["beta"] for p in s["probs"]])
        s["solver"] = mihs.BatchedSolver(
            [(p["A"], p["b"], p["SA"]) for p in s["probs"]],
            torch.as_tensor(np.stack([p["lams"] for p in s["probs"]]), device=DEV),
            torch.as_tensor((1.0 - beta) ** 2, device=DEV), torch.as_tensor(beta, device=DEV),
            eps_sub=case["eps_sub"], tol=case["tol"], max_outer=400, max_inner=2000)
    return s


# ---- one pass --------------------------------------------------------------------

def run(s):
    c = s["case"]
    return globals()["_run_" + c["kind"]](s, c)


def _run_sketch(s, c):
    return mihs.mihs_sketch(s["A"], c["sketch"], c["m"], s["seed"], precision=c["precision"],
                            m2=c["m2"])


def _run_solve(s, c):
    SA = mihs.mihs_sketch(s["A"], c["sketch"], c["m"], s["seed"], precision=c["precision"],
                          m2=c["m2"])
    alpha, beta, out = s["alpha"], s["beta"], {}
    if c["estimate"]:
        sd, _ = mihs.mihs_estimate_sd(SA, s["lam"], T=4, seed=s["seed"] + 1, eps_tr=0.1)
        alpha, beta = mihs.momentum(min(max(sd, 1.0), 0.9 * SA.shape[0]), SA.shape[0])
        out["sd"] = sd
    out["x"], _ = mihs.mihs_solve(s["A"], s["b"], s["lam"], SA, alpha, beta,
                                  eps_sub=c["eps_sub"], tol=c["tol"], max_outer=300,
                                  max_inner=2000, workspace=s["ws"], sync=c["sync"],
                                  inner=c["inner"])
    return out


def _run_dual(s, c):
    SAt = mihs.mihs_sketch(s["A"], c["sketch"], c["m"], s["seed"], precision=c["precision"])
    x, nu, _ = mihs.mihs_solve_dual(s["A"], s["b"], s["lam"], SAt, s["alpha"], s["beta"],
                                    eps_sub=c["eps_sub"], tol=c["tol"], sync=False)
    return {"x": x, "nu": nu}


def _run_pd(s, c):
    Q, WQ = mihs.mihs_sketch_two_stage(s["A"], c["sketch"], c["m"], s["seed"], c["sketch"],
                                       c["m2"], s["seed"] + 1, precision=c["precision"])
    x, _ = mihs.mihs_solve_pd(s["A"], s["b"], s["lam"], Q, WQ, *s["mom"], M=25,
                              eps_sub=c["eps_sub"], tol=c["tol"], max_outer=60,
                              inner=c["inner"], sync=False)
    return x


def _run_diff(s, c):
    SA = mihs.mihs_sketch(s["A"], c["sketch"], c["m"], s["seed"], precision=c["precision"])
    kw = dict(eps_sub=c["eps_sub"], tol=c["tol"], max_outer=300)
    X = mihs.MIHSRidge.apply(s["b"], s["loglam"], s["A"], SA, s["alpha"], s["beta"], kw)
    dB, dl = torch.autograd.grad(X, (s["b"], s["loglam"]), s["gbar"])
    return {"X": X.detach(), "dB": dB, "dloglam": dl}


def _run_batched(s, c):
    for p in s["probs"]:
        mihs.mihs_sketch(p["A"], "gaussian", p["m"], p["seed"], precision=c["precision"],
                         out=p["SA"], workspace=s["sketch_ws"])
    s["solver"].run()
    return s["solver"].X_all


# ---- what a pass cannot do without -----------------------------------------------

def _sketch_work(sketch, n, d, m, m2, ea, es):
    b = n * d * ea + (m2 or m) * d * es
    f = {"gaussian": 2.0 * m * n * d, "srht": n * d * (math.log2(max(n, 2)) + 1),
         "countsketch": float(n * d), "count_gauss": n * d + 2.0 * m * m2 * d}[sketch]
    return b, f


def work(case):
    """A is read once by the sketch and once in every outer iteration, of which Corollary 4's
    rate sqrt(sd / m) needs ln(tol) / ln(rate); the sketch is read once."""
    kind = case["kind"]
    es = 4 if case["precision"] == "mixed" else 8
    if kind == "batched":
        sizes = np.random.default_rng(case["nprob"])
        b = f = 0.0
        for _ in range(case["nprob"]):
            n = int(sizes.integers(case["nmin"], case["nmax"] + 1))
            d = int(sizes.integers(case["dmin"], case["dmax"] + 1))
            its = math.ceil(math.log(case["tol"]) / math.log(0.5))
            m = d  # about 4 sd
            b += n * d * 8 * (1 + its) + m * d * es
            f += 2.0 * m * n * d + its * 4.0 * n * d * case["nlam"]
        return {"bytes": b, "flops": f}
    ea = 8 if case["a"] == "f64" else 4
    n, d, m, m2 = case["n"], case["d"], case["m"], case["m2"]
    if kind == "dual":
        n, d = d, n
    if kind == "pd":
        b, f = _sketch_work(case["sketch"], n, d, m, 0, ea, es)
        b2, f2 = _sketch_work(case["sketch"], d, m, m2, 0, es, es)
        its = math.ceil(math.log(case["tol"]) / math.log(math.sqrt(case["sd"] / m)))
        b += b2 + its * (n * d * ea + 25 * d * m * es)
        return {"bytes": b, "flops": f + f2 + its * (4.0 * n * d + 25 * 4.0 * d * m)}
    b, f = _sketch_work(case["sketch"], n, d, m, m2, ea, es)
    if kind == "sketch":
        return {"bytes": b, "flops": f}
    rows = m2 or m
    its = math.ceil(math.log(case["tol"]) / math.log(math.sqrt(case["sd"] / rows)))
    k = 2 * case["nrhs"] if kind == "diff" else 1
    # right-hand sides share a pass over A, sixteen at a time
    passes = its * ((k + 15) // 16)
    b += passes * n * d * ea + rows * d * es
    return {"bytes": b, "flops": f + its * k * 4.0 * n * d}


# ---- the same results in 64 bits, without the package ----------------------------

M32 = 0xFFFFFFFF


def _murmur(keys, seed):
    """MurmurHash3_x86_32 of 4-byte keys (int64 tensors holding 32-bit values)."""
    def rotl(x, r):
        return ((x << r) | (x >> (32 - r))) & M32
    k = rotl((keys * 0xCC9E2D51) & M32, 15)
    h = rotl((k * 0x1B873593) & M32 ^ (seed & M32), 13)
    h = ((h * 5 + 0xE6546B64) & M32) ^ 4
    h = ((h ^ (h >> 16)) * 0x85EBCA6B) & M32
    h = ((h ^ (h >> 13)) * 0xC2B2AE35) & M32
    return h ^ (h >> 16)


def _mul32(a, c):
    """High and low 32 bits of a * c for 32-bit a, c without leaving int64."""
    p = (a & 0xFFFF) * c
    q = (a >> 16) * c + (p >> 16)
    return (q >> 16) & M32, ((q & 0xFFFF) << 16) | (p & 0xFFFF)


def _gaussian_rows(r0, r1, n, seed, stream):
    """Rows r0..r1 of the standard normal matrix of n columns: Philox-4x32-10 blocks of four
    entries and Box-Muller."""
    first, last = r0 * n, r1 * n
    blk = torch.arange(first // 4, (last + 3) // 4, dtype=torch.int64, device=DEV)
    c0, c1 = blk & M32, blk >> 32
    c2, c3 = torch.full_like(blk, stream), torch.zeros_like(blk)
    k0, k1 = seed & M32, 0
    for _ in range(10):
        h0, l0 = _mul32(c0, 0xD2511F53)
        h1, l1 = _mul32(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    z = []
    for a, b in ((c0, c1), (c2, c3)):
        rad = torch.sqrt(-2.0 * torch.log((a.double() + 0.5) * 2.0 ** -32))
        ang = 2.0 * math.pi * ((b.double() + 0.5) * 2.0 ** -32)
        z += [rad * torch.cos(ang), rad * torch.sin(ang)]
    z = torch.stack(z, dim=1).reshape(-1)
    return z[first % 4:first % 4 + last - first].reshape(r1 - r0, n)


def _exact_gaussian(A, m, seed, stream):
    n, d = A.shape
    A = A.double()
    out = torch.empty((m, d), dtype=torch.float64, device=DEV)
    rows = max(1, (1 << 24) // n)
    for r in range(0, m, rows):
        out[r:r + rows] = _gaussian_rows(r, min(m, r + rows), n, seed, stream) @ A
    return out / math.sqrt(m)


def _exact_sketch(A, sketch, m, m2, seed):
    n, d = A.shape
    if sketch == "gaussian":
        return _exact_gaussian(A, m, seed, 0)
    h = _murmur(torch.arange(n, dtype=torch.int64, device=DEV), seed)
    sign = 1.0 - 2.0 * (h >> 31).double()
    if sketch in ("countsketch", "count_gauss"):
        CA = torch.zeros((m, d), dtype=torch.float64, device=DEV)
        rows = max(1, (1 << 27) // d)
        for r in range(0, n, rows):
            CA.index_add_(0, (h % m)[r:r + rows], A[r:r + rows].double() * sign[r:r + rows, None])
        return CA if sketch == "countsketch" else _exact_gaussian(CA, m2, seed, 1)
    k = _murmur(torch.arange(m, dtype=torch.int64, device=DEV), seed + 0x9E3779B9) & (n - 1)
    out = torch.zeros((m, d), dtype=torch.float64, device=DEV)
    rows = max(1, (1 << 26) // max(m, d))
    for r in range(0, n, rows):
        i = torch.arange(r, min(n, r + rows), dtype=torch.int64, device=DEV)
        v = k[:, None] & i[None, :]
        for sh in (16, 8, 4, 2, 1):
            v = v ^ (v >> sh)
        H = (1 - 2 * (v & 1)).double() * sign[None, r:r + rows]
        out += H @ A[r:r + rows].double()
    return out / math.sqrt(m)


def _ridge(A, lam, B=None, rhs=None):
    """(A^T A + lam I)^-1 (A^T B, or rhs) by Cholesky with two steps of refinement; B or rhs with
    one column per system.  Returns the solution and a solver for more right-hand sides."""
    d = A.shape[1]
    H = torch.zeros((d, d), dtype=torch.float64, device=DEV)
    rows = max(1, (1 << 27) // d)
    for r in range(0, A.shape[0], rows):
        C = A[r:r + rows].double()
        H += C.T.contiguous() @ C
    H += lam * torch.eye(d, dtype=torch.float64, device=DEV)
    L = torch.linalg.cholesky(H)
    del H

    def solve(B, rhs):
        x = torch.zeros((d, (B if B is not None else rhs).shape[1]), dtype=torch.float64, device=DEV)
        for _ in range(3):
            g = -_adjoint(A, _apply(A, x)) + rhs if B is None else _adjoint(A, B - _apply(A, x))
            x = x + torch.cholesky_solve(g - lam * x, L)
        return x
    return solve(B, rhs), solve


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "sketch":
        return _exact_sketch(s["A"], case["sketch"], case["m"], case["m2"], s["seed"])
    if kind == "batched":
        out = []
        for p in s["probs"]:
            xs = [_ridge(p["A"], float(v), B=p["b"][:, None])[0] for v in p["lams"]]
            out.append(torch.cat(xs, dim=1).reshape(-1))
        return torch.cat(out)
    if kind == "dual":
        nu, _ = _ridge(s["A"], s["lam"], rhs=s["b"][:, None])
        return {"x": _apply(s["A"], nu)[:, 0], "nu": nu[:, 0]}
    if kind == "diff":
        X, solve = _ridge(s["A"], s["lam"], B=s["b"])
        W = solve(None, s["gbar"])
        return {"X": X, "dB": _apply(s["A"], W), "dloglam": -s["lam"] * (X * W).sum()}
    x = _ridge(s["A"], s["lam"], B=s["b"][:, None])[0][:, 0]
    if kind == "pd":
        return x
    return {"sd": None, "x": x} if case["estimate"] else {"x": x}
