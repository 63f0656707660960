"""Timed cases of Tr(A^-1) by hierarchical probing on one GPU.

Each case is one call that a program of this library makes: a trace
estimate on a prepared operator (``trace``), the same in one shot from plain
device arrays (``oneshot``), a differentiable estimate with its backward pass
(``grad``), many tori solved together (``batch``), and the operator itself
(``apply``).  Sizes are the library's own workloads (``bench.py``, ``tests/``)
and generic ones between and around them.

``exact`` recomputes every output in 64 bits with plain torch, sharing no code
with the library: the probes from site indices, the operator from rolled
arrays, CG far below the library's tolerance.
"""

import math

import numpy as np
import torch

from paper_1302_4018_amd import autograd as tip_autograd
from paper_1302_4018_amd import binding as tip

SQRT3_2 = 0.8660254037844386          # nearest double to sqrt(3)/2
_KINDS = {"scalar": tip.KIND_SCALAR, "covariant": tip.KIND_COVARIANT}
_MASKS = {"none": tip.MASK_NONE, "z2": tip.MASK_Z2, "z4": tip.MASK_Z4}
_PRECISIONS = {"fp64": tip.PREC_FP64, "mixed": tip.PREC_MIXED}
_PROBES = {"hierarchical": tip.PROBE_HIERARCHICAL, "random": tip.PROBE_RANDOM}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _trace(kind, dims, probes, *, do="trace", precision="fp64", mass=0.1, mass_sigma=0.0, weighted=False, tol=1e-10,
           mask=None, probe="hierarchical"):
    return {"do": do, "kind": kind, "dims": dims, "probes": probes, "precision": precision, "mass": mass,
            "mass_sigma": mass_sigma, "weighted": weighted, "tol": tol,
            "mask": mask or ("z4" if kind == "covariant" else "z2"), "probe": probe}


def _batch(count, precision):
    return {"do": "batch", "kind": "scalar", "count": count, "precision": precision, "tol": 1e-10}


def _apply(kind, dims, nrhs, weighted=False):
    return {"do": "apply", "kind": kind, "dims": dims, "nrhs": nrhs, "mass": 0.1, "mass_sigma": 0.02,
            "weighted": weighted}


def listed():
    return [
        # smallest: every site of a small 2-D torus probed, the exact-recovery check and the
        # call a parameter scan makes thousands of times; latency decides
        {"name": "scalar_16x16_all", **_trace("scalar", "16x16", 256, tol=1e-12)},
        # ordinary 3-D scalar problem: weighted 32^3, 512 probes
        {"name": "scalar_32c_w", **_trace("scalar", "32x32x32", 512, mass=0.05, weighted=True)},
        # scalar problem too large for any one cache: weighted 128^3, one block of probes
        {"name": "scalar_128c_w", **_trace("scalar", "128x128x128", 32, mass=0.05, weighted=True)},
        # ordinary covariant problem, 16^4 with 3 colours, in both precisions
        {"name": "cov_16q", **_trace("covariant", "16x16x16x16", 64)},
        {"name": "cov_16q_mixed", **_trace("covariant", "16x16x16x16", 64, precision="mixed")},
        # the headline operator, 32^4 with 3 colours and a mass field, in both precisions
        {"name": "cov_32q", **_trace("covariant", "32x32x32x32", 32, mass_sigma=0.02)},
        {"name": "cov_32q_mixed", **_trace("covariant", "32x32x32x32", 32, mass_sigma=0.02, precision="mixed")},
        # many uneven 3-D tori (sides 8..48, 16..256 probes each) in one call, in both precisions
        {"name": "tori_16", **_batch(16, "fp64")},
        {"name": "tori_16_mixed", **_batch(16, "mixed")},
        # one ragged torus, odd sides, a probe count that is no power of two, no prepared handle
        {"name": "scalar_odd_oneshot", **_trace("scalar", "21x34x15", 50, do="oneshot", weighted=True)},
        # training through the estimate: forward and backward for mass and couplings
        {"name": "cov_8q_grad", **_trace("covariant", "8x8x8x8", 64, do="grad", mass_sigma=0.02, weighted=True)},
        # the operator alone on sides that are no powers of two
        {"name": "cov_apply", **_apply("covariant", "12x10x14x16", 12)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _volume(dims):
    return math.prod(dims)


def _cost(case):
    """Solver work of a case in site x rhs x iteration units: a covariant site counts as 9 real scalar ones, a complex
    scalar one as 2, one of a torus that is not marched along powers of two twice."""
    if case["do"] == "apply":
        return _rhs(case) * _volume(_dims(case)) * 9
    unit = 9 if case["kind"] == "covariant" else 2 if case.get("mask") == "z4" else 1
    return sum(n * _volume(d) * unit * _iterations(case, d) * (1 if all(k & (k - 1) == 0 for k in d) else 2)
               for d, n in _problems(case))


def draw(rng):
    """One more case of the listed ranges: powers of two and odd sides, small to large, every option."""
    limit = _cost(next(c for c in listed() if c["name"] == "cov_32q"))
    while True:
        do = rng.choice(["trace", "trace", "trace", "trace", "oneshot", "grad", "batch", "apply"])
        if do == "batch":
            case = _batch(rng.randint(2, 24), rng.choice(["fp64", "mixed"]))
        else:
            kind = rng.choice(["scalar", "covariant"])
            nd = rng.choice([2, 3, 3, 4]) if kind == "scalar" else rng.choice([3, 4, 4, 4])
            top = {2: 512, 3: 128, 4: 32}[nd]
            if do in ("trace", "grad") and rng.random() < 0.7:
                dims = [2 ** rng.randint(2, int(math.log2(top))) for _ in range(nd)]
            else:
                dims = [_log_int(rng, 4, top) for _ in range(nd)]
            if not 64 <= _volume(dims) <= (1 << 20 if kind == "covariant" else 1 << 21):
                continue
            text = "x".join(map(str, dims))
            if do == "apply":
                case = _apply(kind, text, _log_int(rng, 1, 32), rng.random() < 0.5)
            else:
                probes = min(_volume(dims), _log_int(rng, 4, 512))
                case = _trace(kind, text, probes, do=do, precision=rng.choice(["fp64", "fp64", "mixed"]) if do != "grad" else "fp64",
                              mass=round(math.exp(rng.uniform(math.log(0.03), math.log(0.3))), 4),
                              mass_sigma=0.005 if rng.random() < 0.4 or do == "grad" else 0.0,
                              weighted=rng.random() < 0.5 or do == "grad",
                              mask=rng.choice(["z2", "z4"]), probe=rng.choice(["hierarchical"] * 4 + ["random"]))
        if _cost(case) <= limit:
            return case


# ---------------------------------------------------------------------------
# inputs, on the GPU, from the seed alone
# ---------------------------------------------------------------------------

def _dims(case):
    return [int(t) for t in case["dims"].split("x")]


def _ncomp(case):
    return 3 if case["kind"] == "covariant" else 1


def _rhs(case):
    return case["nrhs"] if case["do"] == "apply" else case["probes"] * _ncomp(case)


def _tori(case):
    """Sides and probe counts of a batch: the same for every seed, so that a case is one amount of work."""
    rng = np.random.default_rng(1305 + case["count"])
    sides = rng.integers(8, 49, size=(case["count"], 3))
    nvec = 2 ** rng.integers(4, 9, size=case["count"])
    return [([int(v) for v in s], int(n)) for s, n in zip(sides, nvec)]


def _problems(case):
    if case["do"] == "batch":
        return _tori(case)
    return [(_dims(case), _rhs(case))]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _haar_links(n, g):
    """n Haar-random U(3) matrices: Gram-Schmidt on complex Gaussian columns (positive diagonal of R)."""
    z = torch.randn(n, 3, 3, dtype=torch.complex128, device="cuda", generator=g)
    cols = []
    for j in range(3):
        v = z[:, :, j]
        for _ in range(2):
            for u in cols:
                v = v - (u.conj() * v).sum(1, keepdim=True) * u
        cols.append(v / v.abs().square().sum(1, keepdim=True).sqrt())
    return torch.stack(cols, dim=2).contiguous()


def _fields(case, dims, g, mass):
    """(mass_field, coupling, links): None where the case has none."""
    nd, V = len(dims), _volume(dims)
    mf = None
    if case.get("mass_sigma"):
        xi = torch.randn(V, dtype=torch.float64, device="cuda", generator=g).clamp(-3, 3)
        mf = mass + case["mass_sigma"] * xi
    w = 0.5 + torch.rand(nd, V, dtype=torch.float64, device="cuda", generator=g) if case.get("weighted") else None
    U = _haar_links(nd * V, g).reshape(nd, V, 3, 3) if case["kind"] == "covariant" else None
    return mf, w, U


def _inputs(case, seed):
    """Per problem: dims, number of probes or rhs, mass, mass_field, coupling, links; and the input vectors of `apply`."""
    g = _generator(seed)
    if case["do"] == "batch":
        rng = np.random.default_rng(int(seed))
        masses = rng.uniform(0.02, 0.2, size=case["count"])
        return [(dims, n, float(m), *_fields({**case, "weighted": True}, dims, g, m))
                for (dims, n), m in zip(_tori(case), masses)], None
    dims = _dims(case)
    fields = _fields(case, dims, g, case["mass"])
    x = None
    if case["do"] == "apply":
        shape = (case["nrhs"], _volume(dims))
        x = (torch.randn(*shape, 3, dtype=torch.complex128, device="cuda", generator=g) if case["kind"] == "covariant"
             else torch.randn(*shape, dtype=torch.float64, device="cuda", generator=g))
    return [(dims, case.get("probes", 0), case["mass"], *fields)], x


def _mask_seed(seed):
    return 4018 + int(seed)


def prepare(case, seed):
    problems, x = _inputs(case, seed)
    ops = [tip.Operator(dims, _KINDS[case["kind"]], mass=mass, mass_field=mf, coupling=w, links=U)
           for dims, _, mass, mf, w, U in problems]
    state = {"case": case, "seed": _mask_seed(seed), "ops": ops, "probes": [p[1] for p in problems], "x": x}
    if case["do"] == "trace":
        state["handle"] = tip.OpHandle(ops[0])
    if case["do"] == "grad":
        dims, _, mass, mf, w, U = problems[0]
        state["mass_field"] = mf.requires_grad_(True)
        state["coupling"] = w.requires_grad_(True)
        state["links"] = U
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    do = case["do"]
    if do == "apply":
        return tip.tip_apply_operator(state["ops"][0], state["x"])
    precision = _PRECISIONS[case["precision"]]
    if do == "batch":
        out = tip.trace_inv_probe_batch(state["ops"], state["probes"], case["tol"], state["seed"], mask=tip.MASK_Z2,
                                        precision=precision)
        return [{"estimates": est, "quadratures": st["quadratures"]} for est, st in out]
    mask = _MASKS[case["mask"]]
    if do == "grad":
        T = tip_autograd.trace_inv(state["mass_field"], state["coupling"], state["links"], dims=state["ops"][0].dims,
                                   kind=_KINDS[case["kind"]], n_vectors=case["probes"], tol=case["tol"],
                                   seed=state["seed"], mask=mask, precision=precision)
        gm, gw = torch.autograd.grad(T, (state["mass_field"], state["coupling"]))
        return {"estimate": T.detach(), "grad_mass": gm, "grad_coupling": gw}
    kw = dict(mask=mask, precision=precision, probe=_PROBES[case["probe"]])
    if do == "trace":
        est, q, _ = state["handle"].trace_inv_probe(case["probes"], case["tol"], state["seed"], **kw)
    else:
        est, q, _ = tip.trace_inv_probe(state["ops"][0], case["probes"], case["tol"], state["seed"], **kw)
    return {"estimates": est, "quadratures": q}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _iterations(case, dims):
    """CG iterations to the tolerance: half the Chebyshev bound on even sides (even-odd reduction), the bound on odd
    ones.  A Haar-random covariant hop has the spectrum of a tree, |hop| <= 2 sqrt(2d - 1)."""
    d = len(dims)
    m = case.get("mass", 0.08)
    edge = 2.0 * math.sqrt(2 * d - 1) if case["kind"] == "covariant" else 2.0 * d
    kappa = (2 * d + m + edge) / (2 * d + m - edge)
    it = 0.5 * math.sqrt(kappa) * math.log(2.0 / case["tol"])
    if all(n % 2 == 0 for n in dims):
        it *= 0.5
    return max(1, min(int(it), _volume(dims)))


def work(case):
    """Inputs read once, outputs written once; the operator applications and vector updates of the solves."""
    nc = _ncomp(case)
    real = case["kind"] == "scalar" and case.get("mask", "z2") != "z4"
    esz = 8 if real else 16
    bytes_, flops = 0.0, 0.0
    for dims, n in _problems(case):
        V, d = _volume(dims), len(dims)
        field = (d * 9 * 16 if nc == 3 else 0) + (8 * d if case.get("weighted") or case["do"] == "batch" else 0)
        field += 8 if case.get("mass_sigma") else 0
        bytes_ += field * V
        hop = 2 * d * (66 + 6 if nc == 3 else (2 if real else 4))       # one operator application, per site
        vec = nc * (1 if real else 2) * 10                               # x, r, p updates and two dot products
        if case["do"] == "apply":
            bytes_ += 2.0 * n * V * nc * esz
            flops += n * V * hop
            continue
        even = all(k % 2 == 0 for k in dims)
        flops += float(n) * V * _iterations(case, dims) * (hop + (0.5 if even else 1.0) * vec)
        bytes_ += 16.0 * n
        if case["do"] == "grad":
            bytes_ += 8.0 * V * (d + 1)
            flops += float(n) * V * (hop + vec)
    return {"bytes": bytes_, "flops": flops}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, from plain torch
# ---------------------------------------------------------------------------

def _coordinates(dims):
    s = torch.arange(_volume(dims), device="cuda")
    x = []
    for n in dims:
        x.append(s % n)
        s = s // n
    return x


def _popparity(v):
    for k in (32, 16, 8, 4, 2, 1):
        v = v ^ (v >> k)
    return v & 1


def _bitrev(m, bits):
    r = 0
    for _ in range(bits):
        r, m = (r << 1) | (m & 1), m >> 1
    return r


class _Colours:
    """Colour of every site: binary levels (bit m of every side that still has a factor two, first side most
    significant, through the Red-Black order), then one three-colouring level when a side has an odd factor."""

    def __init__(self, dims):
        x = _coordinates(dims)
        two = [(n & -n).bit_length() - 1 for n in dims]
        odd = [k for n, k in zip(dims, two) if n >> k > 1]
        self.levels = min(odd) if odd else max(two)
        self.bits, self.P = 0, torch.zeros_like(x[0])
        for m in range(self.levels):
            active = [j for j in range(len(dims)) if two[j] > m]
            idx = torch.zeros_like(x[0])
            for j in active:
                idx = (idx << 1) | ((x[j] >> m) & 1)
            a = len(active)
            self.P = (self.P << a) | (idx >> 1) | (_popparity(idx) << (a - 1))
            self.bits += a
        self.three = None
        if odd:
            c = torch.zeros_like(x[0])
            for j, n in enumerate(dims):
                sub = n >> self.levels
                if sub > 1:
                    y = x[j] >> self.levels
                    c = c + y + (((y == sub - 1) & ((sub - 1) % 3 == 0)).long())
            self.three = c % 3
        self.gamma = (1 << self.bits) * (3 if odd else 1)


def _i64(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _splitmix(seed, n):
    z = (n + 1) * _i64(0x9E3779B97F4A7C15) + _i64(seed % (1 << 64))
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _probe(col, dims, ncomp, mask, seed, m, comp, kind):
    """b_{m,comp} at every site (complex128)."""
    V = _volume(dims)
    if kind == "random":
        sweep, sign, j3 = m, torch.ones(V, dtype=torch.float64, device="cuda"), 0
    else:
        sweep, j = divmod(m, col.gamma)
        j3 = j >> col.bits
        sign = 1.0 - 2.0 * _popparity(col.P & _bitrev(j & ((1 << col.bits) - 1), col.bits)).double()
    n = (sweep * V + torch.arange(V, device="cuda")) * ncomp + comp
    u = _splitmix(seed, n)
    unit = torch.tensor([1, 1j, -1, -1j], dtype=torch.complex128, device="cuda")
    if mask == "z4":
        z = unit[_shr(u, 62)]
    elif mask == "z2":
        z = unit[_shr(u, 63) * 2]
    else:
        z = unit[torch.zeros_like(u)]
    z = z * sign
    if j3:
        w = torch.tensor([1, complex(-0.5, SQRT3_2), complex(-0.5, -SQRT3_2)], dtype=torch.complex128, device="cuda")
        z = z * w[(col.three * j3) % 3]
    return z


class _Dense:
    """A on arrays x [ncomp][rhs][n_d]...[n_1] by rolls."""

    def __init__(self, dims, mass, mf, w, U):
        self.dims, self.nd = dims, len(dims)
        shape = list(reversed(dims))
        self.mf = (torch.full(shape, mass, dtype=torch.float64, device="cuda") if mf is None else mf.detach().reshape(shape))
        self.w = [None if w is None else w.detach()[mu].reshape(shape) for mu in range(self.nd)]
        self.U = None if U is None else [[[U[mu, :, a, b].reshape(shape).contiguous() for b in range(3)] for a in range(3)]
                                         for mu in range(self.nd)]
        d = self.mf.clone()
        for mu in range(self.nd):
            wm = torch.ones_like(d) if self.w[mu] is None else self.w[mu]
            d += wm + torch.roll(wm, 1, self.axis(mu))
        self.diag = d

    def axis(self, mu):
        return -1 - mu

    def link(self, mu, x, dagger):
        """U_mu x or U_mu^H x at each site, times the coupling."""
        if self.U is None:
            y = [x[0]]
        else:
            y = []
            for a in range(3):
                t = None
                for b in range(3):
                    u = self.U[mu][b][a].conj() if dagger else self.U[mu][a][b]
                    t = u * x[b] if t is None else t.addcmul_(u.expand_as(x[b]), x[b])
                y.append(t)
        return y if self.w[mu] is None else [self.w[mu] * v for v in y]

    def __call__(self, x):
        y = [self.diag * v for v in x]
        for mu in range(self.nd):
            ax = self.axis(mu)
            for c, v in enumerate(self.link(mu, [torch.roll(t, -1, ax) for t in x], False)):
                y[c] -= v
            for c, v in enumerate(self.link(mu, x, True)):
                y[c] -= torch.roll(v, 1, ax)
        return y


def _dot(a, b):
    """Per right-hand side sum over components and sites of conj(a) b."""
    return sum((u.conj() * v).flatten(1).sum(1) for u, v in zip(a, b))


def _solve(A, b, tol=1e-13):
    """CG on every right-hand side; returns x and b - A x."""
    col = lambda s: s.reshape(-1, *([1] * A.nd))                       # noqa: E731
    x = [torch.zeros_like(v) for v in b]
    r, p = [v.clone() for v in b], [v.clone() for v in b]
    rho = _dot(r, r).real
    stop = tol * tol * rho
    for _ in range(5000):
        w = A(p)
        pw = _dot(p, w).real
        alpha = torch.where(rho > stop, rho / pw, torch.zeros_like(rho))
        for c in range(len(b)):
            x[c] += col(alpha) * p[c]
            r[c] -= col(alpha) * w[c]
        new = _dot(r, r).real
        beta = torch.where(rho > stop, new / rho, torch.zeros_like(rho))
        rho = torch.where(rho > stop, new, rho)
        if bool((rho <= stop).all()):
            break
        for c in range(len(b)):
            p[c] = r[c] + col(beta) * p[c]
    Ax = A(x)
    return x, [u - v for u, v in zip(b, Ax)]


def _quadratures(case, problem, seed, mask, grad=False):
    """q_m of one problem and, with grad, the sums over right-hand sides of the two gradients."""
    dims, probes, mass, mf, w, U = problem
    nc, V = (3 if U is not None else 1), _volume(dims)
    A, col = _Dense(dims, mass, mf, w, U), _Colours(dims)
    shape = list(reversed(dims))
    pairs = [(m, c) for m in range(probes) for c in range(nc)]
    real = nc == 1 and mask != "z4" and (col.three is None or probes <= 1 << col.bits or case.get("probe") == "random")
    step = max(1, (1 << 26) // (V * nc))
    q = torch.zeros(probes, dtype=torch.complex128, device="cuda")
    gm, gw = torch.zeros(V, dtype=torch.float64, device="cuda"), torch.zeros(len(dims), V, dtype=torch.float64, device="cuda")
    for k in range(0, len(pairs), step):
        part = pairs[k:k + step]
        b = [torch.zeros(len(part), V, dtype=torch.complex128, device="cuda") for _ in range(nc)]
        for i, (m, c) in enumerate(part):
            b[c][i] = _probe(col, dims, nc, mask, _mask_seed(seed), m, c, case.get("probe", "hierarchical"))
        b = [(v.real.contiguous() if real else v).reshape(-1, *shape) for v in b]
        x, r = _solve(A, b)
        q.index_add_(0, torch.tensor([m for m, _ in part], device="cuda"), (_dot(b, x) + _dot(x, r)).to(torch.complex128))
        if grad:
            gm -= sum(v.abs().square().sum(0).reshape(-1) for v in x)
            unweighted = A.w
            A.w = [None] * A.nd
            for mu in range(A.nd):
                h = A.link(mu, [torch.roll(t, -1, A.axis(mu)) for t in x], False)
                gw[mu] -= sum((u - v).abs().square().sum(0).reshape(-1) for u, v in zip(x, h))
            A.w = unweighted
    return q, gm / probes, gw / probes


def _estimates(q):
    n = q.shape[0]
    sizes = [1 << k for k in range(n.bit_length()) if 1 << k <= n]
    if sizes[-1] != n:
        sizes.append(n)
    q = q.cpu().numpy()
    return np.array([complex(math.fsum(q[:s].real) / s, math.fsum(q[:s].imag) / s) for s in sizes])


def exact(case, seed):
    problems, x = _inputs(case, seed)
    if case["do"] == "apply":
        dims, _, mass, mf, w, U = problems[0]
        A = _Dense(dims, mass, mf, w, U)
        shape = list(reversed(dims))
        v = [x[..., c].reshape(-1, *shape).contiguous() for c in range(3)] if U is not None else [x.reshape(-1, *shape)]
        y = [t.reshape(x.shape[0], -1) for t in A(v)]
        return torch.stack(y, dim=-1) if U is not None else y[0]
    out = []
    for problem in problems:
        q, gm, gw = _quadratures(case, problem, seed, case.get("mask", "z2"), grad=case["do"] == "grad")
        if case["do"] == "grad":
            est = _estimates(q)
            return {"estimate": torch.tensor(est[-1].real, dtype=torch.float64), "grad_mass": gm, "grad_coupling": gw}
        out.append({"estimates": _estimates(q), "quadratures": q.cpu().numpy()})
    return out if case["do"] == "batch" else out[0]
