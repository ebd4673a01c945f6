"""Timed cases of the SOAP library's public entry points.

Every case builds the neighbour list of a structure and computes one kind of
output from it, as a program does that follows a moving structure: the library
context (species, cutoff, basis) is kept, positions come in on the device.

Kinds of call ("call"):
  derivatives   descriptor + analytic Jacobian
  batches       the same in center batches under a memory budget
  compute       descriptor only
  cc            expansion coefficients and their Jacobian
  inner, outer  descriptor averaged over the centers

exact() is a plain float64 evaluation of the same definitions in torch, with
the orthonormalisation of the radial bases in decimal arithmetic (their overlap
matrices are too ill-conditioned for float64).
"""
import decimal
import functools
import math

import numpy as np
import torch

from paper_2609_05709_amd import workloads
from paper_2609_05709_amd.soap import Soap

WATER, CHNO = (1, 8), (1, 6, 7, 8)
QUAD_N = 64  # the library's default Gauss-Legendre order


def _case(name, call, system, size, rbf, n, l, r_cut, sigma, dtype="float32", arith="mixed", periodic=False):
    return dict(name=name, call=call, system=system, size=size, rbf=rbf, n_max=n, l_max=l, r_cut=r_cut, sigma=sigma,
                dtype=dtype, arith=arith, periodic=periodic)


def listed():
    return [
        # a small molecule cluster, one call per step of a trajectory: launches and host latency count
        _case("water64_n4l4", "derivatives", "water", 64, "gto", 4, 4, 5.0, 0.5),
        # the ordinary call: a 3000-atom cluster at a production basis
        _case("water1000_n8l6", "derivatives", "water", 1000, "gto", 8, 6, 6.0, 0.5),
        # the same with float64 positions and outputs, as force fitting with tight residuals asks for
        _case("water1000_n8l6_f64", "derivatives", "water", 1000, "gto", 8, 6, 6.0, 0.5, dtype="float64"),
        # the largest basis of the hyperparameter map: a 7 GB Jacobian
        _case("water1000_n12l12", "derivatives", "water", 1000, "gto", 12, 12, 6.0, 0.5),
        # the polynomial basis at the production size
        _case("water1000_poly_n8l6", "derivatives", "water", 1000, "polynomial", 8, 6, 6.0, 0.5),
        # its Laplace form at another point of the map
        _case("water1000_laplace_n6l8", "derivatives", "water", 1000, "polynomial-laplace", 6, 8, 6.0, 0.5),
        # four species, short rows: an organic condensed phase
        _case("chno4096_poly_n10l10", "derivatives", "chno", 4096, "polynomial", 10, 10, 5.0, 0.4),
        # a periodic box at an odd basis in float64 arithmetic with float32 outputs
        _case("periodic999_n7l3", "derivatives", "water", 999, "gto", 7, 3, 5.5, 0.5, arith="fp64", periodic=True),
        # a larger cluster streamed in center batches under a memory budget
        _case("batches2503_n5l5", "batches", "water", 2503, "gto", 5, 5, 5.0, 0.5),
        # coefficients and their Jacobian, for models that contract them themselves
        _case("water1000_cc_n8l6", "cc", "water", 1000, "gto", 8, 6, 6.0, 0.5),
        # one averaged row per structure, for global models of a mixed phase
        _case("chno4096_inner_n9l5", "inner", "chno", 4096, "gto", 9, 5, 5.0, 0.4),
        # a million atoms, descriptor only: screening a large snapshot
        _case("water333334_desc_n8l6", "compute", "water", 333334, "gto", 8, 6, 5.0, 0.5),
    ]


def draw(rng):
    call = rng.choice(("derivatives",) * 6 + ("batches", "compute", "compute", "cc", "inner", "outer"))
    system = rng.choice(("water", "water", "water", "chno"))
    rbf = rng.choice(("gto", "gto", "polynomial", "polynomial-laplace"))
    n, l = rng.randint(2, 12), rng.randint(2, 12)
    r_cut, sigma = round(rng.uniform(4.5, 6.5), 2), round(rng.uniform(0.4, 0.6), 3)
    dtype = rng.choice(("float32", "float32", "float64"))
    arith = rng.choice(("mixed", "mixed", "fp64")) if dtype == "float32" else "mixed"
    periodic = rng.random() < 0.2
    if system == "chno":  # four species: the largest basis the on-chip plans are meant for
        n, l = min(n, 10), min(l, 10)
        size = int(round(math.exp(rng.uniform(math.log(40), math.log(6000)))))
    else:
        most = 60000 if call in ("compute", "outer", "inner") else 2500
        size = int(round(math.exp(rng.uniform(math.log(16), math.log(most)))))
    c = dict(call=call, system=system, size=size, rbf=rbf, n_max=n, l_max=l, r_cut=r_cut, sigma=sigma, dtype=dtype,
             arith=arith, periodic=periodic)
    # at most a quarter of the largest listed Jacobian (7.3 GB), and a tenth of the million-atom descriptor's sums
    while c["size"] > 16 and (work(c)["bytes"] > 1.8e9 or work(c)["flops"] > 1.0e10):
        c["size"] = c["size"] * 3 // 4
    return c


def _structure(case, seed):
    """Positions (float64, exact float32 values) and atomic numbers."""
    if case["system"] == "chno":
        k = max(1, case["size"] // 8)
        radius = 35.0 * (8 * k / 4096.0) ** (1.0 / 3.0)
        s = workloads.multispecies_sphere(8 * k, seed, radius, 0.9, {1: 4 * k, 6: 2 * k, 7: k, 8: k})
        return s.pos64, s.Z
    if case["size"] <= 4000:
        s = workloads.water_cluster(case["size"], seed)
        return s.pos64, s.Z
    return _large_water(case["size"], seed)


def _large_water(n, seed):
    """n water molecules in a ball at the liquid's density, in random order:
    the generator's rejection sampling takes 17 s for a million atoms, so the
    oxygens sit on a face-centred lattice displaced by up to 0.35 A."""
    rng = np.random.default_rng(seed)
    a = (4.0 / workloads.WATER_DENSITY) ** (1.0 / 3.0)
    m = int(math.ceil((3.0 * n / (4.0 * math.pi * workloads.WATER_DENSITY)) ** (1.0 / 3.0) / a)) + 1
    g = np.stack(np.meshgrid(*[np.arange(-m, m + 1)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    o = (g + np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])).reshape(-1, 3) * a
    o = o[np.argpartition((o * o).sum(1), n)[:n]]
    o = o[rng.permutation(n)] + rng.uniform(-0.35, 0.35, (n, 3))
    u = rng.standard_normal((n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    v = rng.standard_normal((n, 3))
    v -= (u * v).sum(1, keepdims=True) * u
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    half = math.radians(104.52) / 2.0
    pos = np.stack([o, o + 0.9572 * (math.cos(half) * u + math.sin(half) * v),
                    o + 0.9572 * (math.cos(half) * u - math.sin(half) * v)], 1).reshape(-1, 3)
    return pos.astype(np.float32).astype(np.float64), np.tile(np.array([8, 1, 1], np.int32), n)


def _system(case, seed):
    """Positions, atomic numbers, lattice vectors (None: open boundaries)."""
    pos, Z = _structure(case, seed)
    if not case["periodic"]:
        return pos, Z, None
    lo = pos.min(axis=0) - 0.8
    cell = np.diag(np.maximum(pos.max(axis=0) - lo + 0.8, 2.0 * case["r_cut"] + 0.1))
    return (pos - lo).astype(np.float32).astype(np.float64), Z, cell


def prepare(case, seed):
    pos, Z, cell = _system(case, seed)
    dtype = torch.float64 if case["dtype"] == "float64" else torch.float32
    sp = Soap(WATER if case["system"] == "water" else CHNO, case["r_cut"], case["n_max"], case["l_max"],
              case["sigma"], case["rbf"], dtype=case["dtype"], arith=case["arith"])
    if cell is not None:
        sp.set_cell(cell)
    # output arrays kept from step to step, the edges' with room for a changing edge count
    out = [torch.zeros(shape, dtype=dtype, device="cuda") for shape in _shapes(case)]
    return dict(call=case["call"], soap=sp, pos=torch.from_numpy(pos).to("cuda", dtype), Z=torch.from_numpy(Z).cuda(),
                out=out, budget=int(work(case)["bytes"] / 4) + (64 << 20))


def run(state):
    sp, call, out = state["soap"], state["call"], state["out"]
    E = sp.build_neighbors(state["pos"], state["Z"])
    if call == "derivatives":
        desc, edge, own = out
        sp.derivatives(desc, edge[:E], own)
    elif call == "batches":
        desc, edge, own = out
        centers, edges = sp.plan_batches(state["budget"])
        for k in range(len(centers) - 1):
            c0, c1, e0, e1 = centers[k], centers[k + 1], edges[k], edges[k + 1]
            sp.derivatives_batch(c0, c1 - c0, e1 - e0, desc[c0:c1], edge[e0:e1], own[c0:c1])
    elif call == "compute":
        sp.compute(out[0])
    elif call == "cc":
        c, edge, own = out
        sp.coefficient_derivatives(c, edge[:E], own)
    else:
        sp.compute_averaged(call, out[0])
    return out


def _shapes(case):
    """Of the arrays that a call fills; edges get room for 10 % and four per atom more than expected."""
    S, N, E, F, Fe = _sizes(case)
    n, L, call = case["n_max"], (case["l_max"] + 1) ** 2, case["call"]
    room = min(N * (N - 1), int((1.35 if case["periodic"] else 1.1) * E) + 4 * N)
    if call == "cc":
        return [(N, S, n, L), (room, 3, n, L), (N, 3, S, n, L)]
    if call in ("derivatives", "batches"):
        return [(N, F), (room, 3, Fe), (N, 3, F)]
    return [(N, F)] if call == "compute" else [(F,)]


def _sizes(case):
    """(species, atoms, expected edges, features, edge features)"""
    n, lw, r = case["n_max"], case["l_max"] + 1, case["r_cut"]
    if case["system"] == "chno":
        S, N = 4, 8 * max(1, case["size"] // 8)
        R = 35.0 * (N / 4096.0) ** (1.0 / 3.0)
    else:
        S, N = 2, 3 * case["size"]
        R = (3.0 * case["size"] / (4.0 * math.pi * workloads.WATER_DENSITY)) ** (1.0 / 3.0) + 0.5
    x = min(r / R, 2.0)
    # two uniform points of a ball of radius R are within x R of each other with this probability
    E = N * (N - 1) * (x ** 3 * (1.0 - 9.0 * x / 16.0 + x ** 3 / 32.0))
    return S, N, E, lw * S * n * (S * n + 1) // 2, lw * (n * (n + 1) // 2 + (S - 1) * n * n)


def work(case):
    S, N, E, F, Fe = _sizes(case)
    n, l = case["n_max"], case["l_max"]
    L, lw = (l + 1) ** 2, l + 1
    call = case["call"]
    elt = 8 if case["dtype"] == "float64" else 4
    jac = call in ("derivatives", "batches", "cc")
    if case["rbf"] == "gto":
        radial = 2 * n * n * lw + n * lw
    elif case["rbf"] == "polynomial":
        radial = 2 * n * QUAD_N * lw + QUAD_N * (l + 2) + 2 * QUAD_N
    else:
        radial = 8 * n * (n + 3) + 10 * n * lw
    # harmonics, radial factors, sums c (and their gradients)
    flops = E * ((12 * L + 2 * radial + 14 * n * L) if jac else (3 * L + radial + 2 * n * L))
    values = {"compute": N * F, "inner": F, "outer": F, "cc": N * S * n * L * 4 + 3 * E * n * L}.get(
        call, N * 4 * F + 3 * E * Fe)
    if call == "cc":
        pass
    elif call == "inner":
        flops += F * 2 * L / lw + N * S * n * L
    else:
        flops += N * F * 2 * L / lw
    if call in ("derivatives", "batches"):  # precontraction and blocks per edge, center block
        flops += E * (8 * S * n * L + 12 * (Fe + lw * n * (n + 1) // 2) + 3 * Fe)
    return {"bytes": elt * (values + 3 * N) + 4 * N, "flops": flops}


def tolerance(case):
    if case["dtype"] == "float64":
        # sums in float64; the GTO basis amplifies their rounding below n_max 10
        # (up to 1e4 at n_max 8), and its compensated sums from n_max 10 on do not
        return {"rel": 1e-10}
    # float32 outputs, operands rounded to float32 once or twice on the way
    return {"rel": 1e-6}


# ---------------------------------------------------------------------------
# the same definitions in plain float64
# ---------------------------------------------------------------------------

_D = decimal.Decimal


def _inv_sqrt(A):
    """A^(-1/2) of a symmetric positive-definite matrix of Decimals, by the
    coupled Newton iteration (Denman and Beavers, 1976)."""
    n = len(A)

    def inverse(M):
        M = [list(M[i]) + [_D(int(i == j)) for j in range(n)] for i in range(n)]
        for i in range(n):
            p = max(range(i, n), key=lambda r: abs(M[r][i]))
            M[i], M[p] = M[p], M[i]
            d = 1 / M[i][i]
            M[i] = [v * d for v in M[i]]
            for r in range(n):
                if r != i and M[r][i]:
                    f = M[r][i]
                    M[r] = [a - f * b for a, b in zip(M[r], M[i])]
        return [row[n:] for row in M]

    Y, Zm = A, [[_D(int(i == j)) for j in range(n)] for i in range(n)]
    for _ in range(200):
        Yi, Zi = inverse(Y), inverse(Zm)
        Yn = [[(Y[i][j] + Zi[i][j]) / 2 for j in range(n)] for i in range(n)]
        Zn = [[(Zm[i][j] + Yi[i][j]) / 2 for j in range(n)] for i in range(n)]
        change = max(abs(Zn[i][j] - Zm[i][j]) for i in range(n) for j in range(n))
        size = max(abs(v) for row in Zn for v in row)
        Y, Zm = Yn, Zn
        if change < size * _D(10) ** -40:
            break
    return Zm


@functools.lru_cache(maxsize=8)
def _gto_tables(r_cut, n, l_max, sigma):
    """betaC[l][n][k], a'[l][k], on-site c0[n]."""
    with decimal.localcontext() as ctx:
        ctx.prec = 110
        rc, s2, pi = _D(r_cut), _D(sigma) ** 2, _pi()
        z = [_D(1) + k * (rc - 1) / (n - 1) for k in range(n)] if n > 1 else [_D(1)]
        betaC, ap, c0 = [], [], None
        pref = (2 * pi) ** _D("1.5") * s2 * _D(sigma)
        for l in range(l_max + 1):
            al = [(_D(1000).ln() + l * zk.ln()) / zk ** 2 for zk in z]
            g = pi.sqrt()  # Gamma(l + 3/2)
            for k in range(l + 1):
                g = g * (2 * k + 1) / 2
            S = [[g / (2 * ((a + b) ** (l + 1) * (a + b).sqrt())) for b in al] for a in al]
            beta = _inv_sqrt(S)
            q = [1 + 2 * s2 * a for a in al]
            ap.append([float(a / d) for a, d in zip(al, q)])
            betaC.append([[float(pref * beta[i][k] / (q[k] ** (l + 1) * q[k].sqrt())) for k in range(n)]
                          for i in range(n)])
            if l == 0:
                c0 = [float(_D(2).sqrt() * pi * s2 * _D(sigma) *
                            sum(beta[i][k] / (q[k] * q[k].sqrt()) for k in range(n))) for i in range(n)]
    return np.array(betaC), np.array(ap), np.array(c0)


def _pi():
    """pi by Machin's formula at the current precision."""
    def arctan_inv(x):
        t = total = _D(1) / x
        k, sign = 1, -1
        while abs(t) > _D(10) ** -(decimal.getcontext().prec + 5):
            t /= x * x
            k += 2
            total += sign * t / k
            sign = -sign
        return total
    return 4 * (4 * arctan_inv(5) - arctan_inv(239))


@functools.lru_cache(maxsize=8)
def _poly_tables(r_cut, n, sigma):
    """W_nk / N_k, nodes r_q, G[n][q] = w_q r_q^2 g_n(r_q), on-site c0[n]."""
    with decimal.localcontext() as ctx:
        ctx.prec = 110
        rc = _D(r_cut)
        N = [(rc ** (2 * k + 5) / (2 * k + 5)).sqrt() for k in range(1, n + 1)]
        S = [[_D((5 + 2 * a) * (5 + 2 * b)).sqrt() / (5 + a + b) for b in range(1, n + 1)] for a in range(1, n + 1)]
        W = _inv_sqrt(S)
        WN = [[W[i][k] / N[k] for k in range(n)] for i in range(n)]
        t, w = np.polynomial.legendre.leggauss(QUAD_N)
        rq = [rc * (_D(float(v)) + 1) / 2 for v in t]
        G = [[rc * _D(float(w[q])) / 2 * r * r * sum(WN[i][k] * (rc - r) ** (k + 3) for k in range(n))
              for q, r in enumerate(rq)] for i in range(n)]
        G = np.array([[float(v) for v in row] for row in G])
        WN = np.array([[float(v) for v in row] for row in WN])
    rq = np.array([float(r) for r in rq])
    c0 = 4.0 * math.pi / math.sqrt(4.0 * math.pi) * (G * np.exp(-rq * rq / (2.0 * sigma * sigma))).sum(1)
    return WN, rq, G, c0


def _radial(case, r):
    """B[e][n][l], Bh[e][n][l] with c += B r^l Y and grad c = Bh r_vec S + B grad S."""
    n, lw, s2, rc = case["n_max"], case["l_max"] + 1, case["sigma"] ** 2, case["r_cut"]

    def dev(a):
        return torch.as_tensor(a, dtype=torch.float64, device=r.device)
    if case["rbf"] == "gto":
        bc, ap, _ = _gto_tables(rc, n, case["l_max"], case["sigma"])
        bc, ap = dev(bc), dev(ap)
        e = torch.exp(-ap[None] * (r * r)[:, None, None])  # [e][l][k]
        B = torch.stack([e[:, l] @ bc[l].T for l in range(lw)], 2)
        Bh = torch.stack([(-2.0 * ap[l] * e[:, l]) @ bc[l].T for l in range(lw)], 2)
        return B, Bh
    WN, rq, G, _ = _poly_tables(rc, n, case["sigma"])
    ls = torch.arange(lw, dtype=torch.float64, device=r.device)
    if case["rbf"] == "polynomial":
        G, rq, R = dev(G), dev(rq), r[:, None]
        x = rq[None] * R / s2
        w = torch.exp(-(rq[None] - R) ** 2 / (2.0 * s2))
        # ratios i_l / i_{l-1} by the continued fraction, from far above l_max
        top = lw + 2 + int(12.0 * math.sqrt(float(x.max())) + 20)
        ratio = [None] * (lw + 2)
        rho = torch.zeros_like(x)
        for l in range(top, 0, -1):
            rho = 1.0 / (rho + (2 * l + 1) / x)
            if l <= lw:
                ratio[l] = rho
        il = [-torch.expm1(-2.0 * x) / (2.0 * x)]
        for l in range(1, lw + 1):
            il.append(il[-1] * ratio[l])
        f, df = [], []
        for l in range(lw):
            f.append((w * il[l]) @ G.T)
            df.append((w * (-(R / s2) * il[l] + (rq[None] / s2) * (il[l + 1] + (l / x) * il[l]))) @ G.T)
        f, df = 4.0 * math.pi * torch.stack(f, 2), 4.0 * math.pi * torch.stack(df, 2)
    else:
        k = torch.arange(1, n + 1, dtype=torch.float64, device=r.device)
        R, u = r[:, None, None], (rc - r)[:, None, None]
        ll = (ls * (ls + 1.0))[None, :, None]
        pre = (2.0 * math.pi) ** 1.5 * s2 * case["sigma"]
        up = u ** (k + 1.0)[None, None]
        b = (u - ll * s2 * u / (2.0 * R * R) - (k + 2.0) * s2 / R + (k + 2.0) * (k + 1.0) * s2 / (2.0 * u))
        d = (-(k + 2.0) + ll * s2 * u / R ** 3 + (k + 2.0) * (ll + 2.0) * s2 / (2.0 * R * R) +
             (k + 1.0) * (k + 2.0) * s2 / (R * u) - k * (k + 1.0) * (k + 2.0) * s2 / (2.0 * u * u))
        f = pre * ((up * b) @ dev(WN).T).transpose(1, 2)
        df = pre * ((up * d) @ dev(WN).T).transpose(1, 2)
    rl = r[:, None, None] ** ls[None, None]
    R = r[:, None, None]
    return f / rl, (df - ls * f / R) / (rl * R)


def _harmonics(v, l_max):
    """Real solid harmonics S[e][lm] and gradients [e][3][lm], lm = l l + l + m."""
    x, y, z = v[:, 0], v[:, 1], v[:, 2]
    r2, zero, one = (v * v).sum(1), torch.zeros_like(x), torch.ones_like(x)
    L = (l_max + 1) ** 2
    S, dS = [None] * L, [None] * L
    C, Sn, dC, dSn = one, zero, (zero, zero), (zero, zero)  # (x + i y)^m and its x, y derivatives
    for m in range(l_max + 1):
        if m:
            dC, dSn = ((C + x * dC[0] - y * dSn[0], x * dC[1] - Sn - y * dSn[1]),
                       (Sn + x * dSn[0] + y * dC[0], x * dSn[1] + C + y * dC[1]))
            C, Sn = x * C - y * Sn, x * Sn + y * C
        Q0, g0 = zero, (zero, zero, zero)
        Q1, g1 = one * float(math.prod(range(1, 2 * m, 2))), (zero, zero, zero)
        for l in range(m, l_max + 1):
            if l > m:
                a, b = (2 * l - 1) / (l - m), (l + m - 1) / (l - m)
                Q, g = a * z * Q1 - b * r2 * Q0, [a * z * g1[k] - b * (r2 * g0[k] + 2.0 * v[:, k] * Q0)
                                                  for k in range(3)]
                g[2] = g[2] + a * Q1
                Q0, g0, Q1, g1 = Q1, g1, Q, g
            N = math.sqrt((2 * l + 1) / (4.0 * math.pi) * math.factorial(l - m) / math.factorial(l + m))
            for sign, A, dA in ((1, C, dC), (-1, Sn, dSn)) if m else ((1, C, dC),):
                k = N * (math.sqrt(2.0) if m else 1.0)
                S[l * l + l + sign * m] = k * Q1 * A
                dS[l * l + l + sign * m] = torch.stack(
                    [k * (g1[0] * A + Q1 * dA[0]), k * (g1[1] * A + Q1 * dA[1]), k * g1[2] * A], 1)
    return torch.stack(S, 1), torch.stack(dS, 2)


def _edges(case, pos, spec, cell):
    """Center, neighbour atom, vector of every edge, in the library's row
    order: species, then atom, then its images."""
    N, rc2 = pos.shape[0], case["r_cut"] ** 2
    ext, atom = pos, torch.arange(N, device=pos.device)
    if cell is not None:  # cells wider than 2 r_cut: the 26 images around are all that can reach
        a, shifts = np.asarray(cell), [(i, j, k) for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)
                                       if (i, j, k) != (0, 0, 0)]
        s = torch.tensor(np.array([(i * a[0] + j * a[1]) + k * a[2] for i, j, k in shifts]), device=pos.device)
        p = (pos[:, None] + s[None]).reshape(-1, 3)
        if case["dtype"] == "float32":
            p = p.float().double()
        ext = torch.cat([pos, p])
        atom = torch.cat([atom, torch.arange(N, device=pos.device).repeat_interleave(len(shifts))])
        near = ((ext > pos.min(0).values - case["r_cut"]) & (ext < pos.max(0).values + case["r_cut"])).all(1)
        ext, atom = ext[near], atom[near]
    order = torch.sort(spec[atom], stable=True).indices
    out = []
    step = max(1, int(2e8) // ext.shape[0])
    for c0 in range(0, N, step):
        c1 = min(N, c0 + step)
        d = [ext[order, k][None] - pos[c0:c1, k][:, None] for k in range(3)]
        near = ((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]) < rc2
        i, j = near.nonzero(as_tuple=True)
        j = order[j]
        keep = j != i + c0  # the atoms themselves come first in ext
        out.append((i[keep] + c0, j[keep]))
    i, j = torch.cat([o[0] for o in out]), torch.cat([o[1] for o in out])
    return i, atom[j], ext[j] - pos[i]


def exact(case, seed):
    S, N, E, F, Fe = _sizes(case)
    if N > 40000:  # pairs and the intermediates of every edge are formed in full here
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    pos, Z, cell = _system(case, seed)
    n, l_max, call = case["n_max"], case["l_max"], case["call"]
    lw, L = l_max + 1, (l_max + 1) ** 2
    pos = torch.from_numpy(pos).to(dev)
    species = WATER if case["system"] == "water" else CHNO
    spec = torch.from_numpy(np.searchsorted(np.array(species), Z)).to(dev)
    i, j, vec = _edges(case, pos, spec, cell)
    row = torch.zeros(N + 1, dtype=torch.int64, device=dev)
    row[1:] = torch.bincount(i, minlength=N).cumsum(0)
    if case["rbf"] == "gto":
        c0 = _gto_tables(case["r_cut"], n, l_max, case["sigma"])[2]
    else:
        c0 = _poly_tables(case["r_cut"], n, case["sigma"])[3]
    c0 = torch.as_tensor(c0, device=dev)
    pairs = [(a, b) for a in range(S) for b in range(a, S)]
    ia, ib = np.triu_indices(n)
    tri = torch.as_tensor(ia * n + ib, device=dev)
    K = [math.pi * math.sqrt(8.0 / (2 * l + 1)) for l in range(lw)]

    def products(A, B):
        """[..., a, b, l] = K_l sum_m A[..., a, lm] B[..., b, lm]"""
        return torch.stack([K[l] * torch.matmul(A[..., l * l:(l + 1) ** 2],
                                                B[..., l * l:(l + 1) ** 2].transpose(-1, -2).contiguous())
                            for l in range(lw)], -1)

    def section(T, diagonal):
        T = T.flatten(-3, -2)
        return (T[..., tri, :] if diagonal else T).flatten(-2)

    jac = call in ("derivatives", "batches", "cc")
    descs, cs, selfs = [], [], []
    blocks = torch.zeros(_shapes(case)[1], dtype=torch.float64, device=dev) if jac else None
    rows = row.tolist()
    first = 0
    most = max(64, int(1.5e8) // (3 * max(n * L, n * n * lw * S)))
    while first < N:
        last = first + 1
        while last < N and rows[last + 1] - rows[first] <= most:
            last += 1
        e = slice(rows[first], rows[last])
        nc = last - first
        r = vec[e].norm(dim=1)
        B, Bh = _radial(case, r) if e.stop > e.start else (torch.zeros((0, n, lw), device=dev, dtype=torch.float64),) * 2
        Y, dY = _harmonics(vec[e], l_max)
        of_l = torch.tensor([l for l in range(lw) for _ in range(2 * l + 1)], device=dev)
        B, Bh = B[:, :, of_l], Bh[:, :, of_l]
        sj = spec[j[e]]
        at = (i[e] - first) * S + sj
        c = torch.zeros((nc * S, n, L), dtype=torch.float64, device=dev).index_add_(0, at, B * Y[:, None])
        own = torch.arange(nc, device=dev) * S + spec[first:last]
        c[own, :, 0] += c0
        c = c.reshape(nc, S, n, L)
        cs.append(c)
        if call not in ("cc", "inner"):
            descs.append(torch.cat([section(products(c[:, a], c[:, b]), a == b) for a, b in pairs], 1))
        if jac:
            dc = vec[e][:, :, None, None] * (Bh * Y[:, None])[:, None] + B[:, None] * dY[:, :, None]
            D = torch.zeros((nc * S, 3, n, L), dtype=torch.float64, device=dev).index_add_(0, at, dc)
            D = D.reshape(nc, S, 3, n, L)
            if call == "cc":
                blocks[e] = dc
                selfs.append(-D.transpose(1, 2))
            else:
                selfs.append(torch.cat([-section(products(D[:, a], c[:, None, b]) + products(c[:, None, a], D[:, b]),
                                                 a == b) for a, b in pairs], -1))
                ce = c[i[e] - first]
                T = [products(dc, ce[:, None, s]) for s in range(S)]  # dc_a . c^s_b
                for s in range(S):
                    of = (sj == s).nonzero(as_tuple=True)[0]
                    parts = []
                    for a, b in pairs:
                        if s not in (a, b):
                            continue
                        t = T[b if s == a else a][of]
                        if a == b:
                            t = t + t.transpose(-3, -2)
                        elif s == b:
                            t = t.transpose(-3, -2)
                        parts.append(section(t, a == b))
                    blocks[of + e.start] = torch.cat(parts, -1)
        first = last
    c = torch.cat(cs)
    if call == "inner":
        c = c.mean(0)
        return [torch.cat([section(products(c[a], c[b]), a == b) for a, b in pairs])]
    if call == "cc":
        return [c, blocks, torch.cat(selfs)]
    desc = torch.cat(descs)
    if call in ("compute", "outer"):
        return [desc if call == "compute" else desc.mean(0)]
    return [desc, blocks, torch.cat(selfs)]
