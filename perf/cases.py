"""The calls this library is measured on: solves of the Wilson-clover equation from one tiny lattice to twelve
sources on 32^3x64, batches of lattices, a new gauge configuration, the preconditioner and the operator by
themselves.

A case is a dict of plain values.  `prepare` makes a gauge field and sources from a seed on the GPU and a
`ddqcd.Context` set up as a user's program sets it up; `run` is one call (for a new configuration, two) through
the Python binding; `exact` is the same result in plain FP64 torch.  Sizes, masses and solver settings are those
of `paper_1412_2629_amd/configs.py` and the tests, or between them.
"""
import math

import torch

from paper_1412_2629_amd import ddqcd

BC = (1.0, 1.0, 1.0, -1.0)
# (kappa, c_sw, eps) of the smallest workload, of the tests, and of the 16^3x32 and 32^3x64 workloads
PHYSICS = {"small": (0.12, 1.0, 0.3), "test": (0.13, 1.5, 0.5), "mid": (0.1355, 1.5, 0.5), "heavy": (0.1365, 1.7, 0.6)}
LARGEST = 32 ** 3 * 64 * 12   # sites x right-hand sides of the largest solve


def dims(text):
    return tuple(int(v) for v in text.split("x"))


def volume(L):
    return math.prod(L)


def case_lattices(case):
    """[(lattice, domain)] of a case: one, or a batch written "8x8x8x8/4x4x4x4*3 ..." (shape/domain*count)."""
    out = []
    for part in case["lattices"].split():
        shape, count = part.split("*") if "*" in part else (part, 1)
        L, b = shape.split("/")
        out += [(dims(L), dims(b))] * int(count)
    return out


def _case(call, lattices, prec, physics, **more):
    return {"call": call, "lattices": lattices, "prec": prec, "physics": physics, "nrhs": 1, "cycles": 16, "mr": 5,
            "product": "lane", "outer": "fgcr", "restart": 16, "deflate": 0, **more}


def listed():
    return [
        # a first try, a unit test, a thermalisation check: one source on a 4^4 lattice, all in FP64; launches and
        # host round trips are all there is to it
        dict(_case("solve", "4x4x4x4/2x2x2x2", "f64", "small", cycles=8, mr=4), name="solve_4c_f64"),
        # one source on a small lattice of a coarse ensemble, the default precision of production work
        dict(_case("solve", "8x8x8x8/4x4x4x4", "f16", "mid"), name="solve_8c_f16"),
        # extents that only ragged domains fit (288 sites, padded workgroups), with the paper's own outer solver
        dict(_case("solve", "12x12x12x24/6x6x2x4", "f32", "mid", outer="fgmres_dr", restart=8, deflate=4),
             name="solve_12x24_f32_dr"),
        # one source on 16^3x32, FP32 block solves: the middle workload
        dict(_case("solve", "16x16x16x32/8x4x4x4", "f32", "mid"), name="solve_16x32_f32"),
        # one source on the production lattice, FP16 storage
        dict(_case("solve", "32x32x32x64/8x4x4x4", "f16", "heavy"), name="solve_32x64_f16"),
        # a whole point-to-all propagator on the production lattice: the benchmark's default.  Three steps
        # converge, so a basis of four serves, and three such states fit the card.
        dict(_case("solve", "32x32x32x64/4x4x4x4", "f16", "heavy", nrhs=12, product="tile", restart=4),
             name="solve_32x64_12src"),
        # what a measurement run does for each configuration of an ensemble: load the new gauge field, then the
        # twelve sources of its propagator
        dict(_case("newconf", "16x16x16x32/4x4x4x4", "bf16", "mid", nrhs=12, product="tile"),
             name="newconf_16x32_12src"),
        # lattices of several sizes in one call (a parameter scan), domains as the tuner picks them
        dict(_case("batch", "8x8x8x8/4x4x4x4*4 12x12x12x24/2x2x2x2*2 16x16x16x32/8x4x4x4*2 24x24x24x48/4x4x4x4",
                   "f16", "test"), name="batch_uneven"),
        # the preconditioner in FP64 for a user's own Krylov solver (in less precision it runs inside the solves,
        # whose results do not hang on its rounding)
        dict(_case("sap", "16x16x16x32/8x4x4x4", "f64", "mid", nrhs=2), name="sap_16x32_f64"),
        # the operator on the production lattice: residual checks, sequential sources
        dict(_case("apply", "32x32x32x64/4x4x4x4", "f64", "heavy", nrhs=2), name="apply_32x64_f64"),
        # the operator in single precision on an odd-sized lattice, a few vectors at a time: a user's own solver
        dict(_case("apply", "24x12x12x24/6x6x2x4", "f32", "mid", nrhs=3), name="apply_24x12x12x24_f32"),
        # the solver without domain decomposition that results are checked against
        dict(_case("bicgstab", "16x16x16x32/4x4x4x4", "f64", "mid"), name="bicgstab_16x32"),
    ]


DOMAINS = ["2x2x2x2", "4x4x4x4", "4x4x4x4", "8x4x4x4", "4x4x4x8", "6x6x2x4"]


def _draw_lattice(rng, low, high, shapes=DOMAINS):
    """A lattice with an even number of domains in each direction, its sites spread between low and high over
    their logarithm."""
    while True:
        want = math.exp(rng.uniform(math.log(low), math.log(high)))
        b = dims(rng.choice(shapes))
        side = (want / 2) ** 0.25   # about L^3 x 2L
        L = tuple(2 * d * max(1, round(side * (2 if m == 3 else 1) * math.exp(rng.uniform(-0.4, 0.4)) / (2 * d)))
                  for m, d in enumerate(b))
        if want / 2 <= volume(L) <= min(2 * want, high) and max(L) <= 96:
            return "%s/%s" % ("x".join(map(str, L)), "x".join(map(str, b)))


def draw(rng):
    call = rng.choice(["solve", "solve", "solve", "sources", "newconf", "batch", "sap", "apply", "bicgstab"])
    physics = rng.choice(["test", "test", "heavy"])
    if call == "solve":
        lat = _draw_lattice(rng, 512, 2.2e6)
        prec = rng.choice(["f16", "f16", "f32", "f32", "bf16", "f64"])
        if prec == "f64" and lat.endswith("6x6x2x4"):
            prec = "f32"
        outer = {} if rng.random() < 0.75 else dict(outer="fgmres_dr", restart=8, deflate=4)
        return _case("solve", lat, prec, physics, **outer)
    if call in ("sources", "newconf"):
        # sources of one lattice together, in tiles of four and as single workgroups
        tile = rng.random() < 0.75
        nrhs = rng.randint(2, 12)
        most = min(2.2e6, 0.9 * LARGEST / nrhs) if call == "sources" else 3e5
        lat = _draw_lattice(rng, 4096, most, ["4x4x4x4"] if tile else ["4x4x4x4", "8x4x4x4", "2x2x2x2"])
        return _case("solve" if call == "sources" else "newconf", lat, rng.choice(["f16", "f16", "bf16"]), physics,
                     nrhs=nrhs, product="tile" if tile else "lane", restart=4)
    if call == "batch":
        parts = ["%s*%d" % (_draw_lattice(rng, 512, 3e5), rng.randint(1, 3)) for _ in range(rng.randint(2, 4))]
        return _case("batch", " ".join(parts), rng.choice(["f16", "f16", "f32"]), physics, restart=4)
    if call == "sap":
        lat = _draw_lattice(rng, 512, 1e6, ["2x2x2x2", "4x4x4x4", "8x4x4x4", "4x4x4x8"])
        return _case("sap", lat, "f64", physics, nrhs=rng.randint(1, 4), cycles=rng.choice([4, 8, 16]),
                     mr=rng.randint(3, 6))
    if call == "apply":
        return _case("apply", _draw_lattice(rng, 512, 2.2e6), rng.choice(["f64", "f64", "f32", "f16", "bf16"]),
                     physics, nrhs=rng.randint(1, 6))
    return _case("bicgstab", _draw_lattice(rng, 4096, 5e5), "f64", physics)


# ---- inputs ---------------------------------------------------------------------------------------------------

_GELL_MANN = torch.zeros(8, 3, 3, dtype=torch.complex128)
for _k, _i, _j, _v in ((0, 0, 1, 1), (0, 1, 0, 1), (1, 0, 1, -1j), (1, 1, 0, 1j), (2, 0, 0, 1), (2, 1, 1, -1),
                       (3, 0, 2, 1), (3, 2, 0, 1), (4, 0, 2, -1j), (4, 2, 0, 1j), (5, 1, 2, 1), (5, 2, 1, 1),
                       (6, 1, 2, -1j), (6, 2, 1, 1j), (7, 0, 0, 3 ** -0.5), (7, 1, 1, 3 ** -0.5),
                       (7, 2, 2, -2 * 3 ** -0.5)):
    _GELL_MANN[_k, _i, _j] = _v


def _mul(a, b):
    """Products of 3x3 matrices (..., 3, 3)."""
    return sum(a[..., :, k:k + 1] * b[..., k:k + 1, :] for k in range(3))


def random_gauge(V, eps, gen):
    """Links exp(i eps H), H = sum_a w_a lambda_a / 2, w ~ N(0, 1) (the recipe of inputs.random_gauge)."""
    dev = gen.device
    U = torch.empty(V * 4, 3, 3, dtype=torch.complex128, device=dev)
    gm = (_GELL_MANN.to(dev) / 2).reshape(8, 9)
    one = torch.eye(3, dtype=torch.complex128, device=dev)
    for a in range(0, V * 4, 1 << 21):
        n = min(V * 4 - a, 1 << 21)
        w = torch.randn(n, 8, dtype=torch.float64, device=dev, generator=gen)
        X = ((w.to(torch.complex128) @ gm).reshape(n, 3, 3)) * (1j * eps / 16)
        E = one + X / 13
        for k in range(12, 0, -1):   # Horner's form of the exponential series, then four squarings
            E = one + _mul(X, E) / k
        for _ in range(4):
            E = _mul(E, E)
        U[a:a + n] = E
    return U.reshape(V, 4, 3, 3)


def _inputs(case, seed, dev):
    """[(lattice, domain, U, b)]: b is (V, 4, 3), or (nrhs, V, 4, 3) where a case has several right-hand sides."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    eps = PHYSICS[case["physics"]][2]
    out = []
    for L, dom in case_lattices(case):
        V = volume(L)
        U = random_gauge(V, eps, gen)
        n = case["nrhs"]
        if n > 1 and case["call"] in ("solve", "newconf"):
            # point sources: the spins and colours of one site
            b = torch.zeros(n, V, 12, dtype=torch.complex128, device=dev)
            site = int(torch.randint(V, (1,), generator=gen, device=dev))
            for k in range(n):
                b[k, site, k] = 1
            b = b.reshape(n, V, 4, 3)
        else:
            b = torch.randn(n, V, 4, 3, 2, dtype=torch.float64, device=dev, generator=gen)
            b = torch.view_as_complex(b)
            b = b[0] if n == 1 else b
        out.append((L, dom, U, b.contiguous()))
    return out


def _context(case, L, dom):
    kappa, csw, _ = PHYSICS[case["physics"]]
    ctx = ddqcd.Context(L, dom, kappa, csw, BC)
    ctx.set_sap(case["cycles"], case["mr"], case["prec"] if case["call"] not in ("apply", "bicgstab") else "f32",
                case["product"])
    # a solution to check others against is solved further than they are
    ctx.set_solver(case["restart"], 1e-12 if case["call"] == "bicgstab" else 1e-10, 64)
    if case["outer"] != "fgcr":
        ctx.set_outer(case["outer"], case["deflate"])
    return ctx


def prepare(case, seed):
    state = {"case": case, "ctx": [], "U": [], "b": []}
    for L, dom, U, b in _inputs(case, seed, torch.device("cuda")):
        ctx = _context(case, L, dom)
        if case["call"] == "newconf":
            state["U"].append(U)   # the configuration that run() loads
        else:
            ctx.load_gauge(U)
        state["ctx"].append(ctx)
        state["b"].append(b)
    return state


def run(state):
    case, ctx, b = state["case"], state["ctx"][0], state["b"][0]
    call = case["call"]
    if call == "apply":
        return ctx.apply_D(b, case["prec"])
    if call == "sap":
        return ctx.sap(b)
    if call == "batch":
        return ddqcd.solve_batch(state["ctx"], state["b"])[0]
    if call == "bicgstab":
        return ctx.solve_bicgstab(b)[0]
    if call == "newconf":
        ctx.load_gauge(state["U"][0])
    x = ctx.solve(b)[0]
    return list(x) if case["nrhs"] > 1 else x


# ---- what a pass cannot do without ----------------------------------------------------------------------------

STEPS = 3   # outer steps of a solve (three to seven on these fields)


def _sap_flops_per_site(dom, mr):
    """Flops per site of one SAP cycle (both colours): 165 a hop, 504 a clover block application, and the vector
    work of the MR steps; mr + 1 applications of the even-odd operator and its preparation."""
    inside = sum(2 * (d - 1) / d for d in dom)
    hops = (mr + 1) * inside * 165 + (8 - inside) * 165
    return hops + (mr + 1) * 504 + mr * 178 + 48


def work(case):
    nbytes = flops = 0.0
    stored = {"f64": 16, "f32": 8, "f16": 4, "bf16": 4}[case["prec"]]
    for L, dom in case_lattices(case):
        V, n, call = volume(L), case["nrhs"], case["call"]
        nbytes += V * n * 2 * 192            # vectors in and out, FP64
        per_step = 1824
        if call in ("solve", "batch", "newconf", "sap"):
            per_step += case["cycles"] * _sap_flops_per_site(dom, case["mr"])
        if call == "apply":
            nbytes += V * (36 if stored == 16 else 24) * stored + V * 36 * stored
            flops += V * n * 1824
        elif call == "sap":
            nbytes += V * (36 + 36) * 16
            flops += V * n * (per_step - 1824)
        elif call == "bicgstab":
            nbytes += V * (576 + 576)
            flops += V * 340 * 1824          # some 170 iterations of two applications
        else:
            nbytes += V * (576 + 576) + V * 60 * stored
            flops += V * n * STEPS * per_step
        if call == "newconf":
            # the field in, every stored copy of links, clover term and block matrices out; 24 leaves of three
            # 3x3 products a site, the inverse of two 6x6 blocks on the odd ones
            nbytes += V * (576 + 24 * 16 + 2 * 36 * 16 + 2 * 36 * 16)
            flops += V * (24 * 3 * 198 + 0.5 * 2 * 8 * 6 ** 3)
    return {"bytes": nbytes, "flops": flops}


# ---- the same results in plain FP64 -----------------------------------------------------------------------------

# gamma_mu v = phase * v[perm] over the spins, chiral basis
_GAMMA = (((3, 2, 1, 0), (-1j, -1j, 1j, 1j)), ((3, 2, 1, 0), (-1, 1, 1, -1)), ((2, 3, 0, 1), (-1j, 1j, 1j, -1j)),
          ((2, 3, 0, 1), (-1, -1, -1, -1)))


def _gamma_matrix(mu):
    g = torch.zeros(4, 4, dtype=torch.complex128)
    perm, phase = _GAMMA[mu]
    for s in range(4):
        g[s, perm[s]] = phase[s]
    return g


class Exact:
    """A = 1/(2 kappa) - D_w/2 + c_sw (i/8) sum sigma F on fields (Lt, Lz, Ly, Lx, 4, 3), whole or, with every hop
    that leaves a domain left out, restricted to the domains."""

    def __init__(self, L, dom, U, kappa, csw):
        self.L, self.dom = L, dom
        self.dev = U.device
        grid = tuple(reversed(L))
        self.U = [U[:, mu].reshape(*grid, 3, 3) for mu in range(4)]
        self.phase = [torch.tensor(p, dtype=torch.complex128, device=self.dev).reshape(4, 1) for _, p in _GAMMA]
        self.x = torch.meshgrid(*[torch.arange(n, device=self.dev) for n in grid], indexing="ij")[::-1]
        self.C = self._clover(kappa, csw)

    @staticmethod
    def dim(mu):
        return 3 - mu

    def _shift(self, v, mu, step):
        """v at x + step mu, periodic."""
        return torch.roll(v, -step, self.dim(mu))

    def _clover(self, kappa, csw):
        V = volume(self.L)
        C = torch.zeros(V, 12, 12, dtype=torch.complex128, device=self.dev)
        dag = lambda a: a.conj().transpose(-1, -2)  # noqa: E731
        for mu in range(4):
            for nu in range(mu + 1, 4):
                Um, Un = self.U[mu], self.U[nu]
                # the plaquette at x, and the other three leaves as that plaquette seen from x - mu, x - nu, x - mu - nu
                A = _mul(Um, self._shift(Un, mu, 1))
                B = _mul(Un, self._shift(Um, nu, 1))
                Q = _mul(A, dag(B))
                Um_m, Un_m = self._shift(Um, mu, -1), self._shift(Un, mu, -1)
                Um_n, Un_n = self._shift(Um, nu, -1), self._shift(Un, nu, -1)
                B_m = self._shift(B, mu, -1)
                Q = Q + _mul(_mul(_mul(Un, dag(self._shift(Um_m, nu, 1))), dag(Un_m)), Um_m)
                Q = Q + _mul(_mul(dag(self._shift(B_m, nu, -1)), self._shift(Um_m, nu, -1)), Un_n)
                Q = Q + _mul(_mul(_mul(dag(Un_n), Um_n), self._shift(Un_n, mu, 1)), dag(Um))
                F = ((Q - dag(Q)) / 4).reshape(V, 3, 3)
                g, h = _gamma_matrix(mu), _gamma_matrix(nu)
                sigma = 0.5j * (g @ h - h @ g)
                for s in range(4):
                    for t in range(4):
                        if sigma[s, t] != 0:   # both orders of mu and nu
                            C[:, 3 * s:3 * s + 3, 3 * t:3 * t + 3] += 2 * csw * 0.125j * complex(sigma[s, t]) * F
        C[:, range(12), range(12)] += 1 / (2 * kappa)
        return C

    def _site(self, M, v):
        flat = v.reshape(-1, 12)
        out = torch.zeros_like(flat)
        for k in range(12):
            out += M[:, :, k] * flat[:, k:k + 1]
        return out.reshape(v.shape)

    def hops(self, v, local=False):
        """-1/2 D_w v; local: hops inside the domains only."""
        out = torch.zeros_like(v)
        for mu in range(4):
            perm, n, d = list(_GAMMA[mu][0]), self.L[mu], self.dom[mu]
            for step in (1, -1):
                src = v if step == 1 else sum(self.U[mu][..., k, :].conj().unsqueeze(-2) * v[..., k:k + 1]
                                              for k in range(3))
                w = self._shift(src, mu, step)
                at = self.x[mu]
                edge = at == (n - 1 if step == 1 else 0)
                weight = torch.where(edge, BC[mu], 1.0)
                if local:
                    weight = torch.where(at % d == (d - 1 if step == 1 else 0), 0.0, weight)
                w = w * weight[..., None, None]
                w = w - step * self.phase[mu] * w[..., perm, :]
                if step == 1:
                    w = sum(self.U[mu][..., :, k].unsqueeze(-2) * w[..., k:k + 1] for k in range(3))
                out -= 0.5 * w
        return out

    def A(self, v):
        return self._site(self.C, v) + self.hops(v)

    def solve(self, b, tol=2e-14, most=3000):
        """BiCGstab."""
        dot = lambda a, c: torch.vdot(a.reshape(-1), c.reshape(-1))  # noqa: E731
        x = torch.zeros_like(b)
        for _ in range(3):   # restarts from the true residual
            r = b - self.A(x)
            r0, p, v = r.clone(), torch.zeros_like(b), torch.zeros_like(b)
            rho = alpha = omega = 1.0
            goal = tol * float(torch.linalg.vector_norm(b))
            for _ in range(most):
                if float(torch.linalg.vector_norm(r)) <= goal:
                    break
                new = dot(r0, r)
                p = r + (new / rho) * (alpha / omega) * (p - omega * v)
                v = self.A(p)
                rho, alpha = new, new / dot(r0, v)
                s = r - alpha * v
                t = self.A(s)
                omega = dot(t, s) / dot(t, t)
                x = x + alpha * p + omega * s
                r = s - omega * t
        return x

    def _domain_sum(self, v):
        """The sum of a site field over each domain, at each of its sites."""
        Lx, Ly, Lz, Lt = self.L
        bx, by, bz, bt = self.dom
        w = v.reshape(Lt // bt, bt, Lz // bz, bz, Ly // by, by, Lx // bx, bx)
        return w.sum((1, 3, 5, 7), keepdim=True).expand(w.shape).reshape(v.shape)

    def sap(self, eta, cycles, mr):
        """Multiplicative Schwarz, each block by mr minimal-residual steps on its even-site Schur complement."""
        parity = (sum(self.x) % 2)[..., None, None]
        even, odd = parity == 0, parity == 1
        colour = (sum(self.x[m] // self.dom[m] for m in range(4)) % 2)[..., None, None]
        Ci = torch.linalg.inv(self.C)
        hop = lambda v: self.hops(v, local=True)  # noqa: E731
        psi = torch.zeros_like(eta)
        for _ in range(cycles):
            for c in (0, 1):
                rho = torch.where(colour == c, eta - self.A(psi), 0)
                r = torch.where(even, rho - hop(self._site(Ci, torch.where(odd, rho, 0))), 0)
                x = torch.zeros_like(r)
                for _ in range(mr):
                    q = torch.where(odd, self._site(Ci, torch.where(odd, hop(r), 0)), 0)
                    p = torch.where(even, self._site(self.C, r) - hop(q), 0)
                    pr = self._domain_sum((p.conj() * r).sum((-1, -2)))
                    pp = self._domain_sum((p.conj() * p).sum((-1, -2)).real)
                    alpha = torch.where(pp > 0, pr / torch.where(pp > 0, pp, 1), 0)[..., None, None]
                    x, r = x + alpha * r, r - alpha * p
                y = torch.where(odd, self._site(Ci, torch.where(odd, rho - hop(x), 0)), 0)
                psi = psi + torch.where(colour == c, x + y, 0)
        return psi


def exact(case, seed, device=None):
    dev = torch.device(device or ("cuda" if torch.cuda.is_available() else "cpu"))
    kappa, csw, _ = PHYSICS[case["physics"]]
    call, out = case["call"], []
    for L, dom, U, b in _inputs(case, seed, dev):
        E = Exact(L, dom, U, kappa, csw)
        grid = (*reversed(L), 4, 3)
        fields = [v.reshape(grid) for v in b.reshape(-1, volume(L), 4, 3)]
        if call == "apply":
            got = [E.A(v) for v in fields]
        elif call == "sap":
            got = [E.sap(v, case["cycles"], case["mr"]) for v in fields]
        else:
            # two of a call's sources on the large lattices, for time
            most = 2 if volume(L) > 1 << 18 else len(fields)
            got = [E.solve(v) if k < most else None for k, v in enumerate(fields)]
        got = [v if v is None else v.reshape(volume(L), 4, 3) for v in got]
        del E, U
        if call in ("apply", "sap") and case["nrhs"] > 1:
            return torch.stack(got)
        if case["nrhs"] > 1:
            return got
        out.append(got[0])
    return out if call == "batch" else out[0]
