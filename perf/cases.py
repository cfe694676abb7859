"""Workloads that stand for what a user of this framework has it do.

Each case is one call, or the few calls of one step, through the public entry
points of ``paper_2602_20516_amd``: the operator, the solves, the forces, the
smearing, a gauge step and a trajectory, from the 4^4 lattice of the smallest
workload to the 32^3x64 of the largest.  Lattices, couplings and hopping
parameters are those of the workload table (``lgt_inputs.CONFIGS``) and of the
benchmark.  Solves are asked for a true residual at which their own truncation
error lies well below the FP64 parity bars (1e-11 to 1e-12, the tolerances at
which the benchmark and the tests compare forces).

``prepare`` builds inputs with torch alone, from the seed: links
exp(i eps sum_a c_a T_a), Gaussian eta, heat-bath phi = D^dag eta.
``exact`` evaluates the same definitions in complex128 with torch alone:
textbook CG on the full lattice, torch autograd for every force.
"""
from __future__ import annotations

import math

import torch

C128 = torch.complex128
FERMION_BC = -1  # antiperiodic in time


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one operator application on the smallest lattice: launches and host path
        dict(name="dslash_4x4x4x4", kind="dslash", dims="4x4x4x4", eps=0.5, kappa=0.12, dagger=False),
        # heat bath phi = D^dag eta (or a residual) on the large force lattice
        dict(name="dslash_24x24x24x48", kind="dslash", dims="24x24x24x48", eps=0.2, kappa=0.13, dagger=True),
        # FP64 solve of a small ensemble's lattice, X and Y = D X
        dict(name="cg_12x12x12x12_fp64", kind="cg", dims="12x12x12x12", eps=0.3, kappa=0.125,
             precision="fp64", tol=1e-11),
        # the headline: one pseudofermion force of a molecular-dynamics step
        dict(name="force_16x16x16x16_fp32", kind="force", dims="16x16x16x16", eps=0.3, kappa=0.125,
             precision="mixed_fp32", tol=1e-11),
        # the same on a lattice past the caches, BF16-stored inner vectors
        dict(name="force_24x24x24x48_bf16", kind="force", dims="24x24x24x48", eps=0.2, kappa=0.13,
             precision="mixed_bf16", tol=1e-12),
        # even/odd-preconditioned action on a lattice whose extents fit no tile
        dict(name="force_eo_10x14x6x18_fp32", kind="force_eo", dims="10x14x6x18", eps=0.3, kappa=0.125,
             precision="mixed_fp32", tol=1e-11),
        # rational (RHMC) force, 12 shifts over five decades, FP64
        dict(name="rational_16x16x16x16_12", kind="rational", dims="16x16x16x16", eps=0.3, kappa=0.125,
             nshift=12, tol=1e-11),
        # many pseudofermions: three lattices, six kappa, two sources each, in one call
        dict(name="batch_8_12_16_x12", kind="batch", dims="8x8x8x8,12x12x12x12,16x16x16x16", eps=0.3, nrhs=12,
             kappa=0.10, kappa_max=0.135, precision="mixed_fp32", tol=1e-12),
        # quenched update on the largest lattice: gauge kick and link drift, in place
        dict(name="gauge_step_32x32x32x64", kind="gauge_step", dims="32x32x32x64", eps=0.2, beta=6.0, dt=0.02),
        # smearing as an own operator uses it: links forward, gradient back
        dict(name="stout_24x24x24x48_2", kind="stout", dims="24x24x24x48", eps=0.2, rho=0.1, nlevels=2),
        # force of the smeared action on the largest lattice, below its critical kappa
        dict(name="smeared_32x32x32x64_2", kind="smeared", dims="32x32x32x64", eps=0.2, beta=6.0, kappa=0.12,
             rho=0.1, nlevels=2, precision="mixed_fp32", tol=1e-11),
        # a leapfrog trajectory of a small HMC chain, with its Delta H
        dict(name="trajectory_8x8x8x8_fp32", kind="trajectory", dims="8x8x8x8", eps=0.5, beta=5.7, kappa=0.12,
             dt=0.05, nsteps=4, precision="mixed_fp32", tol=1e-12),
    ]


# largest volume a drawn case of each kind may take (sites), and its smallest
_RANGE = {"dslash": (128, 1 << 20), "cg": (256, 1 << 17), "force": (256, 1 << 18), "force_eo": (256, 1 << 18),
          "rational": (256, 1 << 16), "batch": (256, 1 << 16), "gauge_step": (256, 1 << 20),
          "stout": (256, 1 << 18), "smeared": (256, 1 << 18), "trajectory": (256, 1 << 14)}


def _draw_dims(rng, lo, hi):
    """Even extents whose product is near a volume drawn over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = v ** 0.25
    dims = [max(2, 2 * round(0.5 * side * math.exp(rng.uniform(-0.5, 0.5)))) for _ in range(3)]
    dims[0] = max(dims[0], 4)
    dims.append(max(2, 2 * round(0.5 * v / (dims[0] * dims[1] * dims[2]))))
    while math.prod(dims) > hi:
        dims[dims.index(max(dims))] -= 2
    return "x".join(str(d) for d in dims)


def draw(rng):
    kind = rng.choice(sorted(_RANGE))
    c = dict(kind=kind, dims=_draw_dims(rng, *_RANGE[kind]), eps=round(rng.uniform(0.3, 0.5), 3))
    kappa = round(rng.uniform(0.105, 0.125), 4)
    if kind == "dslash":
        c |= dict(kappa=kappa, dagger=rng.random() < 0.5)
    elif kind == "cg":
        c |= dict(kappa=kappa, precision=rng.choice(["fp64", "mixed_fp32", "mixed_bf16"]), tol=1e-12)
    elif kind in ("force", "force_eo"):
        c |= dict(kappa=kappa, precision=rng.choice(["fp64", "mixed_fp32", "mixed_bf16"]), tol=1e-12)
    elif kind == "rational":
        c |= dict(kappa=kappa, nshift=rng.randint(1, 16), tol=1e-12)
    elif kind == "batch":
        c |= dict(nrhs=rng.randint(1, 16), kappa=0.10, kappa_max=kappa, precision=rng.choice(["fp64", "mixed_fp32"]),
                  tol=1e-12)
    elif kind == "gauge_step":
        c |= dict(beta=round(rng.uniform(5.5, 6.5), 2), dt=round(rng.uniform(0.005, 0.02), 4))
    elif kind == "stout":
        c |= dict(rho=round(rng.uniform(0.05, 0.15), 3), nlevels=rng.randint(1, 6))
    elif kind == "smeared":
        c |= dict(beta=6.0, kappa=min(kappa, 0.115), rho=round(rng.uniform(0.05, 0.12), 3), nlevels=rng.randint(1, 4),
                  precision=rng.choice(["fp64", "mixed_fp32"]), tol=1e-12)
    else:
        c |= dict(beta=5.7, kappa=min(kappa, 0.12), dt=0.05, nsteps=rng.randint(1, 4),
                  precision=rng.choice(["fp64", "mixed_fp32"]), tol=1e-12)
    return c


def _dims(text):
    return tuple(int(d) for d in text.split("x"))


def _lattices(case):
    return [_dims(t) for t in case["dims"].split(",")]


def _shifts(n):
    """Shifts 1e-4 to 10, evenly over the logarithm, and residues of a rational function."""
    s = [10.0 ** (-4.0 + 5.0 * i / max(1, n - 1)) for i in range(n)]
    return s, [0.1 * math.sqrt(v) for v in s]


def _kappas(case):
    n, lo, hi = case["nrhs"], case["kappa"], case["kappa_max"]
    m = max(1, (n + 1) // 2)  # two sources a kappa
    return [lo + (hi - lo) * (i // 2) / max(1, m - 1) for i in range(n)]


# ---------------------------------------------------------------------------
# Compulsory work of one pass: inputs read and outputs written once, and the
# arithmetic of the operator applications and link products it stands for.
# ---------------------------------------------------------------------------
_HOP = 1320.0            # flop of one site's eight hops
_D = _HOP + 48.0         # D on one site
_STAPLE = 10800.0        # staple force of one site (four links)
_BILINEAR = 4 * 700.0    # outer products, link product and projection
_LINK, _SPINOR = 576.0, 192.0  # canonical bytes per site


def _iterations(case):
    """CG iterations of the two Schur solves at this tolerance, an estimate."""
    k = case.get("kappa_max", case["kappa"])
    return (120.0 if k <= 0.12 else 160.0 if k <= 0.128 else 400.0 if case["eps"] < 0.25 else 220.0) * \
        (-math.log10(case["tol"]) / 11.0)


def work(case):
    V = sum(math.prod(d) for d in _lattices(case))
    kind = case["kind"]
    iteration = 2 * _D * V  # Mhat^dag Mhat: four half-lattice hops and the updates
    if kind == "dslash":
        return dict(bytes=V * (_LINK + 2 * _SPINOR), flops=V * _D)
    if kind == "cg":
        return dict(bytes=V * (_LINK + 3 * _SPINOR), flops=_iterations(case) * iteration)
    if kind == "batch":
        n = case["nrhs"]
        return dict(bytes=V * (_LINK + 2 * n * _SPINOR), flops=0.7 * n * _iterations(case) * iteration)
    if kind == "force":
        return dict(bytes=V * (2 * _LINK + _SPINOR), flops=_iterations(case) * iteration + V * _BILINEAR)
    if kind == "force_eo":
        return dict(bytes=V * (2 * _LINK + _SPINOR), flops=0.5 * _iterations(case) * iteration + V * _BILINEAR)
    if kind == "rational":
        n = case["nshift"]
        return dict(bytes=V * (2 * _LINK + _SPINOR),
                    flops=(0.5 * _iterations(case) + 2 * n) * iteration + n * V * _BILINEAR)
    if kind == "gauge_step":
        return dict(bytes=V * 4 * _LINK, flops=V * (_STAPLE + 4 * 900.0))
    level = V * 13800.0, V * 43000.0  # smearing of one level, its adjoint
    if kind == "stout":
        return dict(bytes=V * 4 * _LINK, flops=case["nlevels"] * sum(level))
    if kind == "smeared":
        return dict(bytes=V * (2 * _LINK + _SPINOR),
                    flops=case["nlevels"] * sum(level) + V * (_STAPLE + _BILINEAR) + _iterations(case) * iteration)
    n = case["nsteps"]
    return dict(bytes=V * (4 * _LINK + _SPINOR),
                flops=(n + 1) * (V * (_STAPLE + _BILINEAR) + _iterations(case) * iteration) + n * V * 4 * 900.0)


# ---------------------------------------------------------------------------
# Inputs, in plain torch on the GPU
# ---------------------------------------------------------------------------
_AXIS = (3, 2, 1, 0)  # direction x, y, z, t -> axis of the (Lt, Lz, Ly, Lx) site array


def _mul(a, b):
    """Product of stacked 3x3 matrices."""
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _dag(a):
    return a.conj().transpose(-1, -2)


def _su3_algebra(c):
    """i sum_a c_a lambda_a / 2 from coefficients [..., 8]."""
    h = torch.zeros(c.shape[:-1] + (3, 3), dtype=C128, device=c.device)
    r3 = 1.0 / math.sqrt(3.0)
    h[..., 0, 0], h[..., 1, 1], h[..., 2, 2] = c[..., 2] + r3 * c[..., 7], -c[..., 2] + r3 * c[..., 7], -2 * r3 * c[..., 7]
    for i, j, a in ((0, 1, 0), (0, 2, 3), (1, 2, 5)):
        h[..., i, j] = torch.complex(c[..., a], -c[..., a + 1])
        h[..., j, i] = torch.complex(c[..., a], c[..., a + 1])
    return 0.5j * h


def _expm(x):
    """exp of stacked 3x3 matrices of norm up to about 4: Taylor, scaled and squared."""
    one = torch.eye(3, dtype=C128, device=x.device)
    y, s = x / 16.0, one
    for k in range(12, 0, -1):
        s = one + _mul(y, s) / k
    for _ in range(4):
        s = _mul(s, s)
    return s


def _unitary(u):
    """Rows 1, 2 by Gram-Schmidt, row 3 the conjugate cross product."""
    a = u[..., 0, :] / torch.linalg.vector_norm(u[..., 0, :], dim=-1, keepdim=True)
    b = u[..., 1, :] - (a.conj() * u[..., 1, :]).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack((a, b, torch.linalg.cross(a, b).conj()), dim=-2).contiguous()


def _generator(seed, salt):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 64 + salt)


def _shape(dims):
    return tuple(reversed(dims))


def _normals(shape, g):
    return torch.randn(shape, generator=g, dtype=torch.float64, device="cuda")


def _links(dims, eps, g):
    return _unitary(_expm(eps * _su3_algebra(_normals(_shape(dims) + (4, 8), g))))


def _eta(dims, g):
    shape = _shape(dims) + (4, 3)
    return torch.complex(_normals(shape, g), _normals(shape, g)) / math.sqrt(2.0)


def _colour(u, p):
    """U_ij p_sj for every spin s."""
    return sum(u[..., None, :, j] * p[..., :, j, None] for j in range(3))


def _colour_dag(u, p):
    return sum(u[..., None, j, :].conj() * p[..., :, j, None] for j in range(3))


def _b(mu, d, adjoint=False):
    """The off-diagonal block of gamma_mu (upper right; its adjoint: lower left) on two spins d."""
    s = 1j if adjoint else -1j
    d0, d1 = d[..., 0, :], d[..., 1, :]
    if mu == 0:
        v = (s * d1, s * d0)
    elif mu == 1:
        v = (d1, -d0) if adjoint else (-d1, d0)
    elif mu == 2:
        v = (s * d0, -s * d1)
    else:
        return d
    return torch.stack(v, dim=-2)


def _bc_links(u):
    """Links with the fermion boundary sign folded into the last time slice."""
    v = u.clone()
    v[-1, :, :, :, 3] *= FERMION_BC
    return v


def _hop(ub, p, dagger=False):
    """sum_mu (1 - gamma) U p(x+mu) + (1 + gamma) U^dag p(x-mu); dagger flips the gammas.

    ub: links with the boundary sign; leading axes of p before the site axes are batched."""
    out = torch.zeros_like(p)
    for mu in range(4):
        ax = _AXIS[mu] - 6  # counted from the end of [..., t, z, y, x, spin, colour]
        u = ub[..., mu, :, :]
        for forward in (True, False):
            s = (1.0 if dagger else -1.0) * (1.0 if forward else -1.0)
            h = p[..., 0:2, :] + s * _b(mu, p[..., 2:4, :])
            w = _colour(u, torch.roll(h, -1, ax)) if forward else torch.roll(_colour_dag(u, h), 1, ax)
            out[..., 0:2, :] += w
            out[..., 2:4, :] += s * _b(mu, w, adjoint=True)
    return out


def _dslash(ub, p, kappa, dagger=False):
    return p - kappa * _hop(ub, p, dagger)


def _parity(dims, odd):
    grid = sum(torch.arange(n, device="cuda").reshape([-1 if i == k else 1 for k in range(4)])
               for i, n in enumerate(_shape(dims)))
    return ((grid % 2) == (1 if odd else 0)).to(torch.float64)[..., None, None]


def _schur(ub, p, kappa, odd, dagger=False):
    return p - kappa ** 2 * odd * _hop(ub, (1.0 - odd) * _hop(ub, p, dagger), dagger)


def _stout(u, rho, nlevels):
    for _ in range(nlevels):
        x = -rho * _traceless(_mul(u, _staples(u)))
        u = _mul(_expm(x), u)
    return u


def _traceless(a):
    """(A - A^dag)/2 - tr(A - A^dag)/6."""
    h = 0.5 * (a - _dag(a))
    tr = h.diagonal(dim1=-2, dim2=-1).sum(-1) / 3.0
    return h - tr[..., None, None] * torch.eye(3, dtype=C128, device=a.device)


def _staples(u):
    """A_mu(x) with sum of plaquettes through the link = Re tr(U A)."""
    out = []
    for mu in range(4):
        am, um = _AXIS[mu], u[..., mu, :, :]
        total = 0
        for nu in range(4):
            if nu == mu:
                continue
            an, un = _AXIS[nu], u[..., nu, :, :]
            un_m = torch.roll(un, -1, am)
            total = total + _mul(_mul(un_m, _dag(torch.roll(um, -1, an))), _dag(un))
            low = _mul(_mul(_dag(un_m), _dag(um)), un)
            total = total + torch.roll(low, 1, an)
        out.append(total)
    return torch.stack(out, dim=-3)


def _inputs(case, seed):
    """The fields of one case, from the seed alone."""
    kind, out = case["kind"], []
    for n, dims in enumerate(_lattices(case)):
        g = _generator(seed, n)
        d = dict(dims=dims, U=_links(dims, case["eps"], g))
        if kind in ("gauge_step", "trajectory"):
            d["P"] = _su3_algebra(_normals(_shape(dims) + (4, 8), g))
        if kind == "stout":
            d["G"] = torch.complex(_normals(d["U"].shape, g), _normals(d["U"].shape, g))
        if kind == "dslash":
            d["psi"] = _eta(dims, g)
        if kind in ("cg", "force", "trajectory"):
            d["phi"] = _dslash(_bc_links(d["U"]), _eta(dims, g), case["kappa"], dagger=True)
        if kind == "smeared":
            d["phi"] = _dslash(_bc_links(_stout(d["U"], case["rho"], case["nlevels"])), _eta(dims, g), case["kappa"],
                               dagger=True)
        if kind in ("force_eo", "rational"):
            odd = _parity(dims, True)
            d["phi"] = _schur(_bc_links(d["U"]), odd * _eta(dims, g), case["kappa"], odd, dagger=True)
        if kind == "batch":
            ub = _bc_links(d["U"])
            d["phis"] = [_dslash(ub, _eta(dims, g), k, dagger=True) for k in _kappas(case)]
        out.append(d)
    return out


# ---------------------------------------------------------------------------
# The framework
# ---------------------------------------------------------------------------
_handles = {}  # dims -> Lattice: the handles of the current program


def _lattice(dims):
    """The handle for one geometry; a program keeps one and feeds it configuration after configuration."""
    import paper_2602_20516_amd as lgt
    if dims not in _handles:
        if len(_handles) >= 3:
            _handles.clear()
        _handles[dims] = lgt.Lattice(dims, FERMION_BC)
    return _handles[dims]


def _params(case):
    import paper_2602_20516_amd as lgt
    return lgt.Params(precision=case.get("precision", "fp64"), tol=case["tol"])


def prepare(case, seed):
    import paper_2602_20516_amd as lgt
    fields = _inputs(case, seed)
    torch.cuda.empty_cache()  # the inputs' temporaries
    s = dict(case=dict(case), fields=fields, lat=[_lattice(d["dims"]) for d in fields])
    if "tol" in case:
        s["params"] = _params(case)
    if case["kind"] == "batch":
        s["batch"] = lgt.Batch()
    if case["kind"] == "rational":
        s["shifts"] = _shifts(case["nshift"])
    if case["kind"] in ("force", "force_eo", "rational", "smeared"):
        s["out"] = torch.empty_like(fields[0]["U"])
    return s


def run(s):
    c, lat, f = s["case"], s["lat"][0], s["fields"][0]
    kind, U = c["kind"], f["U"]
    if kind == "dslash":
        return lat.dslash(U, f["psi"], c["kappa"], dagger=c["dagger"])
    if kind == "cg":
        X, Y, _ = lat.cg_solve(U, f["phi"], c["kappa"], s["params"])
        return X, Y
    if kind == "force":
        return lat.fermion_force(U, f["phi"], c["kappa"], s["params"], out=s["out"])[0]
    if kind == "force_eo":
        return lat.fermion_force_eo(U, f["phi"], c["kappa"], s["params"], out=s["out"])[:2]
    if kind == "rational":
        return lat.rational_force_eo(U, f["phi"], c["kappa"], *s["shifts"], params=s["params"], out=s["out"])[:2]
    if kind == "batch":
        items = [(l, d["U"], phi, k) for l, d in zip(s["lat"], s["fields"])
                 for phi, k in zip(d["phis"], _kappas(c))]
        return s["batch"].cg_solve(items, s["params"], want_y=False)[0]
    if kind == "gauge_step":
        lat.gauge_force(U, c["beta"], mode="momentum", dt=c["dt"], out=f["P"])
        lat.link_update(U, f["P"], c["dt"])
        return U, f["P"]
    if kind == "stout":
        top = lat.stout_smear(U, c["rho"], c["nlevels"])
        return top, lat.stout_backprop(U, f["G"], c["rho"], c["nlevels"])
    if kind == "smeared":
        return lat.smeared_force(U, f["phi"], c["beta"], c["kappa"], c["rho"], c["nlevels"], s["params"],
                                 out=s["out"])[:2]
    # a trajectory keeps its start for the Metropolis step
    U, P = U.clone(), f["P"].clone()
    dh, _ = lat.md_step(U, P, f["phi"], c["beta"], c["kappa"], c["dt"], c["nsteps"], s["params"])
    return U, P, dh


# ---------------------------------------------------------------------------
# The same in 64 bits, by definition
# ---------------------------------------------------------------------------
_SITES = (-6, -5, -4, -3, -2, -1)


def _dot(a, b):
    """Re <a, b> over the site axes, one value per leading index."""
    return (a.real * b.real + a.imag * b.imag).sum(dim=_SITES, keepdim=True)


def _cg(apply, b, tol=3e-15, most=6000):
    """CG for a Hermitian positive operator, restarted from the true residual until that is at rounding."""
    x = torch.zeros_like(b)
    bb = _dot(b, b)
    for _ in range(3):
        r = b - apply(x)
        p, rr = r, _dot(r, r)
        start = rr
        for n in range(most):
            if n % 8 == 0 and bool((rr <= torch.maximum(tol ** 2 * bb, 1e-26 * start)).all()):
                break
            q = apply(p)
            a = rr / _dot(p, q)
            a = torch.where(rr > 0, a, torch.zeros_like(a))
            x = x + a * p
            r = r - a * q
            new = _dot(r, r)
            p = r + torch.where(rr > 0, new / rr, torch.zeros_like(rr)) * p
            rr = new
    return x


def _solve(ub, phi, kappa):
    """X = (D^dag D)^-1 phi; kappa may be one value per leading index of phi."""
    return _cg(lambda v: _dslash(ub, _dslash(ub, v, kappa), kappa, True), phi)


def _solve_schur(ub, phi, kappa, odd, shift=0.0):
    def normal(v):
        return _schur(ub, _schur(ub, v, kappa, odd), kappa, odd, True) + shift * v
    return _cg(normal, odd * phi)


def _gradient(scalar, u):
    """dS/dRe U + i dS/dIm U of a real scalar function of the links."""
    v = u.detach().clone().requires_grad_(True)
    with torch.enable_grad():
        scalar(v).backward()
    return v.grad


def _to_force(u, grad):
    return -0.5 * _traceless(_mul(u, _dag(grad)))


def _inner(a, b):
    return (a.conj() * b).sum().real


def _fermion_grad(u, x, kappa):
    """Gradient of S_f at the solution x: -2 Re[(D x)^dag (dD) x]."""
    y = _dslash(_bc_links(u), x, kappa)
    return _gradient(lambda v: -2.0 * _inner(y, _dslash(_bc_links(v), x, kappa)), u)


def _gauge_force(u, beta):
    return (beta / 6.0) * _traceless(_mul(u, _staples(u)))


def _gauge_action(u, beta):
    tr = 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a = _mul(u[..., mu, :, :], torch.roll(u[..., nu, :, :], -1, _AXIS[mu]))
            b = _mul(u[..., nu, :, :], torch.roll(u[..., mu, :, :], -1, _AXIS[nu]))
            tr = tr + (a.conj() * b).sum().real
    return beta * (6.0 * math.prod(u.shape[:4]) - tr / 3.0)


def _kinetic(p):
    return -_mul(p, p).diagonal(dim1=-2, dim2=-1).sum().real


def _drift(u, p, dt):
    return _unitary(_mul(_expm(dt * p), u))


def _exact_trajectory(c, f):
    U, P, phi = f["U"], f["P"], f["phi"]
    beta, kappa, dt = c["beta"], c["kappa"], c["dt"]

    def kick(u, p, h):
        x = _solve(_bc_links(u), phi, kappa)
        return p - h * (_gauge_force(u, beta) + _to_force(u, _fermion_grad(u, x, kappa))), _inner(phi, x)

    u, p = U, P
    p, sf0 = kick(u, p, 0.5 * dt)
    for k in range(c["nsteps"]):
        u = _drift(u, p, dt)
        p, sf1 = kick(u, p, 0.5 * dt if k == c["nsteps"] - 1 else dt)
    dh = (_kinetic(p) - _kinetic(P)) + (_gauge_action(u, beta) - _gauge_action(U, beta)) + (sf1 - sf0)
    return u, p, float(dh)


@torch.no_grad()
def exact(case, seed):
    V = sum(math.prod(d) for d in _lattices(case))
    kind = case["kind"]
    if kind == "smeared" and V > 1 << 19:
        return None  # CG and the autograd of the smearing take over 20 seconds
    fs = _inputs(case, seed)
    f, c = fs[0], case
    U = f["U"]
    if kind == "dslash":
        return _dslash(_bc_links(U), f["psi"], c["kappa"], c["dagger"])
    if kind == "cg":
        ub = _bc_links(U)
        X = _solve(ub, f["phi"], c["kappa"])
        return X, _dslash(ub, X, c["kappa"])
    if kind == "force":
        return _to_force(U, _fermion_grad(U, _solve(_bc_links(U), f["phi"], c["kappa"]), c["kappa"]))
    if kind in ("force_eo", "rational"):
        odd, ub = _parity(f["dims"], True), _bc_links(U)
        shifts, residues = _shifts(c["nshift"]) if kind == "rational" else ([0.0], [1.0])
        grad, action = 0.0, 0.0
        for s, a in zip(shifts, residues):
            x = _solve_schur(ub, f["phi"], c["kappa"], odd, s)
            y = _schur(ub, x, c["kappa"], odd)
            grad = grad + a * _gradient(
                lambda v: -2.0 * _inner(y, _schur(_bc_links(v), x, c["kappa"], odd)), U)
            action += a * float(_inner(odd * f["phi"], x))
        return _to_force(U, grad), action
    if kind == "batch":
        out = []
        for d in fs:
            k = torch.tensor(_kappas(c), dtype=torch.float64, device="cuda").reshape(-1, 1, 1, 1, 1, 1, 1)
            out += list(_solve(_bc_links(d["U"]), torch.stack(d["phis"]), k).unbind(0))
        return out
    if kind == "gauge_step":
        P = f["P"] - c["dt"] * _gauge_force(U, c["beta"])
        return _drift(U, P, c["dt"]), P
    if kind in ("stout", "smeared"):
        levels = [U]
        for _ in range(c["nlevels"]):
            levels.append(_stout(levels[-1], c["rho"], 1))
        if kind == "stout":
            grad = f["G"]
        else:
            x = _solve(_bc_links(levels[-1]), f["phi"], c["kappa"])
            grad = _fermion_grad(levels[-1], x, c["kappa"])
        for u in reversed(levels[:-1]):
            g = grad
            grad = _gradient(lambda v: _inner(g, _stout(v, c["rho"], 1)), u)
        if kind == "stout":
            return levels[-1], grad
        return _to_force(U, grad) + _gauge_force(U, c["beta"]), float(_inner(f["phi"], x))
    return _exact_trajectory(c, f)
