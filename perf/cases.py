"""Timed cases of the library: what a Chebyshev-BdG program calls, over the
sizes it calls it with.

Six kinds of pass:
  scf       one iteration of the self-consistency loop's body: the operator
            takes the present order parameter, moments of every site, gap
            update (T > 0: with its coefficients, and the electron density)
  moments   moments of one tile of start sites (real or complex operators,
            FP64 or FP32 recursion)
  ldos      moments of a set of sites and their local density of states
  gradient  moments and gap map (or LDOS) through torch.autograd, forward
            and backward, down to the potential and the order parameter
  jacobian  the rows of a tile of the gap map's Jacobian and one product
            with it (a Newton step's work)
  bond      one iteration of the bond order parameter's loop: neighbour
            moments, bond gap update, bond currents
"""
import math

import numpy as np
import torch

import paper_1007_1609_amd as P
from paper_1007_1609_amd import autograd as AG

DEV = "cuda"


def _case(kind, Lx, Ly, N, n_sites, **kw):
    c = dict(kind=kind, Lx=Lx, Ly=Ly, N=N, n_sites=min(n_sites, Lx * Ly), tile=1024, bc_x=0, bc_y=0, cplx=False, fp32=False, T=0.0,
             n_E=0, lorentz=False, loss="gap")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest solve: a 16x16 lattice with one impurity, every site in one tile
        _case("scf", 16, 16, 256, 256, tile=256, name="scf_16x16"),
        # a periodic supercell of ordinary size at finite temperature, with the density
        _case("scf", 96, 72, 384, 96 * 72, bc_x=1, bc_y=1, T=0.05, name="scf_96x72_thermal"),
        # one tile of the large disordered solve in FP64: the workload that bench.py repeats
        _case("moments", 256, 256, 1024, 1024, name="moments_256x256_fp64"),
        # the same lattice at twice the resolution with the FP32 recursion
        _case("moments", 256, 256, 2048, 1024, fp32=True, name="moments_256x256_fp32"),
        # LDOS map around an impurity of a 150x100 sandwich: sizes that fit no power of two
        _case("ldos", 150, 100, 2048, 441, n_E=201, name="ldos_150x100"),
        # surface LDOS of a wide planar system: few start sites, the Lorentz kernel
        _case("ldos", 400, 500, 2000, 64, bc_y=1, n_E=401, lorentz=True, name="ldos_400x500_surface"),
        # the vortex lattice: flux and d-wave bonds, complex128, a grid of sites
        _case("moments", 512, 512, 256, 256, cplx=True, name="moments_512x512_complex"),
        # a complex operator of ordinary size with the reduced-precision recursion
        _case("moments", 160, 120, 512, 512, cplx=True, fp32=True, name="moments_160x120_complex32"),
        # one tile of the differentiation workload: d(sum of Delta)/dV and /dDelta
        _case("gradient", 128, 128, 512, 1024, name="gradient_128x128"),
        # gradient of LDOS values on a lattice of odd width
        _case("gradient", 91, 70, 256, 300, loss="ldos", n_E=33, name="gradient_91x70_ldos"),
        # a Newton step's rows of the Jacobian, and a product with them
        _case("jacobian", 128, 128, 512, 1024, name="jacobian_128x128"),
        # one iteration of the d-wave bond loop in a field, with the currents
        _case("bond", 48, 40, 256, 48 * 40, cplx=True, name="bond_48x40_dwave"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    cap = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= cap:
            return c


def _draw(rng):
    kind = rng.choice(["scf", "scf", "moments", "moments", "moments", "ldos", "ldos", "gradient", "jacobian", "bond"])
    bc = dict(bc_x=rng.randint(0, 1), bc_y=rng.randint(0, 1))
    if kind == "scf":  # every site of the lattice
        Lx, Ly = _log_int(rng, 12, 130), _log_int(rng, 12, 130)
        return _case(kind, Lx, Ly, _log_int(rng, 128, 512), Lx * Ly, T=rng.choice([0.0, rng.uniform(0.02, 0.2)]),
                     tile=rng.choice([256, 1024]), fp32=rng.random() < 0.25, **bc)
    if kind == "moments":
        cplx = rng.random() < 0.35
        # half of the real lattices a multiple of 64 wide, as large lattices are chosen
        Lx = 64 * rng.choice([1, 2, 4]) if rng.random() < 0.5 and not cplx else _log_int(rng, 24, 512 if cplx else 300)
        Ly = _log_int(rng, 24, 400)
        return _case(kind, Lx, Ly, _log_int(rng, 64, 2048), _log_int(rng, 1, 1024), cplx=cplx, fp32=rng.random() < 0.4,
                     **bc)
    if kind == "ldos":
        return _case(kind, _log_int(rng, 60, 420), _log_int(rng, 60, 520), _log_int(rng, 512, 4096), _log_int(rng, 1, 450),
                     n_E=_log_int(rng, 3, 512), lorentz=rng.random() < 0.5, fp32=rng.random() < 0.2, **bc)
    if kind == "gradient":
        Lx = 64 * rng.choice([1, 2]) if rng.random() < 0.5 else _log_int(rng, 16, 140)
        return _case(kind, Lx, _log_int(rng, 16, 140), _log_int(rng, 32, 512), _log_int(rng, 16, 1024),
                     n_E=_log_int(rng, 1, 64), loss=rng.choice(["gap", "ldos"]), **bc)
    if kind == "jacobian":
        return _case(kind, 64 * rng.choice([1, 2, 4]), _log_int(rng, 32, 160), _log_int(rng, 64, 512),
                     _log_int(rng, 64, 1024), **bc)
    Lx, Ly = _log_int(rng, 8, 56), _log_int(rng, 8, 56)
    return _case("bond", Lx, Ly, _log_int(rng, 64, 384), Lx * Ly, cplx=rng.random() < 0.6, **bc)


# ---------------------------------------------------------------- inputs

U, MU, HOP, ETA = 2.5, -0.4, 1.0, 0.01


def _fields(case, seed):
    """The lattice's coefficients and the start sites, as numpy arrays."""
    rng = np.random.default_rng(seed)
    Lx, Ly, n = case["Lx"], case["Ly"], case["n_sites"]
    L2 = Lx * Ly
    eps = np.zeros(L2)
    where = rng.choice(L2, max(1, L2 // 100), replace=False)
    eps[where] = rng.uniform(-2.0, 2.0, len(where))
    f = dict(eps=eps, delta=0.1 * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, L2)), bond=None, peierls=None)
    if case["cplx"] or case["kind"] == "bond":
        # d-wave bonds, in a field with a winding phase; bonds leaving an open lattice are zero
        x, y = np.tile(np.arange(Lx), Ly), np.repeat(np.arange(Ly), Lx)
        amp = 0.1 * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, (2, L2)))
        amp[1] *= -1.0
        amp[0][(x == Lx - 1) & (case["bc_x"] == 0)] = 0.0
        amp[1][(y == Ly - 1) & (case["bc_y"] == 0)] = 0.0
        f["delta"] = np.zeros(L2)
        f["bond"] = amp
        if case["cplx"]:
            phase = np.arctan2(y - Ly / 2.0 + 0.25, x - Lx / 2.0 + 0.25)
            f["bond"] = amp * np.exp(1j * phase)
            f["delta"] = 0.02 * np.exp(1j * (phase + rng.uniform(-0.1, 0.1, L2)))
            f["peierls"] = np.stack([-np.pi * y / 256.0, np.zeros(L2)])
    if n >= L2:
        f["sites"] = np.arange(L2)
    elif case["kind"] in ("ldos", "moments") and (case["cplx"] or case["lorentz"]):
        f["sites"] = np.sort(rng.choice(L2, n, replace=False))
    else:  # a run of the solve's tiles
        f["sites"] = (int(rng.integers(0, L2 - n + 1)) + np.arange(n)) % L2
    f["sites"] = f["sites"].astype(np.int32)
    # Gershgorin bound with the order parameter raised to its largest iterate
    rows = np.abs(eps - MU) + np.maximum(np.abs(f["delta"]), 0.5 * U) + 4.0 * HOP
    if f["bond"] is not None:
        rows = rows + 4.0 * np.abs(f["bond"]).max()
    f["a"] = float(2.0 * rows.max() / (2.0 - ETA))
    f["cot"] = rng.uniform(0.5, 1.5, (case["n_sites"], max(1, case["n_E"])))
    f["vec"] = rng.standard_normal(L2)
    f["energies"] = np.linspace(-0.6 * f["a"], 0.6 * f["a"], case["n_E"]) if case["n_E"] else None
    return f


def _lam(case, a):  # broadening 0.004 in units of the hopping
    return max(3.0, case["N"] * 0.004 / a)


def prepare(case, seed):
    f = _fields(case, seed)
    cd = torch.complex128 if case["cplx"] else torch.float64
    dev = lambda v, dt: None if v is None else torch.as_tensor(v, dtype=dt, device=DEV).contiguous()  # noqa: E731
    N, n, tile = case["N"], case["n_sites"], min(case["tile"], case["n_sites"])
    prec = P.CBDG_FP32_ACC64 if case["fp32"] else P.CBDG_FP64
    s = dict(case=case, N=N, tile=tile, prec=prec, sites=dev(f["sites"], torch.int32), eps=dev(f["eps"], torch.float64),
             delta=dev(f["delta"], cd), energies=dev(f["energies"], torch.float64),
             w=P.weights(f["a"], 0.0, "lorentz" if case["lorentz"] else "jackson",
                         _lam(case, f["a"]) if case["lorentz"] else 0.0, case["T"]))
    if case["kind"] == "gradient":
        s["geom"] = AG.Geometry(case["Lx"], case["Ly"], HOP, MU, f["a"], 0.0, case["bc_x"], case["bc_y"])
        s["delta_in"] = s["delta"][s["sites"].long()].contiguous()
        s["cot"] = dev(f["cot"] if case["loss"] == "ldos" else f["cot"][:, 0], torch.float64)
        s["eps"].requires_grad_(True)
        s["delta"].requires_grad_(True)
        return s
    bond = dev(None if f["bond"] is None else f["bond"].reshape(-1), cd)
    s["op"] = P.Operator(case["Lx"], case["Ly"], HOP, MU, s["eps"], s["delta"], bond,
                         dev(None if f["peierls"] is None else f["peierls"].reshape(-1), torch.float64),
                         bc_x=case["bc_x"], bc_y=case["bc_y"], complex_=case["cplx"], fixed=(f["a"], 0.0))
    if case["kind"] == "jacobian":
        s["ws"] = P.workspace(P.backward_workspace_bytes(s["op"], tile, N, P.REVERSIBLE, P.CBDG_ALG_DOUBLING), DEV)
        s["ones"] = torch.ones(n, dtype=torch.float64, device=DEV)
        s["jac"] = torch.empty((n, s["op"].L2), dtype=torch.float64, device=DEV)
        s["vec"] = dev(f["vec"], torch.float64)
        return s
    s["out"] = (torch.empty((n, N), dtype=torch.float64, device=DEV), torch.empty((n, N), dtype=cd, device=DEV))
    if case["kind"] == "bond":
        s["ws"] = P.workspace(P.moments_workspace_bytes(s["op"], tile, prec, P.CBDG_ALG_DIRECT), DEV)
        s["bond"] = bond
        s["occ"] = P.sum_coefficients(s["w"], N, P.CBDG_QTY_DENSITY, DEV)
    else:
        s["ws"] = P.workspace(P.moments_workspace_bytes(s["op"], tile, prec), DEV)
    if case["kind"] == "scf":
        s["next"] = torch.empty_like(s["delta"])
        s["resid"] = torch.empty(1, dtype=torch.float64, device=DEV)
        if case["T"] > 0.0:
            s["coeff"] = P.sum_coefficients(s["w"], N, P.CBDG_QTY_GAP, DEV)
            s["occ"] = P.sum_coefficients(s["w"], N, P.CBDG_QTY_DENSITY, DEV)
    return s


def run(s):
    kind, N, tile = s["case"]["kind"], s["N"], s["tile"]
    if kind == "gradient":
        mu_ee, mu_he = AG.moments(s["eps"], s["delta"], s["geom"], s["sites"], N, tile)
        if s["case"]["loss"] == "ldos":
            out = AG.local_dos(mu_ee, s["energies"], s["w"])
        else:
            out = AG.gap_map(mu_he, s["delta_in"], U, s["w"])
        grads = torch.autograd.grad(out, [s["eps"], s["delta"]], s["cot"])
        return {"out": out.detach(), "eps": grads[0], "delta": grads[1]}
    op, w = s["op"], s["w"]
    if kind == "jacobian":
        dmu, _ = P.gap_update_backward(s["ones"], N, w, U, want_delta_in=False)
        P.chebyshev_moments_jacobian(op, s["sites"], N, tile, None, dmu, jac_delta=s["jac"], ws=s["ws"])
        return {"rows": s["jac"], "product": P.jacobian_matvec(s["jac"], s["vec"])}
    if kind == "bond":
        mu_ee, mu_he, nb_ee, nb_he = P.chebyshev_moments_nb(op, s["sites"], N, tile, s["prec"], ws=s["ws"])
        bond, resid = P.bond_gap_update(nb_he, op, w, U, s["bond"])
        cur = P.bond_current(op, nb_ee, w, s["occ"])
        return {"mu_ee": mu_ee, "mu_he": mu_he, "nb_ee": nb_ee, "nb_he": nb_he, "bond": bond, "resid": resid, "current": cur}
    if kind == "scf":
        op.update_delta(s["delta"])
    mu_ee, mu_he = P.chebyshev_moments(op, s["sites"], N, tile, s["prec"], ws=s["ws"], out=s["out"])
    out = {"mu_ee": mu_ee, "mu_he": mu_he}
    if kind == "scf":
        out["delta"], out["resid"] = P.gap_update(mu_he, w, U, s["delta"], delta_out=s["next"], resid=s["resid"],
                                                  coeff=s.get("coeff"))
        if s["case"]["T"] > 0.0:
            out["density"] = P.density(mu_ee, w, s["occ"])
    elif kind == "ldos":
        out["ldos"] = P.ldos(mu_ee, w, s["energies"])
    return out


# ---------------------------------------------------------------- work


def _site_steps(case):
    """Sites of the recursion vectors that can differ from zero, summed over
    steps and start sites: a_n lives within n steps of its start site.  Moment
    doubling takes N/2 steps; neighbour moments need all N - 1."""
    steps = case["N"] - 1 if case["kind"] == "bond" else case["N"] // 2
    m = np.arange(1, steps + 1, dtype=np.float64)
    return float(np.minimum(2 * m * m + 2 * m + 1, case["Lx"] * case["Ly"]).sum()) * case["n_sites"]


def _flops(case):
    """Per site and step: the 2x2 stencil on four neighbours and the doubling
    sums (real 30, complex with bonds 190); backward: the forward vectors again,
    the transposed recursion, its sources and the gradient terms."""
    per = 190.0 if case["cplx"] else (60.0 if case["kind"] == "bond" else 30.0)
    if case["kind"] in ("gradient", "jacobian"):
        per += 80.0
    tail = 2.0 * case["n_sites"] * case["N"] * (2.0 if case["n_E"] == 0 else case["n_E"])
    return per * _site_steps(case) + tail


def _bytes(case):
    L2, n, N = case["Lx"] * case["Ly"], case["n_sites"], case["N"]
    s = 16 if case["cplx"] else 8
    b = L2 * (8 + s) + n * N * (8 + s)
    if case["cplx"] or case["kind"] == "bond":
        b += L2 * (2 * s + 16)
    if case["kind"] == "bond":
        b += 8 * n * N * s + 2 * L2 * s
    if case["kind"] == "jacobian":
        b += n * L2 * 8
    return b + n * case["n_E"] * 8 * (2 if case["kind"] == "gradient" else 1)


def work(case):
    return {"bytes": float(_bytes(case)), "flops": _flops(case)}


def _cost(case):
    """What a pass costs with the vectors streamed once per few steps."""
    f = _site_steps(case) * (6.0 if case["cplx"] else 1.0) * (0.7 if case["fp32"] else 1.0)
    if case["kind"] == "bond":
        f *= 2.0
    if case["kind"] in ("gradient", "jacobian"):
        f *= 6.0
    if case["Lx"] % 64 or case["Lx"] > 256:
        f *= 3.0
    return f


# ---------------------------------------------------------------- reference


def _hamiltonian(case, f):
    """Ht as a sparse matrix on the basis (site, e) = 2 s, (site, h) = 2 s + 1."""
    Lx, Ly, a = case["Lx"], case["Ly"], f["a"]
    L2 = Lx * Ly
    s = np.arange(L2)
    x, y = s % Lx, s // Lx
    rows, cols, vals = [], [], []

    def put(r, c, v):
        rows.append(r)
        cols.append(c)
        vals.append(np.broadcast_to(v, r.shape))

    xi, d = f["eps"] - MU, f["delta"]
    put(2 * s, 2 * s, xi)
    put(2 * s + 1, 2 * s + 1, -xi)
    put(2 * s, 2 * s + 1, d)
    put(2 * s + 1, 2 * s, np.conj(d))
    for axis, (pos, size, bc, step) in enumerate(((x, Lx, case["bc_x"], 1), (y, Ly, case["bc_y"], Lx))):
        keep = np.ones(L2, bool) if bc else pos < size - 1
        i = s[keep]
        j = np.where(pos[keep] < size - 1, i + step, i - (size - 1) * step)
        t = HOP * (np.exp(1j * f["peierls"][axis][keep]) if f["peierls"] is not None else np.ones(len(i)))
        put(2 * i, 2 * j, -t)
        put(2 * j, 2 * i, -np.conj(t))
        put(2 * i + 1, 2 * j + 1, np.conj(t))
        put(2 * j + 1, 2 * i + 1, t)
        if f["bond"] is not None:
            b = f["bond"][axis][keep]
            for p, q in ((i, j), (j, i)):
                put(2 * p, 2 * q + 1, b)
                put(2 * p + 1, 2 * q, np.conj(b))
    dt = torch.complex128 if case["cplx"] else torch.float64
    H = torch.sparse_coo_tensor(torch.as_tensor(np.stack([np.concatenate(rows), np.concatenate(cols)])),
                                torch.as_tensor(np.concatenate(vals)).to(dt) / a, (2 * L2, 2 * L2))
    return H.coalesce().to(DEV).to_sparse_csr()


def _vectors(H, sites, N):
    """a_0 .. a_{N-1} of the start vectors, one [2 L2, sites] block at a time."""
    p = torch.zeros((H.shape[0], len(sites)), dtype=H.dtype, device=DEV)
    p[2 * sites, torch.arange(len(sites), device=DEV)] = 1.0
    yield p
    if N == 1:
        return
    c = torch.sparse.mm(H, p)
    yield c
    for _ in range(2, N):
        p, c = c, 2.0 * torch.sparse.mm(H, c) - p
        yield c


def _chunks(sites, width):
    return [sites[k:k + width] for k in range(0, len(sites), width)]


def _exact_moments(case, H, sites, neighbours=None):
    N, n = case["N"], len(sites)
    ee = torch.empty((n, N), dtype=torch.float64, device=DEV)
    he = torch.empty((n, N), dtype=H.dtype, device=DEV)
    nb = None if neighbours is None else [torch.zeros((n, 4, N), dtype=H.dtype, device=DEV) for _ in range(2)]
    at = 0
    for part in _chunks(sites, 512):
        rows, cols = slice(at, at + len(part)), torch.arange(len(part), device=DEV)
        for k, v in enumerate(_vectors(H, part, N)):
            ee[rows, k] = v[2 * part, cols].real
            he[rows, k] = v[2 * part + 1, cols]
            if nb is not None:
                for d in range(4):
                    j = neighbours[d][part]
                    for c in range(2):
                        nb[c][rows, d, k] = torch.where(j >= 0, v[2 * j.clamp(min=0) + c, cols], torch.zeros_like(he[0, 0]))
        at += len(part)
    return (ee, he) if nb is None else (ee, he, nb[0], nb[1])


def _damping(case, a):
    N = case["N"]
    n = np.arange(N)
    if case["lorentz"]:
        lam = _lam(case, a)
        return np.sinh(lam * (1.0 - n / N)) / np.sinh(lam)
    q = np.pi / (N + 1)
    return ((N - n + 1) * np.cos(q * n) + np.sin(q * n) / np.tan(q)) / (N + 1)


def _coefficients(case, a, gap):
    """g_n c_n of the weight tanh(E/2T) (gap) or f(E) (density)."""
    N, T = case["N"], case["T"]
    n = np.arange(N)
    if T > 0.0:
        M = 1 << 16
        e = a * np.cos(np.pi * (np.arange(M) + 0.5) / M)
        val = np.tanh(e / (2.0 * T)) if gap else 0.5 * (1.0 - np.tanh(e / (2.0 * T)))
        # cosine sums over the Chebyshev points by one real transform
        c = np.real(np.fft.fft(np.concatenate([val, val[::-1]]))[:N] * np.exp(-0.5j * np.pi * n / M)) / M
        c[0] *= 0.5
    else:
        s = np.sin(0.5 * np.pi * n)
        c = np.zeros(N)
        c[1:] = (4.0 if gap else -2.0) * s[1:] / (np.pi * n[1:])
        c[0] = 0.0 if gap else 0.5
    return torch.as_tensor(_damping(case, a) * c, device=DEV)


def _ldos_table(case, f):
    """W[n, m] with LDOS[r, m] = sum_n mu_ee[r, n] W[n, m]."""
    x = f["energies"] / f["a"]
    t = np.cos(np.arange(case["N"])[:, None] * np.arccos(x)[None, :])
    pre = _damping(case, f["a"]) * np.where(np.arange(case["N"]) == 0, 1.0, 2.0)
    return torch.as_tensor(pre[:, None] * t / (np.pi * f["a"] * np.sqrt(1.0 - x * x))[None, :], device=DEV)


def _exact_rows(case, H, sites, a, d_ee, d_he):
    """Per start site the gradient of sum_n (d_ee mu_ee + d_he mu_he) by eps
    and Delta: the transposed recursion over the stored vectors."""
    N, L2 = case["N"], case["Lx"] * case["Ly"]
    width = max(1, min(256, int(16e9 / (16.0 * L2 * N))))
    eps, delta, at = [], [], 0
    for part in _chunks(sites, width):
        cols = torch.arange(len(part), device=DEV)
        vec = list(_vectors(H, part, N))
        l1, l2 = torch.zeros_like(vec[0]), torch.zeros_like(vec[0])
        ge = torch.zeros((L2, len(part)), dtype=torch.float64, device=DEV)
        gd = torch.zeros_like(ge)
        for k in range(N - 1, 0, -1):
            lam = 2.0 * torch.sparse.mm(H, l1) - l2
            if d_ee is not None:
                lam[2 * part, cols] += d_ee[at:at + len(part), k]
            if d_he is not None:
                lam[2 * part + 1, cols] += d_he[at:at + len(part), k]
            v, c = vec[k - 1], (1.0 if k == 1 else 2.0) / a
            ge += c * (lam[0::2] * v[0::2] - lam[1::2] * v[1::2])
            gd += c * (lam[0::2] * v[1::2] + lam[1::2] * v[0::2])
            l1, l2 = lam, l1
        eps.append(ge.T)
        delta.append(gd.T)
        at += len(part)
    return torch.cat(eps), torch.cat(delta)


def _exact_bonds(case, f, mu):
    """Bond order parameter and currents from the neighbour moments of every site."""
    Lx, Ly, a = case["Lx"], case["Ly"], f["a"]
    L2 = Lx * Ly
    ee, he, nb_ee, nb_he = mu
    gap, occ = _coefficients(case, a, True), _coefficients(case, a, False)
    sg, so = (nb_he * gap).sum(-1), (nb_ee * occ).sum(-1)
    nb = _neighbours(case)
    new, cur = [], []
    for axis in range(2):
        j = nb[2 * axis]
        ok = j >= 0
        t = torch.ones(L2, dtype=torch.complex128, device=DEV)
        if f["peierls"] is not None:
            t = torch.exp(1j * torch.as_tensor(f["peierls"][axis], device=DEV))
        d = 0.25 * U * (sg[:, 2 * axis] + sg[j.clamp(min=0), 2 * axis + 1]).conj()
        new.append(torch.where(ok, d, torch.zeros_like(d)))
        cur.append(torch.where(ok, 4.0 * (HOP * t * so[:, 2 * axis]).imag, torch.zeros(L2, dtype=torch.float64, device=DEV)))
    new = torch.cat(new)
    old = torch.as_tensor(f["bond"].reshape(-1), device=DEV)
    return {"mu_ee": ee, "mu_he": he, "nb_ee": nb_ee, "nb_he": nb_he, "bond": new,
            "resid": (new - old).abs().max().reshape(1), "current": torch.stack(cur)}


def _neighbours(case):
    Lx, Ly = case["Lx"], case["Ly"]
    s = torch.arange(Lx * Ly, device=DEV)
    x, y = s % Lx, s // Lx
    out = []
    for pos, size, bc, step in ((x, Lx, case["bc_x"], 1), (y, Ly, case["bc_y"], Lx)):
        wrap = (size - 1) * step
        none = torch.full_like(s, -1)
        out.append(torch.where(pos < size - 1, s + step, s - wrap if bc else none))
        out.append(torch.where(pos > 0, s - step, s + wrap if bc else none))
    return out


def exact(case, seed):
    # vectors over all steps, in 64 bits: cases whose recursion would take too long have no value
    L2, n, N = case["Lx"] * case["Ly"], case["n_sites"], case["N"]
    if 2.0 * L2 * n * N * (3.0 if case["cplx"] else 1.0) * (4.0 if case["kind"] in ("gradient", "jacobian") else 1.0) > 3e11:
        return None
    f = _fields(case, seed)
    H = _hamiltonian(case, f)
    a, kind = f["a"], case["kind"]
    sites = torch.as_tensor(f["sites"], dtype=torch.int64, device=DEV)
    old = torch.as_tensor(f["delta"], device=DEV)[sites]
    if kind == "bond":
        return _exact_bonds(case, f, _exact_moments(case, H, sites, _neighbours(case)))
    if kind == "jacobian":
        d_he = (0.5 * U * _coefficients(case, a, True)).expand(n, N)
        rows = _exact_rows(case, H, sites, a, None, d_he)[1]
        return {"rows": rows, "product": rows @ torch.as_tensor(f["vec"], device=DEV)}
    ee, he = _exact_moments(case, H, sites)
    gap = _coefficients(case, a, True)
    if kind == "gradient":
        cot = torch.as_tensor(f["cot"], device=DEV)
        if case["loss"] == "ldos":
            W = _ldos_table(case, f)
            out, d_ee, d_he = ee @ W, cot @ W.T, None
        else:
            out, d_ee, d_he = 0.5 * U * (he * gap).sum(-1), None, 0.5 * U * gap * cot[:, :1]
        ge, gd = _exact_rows(case, H, sites, a, d_ee, d_he)
        return {"out": out, "eps": ge.sum(0), "delta": gd.sum(0)}
    res = {"mu_ee": ee, "mu_he": he}
    if kind == "scf":
        res["delta"] = 0.5 * U * (he * gap).sum(-1).conj()
        res["resid"] = (res["delta"] - old).abs().max().reshape(1)
        if case["T"] > 0.0:
            res["density"] = 2.0 * (ee * _coefficients(case, a, False)).sum(-1)
    elif kind == "ldos":
        res["ldos"] = ee @ _ldos_table(case, f)
    return res
