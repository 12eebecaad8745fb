"""Performance cases of the Wilson-HMC library: what its users have it do.

Each case is one pass through the public entry points of
``paper_1212_0785_amd.hmc`` on a lattice that a program keeps resident:

* ``mhat``: one application of the even-odd fermion matrix (``hmc_mhat``),
  the unit of every inversion, in each storage precision and both daggers;
* ``solve``: one inversion to a relative residual of 1e-10 (1e-11 with a
  low-precision inner iteration), either the force solve (CG on Mhat^dag
  Mhat) or a Wilson solve of a full source;
* ``refresh``: new momenta and pseudofermions, the start of a trajectory;
* ``md_step``: one integration step around a given solution: gauge force,
  fermion force and link update;
* ``measure``: a stored configuration and a spinor taken up from the canonical
  layout, the plaquette and the global sums a measurement takes of them (the
  norm, an inner product, the sums over time slices), and the configuration
  written back to the canonical layout;
* ``trajectory``: a whole HMC trajectory.

Links are SU(3) with the disorder of a smooth configuration, spinors and
momenta Gaussian; all of it from torch's generator and the seed alone.
``exact`` repeats each pass in plain torch in 64 bits.
"""
import math

import torch

from paper_1212_0785_amd import hmc as H

DEV = "cuda"
PRECS = ("f64", "f32", "f16", "bf16")
SPINOR_BYTES = {"f64": 192, "f32": 96, "f16": 52, "bf16": 48}
LINK_BYTES = {"f64": 144, "f32": 72, "f16": 36, "bf16": 36}
# flops per site of a hopping term, and per link of the other kernels
HOP_FLOPS, GAUGE_FLOPS, FERMION_FLOPS, UPDATE_FLOPS = 1320, 2800, 700, 700
# widest range of a drawn lattice: 4^4 to 48^3x96 sites
V_MIN, V_MAX = 4 ** 4, 48 ** 3 * 96


def _case(name, kind, L, **kw):
    c = {"name": name, "kind": kind, "Lx": L[0], "Ly": L[1], "Lz": L[2], "Lt": L[3], "kappa": 0.13, "disorder": 0.25}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one operator application on the 4^4 lattice of
        # the parity chain, all latency and launches
        _case("mhat_f64_4c4", "mhat", (4, 4, 4, 4), prec="f64", dagger=False),
        # an odd, ragged lattice in single precision
        _case("mhat_f32_18x10x14x26", "mhat", (18, 10, 14, 26), prec="f32", dagger=False),
        # an ordinary production volume in the inner precision of a mixed solve
        _case("mhat_bf16_32c64", "mhat", (32, 32, 32, 64), prec="bf16", dagger=True),
        # the largest volume of the kernel benchmark, FP64
        _case("mhat_f64_48c96", "mhat", (48, 48, 48, 96), prec="f64", dagger=False),
        # the smallest request of the solve service's mix: a Wilson solve
        # with FP32 inner iterations, bound by latency
        _case("solve_f32_8c8", "solve", (8, 8, 8, 8), prec="f32", wilson=True, tol=1e-11, iters=60),
        # the force solve of a small chain
        _case("solve_f64_12c24", "solve", (12, 12, 12, 24), prec="f64", wilson=False, tol=1e-10, iters=75),
        # a Wilson solve of the headline's volume with FP16 inner iterations
        _case("solve_f16_16c32", "solve", (16, 16, 16, 32), prec="f16", wilson=True, tol=1e-11, iters=81),
        # a propagator's Wilson solve at the volume of the precision study
        _case("solve_f64_24c48", "solve", (24, 24, 24, 48), prec="f64", wilson=True, tol=1e-10, iters=76),
        # the start of a trajectory on a volume between the tuned ones
        _case("refresh_20c40", "refresh", (20, 20, 20, 40)),
        # one integration step of a trajectory
        _case("md_step_24c48", "md_step", (24, 24, 24, 48), beta=5.6, eps=0.02),
        # a stored configuration measured, on a ragged lattice
        _case("measure_20x20x22x44", "measure", (20, 20, 22, 44), beta=5.6),
        # the headline: one trajectory of the 16^3x32 chain
        _case("trajectory_16c32", "trajectory", (16, 16, 16, 32), beta=5.6, kappa=0.15, disorder=0.15, tau=1.0, nsteps=20,
              iters=104),
    ]


def _lattice(rng, lo, hi):
    """Even extents, the volume log-uniform in [lo, hi], time usually the longest."""
    for _ in range(1000):
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        stretch = rng.uniform(1.0, 2.6)
        base = (v / stretch) ** 0.25
        L = [2 * max(2, round(base * rng.uniform(0.75, 1.3) / 2)) for _ in range(3)]
        L.append(2 * max(2, round(v / (L[0] * L[1] * L[2]) / 2)))
        if lo <= L[0] * L[1] * L[2] * L[3] <= hi and L[3] <= 128:
            return tuple(L)
    return (8, 8, 8, 16)


def draw(rng):
    kind = rng.choice(["mhat", "mhat", "solve", "solve", "refresh", "md_step", "measure", "trajectory"])
    smooth = {"kappa": round(rng.uniform(0.12, 0.134), 4), "disorder": round(rng.uniform(0.2, 0.3), 3)}
    if kind == "mhat":
        c = _case("", kind, _lattice(rng, V_MIN, V_MAX), prec=rng.choice(PRECS), dagger=rng.random() < 0.5, **smooth)
    elif kind == "solve":
        # BF16 storage is left to the operator: the solutions of its solves
        # agree only to what its own rounding leaves of the tolerance
        prec = rng.choice(PRECS[:3])
        c = _case("", kind, _lattice(rng, V_MIN, 24 ** 3 * 48), prec=prec, wilson=rng.random() < 0.5,
                  tol=1e-10 if prec == "f64" else 1e-11, iters=75, **smooth)
    elif kind == "refresh":
        c = _case("", kind, _lattice(rng, 8 ** 4, V_MAX // 2), **smooth)
    elif kind == "md_step":
        c = _case("", kind, _lattice(rng, 8 ** 4, 32 ** 3 * 64), beta=round(rng.uniform(5.4, 6.2), 2),
                  eps=round(rng.uniform(0.01, 0.05), 3), **smooth)
    elif kind == "measure":
        c = _case("", kind, _lattice(rng, 8 ** 4, 32 ** 3 * 64), beta=round(rng.uniform(5.4, 6.2), 2), **smooth)
    else:
        c = _case("", kind, _lattice(rng, 4 ** 4, 16 ** 3 * 24), beta=round(rng.uniform(5.4, 6.2), 2), tau=0.5,
                  nsteps=rng.randrange(4, 11), iters=60, **smooth)
    del c["name"]
    return c


# ------------------------------------------------------------ inputs


def _extents(case):
    return (case["Lx"], case["Ly"], case["Lz"], case["Lt"])


def _volume(case):
    return case["Lx"] * case["Ly"] * case["Lz"] * case["Lt"]


def _rng(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1) + stream)
    return g


def _links(case, seed):
    """(V, 4, 3, 3) complex128 SU(3) links: 1 + disorder * noise, rows orthonormalised."""
    V = _volume(case)
    g = torch.randn((V, 4, 2, 3, 2), generator=_rng(seed, 1), dtype=torch.float64, device=DEV) * case["disorder"]
    g[:, :, 0, 0, 0] += 1.0
    g[:, :, 1, 1, 0] += 1.0
    g = torch.view_as_complex(g)
    U = torch.empty((V, 4, 3, 3), dtype=torch.complex128, device=DEV)
    a, b = g[:, :, 0], g[:, :, 1]
    a = a / a.abs().square().sum(-1, keepdim=True).sqrt()
    for _ in range(2):
        b = b - (a.conj() * b).sum(-1, keepdim=True) * a
        b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    U[:, :, 0], U[:, :, 1] = a, b
    for k in range(3):
        i, j = (k + 1) % 3, (k + 2) % 3
        U[:, :, 2, k] = (a[..., i] * b[..., j] - a[..., j] * b[..., i]).conj()
    return U


def _spinor(case, seed, stream):
    """(V, 4, 3) complex128 Gaussian spinor."""
    V = _volume(case)
    return torch.randn((V, 4, 3), generator=_rng(seed, stream), dtype=torch.complex128, device=DEV)


def _momenta(case, seed):
    """(V, 4, 3, 3) traceless Hermitian momenta with unit variance per generator."""
    V = _volume(case)
    w = torch.randn((V, 4, 8), generator=_rng(seed, 2), dtype=torch.float64, device=DEV)
    return _hermitian(_algebra(w))


def _algebra(w):
    """sum_a w_a lambda_a / 2 as (P00, P11, P01, P02, P12) parts, (..., 8) reals."""
    s = 1.0 / math.sqrt(3.0)
    return torch.stack([0.5 * (w[..., 2] + s * w[..., 7]), 0.5 * (s * w[..., 7] - w[..., 2]), 0.5 * w[..., 0],
                        -0.5 * w[..., 1], 0.5 * w[..., 3], -0.5 * w[..., 4], 0.5 * w[..., 5], -0.5 * w[..., 6]], -1)


def _hermitian(c):
    P = torch.zeros(c.shape[:-1] + (3, 3), dtype=torch.complex128, device=c.device)
    P[..., 0, 0] = c[..., 0].to(P.dtype)
    P[..., 1, 1] = c[..., 1].to(P.dtype)
    P[..., 2, 2] = (-c[..., 0] - c[..., 1]).to(P.dtype)
    for k, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
        z = torch.complex(c[..., 2 + 2 * k], c[..., 3 + 2 * k])
        P[..., i, j], P[..., j, i] = z, z.conj()
    return P


def _view(buf, case, prec="f64"):
    """The numbers of a device spinor buffer in its storage type."""
    if prec == "f64":
        return buf.view(torch.float64)
    if prec == "f32":
        return buf.view(torch.float32)
    if prec == "bf16":
        return buf.view(torch.bfloat16)
    n = buf.numel() // 52 * 48  # twelve half2 arrays, then one float scale per site
    return buf[:n].view(torch.float16), buf[n:].view(torch.float32)


def _resident(F, which, nbytes):
    off = F.pointer(which) - F.arena.data_ptr()
    return F.arena[off:off + nbytes].view(torch.float64)


def prepare(case, seed):
    L, V, kind = _extents(case), _volume(case), case["kind"]
    low = kind == "mhat" and case["prec"] != "f64" or kind == "solve" and case["prec"] != "f64"
    F = H.Fields(L, case.get("beta", 5.6), case["kappa"], flags=H.FIELDS_LOWPREC if low else 0)
    s = {"case": case, "F": F}
    if kind in ("md_step",):  # handed out before the links are set: the import checks them again
        s["U"] = _resident(F, H.FIELD_GAUGE, V * 576)
    if kind != "measure":
        H.hmc_import_gauge(F, _links(case, seed))
    if kind == "mhat":
        prec = H.PREC_NAMES[case["prec"]]
        x = F.spinor()
        H.hmc_import_spinor(F, x, _spinor(case, seed, 3), 0)
        s["x"] = x
        if low:
            s["x"] = F.spinor(prec)
            H.hmc_convert_spinor(F, s["x"], prec, x, H.F64)
            H.hmc_sync_lowprec(F)
        s["out"] = F.spinor(prec)
    elif kind == "solve":
        full = case["wilson"]
        s["b"], s["x"] = F.spinor(full=full), F.spinor(full=full)
        H.hmc_import_spinor(F, s["b"], _spinor(case, seed, 3), -1 if full else 0)
        if low:
            H.hmc_sync_lowprec(F)
        s["prm"] = H.cg_params(tol=case["tol"], prec=H.PREC_NAMES[case["prec"]],
                               mode=H.CG_WILSON_SOLVE if full else H.CG_NORMAL_MHAT)
    elif kind == "refresh":
        s["out"] = (_resident(F, H.FIELD_MOMENTA, V * 256), _resident(F, H.FIELD_ETA, V * 96),
                    _resident(F, H.FIELD_PHI, V * 96))
        s["seed"], s["traj"] = seed, 0
    elif kind == "md_step":
        H.hmc_import_momenta(F, _momenta(case, seed))
        s["P"] = _resident(F, H.FIELD_MOMENTA, V * 256)
        s["x"] = F.spinor()
        H.hmc_import_spinor(F, s["x"], _spinor(case, seed, 3), 0)
    elif kind == "measure":
        s["gauge"], s["psi"], s["ref"] = _links(case, seed), _spinor(case, seed, 3), F.spinor(full=True)
        H.hmc_import_spinor(F, s["ref"], _spinor(case, seed, 4), -1)
        s["x"], s["written"] = F.spinor(full=True), H.canon_gauge_zeros(L)
        slices = torch.arange(L[3], dtype=torch.int32, device=DEV).repeat_interleave(V // (2 * L[3]))
        s["slices"] = torch.cat([slices, slices]).contiguous()
    elif kind == "trajectory":
        s["out"] = (_resident(F, H.FIELD_MOMENTA, V * 256), _resident(F, H.FIELD_PHI, V * 96),
                    _resident(F, H.FIELD_XE, V * 96))
        s["seed"], s["traj"], s["prm"] = seed, 0, H.cg_params(tol=1e-10)
    return s


def run(s):
    case, F = s["case"], s["F"]
    kind = case["kind"]
    if kind == "mhat":
        H.hmc_mhat(F, s["out"], s["x"], dagger=case["dagger"], prec=H.PREC_NAMES[case["prec"]])
        return _view(s["out"], case, case["prec"])
    if kind == "solve":
        H.hmc_cg_solve(F, s["x"], s["b"], s["prm"])
        return _view(s["x"], case)
    if kind == "refresh":
        H.hmc_refresh(F, s["seed"], s["traj"])
        s["traj"] += 1
        return s["out"]
    if kind == "md_step":
        H.hmc_gauge_force(F, case["eps"])
        H.hmc_fermion_force(F, s["x"], case["eps"])
        H.hmc_exp_update_reunit(F, case["eps"])
        return s["P"], s["U"]
    if kind == "measure":
        H.hmc_import_gauge(F, s["gauge"])
        plaq = H.hmc_plaquette(F)
        H.hmc_import_spinor(F, s["x"], s["psi"], -1)
        n2 = H.hmc_norm2(F, s["x"], 2)
        ip = H.hmc_inner(F, s["ref"], s["x"], 2)
        sums = H.hmc_sum_multi(F, s["x"], 2, s["slices"], case["Lt"])
        H.hmc_export_gauge(F, s["written"])
        return {"plaquette": plaq, "norm2": n2, "inner_re": ip.real, "inner_im": ip.imag, "slices": sums,
                "x": _view(s["x"], case), "written": s["written"]}
    r = H.hmc_trajectory(F, s["seed"], s["traj"], case["tau"], case["nsteps"], s["prm"])
    s["traj"] += 1
    P, phi, X = s["out"]
    return {"H_old": r["H_old"], "H_new": r["H_new"], "plaquette": r["plaquette"], "accepted": r["accepted"],
            "u": r["u"], "momenta": P, "phi": phi, "X_e": X}


def work(case):
    """Bytes and flops of a pass.  An inversion streams its links and vectors
    once per operator application: two of Mhat and one update of the vectors
    in each of its (about) ``iters`` iterations."""
    V, kind = _volume(case), case["kind"]
    mhat_flops = V * (HOP_FLOPS + 48)
    if kind == "mhat":
        return {"bytes": V * (4 * LINK_BYTES[case["prec"]] + SPINOR_BYTES[case["prec"]]), "flops": mhat_flops}
    if kind in ("solve", "trajectory"):
        p = case.get("prec", "f64")
        it = V * (2 * 4 * LINK_BYTES[p] + 4.5 * SPINOR_BYTES[p])
        n = case["iters"] * (1 if kind == "solve" else case["nsteps"] + 1)
        w = {"bytes": n * it + V * (4 * 144 + 2 * 192), "flops": n * (2 * mhat_flops + 96 * V)}
        if kind == "trajectory":
            k = case["nsteps"] + 1
            w["bytes"] += k * V * (3 * 4 * 144 + 6 * 256 + 2 * 192)
            w["flops"] += k * V * 4 * (GAUGE_FLOPS + FERMION_FLOPS + UPDATE_FLOPS)
        return w
    if kind == "refresh":
        return {"bytes": V * (256 + 2 * 96 + 4 * 144), "flops": mhat_flops + V * 44 * 60}
    if kind == "md_step":
        return {"bytes": V * (2 * 4 * 144 + 2 * 256 + 96),
                "flops": V * (4 * (GAUGE_FLOPS + FERMION_FLOPS + UPDATE_FLOPS) + 1.5 * HOP_FLOPS)}
    return {"bytes": V * (2 * 576 + 3 * 192), "flops": V * (6 * 500 + 200)}


# ----------------------------------------------------- 64-bit reference

# Full-lattice arrays of shape (Lt, Lz, Ly, Lx, ...); direction mu is axis 3 - mu.


def _grid(case, a):
    return a.reshape((case["Lt"], case["Lz"], case["Ly"], case["Lx"]) + tuple(a.shape[1:]))


def _odd(case):
    c = [torch.arange(n, device=DEV) for n in (case["Lt"], case["Lz"], case["Ly"], case["Lx"])]
    return (c[0].view(-1, 1, 1, 1) + c[1].view(-1, 1, 1) + c[2].view(-1, 1) + c[3]) % 2 == 1


def _gamma(mu, p):
    p0, p1, p2, p3 = p.unbind(-2)
    q = {0: (1j * p3, 1j * p2, -1j * p1, -1j * p0), 1: (-p3, p2, p1, -p0),
         2: (1j * p2, -1j * p3, -1j * p0, 1j * p1), 3: (p2, p3, p0, p1)}[mu]
    return torch.stack(q, -2)


def _mul(a, b):
    """3x3 matrix times 3xn matrix."""
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.transpose(-1, -2).conj()


def _colour(u, p):
    """u acting on the colour index of a spinor (..., 4, 3)."""
    return (u.unsqueeze(-3) * p.unsqueeze(-2)).sum(-1)


def _up(a, mu):
    return torch.roll(a, -1, 3 - mu)


def _down(a, mu):
    return torch.roll(a, 1, 3 - mu)


def _edge(case, fwd):
    """-1 on the time slice whose hop crosses the boundary."""
    s = torch.ones(case["Lt"], dtype=torch.float64, device=DEV)
    s[-1 if fwd else 0] = -1.0
    return s.view(-1, 1, 1, 1, 1, 1)


def _hop(case, U, p, dagger):
    """D p (or D^dag p)."""
    s = -1.0 if not dagger else 1.0
    out = torch.zeros_like(p)
    for mu in range(4):
        f = _up(p, mu)
        if mu == 3:
            f = f * _edge(case, True)
        out += _colour(U[..., mu, :, :], f + s * _gamma(mu, f))
        b = _colour(_dag(U[..., mu, :, :]), p - s * _gamma(mu, p))
        b = _down(b, mu)
        if mu == 3:
            b = b * _edge(case, False)
        out += b
    return out


def _mhat(case, U, p, dagger):
    """Mhat p for p on the even sites."""
    return p - case["kappa"] ** 2 * _hop(case, U, _hop(case, U, p, dagger), dagger)


def _dot(a, b):
    return torch.view_as_real(a).mul(torch.view_as_real(b)).sum()


def _cg(case, U, b, tol):
    """x = (Mhat^dag Mhat)^-1 b on even sites."""
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = _dot(r, r)
    stop = float(rr) * tol * tol
    for _ in range(4000):
        q = _mhat(case, U, p, False)
        a = rr / _dot(q, q)
        x += a * p
        r -= a * _mhat(case, U, q, True)
        new = _dot(r, r)
        if float(new) <= stop:
            break
        p = r + (new / rr) * p
        rr = new
    return x


def _halves(case, p, *, even=True, odd=False):
    """Component-major half spinors (12, V/2) of a full-lattice spinor, as flat reals."""
    o = _odd(case).reshape(-1)
    p = p.reshape(-1, 12)
    got = [p[~o]] if even else []
    if odd:
        got.append(p[o])
    return torch.cat([torch.view_as_real(h.t().contiguous()).reshape(-1) for h in got])


def _even(case, p):
    return p * (~_odd(case)).view(case["Lt"], case["Lz"], case["Ly"], case["Lx"], 1, 1)


def _by_parity(case, c):
    """(V, 4, n) per-link values as the device's [mu][parity][n][V/2]."""
    o = _odd(case).reshape(-1)
    c = c.reshape((-1,) + tuple(c.shape[-2:]))
    c = torch.stack([c[~o], c[o]])  # parity, site, mu, n
    c = c.permute(2, 0, 3, 1).contiguous()
    return (torch.view_as_real(c) if c.is_complex() else c).reshape(-1)


def _compact(P):
    return torch.stack([P[..., 0, 0].real, P[..., 1, 1].real, P[..., 0, 1].real, P[..., 0, 1].imag, P[..., 0, 2].real,
                        P[..., 0, 2].imag, P[..., 1, 2].real, P[..., 1, 2].imag], -1)


def _i_ta(W):
    """i times the traceless part of W - W^dag."""
    Z = W - _dag(W)
    t = Z.diagonal(dim1=-2, dim2=-1).sum(-1) / 3
    return 1j * (Z - t[..., None, None] * torch.eye(3, dtype=Z.dtype, device=Z.device))


def _gauge_kick(case, U, P, coef):
    """P - coef F_g."""
    P = P.clone()
    for mu in range(4):
        u = U[..., mu, :, :]
        A = torch.zeros_like(u)
        for nu in range(4):
            if nu == mu:
                continue
            v = U[..., nu, :, :]
            vm = _up(v, mu)
            A += _mul(_mul(vm, _dag(_up(u, nu))), _dag(v))
            A += _down(_mul(_mul(_dag(vm), _dag(u)), v), nu)
        P[..., mu, :, :] += coef * case["beta"] / 12 * _i_ta(_mul(u, A))
    return P


def _fermion_kick(case, U, P, Xe, coef):
    """P - coef F_f for the solution Xe on the even sites."""
    P = P.clone()
    Y = _mhat(case, U, Xe, False)
    X = Xe + _hop(case, U, Xe, False)
    Y = Y + _hop(case, U, Y, True)
    for mu in range(4):
        u = U[..., mu, :, :]
        xf, yf = _up(X, mu), _up(Y, mu)
        if mu == 3:
            xf, yf = xf * _edge(case, True), yf * _edge(case, True)
        a = xf - _gamma(mu, xf)
        b = X + _gamma(mu, X)
        M1 = (a.unsqueeze(-1) * Y.conj().unsqueeze(-2)).sum(-3)
        M2 = (b.unsqueeze(-1) * yf.conj().unsqueeze(-2)).sum(-3)
        P[..., mu, :, :] -= coef * case["kappa"] ** 2 / 2 * _i_ta(_mul(u, M1) - _mul(M2, _dag(u)))
    return P


def _link_update(U, P, eps):
    """exp(i eps P) U."""
    U = U.clone()
    for mu in range(4):
        A = 1j * eps * P[..., mu, :, :]
        E = T = torch.eye(3, dtype=U.dtype, device=DEV).expand_as(A)
        n, bound = 1, 1.0
        size = float(A.abs().max()) * 3
        while bound > 1e-18:
            T = _mul(T, A) / n
            E = E + T
            bound *= size / n
            n += 1
        U[..., mu, :, :] = _mul(E, U[..., mu, :, :])
    return U


def _plaquette(case, U):
    s = 0.0
    for mu in range(4):
        for nu in range(mu):
            a = _mul(U[..., mu, :, :], _up(U[..., nu, :, :], mu))
            b = _mul(U[..., nu, :, :], _up(U[..., mu, :, :], nu))
            s = s + float(_dot(a, b))
    return s / (18.0 * _volume(case))


_MASK = 0xFFFFFFFF


def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _mulhi(a, m):
    """High 64 bits of the unsigned product of int64 tensor a and constant m."""
    al, ah = a & _MASK, (a >> 32) & _MASK
    ml, mh = m & _MASK, (m >> 32) & _MASK
    hl, lh = ah * ml, al * mh
    mid = ((al * ml >> 32) & _MASK) + (hl & _MASK) + (lh & _MASK)
    return ah * mh + ((hl >> 32) & _MASK) + ((lh >> 32) & _MASK) + (mid >> 32)


def _philox(block, site, stream, epoch, seed):
    """Philox4x64-10 words (..., 4) of counters (block, site, stream, epoch), key (seed, 0)."""
    m0, m1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    w0, w1 = 0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B
    c0, c1 = torch.full_like(site, block), site
    c2, c3 = torch.full_like(site, stream), torch.full_like(site, epoch)
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0, h1, l1 = _mulhi(c0, m0), c0 * _signed(m0), _mulhi(c2, m1), c2 * _signed(m1)
        c0, c1, c2, c3 = h1 ^ c1 ^ _signed(k0), l1, h0 ^ c3 ^ _signed(k1), l0
        k0, k1 = k0 + w0, k1 + w1
    return c0, c1, c2, c3


def _gaussians(site, n, stream, epoch, seed):
    """n Gaussians per site, consecutive word pairs through Box-Muller."""
    out = []
    for b in range(n // 4):
        w = _philox(b, site, stream, epoch, seed)
        u = [(((v >> 11) & ((1 << 53) - 1)).double() + 0.5) * 2.0 ** -53 for v in w]
        for i in (0, 2):
            r, th = (-2.0 * u[i].log()).sqrt(), 2 * math.pi * u[i + 1]
            out += [r * th.cos(), r * th.sin()]
    return torch.stack(out, -1)


def _refreshed(case, U, seed, traj):
    """Momenta (V, 4, 8) and the even pseudofermions eta, phi."""
    site = torch.arange(_volume(case), dtype=torch.int64, device=DEV)
    c = _algebra(_gaussians(site, 32, 1, traj, seed).reshape(-1, 4, 8))
    g = _gaussians(site, 24, 2, traj, seed).reshape(-1, 4, 3, 2) / math.sqrt(2.0)
    eta = _even(case, _grid(case, torch.view_as_complex(g)))
    return c, eta, _mhat(case, U, eta, True)


def _stored(case, p, prec):
    """A half spinor's exact values in the form the storage type returns them."""
    h = _halves(case, p)
    if prec != "f16":
        return h
    h = h.reshape(12, -1, 2)
    m = h.abs().amax(dim=(0, 2))
    return (h / m[None, :, None]).reshape(-1), m


def exact(case, seed):
    kind = case["kind"]
    canon = _links(case, seed)
    U = _grid(case, canon)
    if kind == "mhat":
        x = _even(case, _grid(case, _spinor(case, seed, 3)))
        return _stored(case, _mhat(case, U, x, case["dagger"]), case["prec"])
    if kind == "solve":
        b = _grid(case, _spinor(case, seed, 3))
        k = case["kappa"]
        if not case["wilson"]:
            return _halves(case, _cg(case, U, _even(case, b), 1e-13))
        be = _even(case, b)
        bo = b - be
        x = _cg(case, U, _mhat(case, U, be + k * _hop(case, U, bo, False), True), 1e-13)
        x = x + bo + k * _hop(case, U, x, False)
        return _halves(case, x, odd=True)
    if kind == "refresh":
        c, eta, phi = _refreshed(case, U, seed, 0)
        return _by_parity(case, c), _halves(case, eta), _halves(case, phi)
    if kind == "md_step":
        eps = case["eps"]
        P = _gauge_kick(case, U, _grid(case, _momenta(case, seed)), eps)
        P = _fermion_kick(case, U, P, _even(case, _grid(case, _spinor(case, seed, 3))), eps)
        U = _link_update(U, P, eps)
        return _by_parity(case, _compact(P)), _by_parity(case, U.flatten(-2))
    if kind == "measure":
        x, ref = _grid(case, _spinor(case, seed, 3)), _grid(case, _spinor(case, seed, 4))
        n = torch.view_as_real(x).square().sum((1, 2, 3, 4, 5, 6))
        return {"plaquette": _plaquette(case, U), "norm2": float(n.sum()), "inner_re": float(_dot(ref, x)),
                "inner_im": float(_dot(1j * ref, x)), "slices": [float(v) for v in n],
                "x": _halves(case, x, odd=True), "written": canon}
    # the trajectory, PQP leapfrog; every solve starts from zero
    if _volume(case) * case["nsteps"] > 16 ** 3 * 32 * 20:
        return None
    n = case["nsteps"]
    eps, V = case["tau"] / n, _volume(case)
    c, eta, phi = _refreshed(case, U, seed, 0)
    P = _hermitian(_grid(case, c))
    U0 = U

    def action(U):
        return case["beta"] * 6.0 * V * (1.0 - _plaquette(case, U))

    h_old = float(_dot(P, P)) + action(U) + float(_dot(eta, eta))
    for k in range(n + 1):
        if k:
            U = _link_update(U, P, eps)
        coef = eps if 0 < k < n else 0.5 * eps
        P = _gauge_kick(case, U, P, coef)
        X = _cg(case, U, phi, 1e-12)
        P = _fermion_kick(case, U, P, X, coef)
    h_new = float(_dot(P, P)) + action(U) + float(_dot(phi, X))
    site = torch.zeros(1, dtype=torch.int64, device=DEV)
    w = int(_philox(0, site, 3, 0, seed)[0])
    u = (((w >> 11) & ((1 << 53) - 1)) + 0.5) * 2.0 ** -53
    dh = h_new - h_old
    taken = dh <= 0.0 or u < math.exp(-dh)
    return {"H_old": h_old, "H_new": h_new, "plaquette": _plaquette(case, U if taken else U0), "accepted": int(taken),
            "u": u, "momenta": _by_parity(case, _compact(P)), "phi": _halves(case, phi), "X_e": _halves(case, X)}
