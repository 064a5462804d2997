"""Timed cases of the screened-interaction library.

Each case is one pass of work that a program has the library do for a molecule
it holds on the GPU, from the molecule to W(omega) or one stage of that way,
through the functions of paper_1101_2065_amd.gw.  The molecules are the paper-
shaped ones of gw_synth (chains and 3-D clusters, 13 orbitals and 4 occupied
states per atom unless said otherwise), cut to a stated number of products so
that the sizes do not depend on the seed.

A case is a dict of plain values:
  kind      solve       response and W = (1 - v chi0)^-1 v on a whole mesh
            compressed  the same in the top-k subspace of v, W at some points
            pair        the same in the paper's pair subspace
            two_window  chi0 and W on a fine and a coarse mesh
            time        A = 1 - v chi0 from the time-domain a0
            sigma       self-energy, exchange, Dyson's equation and the DOS
            batch       several molecules recorded once, replayed
  atoms, n_prod, n_omega, omega_max, eps   molecule and mesh
  and per kind: route ("A" or "chi0"), prec, tol, k, points, ...

One Context serves all molecules of a process, as a user's program keeps it; a
batch has one of its own, since a newer batch on a context retires the older.
Reports are asked for only where a program needs them (none here): a call
returns when its work is enqueued.
"""
import math

import numpy as np
import torch

import gw_synth as gs
from paper_1101_2065_amd import gw

DEVICE = "cuda:0"
PREC = {"fp64": gw.GW_FP64, "fp32": gw.GW_FP32_IR, "bf16x": gw.GW_BF16X_IR}
BATCH_BUDGET = 40 << 30

_shared = []


def _context():
    if not _shared:
        _shared.append(gw.Context(0))
    return _shared[0]


# --------------------------------------------------------------------------
# the cases


def _solve(atoms, n_prod, n_omega, omega_max, eps, route="A", prec="fp64", tol=1e-7, small_atoms=False):
    return {"kind": "solve", "atoms": atoms, "n_prod": n_prod, "n_omega": n_omega, "omega_max": omega_max,
            "eps": eps, "route": route, "prec": prec, "tol": tol, "small_atoms": small_atoms}


def listed():
    return [
        # The smallest molecule anyone runs: four atoms of four orbitals, 64
        # products, 256 points.  Launches and latencies, no arithmetic.
        dict(_solve(4, 64, 256, 4.0, 0.05, small_atoms=True), name="chain4_n64_A"),
        # A small molecule through chi0, all three results kept (the integer
        # histogram, chi0 and W); an odd basis size, the paper's automatic
        # broadening (1.5 mesh spacings) on the 512-point mesh.
        dict(_solve(8, 431, 512, 8.0, 0.046875, route="chi0"), name="chain8_n431_chi0"),
        # The mixed-precision forms, refined down to FP64 accuracy: split-BF16
        # factorisation on the A route, FP32 through chi0.
        dict(_solve(12, 655, 256, 4.0, 0.05, prec="bf16x", tol=1e-10), name="chain12_n655_bf16x_A"),
        dict(_solve(10, 517, 256, 4.0, 0.05, route="chi0", prec="fp32", tol=1e-10), name="chain10_n517_fp32_chi0"),
        # An ordinary molecule through chi0 on the full 1024-point mesh.
        dict(_solve(20, 1100, 1024, 8.0, 0.02, route="chi0"), name="chain20_n1100_chi0"),
        # The headline workload: 40 atoms, 2000 products, 1024 points, A = 1 -
        # v chi0 formed in W's buffer and solved there.
        dict(_solve(40, 2000, 1024, 8.0, 0.02), name="chain40_n2000_A"),
        # A 3-D cluster on the fine 2048-point mesh in the top-k subspace of v,
        # W decompressed at the points the program goes on with.
        {"name": "cluster48_k500", "kind": "compressed", "atoms": 48, "n_prod": 2500, "k": 500, "n_omega": 2048,
         "omega_max": 8.0, "eps": 0.01, "points": 16},
        # The paper's own subspace (pairs below an energy threshold).
        {"name": "cluster64_pair72", "kind": "pair", "atoms": 64, "n_prod": 3100, "k": 72, "threshold": 0.4,
         "n_omega": 1024, "omega_max": 8.0, "eps": 0.02, "points": 16},
        # Two spectral windows, chi0 and W on both meshes.
        {"name": "chain16_n880_2w", "kind": "two_window", "atoms": 16, "n_prod": 880},
        # a0 and A by the paper's time-domain route.
        {"name": "chain24_n1310_time", "kind": "time", "atoms": 24, "n_prod": 1310, "n_omega": 512,
         "omega_max": 8.0, "eps": 0.046875},
        # What comes after W: self-energy, exchange, G and the density of states.
        {"name": "chain16_n870_sigma", "kind": "sigma", "atoms": 16, "n_prod": 870, "n_omega": 512,
         "omega_max": 8.0, "eps": 0.046875},
        # The production batch form: uneven molecules recorded once, W in place.
        {"name": "batch6_chains8to26", "kind": "batch", "atoms": 8, "atoms_last": 26, "molecules": 6, "n_omega": 512,
         "omega_max": 8.0, "eps": 0.046875, "prec": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _products(rng, atoms):
    """A basis size that every chain of so many atoms reaches (40 per atom and
    16 per nearest-neighbour bond), odd as often as even."""
    top = 56 * atoms - 16
    return rng.randint(top - 50, top)


_MESHES = [(256, 4.0, 0.05), (512, 8.0, 0.046875), (1024, 8.0, 0.02)]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "mixed", "compressed", "pair", "two_window", "time",
                       "sigma", "batch"])
    n_omega, top, eps = rng.choice(_MESHES)
    mesh = {"n_omega": n_omega, "omega_max": top, "eps": eps}
    if kind == "solve":
        atoms = _log_int(rng, 4, 30)
        return _solve(atoms, _products(rng, atoms), n_omega, top, eps, route=rng.choice(["A", "chi0"]))
    if kind == "mixed":
        atoms = _log_int(rng, 4, 14)
        return _solve(atoms, _products(rng, atoms), 256, 4.0, 0.05, route=rng.choice(["A", "chi0"]),
                      prec=rng.choice(["fp32", "bf16x"]), tol=1e-10)
    if kind == "compressed":
        atoms = rng.randint(24, 56)
        return {"kind": kind, "atoms": atoms, "n_prod": 48 * atoms + rng.randint(-40, 40),
                "k": _log_int(rng, 200, 600), "points": 16, **mesh}
    if kind == "pair":
        atoms = rng.randint(32, 64)
        return {"kind": kind, "atoms": atoms, "n_prod": 48 * atoms + rng.randint(-40, 40),
                "k": rng.randint(atoms // 2, atoms), "threshold": 0.4, "points": 16, **mesh}
    if kind == "two_window":
        atoms = _log_int(rng, 4, 24)
        return {"kind": kind, "atoms": atoms, "n_prod": _products(rng, atoms)}
    if kind == "time":
        atoms = _log_int(rng, 4, 26)
        return {"kind": kind, "atoms": atoms, "n_prod": _products(rng, atoms), **mesh}
    if kind == "sigma":
        atoms = _log_int(rng, 4, 18)
        return {"kind": kind, "atoms": atoms, "n_prod": _products(rng, atoms), **mesh}
    first = rng.randint(4, 12)
    return {"kind": "batch", "atoms": first, "atoms_last": first + rng.randint(4, 14), "molecules": rng.randint(2, 6),
            "prec": "fp64", "n_omega": 512, "omega_max": 8.0, "eps": 0.046875}


# --------------------------------------------------------------------------
# inputs


def _molecule(case, seed):
    if case["kind"] in ("compressed", "pair"):
        n = case["atoms"]
        mol = gs.cluster_molecule(n, seed, radius=20.0 * (n / 120.0) ** (1.0 / 3.0))
    elif case.get("small_atoms"):
        mol = gs.chain_molecule(case["atoms"], seed, orb_per_atom=4, occ_per_atom=2, prod_per_atom=10, prod_per_bond=8,
                                bond_cutoff=None)
    else:
        mol = gs.chain_molecule(case["atoms"], seed)
    if mol.n_prod < case["n_prod"]:
        raise ValueError("the molecule of seed %d has %d products" % (seed, mol.n_prod))
    return gs.truncate_products(mol, case["n_prod"])


def _batch_atoms(case):
    a, b, n = case["atoms"], case["atoms_last"], case["molecules"]
    return [a + (b - a) * i // (n - 1) for i in range(n)]


def _batch_products(atoms):
    return 56 * atoms - 16


def _batch_molecule(atoms, seed):
    return gs.truncate_products(gs.chain_molecule(atoms, seed), _batch_products(atoms))


def _mesh(case):
    return case["n_omega"], -case["omega_max"], case["omega_max"], case["eps"]


def _empty(*shape, dtype=torch.complex128):
    return torch.empty(shape, dtype=dtype, device=DEVICE)


def _zeros(*shape, dtype):
    """Room for the most bins that a molecule of this kind has on the mesh: the
    rows past a molecule's own bins stay zero."""
    return torch.zeros(shape, dtype=dtype, device=DEVICE)


def _points(case):
    """The mesh points at which a compressed W is decompressed: evenly spaced."""
    return [case["n_omega"] * i // case["points"] for i in range(case["points"])]


def _lowrank_w(mol, case, seed):
    """An interaction v + U diag(c) U^T on the mesh, c(-omega) = c(omega)*."""
    n, N = mol.n_prod, case["n_omega"]
    U, c = gs.lowrank_w_factors(n, N, k_max=int(0.6 * (N // 2)), seed=seed)
    full = np.zeros((N, c.shape[1]), dtype=np.complex128)
    full[N // 2:] = c
    full[1:N // 2] = np.conj(c[:0:-1])
    return U, full


def _vxc(mol, seed):
    a = 0.02 * np.random.default_rng(seed + 77).standard_normal((mol.n_orb, mol.n_orb))
    return a + a.T


def prepare(case, seed):
    if case["kind"] == "batch":
        return _prepare_batch(case, seed)
    mol = _molecule(case, seed)
    st = {"case": case, "ctx": _context(), "mol": gw.DeviceMolecule(mol, device=DEVICE)}
    n = mol.n_prod
    if case["kind"] == "two_window":
        fine, coarse = gs.two_window_grids()
        st["grids"] = [gw.make_grid(g.n_omega, g.omega_min, g.omega_max, g.eps) for g in (fine, coarse)]
        for name in ("chi", "W"):
            st[name] = [_empty(g.n_omega, n, n) for g in (fine, coarse)]
        return st
    N = case["n_omega"]
    st["grid"] = gw.make_grid(*_mesh(case))
    if case["kind"] == "solve":
        st["W"] = _empty(N, n, n)
        if case["route"] == "chi0":
            st["hist"] = _zeros(_bins(case), n * (n + 1) // 2, dtype=torch.int64)
            st["chi"] = _empty(N, n, n)
    elif case["kind"] in ("compressed", "pair"):
        k = case["k"]
        st["U"], st["S"] = _empty(n, k, dtype=torch.float64), _empty(k, k, dtype=torch.float64)
        st["X"] = _empty(N, k, k)
        st["W"] = _empty(case["points"], n, n)
        if case["kind"] == "pair":
            st["Z"], st["R"] = _empty(n, k, dtype=torch.float64), _empty(n, n, dtype=torch.float64)
            st["ones"] = torch.ones(k, dtype=torch.float64, device=DEVICE)
    elif case["kind"] == "time":
        st["a"] = _zeros(_most_time_bins(case), n * (n + 1) // 2, dtype=torch.float64)
        st["A"] = _empty(N, n, n)
    elif case["kind"] == "sigma":
        no = mol.n_orb
        U, c = _lowrank_w(mol, case, seed)
        U = torch.from_numpy(U).to(DEVICE).to(torch.complex128)
        c = torch.from_numpy(c).to(DEVICE)
        W = _empty(N, n, n)
        for j in range(N):
            W[j] = (U * c[j]) @ U.T
        W += st["mol"].v
        st.update(W=W, Vxc=torch.from_numpy(_vxc(mol, seed)).to(DEVICE), Sigma=_empty(N, no, no),
                  Sigma_x=_empty(no, no, dtype=torch.float64), dos=_empty(N, dtype=torch.float64), G=_empty(N, no, no))
    return st


def _prepare_batch(case, seed):
    mols = [_batch_molecule(a, 16 * seed + i) for i, a in enumerate(_batch_atoms(case))]
    dms = [gw.DeviceMolecule(m, device=DEVICE) for m in mols]
    W = [_empty(case["n_omega"], m.n_prod, m.n_prod) for m in mols]
    ctx = gw.Context(0, BATCH_BUDGET)
    batch = ctx.batch_create([d.struct for d in dms], [d.v for d in dms], gw.make_grid(*_mesh(case)), W, W,
                             prec=PREC[case["prec"]])
    return {"case": case, "ctx": ctx, "mols": dms, "W": W, "batch": batch}


# --------------------------------------------------------------------------
# one pass


def run(st):
    case = st["case"]
    return {"solve": _run_solve, "compressed": _run_compressed, "pair": _run_pair, "two_window": _run_two_window,
            "time": _run_time, "sigma": _run_sigma, "batch": _run_batch}[case["kind"]](st, case)


def _run_solve(st, case):
    ctx, m, g, n, N = st["ctx"], st["mol"], st["grid"], case["n_prod"], case["n_omega"]
    prec, tol = PREC[case["prec"]], case["tol"]
    if case["route"] == "chi0":
        ctx.build_chi0(m.struct, g, st["chi"], hist_out=st["hist"], report=False)
        ctx.solve_W(m.v, n, st["chi"], N, st["W"], prec=prec, tol=tol, report=False)
        return {"hist": st["hist"], "chi": st["chi"], "W": st["W"]}
    ctx.build_A(m.struct, m.v, g, st["W"], report=False)
    ctx.solve_W_A(m.v, n, st["W"], N, st["W"], prec=prec, tol=tol, report=False)
    return {"W": st["W"]}


def _decompress(st, case, R=None):
    n, k = case["n_prod"], case["k"]
    for i, j in enumerate(_points(case)):
        st["ctx"].decompress(st["U"], n, k, st["X"][j], st["W"][i], R=R)
    return st["W"]


def _run_compressed(st, case):
    ctx, m, k = st["ctx"], st["mol"], case["k"]
    ctx.compress_basis(m.v, case["n_prod"], k, st["U"], st["S"])
    ctx.build_A_compressed(m.struct, st["S"], st["U"], k, st["grid"], st["X"], report=False)
    ctx.solve_W_A(st["S"], k, st["X"], case["n_omega"], st["X"], report=False)
    return {"W": _decompress(st, case)}


def _run_pair(st, case):
    ctx, m, k = st["ctx"], st["mol"], case["k"]
    rank = ctx.pair_basis(m.struct, m.v, case["threshold"], k, st["Z"], st["U"], st["R"])
    ctx.build_chi0(m.struct, st["grid"], st["X"], basis=st["U"], k=k, report=False)
    ctx.solve_W(st["ones"], k, st["X"], case["n_omega"], st["X"], v_is_diag=True, report=False)
    return {"rank": rank, "W": _decompress(st, case, R=st["R"])}


def _run_two_window(st, case):
    ctx, m, n = st["ctx"], st["mol"], case["n_prod"]
    fine, coarse = st["grids"]
    ctx.build_chi0_2w(m.struct, fine, coarse, st["chi"][0], st["chi"][1], report=False)
    for g, chi, W in zip(st["grids"], st["chi"], st["W"]):
        ctx.solve_W(m.v, n, chi, g.n_omega, W, report=False)
    return {"chi": st["chi"], "W": st["W"]}


def _run_time(st, case):
    m = st["mol"]
    st["ctx"].build_A_time(m.struct, m.v, st["grid"], st["A"], a_out=st["a"], report=False)
    return {"a": st["a"], "A": st["A"]}


def _run_sigma(st, case):
    ctx, m, g = st["ctx"], st["mol"], st["grid"]
    ctx.self_energy(m.struct, g, st["W"], st["Sigma"], v=m.v, Sigma_x_out=st["Sigma_x"], report=False)
    ctx.dyson_dos(m.struct, g, st["dos"], Sigma_c=st["Sigma"], Sigma_x=st["Sigma_x"], Vxc=st["Vxc"], G_out=st["G"],
                  report=False)
    return {"Sigma": st["Sigma"], "Sigma_x": st["Sigma_x"], "G": st["G"], "dos": st["dos"]}


def _run_batch(st, case):
    st["batch"].run(report=False)
    return {"W": st["W"]}


# --------------------------------------------------------------------------
# the work of a pass that no implementation can do without


def _bins(case):
    """The most spectral bins that the pair energies (up to 3 Ha) take."""
    d = 2.0 * case["omega_max"] / case["n_omega"]
    return min(case["n_omega"] // 2, int(3.0 / d) + 2)


def _pairs(atoms, small=False):
    return (2 * atoms) * (2 * atoms) if small else (4 * atoms) * (9 * atoms)


def _response_flops(n, pairs):
    return 2.0 * pairs * n * (n + 1) / 2 * 2


def _inputs_bytes(n, atoms, small=False):
    orb = (4 if small else 13) * atoms
    return 8.0 * (orb * orb + n * n + n * 300)


def _solve_flops(n, solved):
    """LU, and the two substitutions for a symmetric result."""
    return 8.0 * n ** 3 * solved


def _work_A(n, pairs, bins, N, out_bytes=True):
    """Weights, v a0 per bin, transform to the solved half of the mesh."""
    return _response_flops(n, pairs) + 2.0 * n ** 3 * (bins - 1) + 4.0 * n * n * bins * (N // 2 + 1)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for a in _batch_atoms(case):
            w = work(dict(_solve(a, _batch_products(a), case["n_omega"], case["omega_max"], case["eps"])))
            total = {k: total[k] + w[k] for k in total}
        return total
    n, atoms = case["n_prod"], case["atoms"]
    small = bool(case.get("small_atoms"))
    pairs = _pairs(atoms, small)
    inputs = _inputs_bytes(n, atoms, small)
    if kind == "two_window":
        fine, coarse = gs.two_window_grids()
        flops = 0.0
        for g in (fine, coarse):
            flops += _response_flops(n, pairs) + (4.0 + 8.0) * n ** 3 * (g.n_omega // 2 + 1)
        return {"bytes": inputs + 2 * 16.0 * n * n * (fine.n_omega + coarse.n_omega), "flops": flops}
    N, bins = case["n_omega"], _bins(case)
    solved = N // 2 + 1
    full = 16.0 * n * n * N
    if kind == "solve":
        if case["route"] == "A":
            return {"bytes": inputs + full, "flops": _work_A(n, pairs, bins, N) + _solve_flops(n, solved)}
        hist = 8.0 * bins * n * (n + 1) / 2
        return {"bytes": inputs + hist + 2 * full,
                "flops": _response_flops(n, pairs) + 4.0 * n ** 3 * solved + _solve_flops(n, solved)}
    if kind == "compressed":
        k = case["k"]
        flops = 2.0 * n * n * k + 2.0 * k * n * pairs + _work_A(k, pairs, bins, N) + _solve_flops(k, solved)
        return {"bytes": inputs + 16.0 * n * n * case["points"],
                "flops": flops + case["points"] * 4.0 * (n * k * k + n * n * k)}
    if kind == "pair":
        k = case["k"]
        flops = 2.0 * n * n * k + 2.0 * k * n * pairs + _response_flops(k, pairs) + _solve_flops(k, solved)
        return {"bytes": inputs + 16.0 * n * n * case["points"],
                "flops": flops + case["points"] * 4.0 * (n * k * k + n * n * k)}
    if kind == "time":
        times = bins // 2 + 2  # real data: half of the time points
        return {"bytes": inputs + 8.0 * bins * n * (n + 1) / 2 + full,
                "flops": times * n * (n + 1) / 2 * 4.0 * 13 * 13 + _work_A(n, 0, bins, N)}
    orb = 13 * atoms
    times = N // 2
    return {"bytes": inputs + full / 2 + 16.0 * orb * orb * N * 2,
            "flops": times * n * n * 2.0 * 13 * 13 + (8.0 / 3 + 16.0 / 3) * orb ** 3 * N}


# --------------------------------------------------------------------------
# the same in plain torch and numpy, in 64 bits: sums over pairs and levels
# as the method states them, LAPACK's solve


def _pair_vectors(mol):
    """V_mu^{EF} on the GPU, [n_prod][n_occ * n_virt]."""
    out = []
    X = torch.from_numpy(mol.X).to(DEVICE)
    for b in range(mol.n_blk):
        _, _, orbs, mats = mol.block_of(b)
        x = X[torch.from_numpy(np.asarray(orbs, dtype=np.int64)).to(DEVICE)]
        occ, virt = x[:, :mol.n_occ].contiguous(), x[:, mol.n_occ:].contiguous()
        for m in mats:
            out.append((occ.T.contiguous() @ torch.from_numpy(np.ascontiguousarray(m)).to(DEVICE) @ virt).reshape(-1))
    return torch.stack(out)


def _pair_energies(mol):
    return (mol.eig[None, mol.n_occ:] - mol.eig[:mol.n_occ, None]).reshape(-1)


def _split(energy, d):
    """Each pole's two mesh bins and their weights."""
    m = np.floor(energy / d)
    f = energy / d - m
    return [(m, 1.0 - f), (m + 1, f)]


def _cauchy(omega, s, eps):
    return 1.0 / (omega - s + 1j * eps) - 1.0 / (omega + s + 1j * eps)


def _pair_factors(omegas, parts, eps):
    """c_p(omega) = 2 sum over the bins of pair p of weight times kernel;
    parts: (bin position in Ha, weight) arrays over pairs."""
    c = np.zeros((len(omegas), len(parts[0][0])), dtype=np.complex128)
    for s, w in parts:
        c += 2.0 * w[None, :] * _cauchy(omegas[:, None], s[None, :], eps)
    return c


def _weighted(P, c):
    """P diag(c) P^T for a complex c."""
    c = torch.from_numpy(c).to(DEVICE)
    PT = P.T.contiguous()
    return torch.complex((P * c.real) @ PT, (P * c.imag) @ PT)


def _on_mesh(N, omegas, point):
    """point(j) at the upper half of the mesh and its lone lowest point, the
    rest by conjugation."""
    first = point(0)
    out = torch.empty((N,) + tuple(first.shape), dtype=torch.complex128)
    out[0] = first.cpu()
    for j in range(N // 2, N):
        out[j] = point(j).cpu()
        if j > N // 2:
            out[N - j] = out[j].conj()
    return out


def _screened(chi, v):
    n = v.shape[0]
    a = np.eye(n) - v @ chi
    return np.linalg.solve(a, v)


def _exact_mesh(mol, P, N, top, parts, eps, with_w):
    """(chi0, W or None) on a symmetric mesh."""
    d = 2.0 * top / N
    om = -top + d * np.arange(N)
    c = _pair_factors(om, parts, eps) if N * P.shape[1] < 2e7 else None

    def chi_at(j):
        cj = c[j] if c is not None else _pair_factors(om[j:j + 1], parts, eps)[0]
        return _weighted(P, cj)

    chi = _on_mesh(N, om, chi_at)
    if not with_w:
        return chi, None
    W = _on_mesh(N, om, lambda j: torch.from_numpy(_screened(chi[j].numpy(), mol.v)))
    return chi, W


#: LAPACK's solves of a whole mesh stay within seconds up to this many flops.
_MOST_SOLVE = 6e11


def _cheap_solves(n, solved):
    return 12.0 * float(n) ** 3 * solved <= _MOST_SOLVE


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return None
    mol = _molecule(case, seed)
    n = mol.n_prod
    if kind == "sigma":
        return _exact_sigma(case, mol, seed)
    if kind == "two_window":
        return _exact_two_window(mol)
    N, top, eps = case["n_omega"], case["omega_max"], case["eps"]
    d = 2.0 * top / N
    energies = _pair_energies(mol)
    if kind == "time":
        return _exact_time(case, mol, d)
    if kind in ("compressed", "pair"):
        return _exact_points(case, mol)
    with_w = _cheap_solves(n, N // 2 + 1)
    if case["route"] == "A" and not with_w:
        return None
    if 16.0 * n * n * N > 8e9:
        return None
    chi, W = _exact_mesh(mol, _pair_vectors(mol), N, top, [(m * d, w) for m, w in _split(energies, d)], eps, with_w)
    if case["route"] == "A":
        return {"W": W}
    return {"hist": None, "chi": chi, "W": W}


def _exact_points(case, mol):
    """W at the decompressed points.  The top-k form uses v projected on its k
    leading eigenvectors; the pair subspace is an approximation whose own
    basis stands in for the full one, so it has no value here."""
    if case["kind"] == "pair":
        return None
    N, top, eps, k = case["n_omega"], case["omega_max"], case["eps"], case["k"]
    d = 2.0 * top / N
    lam, Q = np.linalg.eigh(mol.v)
    Q, lam = np.ascontiguousarray(Q[:, -k:]), lam[-k:]
    P = torch.from_numpy(np.ascontiguousarray(Q.T)).to(DEVICE) @ _pair_vectors(mol)
    om = -top + d * np.arange(N)
    parts = [(m * d, w) for m, w in _split(_pair_energies(mol), d)]
    W = []
    for j in _points(case):
        chi = _weighted(P, _pair_factors(om[j:j + 1], parts, eps)[0]).cpu().numpy()
        X = np.linalg.solve(np.eye(k) - lam[:, None] * chi, np.diag(lam).astype(np.complex128))
        W.append(Q @ X @ Q.T)
    return {"W": torch.from_numpy(np.stack(W))}


def _exact_two_window(mol):
    fine, coarse = gs.two_window_grids()
    energies = _pair_energies(mol)
    P = _pair_vectors(mol)
    ds, dl = fine.domega, coarse.domega
    edge = math.floor((fine.omega_max - ds) / dl) * dl
    low = (energies < edge).astype(np.float64)
    om = fine.omegas()
    cf = _pair_factors(om, [(m * ds, w * low) for m, w in _split(energies, ds)], fine.eps)
    cf += _pair_factors(om, [(m * dl, w * (1.0 - low)) for m, w in _split(energies, dl)], coarse.eps)
    small = _on_mesh(fine.n_omega, om, lambda j: _weighted(P, cf[j]))
    large, _ = _exact_mesh(mol, P, coarse.n_omega, coarse.omega_max,
                           [(m * dl, w) for m, w in _split(energies, dl)], coarse.eps, False)
    if not _cheap_solves(mol.n_prod, fine.n_omega + 2):
        return {"chi": [small, large], "W": None}
    W = [_on_mesh(g.n_omega, g.omegas(), lambda j, c=c: torch.from_numpy(_screened(c[j].numpy(), mol.v)))
         for g, c in ((fine, small), (coarse, large))]
    return {"chi": [small, large], "W": W}


def _level_split(mol, d):
    empty, occ = _split(mol.eig[mol.n_occ:], d), _split(-mol.eig[:mol.n_occ], d)
    return occ, empty


def _time_bins(mol, case):
    """Bins of the one-particle split: K+ + K- - 1, at most half the mesh."""
    d = 2.0 * case["omega_max"] / case["n_omega"]
    kp = int(math.floor(mol.eig[-1] / d)) + 2
    km = int(math.floor(-mol.eig[0] / d)) + 2
    return min(case["n_omega"] // 2, kp + km - 1)


def _most_time_bins(case):
    d = 2.0 * case["omega_max"] / case["n_omega"]
    return min(case["n_omega"] // 2, int(2.0 / d) + int(1.0 / d) + 3)


def _exact_time(case, mol, d):
    """a0 with each pair on the bins of its two one-particle splits, and A."""
    N, n = case["n_omega"], mol.n_prod
    if 16.0 * n * n * N > 1.6e10:
        return None
    bins = _time_bins(mol, case)
    P = _pair_vectors(mol)
    occ, empty = _level_split(mol, d)
    iu = torch.triu_indices(n, n, device=DEVICE)
    full = torch.zeros((bins, n, n), dtype=torch.float64, device=DEVICE)
    for mo, wo in occ:
        for me, we in empty:
            at = (mo[:, None] + me[None, :]).reshape(-1).astype(np.int64)
            w = 2.0 * (wo[:, None] * we[None, :]).reshape(-1)
            for m in np.unique(at):
                if m < bins:
                    sel = torch.from_numpy(np.nonzero(at == m)[0]).to(DEVICE)
                    p = P[:, sel].contiguous()
                    full[m] += (p * torch.from_numpy(w[at == m]).to(DEVICE)) @ p.T.contiguous()
    a = torch.zeros((_most_time_bins(case), n * (n + 1) // 2), dtype=torch.float64)
    a[:bins] = full[:, iu[0], iu[1]].cpu()
    va = torch.from_numpy(mol.v).to(DEVICE) @ full.permute(1, 0, 2).reshape(n, bins * n)
    va = va.reshape(n, bins, n).permute(1, 0, 2).reshape(bins, n * n).contiguous()
    del full
    om = -case["omega_max"] + d * np.arange(N)
    K = _cauchy(om[:, None], d * np.arange(1, bins)[None, :], case["eps"])
    eye = torch.eye(n, dtype=torch.float64, device=DEVICE)

    def point(j):
        k = torch.from_numpy(K[j:j + 1]).to(DEVICE)
        re, im = k.real.contiguous() @ va[1:], k.imag.contiguous() @ va[1:]
        return torch.complex(eye - re.reshape(n, n), -im.reshape(n, n))

    return {"a": a, "A": _on_mesh(N, om, point)}


def _exact_sigma(case, mol, seed):
    """The spectra level by level: with the low-rank W each level is a short
    sum over ranks; then the Cauchy sum, the exchange and a direct inverse."""
    N, no, top, eps = case["n_omega"], mol.n_orb, case["omega_max"], case["eps"]
    d = 2.0 * top / N
    U, c = _lowrank_w(mol, case, seed)
    rank, half = U.shape[1], N // 2
    gamma = -(d / math.pi) * np.imag(c[half:])
    gamma[0] = 0.0
    # sum over products of U[mu][r] V_mu, then times the eigenvectors
    VU = np.zeros((rank, no, no))
    Xo = np.ascontiguousarray(mol.X[:, :mol.n_occ])
    u = np.zeros((mol.n_prod, no, mol.n_occ))
    for b in range(mol.n_blk):
        p0, cnt, orbs, mats = mol.block_of(b)
        V = np.stack(mats)
        idx = np.ix_(orbs, orbs)
        for r in range(rank):
            VU[r][idx] += np.tensordot(U[p0:p0 + cnt, r], V, axes=1)
        u[p0:p0 + cnt, orbs, :] = V @ Xo[orbs]
    flat = torch.from_numpy(u.reshape(mol.n_prod, -1)).to(DEVICE)
    vu = (torch.from_numpy(mol.v).to(DEVICE) @ flat).reshape(mol.n_prod, no, mol.n_occ)
    uu = flat.reshape(mol.n_prod, no, mol.n_occ).permute(1, 0, 2).reshape(no, -1).contiguous()
    exch = -(uu @ vu.permute(0, 2, 1).reshape(-1, no).contiguous()).cpu().numpy()
    G = np.einsum("rab,bE->Ear", VU, mol.X)  # [state][orbital][rank]
    om = -top + d * np.arange(N)
    Sigma = np.zeros((N, no, no), dtype=np.complex128)
    # per state and rank: s[j] = sum of bins of weight times the kernel
    coef = np.zeros((mol.n_orb, rank, N), dtype=np.complex128)
    k = np.arange(half)
    for E in range(mol.n_orb):
        sign = 1.0 if E >= mol.n_occ else -1.0
        g = np.zeros((half, rank))
        for m, w in _split(np.array([abs(mol.eig[E])]), d):
            at = k + int(m[0])
            ok = at < half
            g[at[ok]] += w[0] * gamma[k[ok]]
        kern = 1.0 / (om[:, None] - sign * d * k[None, :] + 1j * eps)
        coef[E] = (kern @ g).T
    Gf = torch.from_numpy(np.ascontiguousarray(G.transpose(0, 2, 1).reshape(-1, no))).to(DEVICE)
    cf = torch.from_numpy(coef.reshape(-1, N)).to(DEVICE)
    for j in range(N):
        re = (Gf * cf[:, j].real[:, None]).T.contiguous() @ Gf
        im = (Gf * cf[:, j].imag[:, None]).T.contiguous() @ Gf
        Sigma[j] = torch.complex(re, im).cpu().numpy()
    static = (mol.X * mol.eig) @ mol.X.T + exch - _vxc(mol, seed)
    g = np.empty_like(Sigma)
    for j in range(N):
        g[j] = np.linalg.inv((om[j] + 1j * eps) * np.eye(no) - static - Sigma[j])
    dos = -np.imag(np.trace(g, axis1=1, axis2=2)) / math.pi
    return {"Sigma": torch.from_numpy(Sigma), "Sigma_x": torch.from_numpy(exch), "G": torch.from_numpy(g),
            "dos": torch.from_numpy(dos)}
