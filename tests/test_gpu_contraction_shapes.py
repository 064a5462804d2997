"""The time-route and self-energy contractions at the orbital-set and block
sizes where their tiles, groups and pair order change, against the oracle.

Bars as for the workloads: a0 within 1e-12 relative Frobenius, sigma+- and
Sigma within 1e-11 (FP64 on both sides, sums in another order).
"""
import numpy as np
import pytest

import gw_synth as gs
import oracle as o

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


# orbitals per atom (a bond has twice as many): one and two 16-tiles, full and
# ragged, and sets of 30 and 32, for which fewer matrices fit the LDS at once;
# products per atom and bond: fewer than a group, one more than a tile
_SHAPES = [(3, 7, 5), (8, 17, 3), (9, 16, 8), (15, 9, 17), (16, 5, 9)]


def _molecule(orb, per_atom, per_bond):
    return gs.chain_molecule(3, 40 + orb, orb_per_atom=orb, occ_per_atom=max(1, orb // 3), prod_per_atom=per_atom,
                             prod_per_bond=per_bond, bond_cutoff=None)


@pytest.mark.parametrize("shape", _SHAPES)
def test_time_contraction(shape):
    import paper_1101_2065_amd.gw as gw

    mol, grid = _molecule(*shape), gs.config_grid(0)
    ctx = gw.Context(0)
    dm = gw.DeviceMolecule(mol)
    n = mol.n_prod
    nhb = o.level_hist_bins(mol.eig, mol.n_occ, grid.n_omega, grid.domega)
    a = torch.full((nhb, n * (n + 1) // 2), float("nan"), dtype=torch.float64, device="cuda")
    chi = torch.full((grid.n_omega, n, n), float("nan"), dtype=torch.complex128, device="cuda")
    ctx.build_chi0_time(dm.struct, gw.make_grid(grid.n_omega, grid.omega_min, grid.omega_max, grid.eps), chi, a_out=a)
    ref = o.a0_by_pairs(o.pair_vectors(mol), mol.eig, mol.n_occ, grid.domega, nhb)
    assert _rel(a.cpu().numpy(), ref) < 1e-12
    ctx.close()


@pytest.mark.parametrize("shape", _SHAPES)
def test_self_energy_contraction(shape):
    import paper_1101_2065_amd.gw as gw

    mol = _molecule(*shape)
    N, top, eps = 64, 8.0, 0.3
    ctx = gw.Context(0)
    dm = gw.DeviceMolecule(mol)
    U, c = gs.lowrank_w_factors(mol.n_prod, N, k_max=16, seed=3)
    full = np.zeros((N, c.shape[1]), dtype=np.complex128)
    full[N // 2:] = c
    full[1:N // 2] = np.conj(c[:0:-1])
    W = np.einsum("mr,jr,nr->jmn", U, full, U) + mol.v
    no = mol.n_orb
    sig = torch.full((2, N // 2, no, no), float("nan"), dtype=torch.float64, device="cuda")
    Sig = torch.full((N, no, no), float("nan"), dtype=torch.complex128, device="cuda")
    Sx = torch.full((no, no), float("nan"), dtype=torch.float64, device="cuda")
    ctx.self_energy(dm.struct, gw.make_grid(N, -top, top, eps), torch.from_numpy(W).cuda(), Sig, v=dm.v, sigma_out=sig,
                    Sigma_x_out=Sx)
    d = 2 * top / N
    gamma = o.w_spectral(W, N, -top, top)
    sp, sm = o.self_energy_spectra_by_levels(mol, gamma, d, N // 2)
    got = sig.cpu().numpy()
    assert _rel(got[0], sp) < 1e-11 and _rel(got[1], sm) < 1e-11
    assert _rel(Sig.cpu().numpy(), o.self_energy_from_spectra(sp, sm, N, -top, top, eps)) < 1e-11
    assert _rel(Sx.cpu().numpy(), o.exchange_self_energy(mol)) < 1e-12
    ctx.close()
