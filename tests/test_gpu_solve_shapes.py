"""W = A^-1 v at the sizes where the products and panels of the solve change
their tile, their remainder or their variant, against LAPACK.

Tolerance: Gaussian elimination with partial pivoting followed by the
substitutions is normwise backward stable, so the relative error of W is at
most a modest multiple of n eps cond(A); 32 n eps cond(A) allows for pivot
growth and the three-product complex products.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

N_OMEGA = 6  # solved: j = 0 and j >= 3
EPS = 2.0 ** -52


def _inputs(n, seed):
    """v symmetric positive, chi0 complex symmetric with chi0(-w) = chi0(w)*."""
    rng = np.random.default_rng(seed)
    b = rng.standard_normal((n, n)) / np.sqrt(n)
    v = b @ b.T + np.eye(n)
    chi = np.zeros((N_OMEGA, n, n), dtype=np.complex128)
    for j in (0, 3, 4, 5):
        c = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(n)
        chi[j] = c + c.T
    for j in (1, 2):
        chi[j] = np.conj(chi[N_OMEGA - j])
    return v, chi


def _check(W, v, chi):
    n = v.shape[0]
    for j in range(N_OMEGA):
        A = np.eye(n) - v @ chi[j]
        ref = np.linalg.solve(A, v.astype(np.complex128))
        err = np.linalg.norm(W[j] - ref) / np.linalg.norm(ref)
        assert err <= 32 * n * EPS * np.linalg.cond(A), (n, j, err)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 16, 17, 31, 33, 63, 64, 65, 72, 96, 127, 129, 191, 193, 255, 257, 320,
                               333, 449, 511, 513, 577, 1025])
def test_solve_at_every_edge(n):
    import paper_1101_2065_amd.gw as gw

    v, chi = _inputs(n, 100 + n)
    ctx = gw.Context(0)
    vd, cd = torch.from_numpy(v).cuda(), torch.from_numpy(chi).cuda()
    W = torch.empty_like(cd)
    ctx.solve_W(vd, n, cd, N_OMEGA, W)
    _check(W.cpu().numpy(), v, chi)
    # from A, in place
    A = torch.eye(n, dtype=torch.complex128, device="cuda") - torch.stack([vd.to(torch.complex128) @ c for c in cd])
    ctx.solve_W_A(vd, n, A, N_OMEGA, A)
    _check(A.cpu().numpy(), v, chi)
    ctx.close()


@pytest.mark.parametrize("prec", ["FP32_IR", "BF16X_IR"])
@pytest.mark.parametrize("n", [1, 63, 65, 128, 130, 255, 257, 320, 333, 513])
def test_mixed_solve_at_the_block_edges(n, prec):
    """The 32-bit factorisation and substitutions must be good enough for the
    refinement to reach its tolerance by itself (no FP64 fallback)."""
    import paper_1101_2065_amd.gw as gw

    v, chi = _inputs(n, 300 + n)
    ctx = gw.Context(0)
    vd, cd = torch.from_numpy(v).cuda(), torch.from_numpy(chi).cuda()
    W = torch.empty_like(cd)
    rep = ctx.solve_W(vd, n, cd, N_OMEGA, W, prec=getattr(gw, "GW_" + prec), tol=1e-8)
    assert rep.n_fallback == 0
    Wh = W.cpu().numpy()
    for j in range(N_OMEGA):
        A = np.eye(n) - v @ chi[j]
        ref = np.linalg.solve(A, v.astype(np.complex128))
        assert np.linalg.norm(Wh[j] - ref) <= (1e-8 + 32 * n * EPS * np.linalg.cond(A)) * np.linalg.norm(ref), (n, j)
    ctx.close()


@pytest.mark.parametrize("n", [5, 65, 130, 300])
def test_solve_from_pointers_that_are_not_16_byte_aligned(n):
    """double _Complex only asks for 8-byte alignment."""
    import paper_1101_2065_amd.gw as gw

    v, chi = _inputs(n, 7)
    ctx = gw.Context(0)
    size = 2 * N_OMEGA * n * n
    bufs = [torch.zeros(size + 1, dtype=torch.float64, device="cuda") for _ in range(2)]
    vbuf = torch.zeros(n * n + 1, dtype=torch.float64, device="cuda")
    vbuf[1:] = torch.from_numpy(v).cuda().reshape(-1)
    bufs[0][1:] = torch.view_as_real(torch.from_numpy(chi)).reshape(-1).cuda()
    ctx.solve_W(vbuf.data_ptr() + 8, n, bufs[0].data_ptr() + 8, N_OMEGA, bufs[1].data_ptr() + 8)
    W = bufs[1][1:].cpu().numpy().view(np.complex128).reshape(N_OMEGA, n, n)
    _check(W, v, chi)
    assert float(bufs[1][0]) == 0.0
    ctx.close()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 97, 128, 129, 161, 255, 300])
@pytest.mark.parametrize("bins", [2, 5, 64])
def test_spectral_products_at_every_edge(n, bins):
    """A = 1 - v chi0 by both routes on one small molecule whose basis is cut at
    n: the products v a0 and the Cauchy product (odd and even rows, K tails)
    must give 1 - v chi0.  Both sum the same terms in another order: at most
    (n + bins) roundings of entries bounded by |v| |a0| |T|, so 8 (n + bins) eps
    times the largest entry of |v| |chi0| + 1."""
    import gw_synth as gs
    import paper_1101_2065_amd.gw as gw

    mol = gs.truncate_products(gs.chain_molecule(6, 11), n)
    N, top = {2: (16, 16.0), 5: (32, 16.0), 64: (256, 4.0)}[bins]
    g = gw.make_grid(N, -top, top, 0.05)
    ctx = gw.Context(0)
    dm = gw.DeviceMolecule(mol)
    chi = torch.full((N, n, n), float("nan"), dtype=torch.complex128, device="cuda")
    A = torch.full_like(chi, float("nan"))
    ctx.build_chi0(dm.struct, g, chi)
    ctx.build_A(dm.struct, dm.v, g, A)
    ref = torch.eye(n, dtype=torch.complex128, device="cuda") - torch.stack([dm.v.to(torch.complex128) @ c for c in chi])
    scale = float((dm.v.abs() @ chi.abs().amax(0)).amax()) + 1.0
    assert float((A - ref).abs().amax()) <= 8 * (n + bins) * EPS * scale
    ctx.close()
