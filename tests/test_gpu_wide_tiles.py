"""The tiles and panels that carry the large workloads, at sizes they do not
divide: the 128-wide real and complex products, every tile of the batched
driver's long products, the FP32 panels of more than 2048 rows, and the A
route's products beside a histogram in several ranges."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import gw_synth as gs

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EPS = 2.0 ** -52


# n, mesh, products v a0 of how many bins at least side by side.  381: three
# 128s less three, over at least 114 bins, 1024 tiles of 128x128; 1301: 128x64
# (21 64-wide columns are one fewer than eleven 128-wide ones hold) from 5 bins on.
@pytest.mark.parametrize("n, atoms, grid, bins", [(381, 8, (256, -2.0, 2.0, 0.05), 114),
                                                  (1301, 24, (32, -8.0, 8.0, 0.5), 6)])
def test_wide_real_products(n, atoms, grid, bins, monkeypatch):
    """A = 1 - v chi0 from the products v a0 against chi0 itself: the same terms
    in another order, at most (n + bins) roundings of entries bounded by
    |v| |a0| |T|, so 8 (n + bins) eps times the largest entry of |v| |chi0| + 1."""
    import paper_1101_2065_amd.gw as gw

    monkeypatch.setenv("GW_HIST_CHUNKS", "1")
    dm = gw.DeviceMolecule(gs.truncate_products(gs.chain_molecule(atoms, 11), n))
    ctx = gw.Context(0)
    g = gw.make_grid(*grid)
    chi = torch.full((grid[0], n, n), float("nan"), dtype=torch.complex128, device="cuda")
    A = torch.full_like(chi, float("nan"))
    rep = ctx.build_chi0(dm.struct, g, chi)
    assert rep.n_hbins - 1 >= bins
    ctx.build_A(dm.struct, dm.v, g, A)
    peak = 0.0
    bound = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    for j in range(grid[0]):
        c = chi[j]
        ref = torch.eye(n, dtype=torch.complex128, device="cuda") - dm.v.to(torch.complex128) @ c
        peak = max(peak, float((A[j] - ref).abs().amax()))
        bound = torch.maximum(bound, c.abs())
    assert peak <= 8 * (n + rep.n_hbins) * EPS * (float((dm.v.abs() @ bound).amax()) + 1.0)
    ctx.close()


_BATCH = """
import sys
import numpy as np, torch
import gw_synth as gs
from paper_1101_2065_amd import gw
sizes, N = (513, 649, 1025), 16
ctx = gw.Context(0, 16 << 30)
mols = [gw.DeviceMolecule(gs.truncate_products(gs.chain_molecule(a, 5 + a), n)) for a, n in zip((10, 12, 19), sizes)]
chi = [torch.empty(N, n, n, dtype=torch.complex128, device="cuda") for n in sizes]
W = [torch.empty_like(c) for c in chi]
b = ctx.batch_create([m.struct for m in mols], [m.v for m in mols], gw.make_grid(N, -4.0, 4.0, 0.5), chi, W)
b.run()
for m, n, c, w in zip(mols, sizes, chi, W):
    v = m.v.cpu().numpy()
    for j in (0, N // 2, N - 1):
        A = np.eye(n) - v @ c[j].cpu().numpy()
        ref = np.linalg.solve(A, v.astype(complex))
        err = np.linalg.norm(w[j].cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 32 * n * 2.0 ** -52 * np.linalg.cond(A), (n, j, err)
print("OK")
"""


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
def test_long_products_of_a_batch_by_every_tile(tile, tmp_path):
    """A recorded batch whose tuner table names the tile (64x64, 128x64, 64x32,
    32x32): trailing updates with an edge of one row and column (513), products
    of inner dimension 137 (649), several blocks (1025); against LAPACK, within
    the backward error of elimination, 32 n eps cond(A)."""
    table = tmp_path / "tune.json"
    table.write_text(json.dumps({"zgemm_lds_fp64_n%d" % c: tile for c in (768, 1280)}))
    env = dict(os.environ, GW_TUNE_FILE=str(table), PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", _BATCH], env=env, cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-2000:] + r.stderr[-2000:]
    assert json.loads(table.read_text()) == {"zgemm_lds_fp64_n%d" % c: tile for c in (768, 1280)}  # nothing measured


@pytest.mark.parametrize("prec", ["FP32_IR", "BF16X_IR"])
@pytest.mark.parametrize("n", [2600, 3500])
def test_tall_float_panels(n, prec):
    """Six and eight rows a thread in FP32: the factorisation must be good enough
    for the refinement to reach W within 1e-8 by itself.  Then |A W - v| is at
    most |A| |W| 1e-8 beside the rounding of the check."""
    import paper_1101_2065_amd.gw as gw

    g = torch.Generator(device="cuda")
    g.manual_seed(n)

    def rand():
        return torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5

    b = rand()
    v = b @ b.T + torch.eye(n, device="cuda", dtype=torch.float64)
    chi = torch.empty(2, n, n, dtype=torch.complex128, device="cuda")
    for j in range(2):
        x = torch.complex(rand(), rand())
        chi[j] = x + x.T
    W = torch.empty_like(chi)
    ctx = gw.Context(0)
    rep = ctx.solve_W(v, n, chi, 2, W, prec=getattr(gw, "GW_" + prec), tol=1e-8)
    ctx.close()
    assert rep.n_solved == 2 and rep.n_fallback == 0
    vc = v.to(torch.complex128)
    for j in range(2):
        A = torch.eye(n, dtype=torch.complex128, device="cuda") - vc @ chi[j]
        r = (A @ W[j] - vc).norm()
        assert float(r) <= (1e-8 + 4 * n * EPS) * float(A.norm() * W[j].norm()), j


def test_histogram_ranges_beside_the_products(monkeypatch):
    """A small molecule takes one range by itself; four (what a large one takes)
    and sixteen give the same A bit for bit."""
    import paper_1101_2065_amd.gw as gw

    monkeypatch.delenv("GW_A_TRANSFORM", raising=False)
    n, N = 301, 256
    dm = gw.DeviceMolecule(gs.truncate_products(gs.chain_molecule(6, 2), n))
    ctx = gw.Context(0)
    got = {}
    for chunks in (None, "1", "4", "16"):
        if chunks is None:
            monkeypatch.delenv("GW_HIST_CHUNKS", raising=False)
        else:
            monkeypatch.setenv("GW_HIST_CHUNKS", chunks)
        A = torch.full((N, n, n), float("nan"), dtype=torch.complex128, device="cuda")
        rep = ctx.build_A(dm.struct, dm.v, gw.make_grid(N, -4.0, 4.0, 0.05), A)
        assert rep.n_hbins > 32
        got[chunks] = A
    ctx.close()
    for chunks, A in got.items():
        assert torch.equal(A, got["1"]), chunks
