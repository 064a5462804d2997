"""Where the 32-bit factorisation and substitutions round.

The matrices make every product of a sum a small multiple of a power of two and
the sum cancel: 2^24 - 2^24 with 62 quarters in between.  Each entry of the
result, and every sum of whole products, fits a float, so arithmetic that rounds
once per sum gives W exactly and the refinement finds a residual of exactly
zero; with a rounding per few products the quarters are lost beside 2^24 (whose
neighbour is 2 away) and the first update is not zero.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

N_OMEGA = 4  # solved: j = 0, 2, 3
B = 64       # panel


def _first_update(A, v, W, prec):
    """The first solution and its update: a tolerance that stops after one step."""
    import paper_1101_2065_amd.gw as gw

    n = v.shape[0]
    ctx = gw.Context(0)
    Ad = torch.from_numpy(np.stack([A] * N_OMEGA)).cuda()
    vd = torch.from_numpy(np.ascontiguousarray(v)).cuda()
    out = torch.empty_like(Ad)
    rep = ctx.solve_W_A(vd, n, Ad, N_OMEGA, out, prec=getattr(gw, "GW_" + prec), tol=1.0)
    ctx.close()
    assert rep.n_fallback == 0 and rep.max_iter == 1
    got = out.cpu().numpy()
    for j in (0, 2, 3):
        np.testing.assert_array_equal(got[j], W)
    assert rep.max_rel_update == 0.0


@pytest.mark.parametrize("prec", ["FP32_IR", "BF16X_IR"])
@pytest.mark.parametrize("upper", [False, True])
def test_substitution_rounds_once_per_panel(upper, prec):
    """Two panels, T_10 (T_01) = 1/4 (1 + i) everywhere, unit diagonal blocks."""
    P = np.ones((B, B))
    P[0], P[-1] = 2.0 ** 26, -2.0 ** 26
    A = np.eye(2 * B, dtype=np.complex128)
    v = np.zeros((2 * B, 2 * B))
    if upper:
        A[:B, B:] = 0.25 + 0.25j
        v[B:, :B], v[:B, B:] = P, P.T
        W = v.astype(np.complex128)
        W[:B, :B] = -(0.25 + 0.25j) * P.sum(0)
    else:
        A[B:, :B] = 0.25 + 0.25j
        v[:B, B:], v[B:, :B] = P, P.T
        W = v.astype(np.complex128)
        W[B:, B:] = -(0.25 + 0.25j) * P.sum(0)
    _first_update(A, v, W, prec)


@pytest.mark.parametrize("prec", ["FP32_IR", "BF16X_IR"])
@pytest.mark.parametrize("n", [64, 600, 1100])
def test_panel_update_rounds_once_per_chunk(n, prec):
    """The last 16 columns of the first panel against its first 48: L = 1/2 on
    rows 48 .. 63, U = (2^25, 1/2, ..., 1/2, -2^25), so that A = L U has 1/2 *
    46 * 1/2 there.  v = A S A^T with S = 1 on those 16 columns, so W = S A^T
    (64, 600, 1100: one, two, four rows a thread)."""
    k = 48
    u = np.full(k, 0.5)
    u[0], u[-1] = 2.0 ** 25, -2.0 ** 25
    A = np.eye(n)
    A[k:B, :k] = 0.5
    A[:k, k:B] = u[:, None]
    A[k:B, k:B] += 0.5 * u.sum()
    S = np.zeros((n, n))
    S[range(k, B), range(k, B)] = 1.0
    _first_update(A.astype(np.complex128), A @ S @ A.T, S @ A.T, prec)
