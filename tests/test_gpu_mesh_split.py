"""W at a frequency does not depend on how the mesh was cut into batches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 129, 301, 513])
def test_w_does_not_depend_on_the_other_mesh_points(n):
    """Eight points at once (a lone point and a batch of four) and two at a time:
    1 - v chi0, whose product takes another kernel where v's odd rows find no
    room to be padded, and the solve give the same bits."""
    import paper_1101_2065_amd.gw as gw

    N = 8
    rng = np.random.default_rng(n)
    b = rng.standard_normal((n, n)) / np.sqrt(n)
    chi = rng.standard_normal((N, n, n)) + 1j * rng.standard_normal((N, n, n))
    chi = (chi + chi.transpose(0, 2, 1)) / np.sqrt(n)
    ctx = gw.Context(0)
    v = torch.from_numpy(b @ b.T + np.eye(n)).cuda()
    c = torch.from_numpy(chi).cuda()
    W = torch.empty_like(c)
    ctx.solve_W(v, n, c, N, W)
    for j, k in ((0, 4), (5, 6), (7, 0)):
        pair = torch.stack([c[j], c[k]])
        Wp = torch.empty_like(pair)
        ctx.solve_W(v, n, pair, 2, Wp)
        assert torch.equal(Wp[0], W[j]) and torch.equal(Wp[1], W[k]), (j, k)
    ctx.close()
