"""Complex FP64 arrays on 8-byte boundaries (all that double _Complex asks for):
the panels and products load through registers there instead of by 16-byte
direct copies, in the same order."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _system(n, n_omega):
    """A = 1 + small on every mesh point, v = 1 + small symmetric; A at each
    offset of a buffer with room for one value more."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    b = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) / n
    v = torch.eye(n, device="cuda", dtype=torch.float64) + b + b.T
    A = torch.randn(n_omega, n, n, 2, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5
    A[..., 0] += torch.eye(n, device="cuda", dtype=torch.float64)
    return v, A.reshape(-1)


def _buffer(size):
    return torch.full((size + 1,), float("nan"), device="cuda", dtype=torch.float64)


def _solve(ctx, n, n_omega, v, A, off_a, off_w):
    a, w = _buffer(A.numel()), _buffer(A.numel())
    a[off_a:off_a + A.numel()] = A
    ctx.solve_W_A(v, n, a.data_ptr() + 8 * off_a, n_omega, w.data_ptr() + 8 * off_w)
    assert bool(torch.isnan(w[-1 if off_w == 0 else 0]))  # the value beside W is untouched
    return w[off_w:off_w + A.numel()]


@pytest.mark.parametrize("n", [7, 130, 600, 1100, 2100, 3100])
def test_w_is_the_same_bit_for_bit(n):
    """One size for each number of rows a panel's thread holds (1, 2, 4, 6, 8)."""
    import paper_1101_2065_amd.gw as gw

    ctx = gw.Context(0)
    v, A = _system(n, 4)
    ref = _solve(ctx, n, 4, v, A, 0, 0)
    assert bool(torch.isfinite(ref).all())
    for off_a, off_w in ((1, 1), (1, 0), (0, 1)):
        assert torch.equal(_solve(ctx, n, 4, v, A, off_a, off_w), ref), (off_a, off_w)
    ctx.close()


def test_panels_stay_in_registers():
    """The panels from 8-byte boundaries add the staging of their loads; the
    column-by-column panel in memory, for more than 4096 rows only, would take
    four times as long at this size."""
    import paper_1101_2065_amd.gw as gw

    n, n_omega = 431, 256
    ctx = gw.Context(0)
    v, A = _system(n, n_omega)
    ms = {0: [], 1: []}
    for off in (0, 1, 0, 1, 0, 1):
        ctx.profile_begin()
        _solve(ctx, n, n_omega, v, A, off, off)
        ms[off].append({k["name"]: k["ms"] for k in ctx.profile_read()}["lu_panel"])
        ctx.profile_end()
    ctx.close()
    assert min(ms[1]) < 2 * min(ms[0]), ms
