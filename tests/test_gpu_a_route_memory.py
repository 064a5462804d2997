"""The A route's workspace at an odd number of products."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _kept(n):
    """Device memory that a context keeps after one build of A, a mesh of 16
    points: few bins, so that the workspace is mostly pair vectors and products."""
    import gw_synth as gs
    import paper_1101_2065_amd.gw as gw

    dm = gw.DeviceMolecule(gs.truncate_products(gs.chain_molecule(29, 5), n))
    A = torch.empty(16, n, n, dtype=torch.complex128, device="cuda")
    ctx = gw.Context(0, 8 << 30)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx.build_A(dm.struct, dm.v, gw.make_grid(16, -16.0, 16.0, 0.5), A)
    torch.cuda.synchronize()
    kept = before - torch.cuda.mem_get_info()[0]
    ctx.close()
    return kept


def test_an_odd_size_takes_no_more_than_the_next_even_one():
    """v's rows, which are padded at odd n, find room in the workspace: a copy
    of 8 n (n + 1) bytes would be 20 MB more.  (2 MB: the size of an allocation.)"""
    _kept(1602)  # what the first call of a process allocates for itself
    even, odd = _kept(1602), _kept(1601)
    assert odd <= even + (2 << 20), (odd, even)
