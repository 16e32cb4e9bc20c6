"""The transform kernels where they can go wrong: rows that follow one another in a workgroup.  Exact residues."""
import pytest

from paper_1908_04172_amd import he as he_mod
from paper_1908_04172_amd import workloads as wl

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def he():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    he_mod.lib()
    return he_mod


@pytest.mark.gpu
@pytest.mark.parametrize("log2N,polys", [(13, 700), (14, 300)])
def test_inverse_rows_that_follow_one_another(he, log2N, polys):
    """Several rows per workgroup, inverse direction, several times over: a row's first regrouping must not overtake the
    last one of the row before."""
    N = 1 << log2N
    q = wl.modulus_chain([60, 50, 40], N)
    ctx = he.Context(log2N, q)
    a = wl.uniform_residues_torch((polys,), q, N, 7, "cuda")
    x = a.clone()
    ctx.ntt_fwd(x)
    for _ in range(6):
        y = x.clone()
        ctx.ntt_inv(y)
        assert torch.equal(y, a)


@pytest.mark.gpu
def test_packed_inverse_rows_that_follow_one_another(he):
    N = 1 << 13
    q = wl.modulus_chain([30, 30], N)
    ctx = he.Context(13, q)
    a = ctx.pack32(wl.uniform_residues_torch((3000,), q, N, 8, "cuda"))
    x = a.clone()
    ctx.ntt_fwd32(x)
    for _ in range(6):
        y = x.clone()
        ctx.ntt_inv32(y)
        assert torch.equal(y, a)
