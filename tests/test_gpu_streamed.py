"""Calls larger than the memory-side cache, whose rows pass by the caches, against the same call in slices that fit it; and
rescales of every number of kept limbs, whose intermediate coefficients lie partly in the LDS and partly in the output."""
import numpy as np
import pytest
import torch

import oracle
from paper_1908_04172_amd import he, workloads as wl

pytestmark = pytest.mark.gpu


def residues(outer, q, N, seed):
    return wl.uniform_residues_torch(outer, q, N, seed, "cuda", chunk=2048)


# ciphertexts just beyond 256 MiB of input
@pytest.mark.parametrize("log2N,bits,n", [(10, [30, 30], 8200), (12, [60, 40], 2060), (13, [60, 50, 50], 690), (14, [60, 55, 50], 345)])
def test_large_calls_equal_their_slices(log2N, bits, n):
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q, device=0)
    x = residues((n, 2), q, N, 5)
    assert x.numel() * 8 > 256 << 20
    third = n // 3
    want = torch.cat([ctx.rescale(x[k:k + third].contiguous()) for k in range(0, n, third)])
    assert torch.equal(ctx.rescale(x), want)
    rows = x.clone()
    parts = [x[k:k + third].clone() for k in range(0, n, third)]
    ctx.ntt_fwd(rows)
    for p in parts:
        ctx.ntt_fwd(p)
    assert torch.equal(rows, torch.cat(parts))
    ctx.ntt_inv(rows)
    assert torch.equal(rows, x)


@pytest.mark.parametrize("log2N,l,n", [(12, 3, 1000), (13, 4, 280)])
def test_large_squares_equal_their_slices(log2N, l, n):
    N = 1 << log2N
    q = wl.modulus_chain([60] + [50] * (l - 1) + [60], N)
    ctx = he.Context(log2N, q, device=0)
    ct, evk = residues((n, 2), q[:l], N, 6), residues((l, 2), q, N, 7)
    assert n * l * l * N * 8 > 256 << 20  # the expanded digits
    third = -(-n // 3)
    want = torch.cat([ctx.ct_square_relin(ct[k:k + third].contiguous(), evk) for k in range(0, n, third)])
    assert torch.equal(ctx.ct_square_relin(ct, evk), want)


# (the squares' inverse transforms are 256 MiB of rows and more, the digits a multiple of that)
@pytest.mark.parametrize("log2N,l,n", [(12, 2, 4100), (13, 3, 1400)])
def test_larger_squares_equal_their_slices(log2N, l, n):
    N = 1 << log2N
    q = wl.modulus_chain([60] + [50] * (l - 1) + [60], N)
    ctx = he.Context(log2N, q, device=0)
    ct, evk = residues((n, 2), q[:l], N, 6), residues((l, 2), q, N, 7)
    assert n * l * N * 8 > 256 << 20
    got, eighth = ctx.ct_square_relin(ct, evk), -(-n // 8)
    for k in range(0, n, eighth):
        assert torch.equal(got[k:k + eighth], ctx.ct_square_relin(ct[k:k + eighth].contiguous(), evk))


def test_large_calls_at_the_largest_ring_degree_equal_their_slices():
    """Half rows beyond 256 MiB, in place and (the rescale's inverse transforms) from the input."""
    N, n = 1 << 15, 530
    q = wl.modulus_chain([60, 50, 50], N)
    ctx = he.Context(15, q, device=0)
    x = residues((n, 2), q, N, 5)
    assert n * 2 * N * 8 > 256 << 20
    third = -(-n // 3)
    got = ctx.rescale(x)
    for k in range(0, n, third):
        assert torch.equal(got[k:k + third], ctx.rescale(x[k:k + third].contiguous()))
    rows = x.clone()
    ctx.ntt_fwd(rows)
    for k in range(0, n, third):
        part = x[k:k + third].clone()
        ctx.ntt_fwd(part)
        assert torch.equal(rows[k:k + third], part)
    ctx.ntt_inv(rows)
    assert torch.equal(rows, x)


WIDTHS = [60, 40, 50, 30, 55, 61, 45, 50, 62, 40, 58, 50, 60, 30, 50, 61]


@pytest.mark.parametrize("log2N", [10, 11, 12, 13, 14])
@pytest.mark.parametrize("limbs", range(2, 17))
def test_rescale_of_every_number_of_kept_limbs(log2N, limbs):
    """More polynomials than the chip holds workgroups, so that one workgroup takes all kept limbs."""
    N = 1 << log2N
    q = wl.modulus_chain(WIDTHS[:limbs], N)
    ctx = he.Context(log2N, q, device=0)
    n = 1 + (256 * 16 * 1024 // N) // 2
    x = residues((n, 2), q, N, 8)
    out = ctx.rescale(x)
    pick = [0, n // 2, n - 1]
    got = out[pick].cpu().numpy().view(np.uint64)
    want = oracle.rescale(x[pick].cpu().numpy().view(np.uint64), q, oracle.find_psis(q, N))
    assert np.array_equal(got, want)
