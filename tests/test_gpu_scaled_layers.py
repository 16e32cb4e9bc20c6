"""Layers whose sums have one term each (an elementwise scaling with bias and rescale): one kernel multiplies the rows as it
reads them.  Against the oracle, and against the same layer in two calls."""
import numpy as np
import pytest
import torch

import oracle
from paper_1908_04172_amd import he, workloads as wl

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def plan_of(ctx, term_ct, term_pt, n_in, n_pt):
    n = len(term_ct)
    off = np.arange(n + 1, dtype=np.uint32)
    term_ct, term_pt = np.asarray(term_ct, np.uint32), np.asarray(term_pt, np.uint32)
    return ctx.plan(n_in, n, n_pt, off, term_ct, term_pt), (off, term_ct, term_pt)


CHAINS = [[30, 30], [60, 40, 40], [61, 62, 58, 50, 45, 61], [62, 55, 50, 30], [50, 60, 62]]


@pytest.mark.parametrize("log2N", [10, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("bits", CHAINS)
@pytest.mark.parametrize("with_bias", [False, True])
def test_one_term_each(log2N, bits, with_bias):
    """Inputs in any order, some read by several outputs that do not follow one another, plaintexts shared or not, extreme
    residues, both levels; ring degree 2^15 takes the two launches."""
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q, device=0)
    rng = np.random.default_rng(log2N * 16 + len(bits))
    term_ct, term_pt = [3, 0, 2, 0, 1, 3, 4], [0, 1, 1, 3, 2, 4, 0]
    hp, (off, tc, tp) = plan_of(ctx, term_ct, term_pt, 5, 5)
    for L in sorted({len(q), max(2, len(q) - 1)}):
        ct = np.stack([rng.integers(0, m, (5, 2, N), dtype=np.uint64) for m in q[:L]], axis=2)
        pt = np.stack([rng.integers(0, m, 5, dtype=np.uint64) for m in q[:L]], axis=1)
        b = np.stack([rng.integers(0, m, 7, dtype=np.uint64) for m in q[:L]], axis=1)
        for i, m in enumerate(q[:L]):
            ct[0, 0, i, ::2], ct[0, 1, i, 1::3] = m - 1, 0
            pt[0, i], pt[1, i], b[2, i], b[1, i] = m - 1, 0, m - 1, 0
        bias = b if with_bias else None
        psi = oracle.find_psis(q[:L], N)
        want, _ = oracle.layer(ct, q[:L], psi, off, tc, tp, pt, oracle.PT_SCALAR, bias)
        x, w, bd = dev(ct), dev(pt), dev(b) if with_bias else None
        got = ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=bd, flags=he.RESCALE)
        assert np.array_equal(got.cpu().numpy().view(np.uint64), want)
        two_calls = ctx.rescale(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=bd))
        assert torch.equal(got, two_calls)


@pytest.mark.parametrize("log2N,bits,n", [(10, [60, 40], 2100), (12, [30, 30], 2060), (13, [60, 55, 50], 700), (14, [60, 50, 40], 345)])
def test_many_outputs(log2N, bits, n):
    """More polynomials than the chip holds workgroups, and inputs beyond the memory-side cache: against two calls."""
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q, device=0)
    rng = np.random.default_rng(n)
    hp, _ = plan_of(ctx, rng.permutation(n), np.arange(n) % 7, n, 7)
    x = wl.uniform_residues_torch((n, 2), q, N, 3, "cuda", chunk=2048)
    w = wl.uniform_residues_torch((7,), q, 1, 4, "cuda")[..., 0].contiguous()
    b = wl.uniform_residues_torch((n,), q, 1, 5, "cuda")[..., 0].contiguous()
    got = ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.RESCALE)
    assert torch.equal(got, ctx.rescale(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b)))


@pytest.mark.parametrize("log2N,bits,n,n_in", [(12, [60, 40], 2100, 2048), (12, [60, 40], 2100, 2049), (12, [60, 40], 2100, 3), (13, [60, 50, 50], 700, 60)])
def test_many_outputs_of_shared_inputs(log2N, bits, n, n_in):
    """Inputs that several outputs read: on both sides of the memory-side cache's size (2048 ciphertexts of 128 KiB), and few of them."""
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q, device=0)
    hp, _ = plan_of(ctx, np.arange(n) % n_in, np.arange(n) % 5, n_in, 5)
    x = wl.uniform_residues_torch((n_in, 2), q, N, 3, "cuda", chunk=2048)
    w = wl.uniform_residues_torch((5,), q, 1, 4, "cuda")[..., 0].contiguous()
    b = wl.uniform_residues_torch((n,), q, 1, 5, "cuda")[..., 0].contiguous()
    got = ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.RESCALE)
    assert torch.equal(got, ctx.rescale(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b)))
