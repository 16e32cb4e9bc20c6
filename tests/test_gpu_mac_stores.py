"""Sums that are written past the caches: on both sides of each line at which that begins, with every flag, against the same
outputs in a call of their own that is small enough for the caches."""
import numpy as np
import pytest
import torch

from paper_1908_04172_amd import he, workloads as wl

pytestmark = pytest.mark.gpu


def residues(outer, q, N, seed):
    return wl.uniform_residues_torch(outer, q, N, seed, "cuda", chunk=2048)


# Two limbs of 2^12: 128 KiB a ciphertext (packed: 64), so that 2048 (4096) of them are the 256 MiB of the memory-side cache and 256
# (512) the 32 MiB of the L2s.
@pytest.mark.parametrize("packed,K,M,streamed", [(False, 16, 2032, False), (False, 16, 2033, True), (False, 11, 2037, False),
                                                 (False, 12, 2037, True), (False, 1900, 256, False), (False, 1900, 257, True),
                                                 (True, 100, 3996, False), (True, 100, 3997, True), (True, 3700, 512, False),
                                                 (True, 3700, 517, True)])
def test_sums_around_the_sizes_of_the_caches(packed, K, M, streamed):
    N = 1 << 12
    q = wl.modulus_chain([30, 30] if packed else [60, 40], N)
    ctx = he.Context(12, q, device=0)
    mac = ctx.ct_pt_mac32 if packed else ctx.ct_pt_mac
    whole = wl.dense_plan(K, M)
    hp = ctx.plan(whole.n_in, M, whole.n_pt, whole.off, whole.term_ct, whole.term_pt)
    for flags in (0, he.RESCALE, he.ACCUMULATE):
        assert bool(hp.mac_form(2, 16, packed, flags) & he.FORM_PAST_CACHES) == streamed
    tail = 16 + M % 16  # the last whole group and what is left over
    part = wl.dense_plan(K, tail)
    few = ctx.plan(K, tail, part.n_pt, part.off, part.term_ct, part.term_pt)
    assert not few.mac_form(2, 16, packed) & he.FORM_PAST_CACHES
    x, w = residues((K, 2), q, N, 1), residues((whole.n_pt,), q, 1, 2)[..., 0].contiguous()
    b, acc = residues((M,), q, 1, 3)[..., 0].contiguous(), residues((M, 2), q, N, 4)
    if packed:
        x, acc = ctx.pack32(x), ctx.pack32(acc)
    w_tail, b_tail, acc_tail = w.view(K, M, -1)[:, M - tail:].reshape(K * tail, -1).contiguous(), b[M - tail:].contiguous(), acc[M - tail:].clone()
    for flags in (0, he.RESCALE):
        assert torch.equal(mac(hp, x, w, he.PT_SCALAR, bias=b, flags=flags)[M - tail:], mac(few, x, w_tail, he.PT_SCALAR, bias=b_tail, flags=flags))
    mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.ACCUMULATE, out=acc)
    mac(few, x, w_tail, he.PT_SCALAR, bias=b_tail, flags=he.ACCUMULATE, out=acc_tail)
    assert torch.equal(acc[M - tail:], acc_tail)


def windows(n, terms):
    """Output o is the sum of `terms` inputs from input o on, round the end: no two share all their inputs."""
    off = np.arange(n + 1, dtype=np.uint32) * terms
    term_ct = ((np.arange(n)[:, None] + np.arange(terms)) % n).astype(np.uint32).reshape(-1)
    return wl.Plan(n, n, n * terms, off, term_ct, np.arange(n * terms, dtype=np.uint32))


# (128 KiB a ciphertext again, as many inputs as outputs)
@pytest.mark.parametrize("n,terms,streamed", [(1024, 2, False), (1025, 1, True), (1500, 5, True), (2048, 2, True),
                                              (2049, 1, False), (2049, 2, False), (2049, 3, True)])
def test_sums_of_their_own_around_the_sizes_of_the_cache(n, terms, streamed):
    N = 1 << 12
    q = wl.modulus_chain([60, 40], N)
    ctx = he.Context(12, q, device=0)
    p = windows(n, terms)
    hp = ctx.plan(p.n_in, p.n_out, p.n_pt, p.off, p.term_ct, p.term_pt)
    assert [bool(hp.mac_form(2, 1, False, flags) & he.FORM_PAST_CACHES) for flags in (0, he.ACCUMULATE, he.RESCALE)] == [streamed, streamed, False]
    x, w = residues((n, 2), q, N, 1), residues((p.n_pt,), q, 1, 2)[..., 0].contiguous()
    b, acc = residues((n,), q, 1, 3)[..., 0].contiguous(), residues((n, 2), q, N, 4)
    # the same outputs in three calls that fit the cache: inputs [first, first + count + terms - 1), round the end
    sums, third = torch.empty_like(acc), -(-n // 3)
    for first in range(0, n, third):
        count = min(third, n - first)
        off = np.arange(count + 1, dtype=np.uint32) * terms
        term_ct = (np.arange(count)[:, None] + np.arange(terms)).astype(np.uint32).reshape(-1)
        few = ctx.plan(count + terms - 1, count, count * terms, off, term_ct, np.arange(count * terms, dtype=np.uint32))
        assert not few.mac_form(2, 1) & he.FORM_PAST_CACHES
        at = (torch.arange(first, first + count + terms - 1) % n).cuda()
        sums[first:first + count] = ctx.ct_pt_mac(few, x[at], w[first * terms:(first + count) * terms].contiguous(), he.PT_SCALAR,
                                                  bias=b[first:first + count].contiguous())
    assert torch.equal(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b), sums)
    assert torch.equal(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.RESCALE), ctx.rescale(sums))
    moduli = torch.tensor([int(m) for m in q], dtype=torch.int64, device="cuda").view(1, 1, -1, 1)
    want = acc + sums
    want -= torch.where(want >= moduli, moduli, torch.zeros_like(moduli))
    assert torch.equal(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.ACCUMULATE, out=acc), want)
