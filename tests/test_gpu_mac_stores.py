"""Sums that are written past the caches: on both sides of each line at which that begins, with every flag, against the same
outputs in a call of their own that is small enough for the caches."""
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
