"""Convolutions whose windows share most of their inputs and one table of plaintexts: the wavefronts of a workgroup take
neighbouring windows.  Every output against the oracle, for window counts that leave wavefronts without a window at the end of
a run, runs of one and of several windows per wavefront, and the longest sums whose table stays on chip; and for convolutions that
are just not taken that way: longer sums, too few windows, windows that share less than a third of their inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_1908_04172_amd import he, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,C,KH,OC,stride,abreast", [(5, 1, 3, 2, 1, True), (6, 1, 3, 5, 1, True), (7, 2, 3, 3, 1, True), (9, 1, 5, 12, 1, True),
                                                      (19, 1, 3, 2, 1, True), (21, 2, 5, 9, 2, True), (12, 1, 8, 4, 1, True), (40, 1, 5, 2, 1, True),
                                                      (13, 1, 9, 4, 1, False), (4, 1, 3, 4, 1, False), (21, 3, 3, 9, 2, False)])
@pytest.mark.parametrize("log2N,bits", [(10, [60, 40]), (11, [30, 50, 61])])
def test_windows_abreast(H, C, KH, OC, stride, abreast, log2N, bits):
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q, device=0)
    p = wl.conv_plan(H, H, C, KH, KH, OC, stride, "valid")
    hp = ctx.plan(p.n_in, p.n_out, p.n_pt, p.off, p.term_ct, p.term_pt)
    assert bool(hp.mac_form(len(q), OC) & he.FORM_ABREAST) == abreast
    assert not abreast or hp.groups_per_workgroup(len(q), OC) % 4 == 0
    x = wl.uniform_residues_torch((p.n_in, 2), q, N, 11, "cuda")
    w = wl.uniform_residues_torch((p.n_pt,), q, 1, 12, "cuda")[..., 0].contiguous()
    b = wl.uniform_residues_torch((p.n_out,), q, 1, 13, "cuda")[..., 0].contiguous()
    out = torch.full((p.n_out, 2, len(q), N), -1, dtype=torch.int64, device="cuda")
    ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, out=out)
    host = lambda t: t.cpu().numpy().view(np.uint64)
    want = oracle.mac(host(x), q, p.off, p.term_ct, p.term_pt, host(w), oracle.PT_SCALAR, host(b))
    assert np.array_equal(host(out), want)
    ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.ACCUMULATE, out=out)
    moduli = np.array(q, dtype=np.uint64).reshape(1, 1, -1, 1)
    assert np.array_equal(host(out), (want + want) % moduli)
    layer, _ = oracle.layer(host(x), q, ctx.psi, p.off, p.term_ct, p.term_pt, host(w), oracle.PT_SCALAR, host(b))
    assert np.array_equal(host(ctx.ct_pt_mac(hp, x, w, he.PT_SCALAR, bias=b, flags=he.RESCALE)), layer)
