"""Plans over far more inputs than their terms name: the number of inputs is a bare number of the caller's, with no array behind
it, and costs neither host memory nor time.  Plans are host code around a few uploads; results against the oracle."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_1908_04172_amd import he, workloads as wl

pytestmark = pytest.mark.gpu

# (in a process of its own: the peak of this one may already be high)
GROWTH = """
import resource
import numpy as np
from paper_1908_04172_amd import he, workloads as wl
ctx = he.Context(10, wl.modulus_chain([40, 30], 1 << 10), device=0)
def plan(n_in, first, outputs, terms=3, groups=3):
    n_out = groups * outputs
    term_ct = np.concatenate([first + (g + np.arange(terms)) % 5 for g in range(groups) for _ in range(outputs)]).astype(np.uint32)
    return ctx.plan(n_in, n_out, n_out * terms, np.arange(n_out + 1, dtype=np.uint32) * terms, term_ct, np.arange(n_out * terms, dtype=np.uint32))
plan(5, 0, 16)
for first in (0, (1 << 30) - 5):
    for outputs in (1, 4, 16):  # sums of their own, groups of four, groups of 16
        before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
        plan(1 << 30, first, outputs)
        print("grown by", resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before >> 10, "MiB", flush=True)
"""


def test_a_plan_costs_memory_by_its_terms():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", GROWTH], cwd=root, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr
    grown = [int(line.split()[2]) for line in run.stdout.splitlines() if line.startswith("grown by")]
    assert len(grown) == 6 and max(grown) < 64, grown  # a word per input would be 4096


def test_inputs_named_far_apart():
    """The same sums through inputs that lie next to one another and far apart: windows that share inputs, so that what a plan
    finds out about its neighbours matters."""
    N = 1 << 10
    q = wl.modulus_chain([60, 40], N)
    ctx = he.Context(10, q, device=0)
    p = wl.conv_plan(6, 6, 1, 3, 3, 2, 1, "valid")
    spread = 40  # more than four times as far as there are terms
    n_in = p.n_in * spread
    assert n_in > 4 * 16 * 9
    ct = wl.uniform_residues((p.n_in, 2), q, N, 1)
    w = wl.uniform_residues((p.n_pt,), q, 1, 2)[..., 0]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()
    want = oracle.mac(ct, q, p.off, p.term_ct, p.term_pt, w, oracle.PT_SCALAR, None)
    x = torch.zeros((n_in,) + ct.shape[1:], dtype=torch.int64, device="cuda")
    x[::spread] = dev(ct)
    far = ctx.plan(n_in, p.n_out, p.n_pt, p.off, p.term_ct * np.uint32(spread), p.term_pt)
    near = ctx.plan(p.n_in, p.n_out, p.n_pt, p.off, p.term_ct, p.term_pt)
    assert far.mac_form(2, 2) == near.mac_form(2, 2) == he.FORM_ABREAST
    assert far.groups_per_workgroup(2, 2) == near.groups_per_workgroup(2, 2)
    for hp, ins in ((near, dev(ct)), (far, x)):
        assert np.array_equal(ctx.ct_pt_mac(hp, ins, dev(w), he.PT_SCALAR).cpu().numpy().view(np.uint64), want)
