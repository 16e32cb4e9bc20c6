"""The scalar MAC on the matrix cores at the sizes where it can go wrong: group sizes around its tiles of four outputs and
its classes, term counts around its chunks of 16, around what it keeps in the LDS (64) and beyond what its 32-bit sums take
(4080), moduli of every width class, extreme operands; and tables that are worked off in slices.  Exact residues."""
import numpy as np
import pytest

import oracle
from paper_1908_04172_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def he():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04172_amd import he as he_mod
    he_mod.lib()
    return he_mod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def host(t):
    return t.cpu().numpy().view(np.uint64)


def groups_plan(groups, n_in, n_pt, seed):
    """One group of `count` outputs over `terms` random ciphertexts per (count, terms)."""
    rng = np.random.default_rng(seed)
    off, tc, tp = [0], [], []
    for count, terms in groups:
        cts = rng.integers(0, n_in, terms)
        for _ in range(count):
            tc.append(cts)
            tp.append(rng.integers(0, n_pt, terms))
            off.append(off[-1] + terms)
    cat = lambda xs: np.concatenate(xs).astype(np.uint32)
    return wl.Plan(n_in, len(off) - 1, n_pt, np.asarray(off, np.uint32), cat(tc), cat(tp))


def operands(plan, q, N, seed, extreme):
    ct = wl.uniform_residues((plan.n_in, 2), q, N, seed)
    w = wl.uniform_residues((plan.n_pt,), q, 1, seed + 1)[..., 0]
    b = wl.uniform_residues((plan.n_out,), q, 1, seed + 2)[..., 0]
    if extreme:  # q - 1, and residues whose digits are all -128 or next to it, against weights q - 1 and around q / 2
        for i, qi in enumerate(q):
            digits = [0x8080808080808080 % qi, 0x7F7F7F7F7F7F7F7F % qi, qi - 1, 0]
            for c in range(plan.n_in):
                ct[c, :, i, :] = digits[c % 4] if c % 4 < 3 else ct[c, :, i, :]
            w[0::3, i], w[1::3, i] = qi - 1, qi // 2 + 1
            b[:, i] = qi - 1
    return ct, w, b


def run(he, ctx, plan, ct, w, b, **kw):
    hp = ctx.plan(plan.n_in, plan.n_out, plan.n_pt, plan.off, plan.term_ct, plan.term_pt)
    return host(ctx.ct_pt_mac(hp, dev(ct), dev(w), he.PT_SCALAR, bias=None if b is None else dev(b), **kw))


@pytest.mark.parametrize("bits", [[20, 24, 30], [31, 32, 33, 39], [40, 41, 47, 48], [49, 50, 55, 56], [57, 60, 61, 62]], ids=str)
@pytest.mark.parametrize("extreme", [False, True])
def test_group_sizes_and_term_counts_on_moduli_of_every_width(he, bits, extreme):
    N = 1 << 10
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(10, q)
    groups = [(c, t) for c in (2, 4, 5, 8, 9, 16) for t in (1, 16, 17)] + [(3, 15), (7, 64), (16, 65), (2, 129), (16, 128)]
    plan = groups_plan(groups, 40, 50, sum(bits))
    ct, w, b = operands(plan, q, N, 7 + sum(bits), extreme)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b), want)
    layer, _ = oracle.layer(ct, q, ctx.psi, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b, flags=he.RESCALE), layer)


@pytest.mark.parametrize("groups", [[(16, 1)], [(8, 4)], [(2, 3), (4, 4)], [(16, 4), (9, 2), (5, 1), (8, 3), (2, 4), (3, 0), (12, 0), (1, 7)],
                                    [(c, 1 + k % 4) for k, c in enumerate([2, 3, 7, 16, 13, 4, 1] * 40)]], ids=lambda g: f"{len(g)}-{g[0]}")
@pytest.mark.parametrize("extreme", [False, True])
def test_plans_of_short_sums(he, groups, extreme):
    """No group of outputs with more than four terms: tables of one block.  (The longest plan chains groups in a workgroup.)"""
    N = 1 << 11
    q = wl.modulus_chain([60, 50, 40, 61], N)
    ctx = he.Context(11, q)
    plan = groups_plan(groups, 40, 50, len(groups))
    ct, w, b = operands(plan, q, N, 9, extreme)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    out = dev(want)
    got = run(he, ctx, plan, ct, w, b)
    assert np.array_equal(got, want)
    run(he, ctx, plan, ct, w, b, flags=he.ACCUMULATE, out=out)
    assert np.array_equal(host(out), (2 * want.astype(object) % np.asarray(q, object)[:, None]).astype(np.uint64))
    if plan.n_out < 500:
        layer, _ = oracle.layer(ct, q, ctx.psi, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
        assert np.array_equal(run(he, ctx, plan, ct, w, b, flags=he.RESCALE), layer)


@pytest.mark.parametrize("log2N", [10, 11, 13])
@pytest.mark.parametrize("terms", [[1], [2, 1, 0], [3, 1, 2]], ids=str)
def test_single_outputs_of_few_terms(he, log2N, terms):
    """Outputs that share their inputs with no other: the forms of the streaming kernel."""
    N = 1 << log2N
    q = wl.modulus_chain([60, 50, 30], N)
    ctx = he.Context(log2N, q)
    plan = groups_plan([(1, t) for t in terms * 5], 7, 9, log2N)
    ct, w, b = operands(plan, q, N, 70 + log2N, True)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b), want)
    layer, _ = oracle.layer(ct, q, ctx.psi, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b, flags=he.RESCALE), layer)


@pytest.mark.parametrize("terms", [4079, 4080, 4081, 8161])
def test_sums_beyond_the_range_of_the_32_bit_accumulators(he, terms):
    N = 1 << 10
    q = wl.modulus_chain([62, 50, 30], N)
    ctx = he.Context(10, q)
    plan = groups_plan([(16, terms), (5, 3), (2, terms), (1, terms)], 4, 6, terms)
    ct, w, b = operands(plan, q, N, terms, True)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b), want)
    layer, _ = oracle.layer(ct, q, ctx.psi, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b, flags=he.RESCALE), layer)


def dev32(a):
    return torch.from_numpy(np.ascontiguousarray(a).astype(np.uint32).view(np.int32)).cuda()


def host32(t):
    return t.cpu().numpy().view(np.uint32).astype(np.uint64)


@pytest.mark.parametrize("bits,groups", [
    ([17, 24, 29, 30], [(c, t) for c in (2, 4, 5, 8, 9, 16) for t in (1, 16, 17)] + [(3, 15), (7, 64), (16, 65), (2, 129), (1, 20)]),
    ([30, 30], [(16, 4080), (16, 4081), (3, 8161), (8, 7), (1, 4097)]),
    # classes of few terms run on the vector ALU: the most that it takes, one more, and one class of three
    ([30, 29, 20], [(c, t) for c in (2, 3, 4) for t in (1, 3, 15, 16, 39, 40)] + [(c, t) for c in (5, 6) for t in (1, 4, 17, 18)]
     + [(c, t) for c in (9, 12) for t in (2, 5, 13, 18)] + [(1, 30)]),
    ([30, 30], [(4, 41), (2, 5), (8, 12), (7, 1), (5, 11), (16, 13), (9, 2)]),
    ([17, 30], [(4, 40), (6, 19), (5, 2), (16, 12), (13, 1), (10, 12), (3, 0), (2, 0)]),
], ids=["sizes", "long", "few terms", "one class of few terms", "two classes of few terms"])
@pytest.mark.parametrize("extreme", [False, True])
def test_packed_group_sizes_and_term_counts(he, bits, groups, extreme):
    N = 1 << 10
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(10, q)
    plan = groups_plan(groups, 40, 50, len(groups))
    ct, w, b = operands(plan, q, N, 3 + len(groups), extreme)
    hp = ctx.plan(plan.n_in, plan.n_out, plan.n_pt, plan.off, plan.term_ct, plan.term_pt)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    out = ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, bias=dev(b))
    assert np.array_equal(host32(out), want)
    ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, flags=he.ACCUMULATE, out=out)
    twice = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR)
    assert np.array_equal(host32(out), (want + twice) % np.asarray(q, np.uint64)[:, None])
    layer, _ = oracle.layer(ct, q, ctx.psi, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(host32(ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, bias=dev(b), flags=he.RESCALE)), layer)


def runs_of_long_sums(classes, groups, seed):
    """`groups` groups of each of the output counts, most with sums beyond the 64 terms whose tables stay in the LDS, shorter
    ones among them and, at the front of the first class, a whole run of those."""
    rng = np.random.default_rng(seed)
    terms = [int(t) for t in rng.choice([65, 66, 80, 96, 129, 160, 1, 16, 40, 64], groups, p=[.15, .1, .15, .1, .1, .1, .05, .1, .05, .1])]
    terms[:2], terms[2:5], terms[-3:] = [30, 64], [65, 7, 81], [70, 12, 90]
    return [(c, t + (k if t > 64 else 0)) for t in terms for k, c in enumerate(classes)]


@pytest.mark.parametrize("log2N,bits,classes,groups,per_wg", [(11, [60, 50, 40, 55], (16, 7, 3), 97, 2), (11, [62, 30], (9, 2), 131, 2),
                                                              (12, [60, 60, 50, 50, 50, 50, 46, 50], (4, 16), 69, 8)])
@pytest.mark.parametrize("extreme", [False, True])
def test_long_sums_of_several_groups_in_one_workgroup(he, log2N, bits, classes, groups, per_wg, extreme):
    """The stream of chunks that brings its tables along runs on from one group into the next (lists, inputs and tables of the
    next group are requested during the last chunk of the one before), past shorter groups too and into a ragged last run."""
    N = 1 << log2N
    q = wl.modulus_chain(bits, N)
    ctx = he.Context(log2N, q)
    plan = groups_plan(runs_of_long_sums(classes, groups, log2N), 11, 13, groups)
    hp = ctx.plan(plan.n_in, plan.n_out, plan.n_pt, plan.off, plan.term_ct, plan.term_pt)
    assert [hp.groups_per_workgroup(len(q), c) for c in classes] == [per_wg] * len(classes)
    ct, w, b = operands(plan, q, N, groups, extreme)
    first = np.cumsum([0] + [c for _ in range(groups) for c in classes])[:-1]        # a group's first output, and of some all
    some = sorted(set(first.tolist()) | set(range(40)) | set(range(plan.n_out - 40, plan.n_out)))[::1 if groups > 90 else 3]
    sub = plan.subset(some)
    want = oracle.mac(ct, q, sub.off, sub.term_ct, sub.term_pt, w, oracle.PT_SCALAR, b[some])
    out = run(he, ctx, plan, ct, w, b)
    assert np.array_equal(out[some], want)
    twice = dev(out)
    run(he, ctx, plan, ct, w, b, flags=he.ACCUMULATE, out=twice)
    qa = np.asarray(q, np.uint64)[:, None]
    assert np.array_equal(host(twice), (out + out) % qa)             # (below 2^63)
    few = some[::7]
    layer, _ = oracle.layer(ct, q, ctx.psi, *(lambda s: (s.off, s.term_ct, s.term_pt))(plan.subset(few)), w, oracle.PT_SCALAR, b[few])
    assert np.array_equal(run(he, ctx, plan, ct, w, b, flags=he.RESCALE)[few], layer)


@pytest.mark.parametrize("classes,groups,per_wg", [((16, 11), 200, 4), ((8, 7), 131, 4), ((3,), 150, 2), ((16, 6, 2), 129, 2)])
def test_packed_long_sums_of_several_groups_in_one_workgroup(he, classes, groups, per_wg):
    N = 1 << 11
    q = wl.modulus_chain([30, 29, 30, 24], N)
    ctx = he.Context(11, q)
    plan = groups_plan(runs_of_long_sums(classes, groups, 5), 11, 13, groups)
    hp = ctx.plan(plan.n_in, plan.n_out, plan.n_pt, plan.off, plan.term_ct, plan.term_pt)
    assert [hp.groups_per_workgroup(len(q), c, packed=True) for c in classes] == [per_wg] * len(classes)
    ct, w, b = operands(plan, q, N, groups, True)
    first = np.cumsum([0] + [c for _ in range(groups) for c in classes])[:-1]
    some = sorted(set(first.tolist()) | set(range(40)) | set(range(plan.n_out - 40, plan.n_out)))
    sub = plan.subset(some)
    want = oracle.mac(ct, q, sub.off, sub.term_ct, sub.term_pt, w, oracle.PT_SCALAR, b[some])
    out = ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, bias=dev(b))
    once = host32(out)
    assert np.array_equal(once[some], want)
    ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, bias=dev(b), flags=he.ACCUMULATE, out=out)
    assert np.array_equal(host32(out), 2 * once % np.asarray(q, np.uint64)[:, None])
    few = some[::7]
    layer, _ = oracle.layer(ct, q, ctx.psi, *(lambda s: (s.off, s.term_ct, s.term_pt))(plan.subset(few)), w, oracle.PT_SCALAR, b[few])
    assert np.array_equal(host32(ctx.ct_pt_mac32(hp, dev32(ct), dev(w), he.PT_SCALAR, bias=dev(b), flags=he.RESCALE))[few], layer)


@pytest.mark.parametrize("K,M,rescale", [(9000, 16, True), (600, 528, False)])
def test_tables_larger_than_the_fixed_scratch_are_worked_off_in_slices(he, K, M, rescale):
    """One table that does not fit (passes over its terms), and many (ranges of groups)."""
    N = 1 << 10
    q = wl.modulus_chain([60, 50, 50, 40], N)
    ctx = he.Context(10, q)
    n_in = 5
    tc = np.random.default_rng(K).integers(0, n_in, K)
    rng = np.random.default_rng(M)
    plan = wl.Plan(n_in, M, 64, (np.arange(M + 1) * K).astype(np.uint32), np.tile(tc, M).astype(np.uint32),
                   rng.integers(0, 64, K * M).astype(np.uint32))
    hp = ctx.plan(plan.n_in, plan.n_out, plan.n_pt, plan.off, plan.term_ct, plan.term_pt)
    flags = he.RESCALE if rescale else 0
    assert hp.workspace_bytes(4, he.PT_SCALAR, flags) > he.STATIC_SCRATCH_BYTES
    ct, w, b = operands(plan, q, N, K, False)
    out = torch.full((M, 2, 4 - rescale, N), -1, dtype=torch.int64, device="cuda")
    ctx.ct_pt_mac_static(hp, dev(ct), dev(w), he.PT_SCALAR, out, bias=dev(b), flags=flags)
    assert torch.equal(out, ctx.ct_pt_mac(hp, dev(ct), dev(w), he.PT_SCALAR, bias=dev(b), flags=flags))
    some = [0, 1, M // 2, M - 1]
    sub = plan.subset(some)
    if rescale:
        want, _ = oracle.layer(ct, q, ctx.psi, sub.off, sub.term_ct, sub.term_pt, w, oracle.PT_SCALAR, b[some])
    else:
        want = oracle.mac(ct, q, sub.off, sub.term_ct, sub.term_pt, w, oracle.PT_SCALAR, b[some])
    assert np.array_equal(host(out[some]), want)


@pytest.mark.parametrize("M", [20, 37, 68, 85])
@pytest.mark.parametrize("K", [5, 70])
def test_order_of_the_groups_of_several_classes(he, K, M):
    """Launches of 384 (one wave of workgroups), 576 and 960 (less than two: the groups of a slice side by side where the classes
    are close in size, the largest class first where it is four fifths of the launch) and 1152 workgroups."""
    N = 1 << 11
    q = wl.modulus_chain([60, 50, 40] * 4, N)
    ctx = he.Context(11, q)
    plan = wl.dense_plan(K, M)
    ct, w, b = operands(plan, q, N, M, False)
    want = oracle.mac(ct, q, plan.off, plan.term_ct, plan.term_pt, w, oracle.PT_SCALAR, b)
    assert np.array_equal(run(he, ctx, plan, ct, w, b), want)
