"""Device pointers are 8-byte aligned by contract and no more: every call on tensors and workspaces that start 8 bytes behind a
16-byte boundary gives what it gives on aligned ones."""
import numpy as np
import pytest

from paper_1908_04172_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LOG2N, N = 11, 1 << 11


@pytest.fixture(scope="module")
def he():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04172_amd import he as he_mod
    he_mod.lib()
    return he_mod


def shifted(t):
    """A copy of t (or room like it) whose first byte lies 8 bytes behind a 16-byte boundary."""
    skip = 8 // t.element_size()
    room = torch.empty(t.numel() + skip, dtype=t.dtype, device="cuda")
    view = room[skip:].view(t.shape)
    assert view.data_ptr() % 16 == 8 and view.is_contiguous()
    view.copy_(t)
    return view


def blank(t):
    return shifted(torch.zeros_like(t))


def room(n_bytes):
    return shifted(torch.empty(max(n_bytes, 256), dtype=torch.uint8, device="cuda"))


def residues(outer, q, seed, n=N):
    return wl.uniform_residues_torch(outer, q, n, seed, "cuda")


def plan_of(ctx):
    """Single outputs, and groups of every class with short and long sums."""
    rng = np.random.default_rng(3)
    off, tc, tp = [0], [], []
    for count, terms in [(1, 1), (1, 5), (2, 3), (3, 70), (6, 17), (12, 20), (16, 70), (8, 2)]:
        cts = rng.integers(0, 9, terms)
        for _ in range(count):
            tc.append(cts)
            tp.append(rng.integers(0, 11, terms))
            off.append(off[-1] + terms)
    cat = lambda xs: np.concatenate(xs).astype(np.uint32)
    return ctx.plan(9, len(off) - 1, 11, np.asarray(off, np.uint32), cat(tc), cat(tp)), len(off) - 1


def test_64_bit_calls(he):
    q = wl.modulus_chain([60, 50, 45, 60], N)
    ctx = he.Context(LOG2N, q)
    plan, n_out = plan_of(ctx)
    ct, w, b = residues((9, 2), q, 1), residues((11,), q, 2, 1)[..., 0].contiguous(), residues((n_out,), q, 3, 1)[..., 0].contiguous()
    poly = residues((11,), q, 4)
    for kind, pt in ((he.PT_SCALAR, w), (he.PT_POLY, poly)):
        for flags in (0, he.RESCALE, he.ACCUMULATE):
            want = torch.zeros((n_out, 2, 4 - (flags == he.RESCALE), N), dtype=torch.int64, device="cuda")
            out = shifted(want)
            ctx.ct_pt_mac(plan, ct, pt, kind, bias=b, flags=flags, out=want)
            ctx.ct_pt_mac(plan, shifted(ct), shifted(pt), kind, bias=shifted(b), flags=flags, out=out,
                          workspace=room(plan.workspace_bytes(4, kind, flags)))
            assert torch.equal(out, want), (kind, flags)
    for kind, pt in ((he.PT_SCALAR, w[:9].contiguous()), (he.PT_POLY, poly[:9].contiguous())):
        want, got = ct.clone(), shifted(ct)
        ctx.ct_pt_add(want, pt, kind)
        ctx.ct_pt_add(got, shifted(pt), kind)
        assert torch.equal(got, want)
    assert torch.equal(ctx.rescale(shifted(ct), out=blank(ctx.rescale(ct))), ctx.rescale(ct))
    want, got = poly.clone(), shifted(poly)
    for call in (ctx.ntt_fwd, ctx.ntt_inv):
        call(want)
        call(got)
        assert torch.equal(got, want)
    evk, low = residues((3, 2), q, 5), residues((9, 2), q[:3], 6)
    got = ctx.ct_square_relin(shifted(low), shifted(evk), out=blank(low), workspace=room(ctx.square_relin_workspace_bytes(3, 9)))
    assert torch.equal(got, ctx.ct_square_relin(low, evk))


def test_packed_calls(he):
    q = wl.modulus_chain([30, 29, 30], N)
    ctx = he.Context(LOG2N, q)
    plan, n_out = plan_of(ctx)
    wide = residues((9, 2), q, 1)
    w, b = residues((11,), q, 2, 1)[..., 0].contiguous(), residues((n_out,), q, 3, 1)[..., 0].contiguous()
    ct, poly = ctx.pack32(wide), ctx.pack32(residues((11,), q, 4))
    assert torch.equal(ctx.pack32(shifted(wide)), ct) and torch.equal(ctx.unpack32(shifted(ct)), wide)
    for kind, pt in ((he.PT_SCALAR, w), (he.PT_POLY, poly)):
        for flags in (0, he.RESCALE, he.ACCUMULATE):
            want = torch.zeros((n_out, 2, 3 - (flags == he.RESCALE), N), dtype=torch.int32, device="cuda")
            out = shifted(want)
            ctx.ct_pt_mac32(plan, ct, pt, kind, bias=b, flags=flags, out=want)
            ctx.ct_pt_mac32(plan, shifted(ct), shifted(pt), kind, bias=shifted(b), flags=flags, out=out,
                            workspace=room(plan.workspace_bytes(3, kind, flags)))
            assert torch.equal(out, want), (kind, flags)
    want, got = ct.clone(), shifted(ct)
    ctx.ct_pt_add32(want, poly[:9].contiguous(), he.PT_POLY)
    ctx.ct_pt_add32(got, shifted(poly[:9].contiguous()), he.PT_POLY)
    assert torch.equal(got, want)
    assert torch.equal(ctx.rescale32(shifted(ct), out=blank(ctx.rescale32(ct))), ctx.rescale32(ct))
    for call in (ctx.ntt_fwd32, ctx.ntt_inv32):
        call(want)
        call(got)
        assert torch.equal(got, want)


def test_vector_encoding(he):
    """(Slots to encode are 16-byte aligned by contract.)"""
    q = wl.modulus_chain([60, 40], N)
    ctx = he.Context(LOG2N, q)
    gen = torch.Generator(device="cuda").manual_seed(7)
    slots = torch.view_as_complex(torch.rand((5, N // 2, 2), dtype=torch.float64, device="cuda", generator=gen) * 2 - 1)
    poly = ctx.encode_vector(slots, 2.0**30)
    assert torch.equal(ctx.encode_vector(slots, 2.0**30, out=blank(poly)), poly)
    assert torch.equal(ctx.decode_vector(shifted(poly), 2.0**30, workspace=room(poly.numel() * 8)), ctx.decode_vector(poly, 2.0**30))
