"""CPU-only checks of the library: it loads, exports every symbol include/*.h declares, and its host
logic (modulus validation, root choice, the device arithmetic compiled for the host, scalar
encoding) agrees with Python integers and with the oracle.  No kernel is launched here."""
import os
import random
import re

import numpy as np
import pytest

import oracle
from paper_1908_04172_amd import he
from paper_1908_04172_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    declared = set()
    for name in ("he.h", "he_test.h"):                      # the product ABI and the test / measurement hooks
        header = open(os.path.join(ROOT, "include", name)).read()
        declared |= set(re.findall(r"\b(he_[a-z0-9_]+)\s*\(", header))
    product = set(re.findall(r"\b(he_[a-z0-9_]+)\s*\(", open(os.path.join(ROOT, "include", "he.h")).read()))
    assert not any(n.startswith("he_host_") or n == "he_measure_rate" for n in product)
    assert declared == set(he.EXPORTS)
    L = he.lib()
    for name in declared:
        assert getattr(L, name) is not None
    assert he.lib().he_strerror(0) == b"ok"
    assert b"modulus" in he.lib().he_strerror(-2)


def primes():
    return [wl.ntt_primes(b, 1 << 14, 1)[0] for b in (30, 40, 50, 58, 60, 61, 62)]


def test_barrett_and_shoup_equal_python_mod():
    rnd = random.Random(3)
    for q in primes():
        edge = [0, 1, q - 1, q - 2, q // 2]
        for _ in range(200):
            a, b = rnd.choice(edge + [rnd.randrange(q)]), rnd.choice(edge + [rnd.randrange(q)])
            assert he.host_mulmod(a, b, q) == a * b % q
            assert he.host_shoup_mulmod(a, b, q) == a * b % q
        # the Shoup product takes any 64-bit left operand (lazy butterflies feed it values up to 4q)
        for y in (2**64 - 1, 4 * q - 1, 2 * q, 2 * q + 1):
            w = rnd.randrange(q)
            assert he.host_shoup_mulmod(y, w, q) == y * w % q
        # any 128-bit input
        for z in [0, q, q - 1, (q - 1) ** 2, 2**64 - 1, 2**64, 2**128 - 1, 2**127] + [rnd.randrange(2**128) for _ in range(200)]:
            assert he.host_reduce128(z >> 64, z & (2**64 - 1), q) == z % q


def test_lazy_shoup_products_stay_in_their_ranges():
    """The butterflies' unreduced products: congruent to y*w for any 64-bit y, below 2q with the exact
    quotient estimate and below 4q with the cheap one."""
    rnd = random.Random(5)
    for q in primes() + [wl.ntt_primes(b, 1 << 14, 1)[0] for b in (58, 61)]:
        ys = [0, 1, q - 1, q, 2 * q, 4 * q - 1, 2**32 - 1, 2**32, 2**64 - 1, 2**63, 57 * q if 57 * q < 2**64 else 2**64 - 2]
        ys += [rnd.randrange(2**64) for _ in range(300)] + [rnd.randrange(min(8 * q, 2**64)) for _ in range(300)]
        ws = [0, 1, q - 1, q // 2] + [rnd.randrange(q) for _ in range(4)]
        for w in ws:
            for y in ys:
                exact = he.host_shoup_lazy(y, w, q, False)
                cheap = he.host_shoup_lazy(y, w, q, True)
                assert exact % q == y * w % q and exact < 2 * q, (q, y, w)
                assert cheap % q == y * w % q and cheap < 4 * q and cheap >= exact, (q, y, w)


def test_mac_accumulator_fold_and_reduce_schedule():
    rnd = random.Random(4)
    for q in primes():
        for n in (0, 1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 63, 64, 65, 255, 256, 257, 1000, 4095, 4096, 4097, 9000):
            for mode in ("max", "rand"):
                x = [q - 1] * n if mode == "max" else [rnd.randrange(q) for _ in range(n)]
                w = [q - 1] * n if mode == "max" else [rnd.randrange(q) for _ in range(n)]
                want = sum(a * b for a, b in zip(x, w)) % q
                assert he.host_mac_accumulate(x, w, q) == want, (q, n, mode)
                # the final step with an addend (the bias of Alg. 4), extreme and random
                for b in (q - 1, 1, rnd.randrange(q)):
                    assert he.host_mac_accumulate(x, w, q, b) == (want + b) % q, (q, n, mode, b)


def test_unreduced_mac_result_is_congruent_and_small():
    """What the MAC of a fused layer hands to the rescale kernel on kept limbs: congruent to sum + addend, below 4q on limbs
    whose combine step runs on doubles and below 6q on the others."""
    rnd = random.Random(14)
    for q in primes():
        for n in (0, 1, 2, 5, 12, 27, 28, 64, 255, 845, 4096, 9000):
            for mode in ("max", "rand"):
                x = [q - 1] * n if mode == "max" else [rnd.randrange(q) for _ in range(n)]
                w = [q - 1] * n if mode == "max" else [rnd.randrange(q) for _ in range(n)]
                for addend in (0, q - 1, 2 * q - 1, rnd.randrange(2 * q)):
                    got = he.host_mac_accumulate_lazy(x, w, q, addend)
                    assert got % q == (sum(a * b for a, b in zip(x, w)) + addend) % q, (q, n, mode)
                    assert got < (4 if q < 1 << 50 else 6) * q, (q, n, mode, got // q)


def test_context_validates_moduli():
    N = 1 << 12
    good = wl.modulus_chain([30, 30], N)
    he.Context(12, good, device=None).close()
    he.Context(15, wl.modulus_chain([30, 60], 1 << 15), device=None).close()      # the largest ring degree
    bad_sets = [
        [good[0], good[0]],                      # repeated
        [good[0], good[1] + 2 * N],              # = 1 mod 2N but (here) composite
        [good[0], 1073741827],                   # prime, but not 1 mod 2N
        [good[0], (1 << 62) + 1],                # too large
    ]
    assert not oracle.is_prime(good[1] + 2 * N) and oracle.is_prime(1073741827)
    for mods in bad_sets:
        with pytest.raises(he.HeError) as e:
            he.Context(12, mods, device=None)
        assert e.value.status == -2
    for log2N in (9, 16):
        with pytest.raises(he.HeError) as e:
            he.Context(log2N, good, device=None)
        assert e.value.status == -1


@pytest.mark.parametrize("cfg", [1, 2, 4])
def test_root_choice_matches_oracle(cfg):
    c = wl.config(cfg)
    ctx = he.Context(c.log2N, c.q, device=None)
    assert ctx.psi == oracle.find_psis(c.q, c.N)


def test_encode_scalar_host_matches_oracle():
    c = wl.config(4)
    ctx = he.Context(c.log2N, c.q, device=None)
    rnd = random.Random(6)
    vals = [0.0, -0.0, 0.5, -0.5, 1.5, 2.5, -2.5, 0.49999999999999994, 1e-30, 3.0, -3.0, 2.0**52 + 1]
    vals += [rnd.gauss(0, 0.1) for _ in range(200)] + [rnd.randrange(-999, 999) + 0.5 for _ in range(50)]
    for scale in (1.0, 2.0**24, 2.0**50, 2.0**62, 2.0**63, 2.0**80, 2.0**100):
        got = ctx.encode_scalar_host(vals, scale)
        assert got.shape == (len(vals), c.L) and got.nbytes == 8 * c.L * len(vals)   # 8*L bytes per scalar
        for v, row in zip(vals, got):
            assert row.tolist() == oracle.encode_scalar(v, scale, c.q).tolist(), (v, scale)
    # depth-aware encoding: a lower level is a prefix of the limbs
    assert np.array_equal(ctx.encode_scalar_host(vals, 2.0**50, limbs=3), ctx.encode_scalar_host(vals, 2.0**50)[:, :3])
    with pytest.raises(he.HeError):
        ctx.encode_scalar_host([float("nan")], 1.0)
    with pytest.raises(he.HeError) as e:
        ctx.encode_scalar_host([1.0], 1.0, limbs=9)
    assert e.value.status == -3


def test_device_calls_fail_loudly_on_a_host_only_context():
    c = wl.config(1)
    ctx = he.Context(c.log2N, c.q, device=None)
    p = c.plan
    with pytest.raises(he.HeError) as e:
        ctx.plan(p.n_in, p.n_out, p.n_pt, p.off, p.term_ct, p.term_pt)
    assert e.value.status == -5
    dummy = np.zeros(2 * c.N, dtype=np.uint64)  # (whole, so that it shares no memory with the other one wherever the two lie)
    other = np.zeros(2 * 2 * c.N, dtype=np.uint64)
    assert he.lib().he_rescale(ctx._h, 2, other.ctypes.data, dummy.ctypes.data, 1, None) == -5
    # output sharing memory with the input is refused before anything is launched
    assert he.lib().he_rescale(ctx._h, 2, other.ctypes.data, other.ctypes.data + 8 * c.N, 1, None) == -1
    assert he.lib().he_rescale(ctx._h, 1, dummy.ctypes.data, dummy.ctypes.data, 1, None) == -3
    assert he.lib().he_ntt_fwd(ctx._h, 3, dummy.ctypes.data, 1, None) == -3
    with pytest.raises(he.HeError) as e:
        ctx.measure_rate(he.RATE_MAD32)
    assert e.value.status == -5
    for bad in (dict(kind=99), dict(kind=0, limb=c.L), dict(kind=0, iters=0), dict(kind=0, iters=(1 << 20) + 1)):
        with pytest.raises(he.HeError) as e:
            ctx.measure_rate(**bad)
        assert e.value.status == -1


def test_packed32_primitives_against_python_integers():
    """Alg. 6 (BarrettReduction64) and the lazy 32-bit Shoup product, compiled for the host, on the
    extremes and on random operands, for the smallest and the largest moduli the packed path takes."""
    rng = np.random.default_rng(32)
    for q in (3, 12289, 1073479681, 2**30 - 35, 2**29 + 11):
        zs = [0, 1, q - 1, q, q + 1, 2**64 - 1, 2**64 - q, (q - 1) ** 2, 16 * (q - 1) ** 2 % 2**64]
        zs += [int(z) for z in rng.integers(0, 2**64, 2000, dtype=np.uint64)]
        for z in zs:
            assert he.host_barrett64(z, q) == z % q
        ws = [0, 1, q - 1] + [int(w) for w in rng.integers(0, q, 40)]
        ys = [0, 1, q - 1, 2 * q - 1, 2**32 - 1] + [int(y) for y in rng.integers(0, 2**32, 60, dtype=np.uint64)]
        for w in ws:
            for y in ys:
                if y >= 2**32:
                    continue
                r = he.host_shoup32(y, w, q)
                assert r < 2 * q and r % q == y * w % q


DIGIT_TERMS = 4080                                              # the most terms that the 32-bit sums of the matrix cores take


def primes_of_width(b):
    """The smallest and the largest prime of b bits."""
    low, high = (1 << (b - 1)) + 1, (1 << b) - 1
    while not oracle.is_prime(low):
        low += 2
    while not oracle.is_prime(high):
        high -= 2
    return low, high


def digit_shape(q):
    """Where digit k of a plaintext residue goes: R_k below the cut kappa, R_(4 + k - kappa) above, d of them there."""
    b = q.bit_length()
    kappa = 0 if b < 32 else (b - 32) // 8 + 1
    return kappa, b // 8 + 1 - kappa


def check_forms(got, value, q):
    """got(form): the reduction of a sum whose value is given, in every form that q has."""
    assert got(he.DIGITS_CANONICAL) == value % q
    lazy = got(he.DIGITS_BELOW_6Q)
    assert lazy % q == value % q and (lazy < 6 * q if q < 1 << 60 else 5 * lazy < 16 * q), lazy / q
    if q < 1 << 61:
        lazy = got(he.DIGITS_BELOW_4Q)
        assert lazy % q == value % q and lazy < 4 * q, lazy / q


@pytest.mark.parametrize("bits", range(12, 63))
def test_final_reduction_of_the_matrix_core_sums(bits):
    """The sums of the int8 products at the ends of their range (4080 terms of 2^17, packed 2^16) and anywhere in it, every
    width of modulus: congruent, below 6q and 4q in the unreduced forms (3.2q from 2^60 on), canonical in the others."""
    rnd = random.Random(bits)
    for q in primes_of_width(bits):
        kappa, d = digit_shape(q)
        top = DIGIT_TERMS << 17
        for trial in range(120):
            sums = [0] * 8
            for m in list(range(kappa)) + list(range(4, 4 + d)):
                sums[m] = {0: top, 1: -top, 2: rnd.choice([top, -top])}.get(trial, rnd.choice([top, -top, rnd.randint(-top, top)]))
            value = sum(v << 8 * (m if m < 4 else m - 4 + kappa) for m, v in enumerate(sums))
            addend = rnd.choice([0, q - 1, rnd.randrange(q)])
            check_forms(lambda form: he.host_digit_reduce(sums, q, addend, form), value + addend, q)
            if q < 1 << 30:
                four = [v >> 1 for v in sums[4:]]
                value = sum(v << 8 * m for m, v in enumerate(four)) + addend
                assert he.host_digit_reduce(four, q, addend, he.DIGITS_PACKED) == value % q


@pytest.mark.parametrize("bits", range(12, 63))
def test_matrix_core_mac_on_the_host(bits):
    """Digits of both operands, products and reduction: sums of one term to the most that the 32-bit sums take, of operands
    whose digits are extreme (-128 and 127 throughout, q - 1 and its neighbours, around q / 2) and of random ones."""
    rng = np.random.default_rng(bits)
    for q in primes_of_width(bits):
        extreme = [0, 1, q - 1, q - 2, q // 2, q // 2 + 1, 0x8080808080808080 % q, 0x7F7F7F7F7F7F7F7F % q,
                   int("80" * 8, 16) & ((1 << (bits - 1)) - 1), int("7f" * 8, 16) & ((1 << (bits - 1)) - 1)]
        for n in (0, 1, 2, 17, 300, DIGIT_TERMS):
            for kind in ("extreme", "random", "top"):
                x = rng.choice(extreme, n) if kind == "extreme" else rng.integers(0, q, n) if kind == "random" else np.full(n, q - 1)
                w = rng.choice(extreme, n) if kind == "extreme" else rng.integers(0, q, n) if kind == "random" else np.full(n, q - 1)
                addend = int(rng.choice([0, q - 1]))
                value = sum(int(a) * int(b) for a, b in zip(x, w)) + addend
                check_forms(lambda form: he.host_mac_digits(x, w, q, addend, form), value, q)
                if q < 1 << 30:
                    assert he.host_mac_digits(x, w, q, addend, he.DIGITS_PACKED) == value % q
        too_many = np.zeros(DIGIT_TERMS + 1, dtype=np.uint64)
        assert he.host_mac_digits(too_many, too_many, q) == 2**64 - 1


@pytest.mark.parametrize("log2N,bits", [(10, 50), (11, 48), (12, 47), (13, 49), (14, 50), (10, 46), (14, 46), (14, 30)])
def test_double_precision_transform_of_a_digit_on_the_host(log2N, bits):
    """The digit expansion of a key switch feeds the double-precision transform values up to twice the modulus: exact, and
    below the 6.62 q that the first pass then reaches (9.93 q where nothing is reduced between the stages)."""
    N = 1 << log2N
    q = wl.ntt_primes(bits, N, 1)[0]
    ctx = he.Context(log2N, [wl.ntt_primes(60, N, 1)[0], q], device=None)
    rng = np.random.default_rng(log2N + bits)
    for v in (rng.integers(0, 2 * q, N), np.full(N, 2 * q - 1), np.where(rng.integers(0, 2, N) == 1, 2 * q, -2 * q),
              np.where(np.arange(N) % 2 == 0, 2 * q - 1, 0)):
        got, worst = ctx.host_ntt_forward_fp64(1, v, expand=True)
        assert np.array_equal(got, oracle.ntt_fwd(np.mod(v, q).astype(np.uint64)[None, :], [q], [ctx.psi[1]])[0])
        assert worst < (9.93 if bits <= 46 else 6.62)
    with pytest.raises(he.HeError):
        ctx.host_ntt_forward_fp64(1, np.full(N, 2 * q + 1), expand=True)


@pytest.mark.parametrize("log2N,bits", [(10, 50), (11, 49), (12, 40), (13, 50), (14, 50), (14, 31)])
def test_double_precision_forward_transform_on_the_host(log2N, bits):
    """The forward transform on double-precision FMAs (moduli below 2^50), compiled for the host, against the oracle's
    direct transform: inputs of either sign up to q in magnitude, extreme and random; every intermediate an exact
    integer, and none beyond the 6.22 q that the kernels' reduction points are placed for."""
    N = 1 << log2N
    q = wl.ntt_primes(bits, N, 1)[0]
    big = wl.ntt_primes(60, N, 1)[0]
    ctx = he.Context(log2N, [big, q], device=None)
    psi = ctx.psi[1]
    rng = np.random.default_rng(log2N * 100 + bits)
    cases = [rng.integers(-q, q + 1, N), np.full(N, q), np.full(N, -q), np.where(rng.integers(0, 2, N) == 1, q, -q),
             np.where(np.arange(N) % 2 == 0, q // 2, -(q // 2)), np.zeros(N, dtype=np.int64)]
    for k, v in enumerate(cases):
        got, worst = ctx.host_ntt_forward_fp64(1, v)
        want = oracle.ntt_fwd(np.mod(v, q).astype(np.uint64)[None, :], [q], [psi])[0]
        assert np.array_equal(got, want), (log2N, bits, k)
        assert worst < 6.22, (log2N, bits, k, worst)
    # the inverse transform: canonical inputs, extreme and random; sums, differences and products stay below 4.001 q
    for k, v in enumerate([rng.integers(0, q, N), np.full(N, q - 1), np.where(np.arange(N) % 2 == 0, q - 1, 0),
                           np.where(rng.integers(0, 2, N) == 1, (q - 1) // 2, (q + 1) // 2), np.zeros(N, dtype=np.int64)]):
        v = v.astype(np.uint64)
        got, worst = ctx.host_ntt_inverse_fp64(1, v)
        assert np.array_equal(got, oracle.ntt_inv(v[None, :], [q], [psi])[0]), (log2N, bits, k)
        assert worst < 4.001, (log2N, bits, k, worst)
    with pytest.raises(he.HeError) as e:                       # the 60-bit limb has no such form
        ctx.host_ntt_forward_fp64(0, np.zeros(N, dtype=np.int64))
    assert e.value.status == -2
    with pytest.raises(he.HeError):                            # an input beyond q in magnitude
        ctx.host_ntt_forward_fp64(1, np.full(N, q + 1))


def test_double_precision_butterfly_bounds():
    """The growth bound that places the reductions of the double-precision transform: with |W| <= q/2 and
    |Y| <= B q the quotient estimate is off by less than 0.1875 B, so a butterfly takes B to 0.5 + 1.1875 B;
    from 1 four stages, and from 0.5001 six, stay below 2^53 / 2^50 = 8."""
    def after(b, stages):
        for _ in range(stages):
            b = 0.5 + 1.1875 * b
        return b
    assert after(1.0, 4) < 4.63 and after(0.5001, 4) < 3.64 and after(0.5001, 6) < 6.22 and after(0.5001, 7) < 7.88
    assert after(0.5001, 8) > 8
    # inverse butterflies: sums double, products of differences bounded by 2B start again at 0.5 + 0.375 B
    b = 0.5001
    sums, prods = 2 * b, 0.5 + 0.375 * b                      # first stage
    sums, prods = 2 * max(sums, prods), 0.5 + 0.375 * max(sums, prods)
    assert sums < 2.0005
    three = 2 * max(sums, prods)
    assert three < 4.001                                       # a three-stage pass ends here
    m = max(0.5001, prods)                                     # four stages: the second stage's sums are reduced
    sums, prods = 2 * m, 0.5 + 0.375 * m
    m = max(sums, prods)
    assert 2 * m < 3.501 and 0.5 + 0.375 * m < 1.16
    # the estimate's error: three roundings of 2^-53 on a value below B * 2^49
    assert 3 * 2.0 ** -53 * 2.0 ** 49 == 0.1875
