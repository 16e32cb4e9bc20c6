"""The work that a user of the library has it do, as cases to time: whole layer calls and the calls around them,
through the public entry points of `paper_1908_04172_amd.he`, on seeded synthetic inputs of the shapes in
`paper_1908_04172_amd.workloads` and bench.py.

A case is a dict of plain values.  "bits" is the modulus chain as text, one bit size per limb, the last limb being
the one that a rescale drops (or the special prime of a relinearisation).  Kinds:

  layer    a dense or convolution layer with scalar plaintexts: weights and bias (doubles on the GPU) are encoded at
           the level in use and one he_ct_pt_mac(RESCALE) call computes MAC, bias and the lazy rescale
  packed   the same dense layer on packed 32-bit residues
  poly     a dense layer whose weights differ per slot: full-polynomial plaintexts, encoded ahead of time
  split    a dense layer whose terms arrive in two calls (partial sums), then a full-polynomial bias, then the rescale
  scale    one scalar multiply, a bias and a rescale per ciphertext (a batch normalisation that is not folded)
  square   the x^2 activation: square, relinearise, rescale
  encode   complex slot vectors to plaintext polynomials (what a client does with its inputs)
  decode   plaintext polynomials back to complex slots (what a client does with the results)

Residues are integers and have to be the same whole numbers whatever computes them.  So have the encoder's (its
doubles are rounded to integers before a transform that spreads one different integer over a whole row); the
decoder's results are doubles.
"""
import math

import torch

from paper_1908_04172_amd import he, workloads as wl

DEVICE = "cuda"


def listed():
    return [
        # the smallest layer of the benchmark configurations: launches and latency count
        {"name": "dense_64_16", "kind": "layer", "log2N": 12, "bits": "30 30", "layer": "dense", "K": 64, "M": 16,
         "log2_scale": 24},
        # CryptoNets' convolution over a 28x28 image, five filters
        {"name": "conv_28x28x1_5", "kind": "layer", "log2N": 13, "bits": "60 40 40 40", "layer": "conv", "H": 28, "C": 1,
         "KH": 5, "OC": 5, "stride": 2, "padding": "valid", "log2_scale": 40},
        # CryptoNets' dense layer: long sums, an output count that is not a multiple of anything
        {"name": "dense_845_100", "kind": "layer", "log2N": 13, "bits": "60 40 40 40", "layer": "dense", "K": 845, "M": 100,
         "log2_scale": 40},
        # a convolution over an RGB image: the largest layer with scalar plaintexts
        {"name": "conv_32x32x3_16", "kind": "layer", "log2N": 14, "bits": "60 60 50 50 50 50 50 50", "layer": "conv", "H": 32,
         "C": 3, "KH": 3, "OC": 16, "stride": 2, "padding": "same", "log2_scale": 50},
        # the largest ring degree, whose rows do not fit a compute unit's local memory
        {"name": "dense_96_24_ring15", "kind": "layer", "log2N": 15, "bits": "60 60 50 50 50 50 50 50", "layer": "dense",
         "K": 96, "M": 24, "log2_scale": 50},
        # weights that differ per slot
        {"name": "poly_256_64", "kind": "poly", "log2N": 14, "bits": "60 60 50 50 50 50 50 50", "K": 256, "M": 64},
        # 30-bit moduli in 32-bit storage
        {"name": "packed_1024_256", "kind": "packed", "log2N": 12, "bits": "30 30", "K": 1024, "M": 256, "log2_scale": 24},
        # a layer whose terms arrive in two parts of odd sizes, with a bias that differs per slot
        {"name": "split_200_113_37", "kind": "split", "log2N": 13, "bits": "60 50 50", "K": 200, "K2": 113, "M": 37,
         "log2_scale": 45},
        # elementwise scaling of a feature map: streaming
        {"name": "scale_845", "kind": "scale", "log2N": 13, "bits": "60 40 40", "n": 845, "log2_scale": 40},
        # the activation of a hidden layer
        {"name": "square_256", "kind": "square", "log2N": 14, "bits": "60 50 50 50 50 50 50 60", "n": 256},
        {"name": "encode_784", "kind": "encode", "log2N": 13, "bits": "60 40 40 40", "n": 784, "log2_scale": 40},
        {"name": "decode_100", "kind": "decode", "log2N": 13, "bits": "60 40", "n": 100, "log2_scale": 40},
    ]


def _log_int(rng, low, high):
    """low..high, spread over the logarithm; odd sizes as they come."""
    return min(high, max(low, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def _chain(rng, min_limbs=2):
    """A modulus chain of the families in use: one or two large primes, then equal ones near the scale."""
    first, rest, most, scale = rng.choice([("30", "30", 4, 24), ("60", "40", 5, 40), ("60", "45", 5, 42), ("60 60", "50", 8, 50),
                                           ("60", "55", 4, 50), ("58", "50", 4, 48)])
    n = rng.randint(max(min_limbs, len(first.split()) + 1), max(most, min_limbs))
    return " ".join([first] + [rest] * (n - len(first.split()))), scale


def _draw_once(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "poly", "packed", "split", "scale", "square", "encode", "decode"])
    log2N = rng.choice([12, 13, 13, 14, 14])
    if kind == "packed":
        return {"kind": kind, "log2N": log2N, "bits": " ".join(["30"] * rng.randint(2, 4)), "K": _log_int(rng, 16, 1024),
                "M": _log_int(rng, 2, 256), "log2_scale": 24}
    if kind == "square":
        limbs = rng.randint(2, 7)
        return {"kind": kind, "log2N": log2N, "bits": " ".join(["60"] + ["50"] * (limbs - 1) + ["60"]), "n": _log_int(rng, 4, 256)}
    bits, scale = _chain(rng)
    case = {"kind": kind, "log2N": log2N, "bits": bits}
    if kind in ("encode", "decode"):
        return dict(case, n=_log_int(rng, 4, 1024), log2_scale=min(scale, 40))
    if kind == "poly":
        return dict(case, K=_log_int(rng, 16, 256), M=_log_int(rng, 2, 64))
    if kind == "split":
        return dict(case, K=_log_int(rng, 32, 400), K2=_log_int(rng, 16, 200), M=_log_int(rng, 8, 128), log2_scale=scale)
    if kind == "scale":
        return dict(case, n=_log_int(rng, 32, 2048), log2_scale=scale)
    if rng.random() < 0.15:
        case["log2N"] = 15
    if rng.random() < 0.5:
        return dict(case, layer="dense", K=_log_int(rng, 16, 1024), M=_log_int(rng, 4, 256), log2_scale=scale)
    KH = rng.choice([1, 3, 3, 5])
    return dict(case, layer="conv", H=rng.randint(max(8, KH), 40), C=rng.randint(1, 8), KH=KH, OC=_log_int(rng, 2, 32),
                stride=1 if KH == 1 else rng.choice([1, 2]), padding=rng.choice(["valid", "same"]), log2_scale=scale)


def draw(rng):
    """One more case; none costs more than the largest of listed()."""
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["bytes"] < 1.2e10 and w["flops"] < 8e10:
            return case


# --------------------------------------------------------------------------------------------------------------

_plans = {}


def _plan(case):
    """The case's MAC plan or plans (host arrays; kept, because building a large convolution's takes a while)."""
    if case["kind"] in ("poly", "packed"):
        key = ("dense", case["K"], case["M"])
    elif case["kind"] == "split":
        key = ("dense", case["K"], case["M"])
    elif case["kind"] == "scale":
        key = ("scale", case["n"])
    elif case["layer"] == "dense":
        key = ("dense", case["K"], case["M"])
    else:
        key = ("conv", case["H"], case["C"], case["KH"], case["OC"], case["stride"], case["padding"])
    if key not in _plans:
        if len(_plans) > 16:
            _plans.clear()
        if key[0] == "dense":
            _plans[key] = wl.dense_plan(key[1], key[2])
        elif key[0] == "conv":
            _, H, C, KH, OC, stride, padding = key
            _plans[key] = wl.conv_plan(H, H, C, KH, KH, OC, stride, padding)
        else:
            import numpy as np
            each = np.arange(key[1], dtype=np.uint32)
            _plans[key] = wl.Plan(key[1], key[1], key[1], np.arange(key[1] + 1, dtype=np.uint32), each, each)
    return _plans[key]


def _shape(case):
    """(inputs, outputs, plaintexts, terms) of a MAC case, without building its plan."""
    kind = case["kind"]
    if kind == "scale":
        return case["n"], case["n"], case["n"], case["n"]
    if kind == "layer" and case["layer"] == "conv":
        H, C, KH, OC, s = case["H"], case["C"], case["KH"], case["OC"], case["stride"]
        out = (H - KH) // s + 1 if case["padding"] == "valid" else -(-H // s)
        return H * H * C, out * out * OC, KH * KH * C * OC, out * out * OC * KH * KH * C
    K, M = case["K"] + case.get("K2", 0), case["M"]
    return K, M, K * M, K * M


def work(case):
    """Bytes: every input residue or double once, every output once.  Operations: a multiply and an addition per residue
    and MAC term, three per butterfly (a rescale: one inverse transform and one forward transform per kept limb)."""
    N, L, kind = 1 << case["log2N"], len(case["bits"].split()), case["kind"]
    transform = 3 * (N // 2) * case["log2N"]  # operations of one row
    if kind == "encode":
        return {"bytes": case["n"] * (N // 2 * 16 + L * N * 8), "flops": case["n"] * (L + 1) * transform}
    if kind == "decode":
        return {"bytes": case["n"] * (N // 2 * 16 + L * N * 8), "flops": case["n"] * (L + 1) * transform}
    if kind == "square":
        n, l = case["n"], L - 1
        return {"bytes": 8 * N * (n * 2 * l + n * 2 * (l - 1) + l * 2 * L),
                "flops": n * ((l + l * l + 2 * L + 2 * l) * transform + (4 * l + 4 * l * L) * N)}
    n_in, n_out, n_pt, terms = _shape(case)
    word = 4 if kind == "packed" else 8
    residues = n_in * 2 * L * N + n_out * 2 * (L - 1) * N
    if kind == "poly":
        residues += n_pt * L * N
    if kind == "split":
        residues += n_out * L * N
    plain = 0 if kind == "poly" else 8 * (n_pt + n_out)
    return {"bytes": residues * word + plain, "flops": 2 * terms * 2 * L * N + n_out * 2 * L * transform}


def tolerance(case):
    # the decoder computes in doubles: against the same map in long double its results are off by 2.5e-16 (2-norm) and by
    # at most 1.0e-15 of their root mean square (log2N = 12 to 14, scales 2^24 to 2^50); four times that
    return {"rel": 1e-15, "max": 4e-15} if case["kind"] == "decode" else "exact"


# --------------------------------------------------------------------------------------------------------------

def _residues(outer, q, N, seed):
    return wl.uniform_residues_torch(outer, q, N, seed, DEVICE, chunk=2048)


def _normal(n, sigma, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device=DEVICE, generator=gen) * sigma


def _device_plan(ctx, p):
    return ctx.plan(p.n_in, p.n_out, p.n_pt, p.off, p.term_ct, p.term_pt)


def _empty(*shape, dtype=torch.int64):
    return torch.empty(shape, dtype=dtype, device=DEVICE)


def _workspace(n_bytes):
    return torch.empty(max(n_bytes, 256), dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    """What the program holds before the call: context, plan, buffers for outputs and workspace, and the inputs (uniform
    residues as ciphertexts, Gaussian weights and biases, slots in [-1, 1])."""
    kind, log2N = case["kind"], case["log2N"]
    N = 1 << log2N
    bits = [int(b) for b in case["bits"].split()]
    q = wl.modulus_chain(bits, N)
    L = len(q)
    ctx = he.Context(log2N, q, device=0)
    s = {"kind": kind, "ctx": ctx, "limbs": L, "scale": 2.0 ** case.get("log2_scale", 0)}
    seed = seed * 16 + 1
    if kind == "encode":
        n = case["n"]
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(seed)
        s["slots"] = torch.view_as_complex(torch.rand((n, N // 2, 2), dtype=torch.float64, device=DEVICE, generator=gen) * 2 - 1)
        s["out"] = _empty(n, L, N)
    elif kind == "decode":
        n = case["n"]
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(seed)
        slots = torch.view_as_complex(torch.rand((n, N // 2, 2), dtype=torch.float64, device=DEVICE, generator=gen) * 2 - 1)
        s["poly"] = ctx.encode_vector(slots, s["scale"])
        s["out"] = _empty(n, N // 2, dtype=torch.complex128)
        s["ws"] = _workspace(n * L * N * 8)
    elif kind == "square":
        n, l = case["n"], L - 1
        s["ct"] = _residues((n, 2), q[:l], N, seed)
        s["evk"] = _residues((l, 2), q, N, seed + 1)
        s["square"], s["out"] = _empty(n, 2, l, N), _empty(n, 2, l - 1, N)
        s["ws"] = _workspace(ctx.square_relin_workspace_bytes(l, n))
    else:
        p = _plan(case)
        s["plan"] = _device_plan(ctx, p)
        s["ct"] = _residues((p.n_in, 2), q, N, seed)
        s["out"] = _empty(p.n_out, 2, L - 1, N)
        if kind == "poly":
            s["pt"] = _residues((p.n_pt,), q, N, seed + 1)
            s["ws"] = _workspace(s["plan"].workspace_bytes(L, he.PT_POLY, he.RESCALE))
            return s
        s["w"], s["b"] = _normal(p.n_pt, 0.1, seed + 1), _normal(p.n_out, 0.1, seed + 2)
        s["w_enc"], s["b_enc"] = _empty(p.n_pt, L), _empty(p.n_out, L)
        s["ws"] = _workspace(s["plan"].workspace_bytes(L, he.PT_SCALAR, he.RESCALE))
        if kind == "packed":
            s["ct"] = ctx.pack32(s["ct"])
            s["out"] = _empty(p.n_out, 2, L - 1, N, dtype=torch.int32)
        elif kind == "split":
            p2 = wl.dense_plan(case["K2"], case["M"])
            s["plan2"] = _device_plan(ctx, p2)
            s["ct2"] = _residues((p2.n_in, 2), q, N, seed + 3)
            s["w2"], s["w2_enc"] = _normal(p2.n_pt, 0.1, seed + 4), _empty(p2.n_pt, L)
            s["bias"] = _residues((p.n_out,), q, N, seed + 5)
            s["sum"] = _empty(p.n_out, 2, L, N)
            s["ws"] = _workspace(max(s["plan"].workspace_bytes(L, he.PT_SCALAR, 0),
                                     s["plan2"].workspace_bytes(L, he.PT_SCALAR, he.ACCUMULATE)))
    return s


def run(s):
    """One pass: what a program calls for this layer or tensor, on the current stream."""
    ctx, kind, L = s["ctx"], s["kind"], s["limbs"]
    if kind == "encode":
        return ctx.encode_vector(s["slots"], s["scale"], out=s["out"])
    if kind == "decode":
        return ctx.decode_vector(s["poly"], s["scale"], out=s["out"], workspace=s["ws"])
    if kind == "square":
        ctx.ct_square_relin(s["ct"], s["evk"], out=s["square"], workspace=s["ws"])
        return ctx.rescale(s["square"], out=s["out"])
    if kind == "poly":
        return ctx.ct_pt_mac(s["plan"], s["ct"], s["pt"], he.PT_POLY, flags=he.RESCALE, out=s["out"], workspace=s["ws"])
    ctx.encode_scalar(s["w"], s["scale"], L, out=s["w_enc"])
    if kind == "split":
        ctx.encode_scalar(s["w2"], s["scale"], L, out=s["w2_enc"])
        ctx.ct_pt_mac(s["plan"], s["ct"], s["w_enc"], he.PT_SCALAR, out=s["sum"], workspace=s["ws"])
        ctx.ct_pt_mac(s["plan2"], s["ct2"], s["w2_enc"], he.PT_SCALAR, flags=he.ACCUMULATE, out=s["sum"], workspace=s["ws"])
        ctx.ct_pt_add(s["sum"], s["bias"], he.PT_POLY)
        ctx.rescale(s["sum"], out=s["out"])
        return s["out"], s["sum"]
    ctx.encode_scalar(s["b"], s["scale"], L, out=s["b_enc"])
    mac = ctx.ct_pt_mac32 if kind == "packed" else ctx.ct_pt_mac
    return mac(s["plan"], s["ct"], s["w_enc"], he.PT_SCALAR, bias=s["b_enc"], flags=he.RESCALE, out=s["out"], workspace=s["ws"])
