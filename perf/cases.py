"""Performance cases of the library's four calls on one GPU.

A case is one call (or one layer step of three calls) through the public
binding, with everything a user's program holds before it already made: the
context, the compiled plan, the NTT tables and workspaces, the rotation keys in
the library's layout, and the output buffer.  Values are uniform residues, as
ciphertexts and NTT-domain plaintexts are; signs are +1 / -1 / 0 with
probability 0.35 / 0.35 / 0.3 and scales uniform in [1, 2^20), as a ternary
layer's are.  Every result is a residue and has one right value, so the
tolerance is "exact".
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_35352_amd as fiona

SCALE_BITS = 20


# ----------------------------------------------------------------------------
# The cases
# ----------------------------------------------------------------------------

def _sum(name, N, L, n_in, n_out, T, g, ternary, pool=0, pitch=True, op="sum"):
    c = dict(op=op, N=N, L=L, n_in=n_in, n_out=n_out, T=T, g=g, ternary=ternary, pool=pool, pitch=pitch)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The weighted sum.
        # One packed output over 64 inputs at a small ring: the smallest call, where launches count.
        _sum("sum_tiny", 1 << 12, 3, 64, 1, 64, 8, 0.5, pitch=False),
        # A ragged ring (the weighted sum takes any N), odd counts, a remainder of raw terms per output.
        _sum("sum_ragged", 12001, 5, 37, 19, 203, 7, 0.5, pool=4, pitch=False),
        # A 3x3 convolution of 512 channels at N = 2^16: many outputs of few terms.
        _sum("sum_conv", 1 << 16, 8, 64, 128, 64, 8, 0.53),
        # A 768 x 768 projection in diagonal packing, signed sums shared across outputs.
        _sum("sum_projection", 1 << 16, 10, 24, 24, 768, 16, 0.65, pool=16),
        # A feed-forward up-projection: mostly ternary, little shared (a third of its outputs).
        _sum("sum_ffn", 1 << 16, 12, 32, 32, 768, 16, 0.795),
        # A 4096 x 4096 product (one chunk of its outputs): the longest sums, the largest call.
        _sum("sum_matmul", 1 << 16, 16, 128, 4, 4096, 32, 0.70, pool=16),
        # More inputs than one tile holds: passes over input ranges.
        _sum("sum_many_inputs", 1 << 14, 6, 320, 24, 320, 16, 0.6),
        # The rescale that follows a layer: a few ciphertexts at a small ring, and a convolution's outputs.
        dict(name="rescale_small", op="rescale", N=1 << 13, L=4, n_ct=4),
        dict(name="rescale_conv", op="rescale", N=1 << 16, L=8, n_ct=128),
        # The baby-step rotations that make a layer's inputs: a few at a small ring, and a convolution's.
        dict(name="rotate_small", op="rotate", N=1 << 13, L=4, n_rot=7),
        dict(name="rotate_conv", op="rotate", N=1 << 16, L=8, n_rot=63),
        # One whole layer step at a medium ring: rotations, weighted sum, rescale.
        _sum("layer_projection", 1 << 14, 6, 24, 24, 192, 16, 0.65, pool=16, op="layer"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["sum", "rescale", "rotate", "layer"], [5, 2, 2, 1])[0]
    while True:
        logn = rng.randint(12, 16)
        L = rng.randint(3, 16)
        if op in ("rescale", "rotate"):
            c = dict(op=op, N=1 << logn, L=L)
            c["n_ct" if op == "rescale" else "n_rot"] = _log_int(rng, 1, 128 if op == "rescale" else 127)
        else:
            N = 1 << logn
            if op == "sum" and rng.random() < 0.3:   # a ring that is not a power of two
                N = _log_int(rng, 1000, 1 << 16)
            n_in = _log_int(rng, 8, 320 if op == "sum" else 64)
            T = _log_int(rng, 32, 2048)
            c = _sum(None, N, L, n_in, _log_int(rng, 1, 128), T, rng.choice([7, 8, 16, 32]),
                     round(rng.uniform(0.0, 0.95), 3), rng.choice([0, 0, 4, 16]), rng.random() < 0.7, op)
        if op in ("sum", "layer") and c["n_out"] * c["T"] > 30000:   # at most about 30,000 terms
            continue
        if work(c)["bytes"] <= 16e9:
            return c


def tolerance(case):
    return "exact"


def _terms(case):
    """Ternary blocks per output, and raw terms of the whole layer."""
    k = int(round(case["ternary"] * (case["T"] // case["g"])))
    return k, case["n_out"] * (case["T"] - k * case["g"])


def work(case):
    """Words read and written once; modular operations (a product or a sum of residues counts one)."""
    N, L = case["N"], case["L"]
    ntt = 1.5 * N * math.log2(N)   # a product, a sum and a difference per butterfly
    if case["op"] == "rescale":
        v = 2 * case["n_ct"]
        return {"bytes": 8.0 * N * v * (2 * L - 1), "flops": v * (L * ntt + 2 * (L - 1) * N)}
    words = ops = 0.0
    if case["op"] in ("rotate", "layer"):
        n_rot = case["n_rot"] if case["op"] == "rotate" else case["n_in"] - 1
        words += 2 * L * N + n_rot * 2 * L * (L + 1) * N
        ops += (L * (L + 2) + 2 * n_rot * (L + 1)) * ntt + n_rot * (4 * L * (L + 1) + 5 * L) * N
        if case["op"] == "rotate":
            words += n_rot * 2 * L * N
    if case["op"] in ("sum", "layer"):
        k, raw = _terms(case)
        groups = k * case["n_out"]
        words += raw * L * N
        ops += L * N * (4.0 * raw + groups * (2 * 0.7 * case["g"] + 4))
        if case["op"] == "sum":
            words += L * N * 2 * (case["n_in"] + case["n_out"])
        else:
            v = 2 * case["n_out"]
            words += v * (L - 1) * N
            ops += v * (L * ntt + 2 * (L - 1) * N)
    return {"bytes": 8.0 * words, "flops": ops}


# ----------------------------------------------------------------------------
# Inputs, from the case and the seed alone
# ----------------------------------------------------------------------------

def _is_prime(n):
    for p in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if n % p == 0:
            return n == p
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def _primes(N, count):
    """The first primes below 2^50 that are 1 modulo 2 N (N rounded up to a power of two)."""
    step = 2 << (N - 1).bit_length()
    q, out = ((1 << 50) - 2) // step * step + 1, []
    while len(out) < count:
        if _is_prime(q):
            out.append(q)
        q -= step
    return out


def _galois(N, n_rot):
    return [pow(5, r, 2 * N) for r in range(1, n_rot + 1)]


def _layer(case, seed):
    """The layer's description: term t of an output reads input t mod n_in; g consecutive terms are a
    ternary group with one scale, or raw terms; with a pool, signs recur (up to a flip) across outputs."""
    rng = np.random.default_rng([seed, 1])
    n_in, n_out, T, g, pool = (case[k] for k in ("n_in", "n_out", "T", "g", "pool"))
    blocks, (k, _) = T // g, _terms(case)
    draw_signs = lambda shape: rng.choice(np.array([1, -1, 0], np.int8), shape, p=[0.35, 0.35, 0.3])
    signs_of = {s: draw_signs((pool, g)) for s in sorted({b * g % n_in for b in range(blocks)})} if pool else {}
    pm_off, grp_off, pm_input, mem_input, mem_sign = [0], [0], [], [], []
    for _ in range(n_out):
        ternary = np.zeros(blocks, bool)
        ternary[rng.permutation(blocks)[:k]] = True
        raw = np.concatenate([np.repeat(~ternary, g), np.ones(T - blocks * g, bool)])
        pm_input.append(np.flatnonzero(raw) % n_in)
        for b in np.flatnonzero(ternary):
            mem_input.append(np.arange(b * g, (b + 1) * g) % n_in)
            if pool:
                mem_sign.append(signs_of[b * g % n_in][rng.integers(pool)] * np.int8(1 - 2 * rng.integers(2)))
            else:
                mem_sign.append(draw_signs(g))
        pm_off.append(pm_off[-1] + int(raw.sum()))
        grp_off.append(grp_off[-1] + k)
    groups = grp_off[-1]
    cat = lambda xs, dt: np.concatenate(xs).astype(dt) if xs else np.zeros(0, dt)
    return dict(pm_off=pm_off, pm_input=cat(pm_input, np.uint32), pm_pt=np.arange(pm_off[-1]), grp_off=grp_off,
                grp_mem_off=np.arange(groups + 1) * g, mem_input=cat(mem_input, np.uint32),
                mem_sign=cat(mem_sign, np.int8), grp_scale=np.arange(groups),
                scales=rng.integers(1, 1 << SCALE_BITS, groups))


def _residues(shape, moduli, gen, pitch=0):
    """Uniform residues [...][limb][N]; rows of the first axis `pitch` words apart if given."""
    n, N = int(np.prod(shape[:-2])), shape[-1]
    row = max(pitch, len(moduli) * N)
    make = torch.zeros if pitch > len(moduli) * N else torch.empty
    flat = make(n * row, dtype=torch.int64, device="cuda")
    rows = flat.view(n, row)
    for l, q in enumerate(moduli):
        rows[:, l * N:(l + 1) * N].random_(0, q, generator=gen)
    return flat if pitch else flat.view(shape)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    op, N, L = case["op"], case["N"], case["L"]
    d = {"moduli": _primes(N, L + 1)}
    q = d["moduli"][:L]
    if op in ("sum", "layer"):
        d["layer"] = la = _layer(case, seed)
        d["pitch"] = (L * N + 63) // 64 * 64 + 128 if case["pitch"] else L * N
        d["pt"] = _residues((len(la["pm_pt"]), L, N), q, gen, d["pitch"])
        d["sign"] = torch.from_numpy(la["mem_sign"]).cuda()
        d["scale"] = torch.from_numpy(la["scales"]).cuda()
    if op in ("rotate", "layer"):
        n_rot = case["n_rot"] if op == "rotate" else case["n_in"] - 1
        d["galois"] = _galois(N, n_rot)
        d["ct"] = _residues((1, 2, L, N), q, gen)
        d["keys"] = _residues((n_rot, L, 2, L + 1, N), d["moduli"], gen)   # natural order
    else:
        n = case["n_in"] if op == "sum" else case["n_ct"]
        d["x"] = _residues((n, 2, L, N), q, gen)
    return d


def prepare(case, seed):
    s = _inputs(case, seed)
    op, N, L = case["op"], case["N"], case["L"]
    s["op"] = op
    s["ctx"] = ctx = fiona.Ctx(N, L, s["moduli"][:L])
    empty = lambda *shape: torch.empty(shape, dtype=torch.int64, device="cuda")
    if op in ("sum", "layer"):
        la = s["layer"]
        s["plan"] = fiona.Plan(ctx, case["n_in"], case["n_out"], len(la["pm_pt"]), len(la["scales"]), la["pm_off"],
                               la["pm_input"], la["pm_pt"], la["grp_off"], la["grp_mem_off"], la["mem_input"],
                               la["mem_sign"], la["grp_scale"], pt_pitch=s["pitch"])
        s["out"] = empty(case["n_out"], 2, L, N)
    if op in ("rotate", "layer"):
        s["rotator"] = rot = fiona.Rotator(ctx, s["moduli"][L], len(s["galois"]))
        natural, s["keys"] = s["keys"], empty(*s["keys"].shape)
        for r, g in enumerate(s["galois"]):
            fiona.rotation_key_layout(rot, g, natural[r], s["keys"][r])
        torch.cuda.synchronize()
        # a layer's inputs: step 0 is the ciphertext itself, the rotations follow it
        s["x"] = empty(len(s["galois"]) + 1, 2, L, N)
        s["x"][0] = s["ct"][0]
    if op in ("rescale", "layer"):
        n = case["n_ct"] if op == "rescale" else case["n_out"]
        s["rescaler"] = fiona.Rescaler(ctx, n)
        s["n_ct"] = n
        s["res"] = empty(n, 2, L - 1, N)
    return s


def run(s):
    op = s["op"]
    if op == "sum":
        fiona.hybrid_linear(s["plan"], s["x"], s["pt"], s["sign"], s["scale"], s["out"])
        return s["out"]
    if op == "rescale":
        fiona.rescale(s["rescaler"], s["x"], s["n_ct"], s["res"])
        return s["res"]
    fiona.hoisted_rotate(s["rotator"], s["x"][0], s["galois"], s["keys"], s["x"][1:])
    if op == "rotate":
        return s["x"][1:]
    fiona.hybrid_linear(s["plan"], s["x"], s["pt"], s["sign"], s["scale"], s["out"])
    fiona.rescale(s["rescaler"], s["out"], s["n_ct"], s["res"])
    return s["res"]


# ----------------------------------------------------------------------------
# The same results in plain 64-bit torch
# ----------------------------------------------------------------------------

def _mul(a, b, q):
    """a b mod q for residues of q < 2^50: the quotient in float64 (off by at most one), the rest in
    64-bit integers that wrap."""
    k = (a.double() * (b.double() if torch.is_tensor(b) else float(b)) / q).round().long()
    return (a * b - k * q) % q


def _powers(w, n, q):
    t = torch.ones(1, dtype=torch.int64, device="cuda")
    while t.numel() < n:
        t = torch.cat([t, _mul(t, pow(w, t.numel(), q), q)])
    return t[:n]


def _dft(x, w, q):
    """sum_n x_n w^(n k) along the last axis, natural order in and out (w of order N)."""
    lead, N = x.shape[:-1], x.shape[-1]
    x, n, s, pw = x.reshape(-1, N), N, 1, _powers(w, N, q)
    while n > 1:
        m = n // 2
        a, b = x.reshape(-1, 2, m, s).unbind(1)
        x = torch.stack([(a + b) % q, _mul((a - b) % q, pw[: m * s : s, None], q)], 2).reshape(-1, N)
        n, s = m, 2 * s
    return x.reshape(*lead, N)


def _psi(N, q):
    x = 2
    while pow(x, (q - 1) // 2, q) != q - 1:
        x += 1
    return pow(x, (q - 1) // (2 * N), q)


def _ntt(x, q):
    """a_k = sum_n x_n psi^((2 k + 1) n)."""
    N, psi = x.shape[-1], _psi(x.shape[-1], q)
    return _dft(_mul(x, _powers(psi, N, q), q), psi * psi % q, q)


def _intt(x, q):
    N = x.shape[-1]
    inv = pow(_psi(N, q), -1, q)
    return _mul(_mul(_dft(x, inv * inv % q, q), _powers(inv, N, q), q), pow(N, -1, q), q)


def _divide(x, moduli):
    """round(x / last modulus), x [..., limbs, N] in the NTT domain."""
    t = moduli[-1]
    r = _intt(x[..., -1, :], t)
    r = torch.where(r > t // 2, r - t, r)
    return torch.stack([_mul((x[..., l, :] - _ntt(r % q, q)) % q, pow(t, -1, q), q)
                        for l, q in enumerate(moduli[:-1])], -2)


def _exact_sum(case, d, x):
    la, L, N = d["layer"], case["L"], case["N"]
    q = torch.tensor(d["moduli"][:L], device="cuda")[:, None]
    pt = d["pt"].view(-1, d["pitch"])
    out = torch.zeros(case["n_out"], 2, L, N, dtype=torch.int64, device="cuda")
    for j in range(case["n_out"]):
        acc = out[j]
        for p in range(la["pm_off"][j], la["pm_off"][j + 1]):
            acc += _mul(x[int(la["pm_input"][p])], pt[p, : L * N].view(L, N), q)   # below 2^50 a term
        acc %= q
        for g in range(la["grp_off"][j], la["grp_off"][j + 1]):
            u = torch.zeros_like(acc)
            for m in range(int(la["grp_mem_off"][g]), int(la["grp_mem_off"][g + 1])):
                if la["mem_sign"][m]:
                    u.add_(x[int(la["mem_input"][m])], alpha=int(la["mem_sign"][m]))
            acc += _mul(u % q, int(la["scales"][g]), q)
        acc %= q
    return out


def _exact_rotate(case, d):
    """Hoisted: digits of c1 by limb, the automorphism as a slot gather, the keys, the division by P."""
    L, N, mods = case["L"], case["N"], d["moduli"]
    c0, c1 = d["ct"][0]
    digits = [_intt(c1[j], mods[j]) for j in range(L)]
    hat = torch.stack([torch.stack([_ntt(dj % q, q) for q in mods]) for dj in digits])   # [digit][modulus][N]
    q = torch.tensor(mods, device="cuda")[:, None]
    slots, out = torch.arange(N, device="cuda"), []
    for r, g in enumerate(d["galois"]):
        pi = (slots * g + (g - 1) // 2) % N
        v = sum(_mul(d["keys"][r, j], hat[j][:, pi], q) for j in range(L)) % q
        y = _divide(v, mods)
        y[0] = (y[0] + c0[:, pi]) % q[:L]
        out.append(y)
    return torch.stack(out)


def exact(case, seed):
    d = _inputs(case, seed)
    moduli = d["moduli"][: case["L"]]
    if case["op"] == "rescale":
        return _divide(d["x"], moduli)
    if case["op"] == "sum":
        return _exact_sum(case, d, d["x"])
    rot = _exact_rotate(case, d)
    if case["op"] == "rotate":
        return rot
    return _divide(_exact_sum(case, d, torch.cat([d["ct"], rot])), moduli)
