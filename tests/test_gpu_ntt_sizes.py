"""GPU parity of the NTT kernels at every size they are built for: rescales and
rotations at N = 2^8 .. 2^17 (whole transforms up to 2^14, passes from 2^13 on;
both splits, even and odd log N), with uniform residues, residues at the ends of
their range and moduli of very different sizes, bit-exact against the oracle's
integer arithmetic."""
import sys

import numpy as np
import pytest

import synth
import paper_2609_35352_amd as fiona
from oracle import rescale as rs
from oracle import rotate as ro

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fiona.lib()
    return torch.device("cuda:0")


def _moduli(N, mixed):
    """Three moduli: the largest below 2^50, or a small one, a large one and a large last one."""
    big = synth.ntt_primes(N, 3)
    return big if not mixed else [synth.ntt_primes(N, 1, bits=26)[0], big[0], big[1]]


def _cts(N, moduli, n_ct, seed):
    rng = np.random.default_rng(seed)
    cts = np.zeros((n_ct, 2, len(moduli), N), dtype=np.uint64)
    for l, q in enumerate(moduli):
        cts[:, :, l] = rng.integers(0, q, (n_ct, 2, N), dtype=np.uint64)
        cts[0, 0, l] = q - 1                                        # the ends of the range
        cts[0, 1, l, ::2] = q - 1
        cts[0, 1, l, 1::2] = 0
    return cts


def _t(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).reshape(-1).view(np.int64)).to(dev)


@pytest.mark.parametrize("log_n", range(8, 18))
@pytest.mark.parametrize("mixed", [False, True])
def test_rescale_every_size(dev, log_n, mixed):
    import torch
    N, n_ct = 1 << log_n, 2 if log_n > 14 else 3
    _say("[ntt sizes] rescale N=2^%d mixed=%s" % (log_n, mixed))
    moduli = _moduli(N, mixed)
    cts = _cts(N, moduli, n_ct, log_n)
    r = fiona.Rescaler(fiona.Ctx(N, 3, moduli), n_ct)
    out = torch.full((n_ct * 2 * 2 * N,), -1, dtype=torch.int64, device=dev)
    fiona.rescale(r, _t(cts, dev), n_ct, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint64).reshape(n_ct, 2, 2, N)
    for c in range(n_ct if log_n <= 14 else 1):
        assert np.array_equal(got[c], rs.rescale(cts[c], moduli)), "ciphertext %d differs" % c


@pytest.mark.parametrize("log_n", [8, 9, 10, 13, 14, 15])
def test_rotate_every_size(dev, log_n):
    _rotate(dev, log_n, [5, 2 * (1 << log_n) - 1, 1], range(3))


@pytest.mark.parametrize("n_rot", [64, 65, 130])
def test_rotate_round_edges(dev, n_rot):
    """The inner product's rounds of buffered outputs: one of 64, 33 + 32, 44 + 43 + 43."""
    galois = [pow(5, 1 + r, 512) for r in range(n_rot)]
    _rotate(dev, 8, galois, [r for r in (0, 32, 33, 43, 44, 63, 64, 87, 88, 129) if r < n_rot])


@pytest.mark.parametrize("n_rot", [33, 63])
def test_rotate_long_chain(dev, n_rot):
    """L = 32: 63 rotations fill the inner product's LDS (33 and 63 take more of it than 64, two rounds of 32)."""
    _rotate(dev, 8, [pow(5, 1 + r, 512) for r in range(n_rot)], [0, n_rot - 1], L=32)


def _rotate(dev, log_n, galois, check, L=2):
    import torch
    N = 1 << log_n
    _say("[ntt sizes] rotate N=2^%d, L=%d, %d rotations" % (log_n, L, len(galois)))
    chain = synth.ntt_primes(N, L + 1)
    moduli, P = chain[:L], chain[L]
    ct = _cts(N, moduli, 1, 40 + log_n)[0]
    rng = np.random.default_rng(log_n)
    ctx = fiona.Ctx(N, L, moduli)
    rot = fiona.Rotator(ctx, P, len(galois))
    keys = np.zeros((len(galois), L, 2, L + 1, N), dtype=np.uint64)
    for m, q in enumerate(chain):
        keys[:, :, :, m] = rng.integers(0, q, (len(galois), L, 2, N), dtype=np.uint64)
    lib = torch.empty(keys.size, dtype=torch.int64, device=dev)
    for r, g in enumerate(galois):
        fiona.rotation_key_layout(rot, g, _t(keys[r], dev), lib[r * rot.key_words():(r + 1) * rot.key_words()])
    out = torch.full((len(galois) * 2 * L * N,), -1, dtype=torch.int64, device=dev)
    fiona.hoisted_rotate(rot, _t(ct, dev), galois, lib, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint64).reshape(len(galois), 2, L, N)
    for r in check:
        want = ro.rotate(ct, galois[r], keys[r], moduli, P)
        assert np.array_equal(got[r], want), "rotation %d (element %d) differs" % (r, galois[r])


@pytest.mark.parametrize("log_n,L,n_ct", [(8, 2, 1), (9, 4, 40), (10, 7, 3), (12, 6, 33), (13, 3, 1), (14, 3, 39), (14, 3, 40)])
def test_rescale_groups_of_limbs(dev, log_n, L, n_ct):
    """Whole transforms with one and several limbs a workgroup, and the edge
    of their use at N = 2^14 (160 forward transforms)."""
    import torch
    N = 1 << log_n
    _say("[ntt sizes] rescale N=2^%d L=%d n_ct=%d" % (log_n, L, n_ct))
    moduli = synth.ntt_primes(N, L)
    cts = _cts(N, moduli, n_ct, 7 * log_n + L)
    r = fiona.Rescaler(fiona.Ctx(N, L, moduli), n_ct)
    out = torch.full((n_ct * 2 * (L - 1) * N,), -1, dtype=torch.int64, device=dev)
    fiona.rescale(r, _t(cts, dev), n_ct, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(np.uint64).reshape(n_ct, 2, L - 1, N)
    for c in sorted({0, n_ct // 2, n_ct - 1}):
        assert np.array_equal(got[c], rs.rescale(cts[c], moduli)), "ciphertext %d differs" % c


@pytest.mark.parametrize("log_n,n_rot", [(12, 3), (13, 63), (13, 64)])
def test_rotate_division_edges(dev, log_n, n_rot):
    """The division whole up to N = 2^12, and at 2^13 from 256 forward transforms on (L = 2: 64 rotations)."""
    galois = [pow(5, 1 + r, 2 << log_n) for r in range(n_rot)]
    _rotate(dev, log_n, galois, sorted({0, n_rot // 2, n_rot - 1}))


def _residues(moduli, shape, seed, dev):
    """Uniform residues [...][limb][N] on the device."""
    import torch
    gen = torch.Generator(device=dev).manual_seed(seed)
    x = torch.empty(shape, dtype=torch.int64, device=dev)
    for l, q in enumerate(moduli):
        x[..., l, :].random_(0, q, generator=gen)
    return x


def _np(x):
    return x.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n_ct", [240, 243])
def test_rescale_chunks(dev, n_ct):
    """Intermediates of just within 256 MiB (one chunk) and just over (chunks of 122 and 121 ciphertexts)."""
    import torch
    N, L = 1 << 15, 3
    _say("[ntt sizes] rescale chunks n_ct=%d" % n_ct)
    moduli = _moduli(N, False)
    cts = _residues(moduli, (n_ct, 2, L, N), n_ct, dev)
    out = torch.full((n_ct, 2, L - 1, N), -1, dtype=torch.int64, device=dev)
    fiona.rescale(fiona.Rescaler(fiona.Ctx(N, L, moduli), n_ct), cts, n_ct, out)
    torch.cuda.synchronize()
    for c in (0, 121, 122, n_ct - 1):
        assert np.array_equal(_np(out[c]), rs.rescale(_np(cts[c]), moduli)), "ciphertext %d differs" % c


@pytest.mark.parametrize("log_n,n_ct", [(15, 3), (15, 4), (15, 30), (15, 31), (14, 12), (16, 6), (17, 3)])
def test_rescale_store_policies(dev, log_n, n_ct):
    """Intermediates of just under 4 MiB and just over 32 (stores of the default policy), just within
    (nontemporal), and within at every pair of sides."""
    import torch
    N, L = 1 << log_n, 3
    _say("[ntt sizes] rescale store policy N=2^%d n_ct=%d" % (log_n, n_ct))
    moduli = _moduli(N, False)
    cts = _residues(moduli, (n_ct, 2, L, N), n_ct, dev)
    out = torch.full((n_ct, 2, L - 1, N), -1, dtype=torch.int64, device=dev)
    fiona.rescale(fiona.Rescaler(fiona.Ctx(N, L, moduli), n_ct), cts, n_ct, out)
    torch.cuda.synchronize()
    for c in (0, n_ct - 1):
        assert np.array_equal(_np(out[c]), rs.rescale(_np(cts[c]), moduli)), "ciphertext %d differs" % c


def test_rotate_division_chunks(dev):
    """The division in three chunks of 132, 132 and 130 vectors, the second over both polynomials."""
    import torch
    N, L, n_rot = 1 << 15, 8, 197
    _say("[ntt sizes] rotate chunks")
    chain = synth.ntt_primes(N, L + 1)
    ct = _residues(chain[:L], (2, L, N), 5, dev)
    key = _residues(chain, (L, 2, L + 1, N), 6, dev)
    rot = fiona.Rotator(fiona.Ctx(N, L, chain[:L]), chain[L], n_rot)
    galois = [pow(5, 1 + r, 2 * N) for r in range(n_rot)]
    keys = torch.empty(n_rot, rot.key_words(), dtype=torch.int64, device=dev)   # one key under every element
    for r, g in enumerate(galois):
        fiona.rotation_key_layout(rot, g, key, keys[r])
    out = torch.full((n_rot, 2, L, N), -1, dtype=torch.int64, device=dev)
    fiona.hoisted_rotate(rot, ct, galois, keys, out)
    torch.cuda.synchronize()
    for r in (0, 66, 67, 131, 132, 196):   # vectors r and 197 + r
        assert np.array_equal(_np(out[r]), ro.rotate(_np(ct), galois[r], _np(key), chain[:L], chain[L])), \
            "rotation %d differs" % r
