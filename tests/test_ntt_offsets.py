"""Host replay of every memory access of the NTT kernels (no device).

fiona_check_ntt_offsets lays a rescaler or rotator out at fake device
addresses, records one call's launches instead of issuing them, and
recomputes every global access of every workgroup and thread of the NTT passes
and of the whole transforms with the kernels' own offset helpers.  Each access
must fall inside the buffer that holds its descriptor's base (the twiddle
tables each on their own), offsets must stay below 2^32 bytes, and every
descriptor's end must be its buffer's end.  The whole transforms' LDS words are
recomputed too: every step must touch each word of the vector once; and their
workgroups must write each output vector once.  The inner product and the
transpose are checked by the byte ranges they touch.  Every fake buffer starts
with bit 31 of its low address half set, and the replay rebuilds each
descriptor base from its two halves as the kernels do (a signed low half would
spill into the high half).

The shapes are those of the GPU tests and of bench.py: rings 2^8 .. 2^17 (whole
transforms up to 2^14, passes from 2^13 on), L up to 16, one and several groups
of limbs, the shared input order of pass A, the transposed outputs, c0 in
natural order and transposed, one and several chunks, 1 .. 256 rotations.
"""
import os

import pytest

import synth
import paper_2609_35352_amd as fiona

pytestmark = pytest.mark.skipif(not os.path.exists(fiona.LIB_PATH), reason="libfiona.so not built")

RESCALE = [  # N, L, max_ct, n_ct
    # whole transforms: one limb and all limbs a workgroup, and some; each ring
    (256, 2, 3, 2), (1 << 12, 3, 4, 3), (1 << 13, 5, 3, 2), (1 << 11, 4, 2, 1), (512, 4, 40, 40), (1024, 7, 3, 3),
    (256, 5, 16384, 3), (256, 5, 10000, 3), (256, 3, 32767, 32767), (1 << 12, 3, 1, 1), (1 << 12, 6, 33, 33),
    (1 << 14, 3, 40, 40), (1 << 14, 6, 128, 128),
    # passes
    (1 << 14, 3, 40, 39), (1 << 14, 2, 1, 1), (1 << 15, 3, 31, 30), (1 << 15, 6, 3, 3), (1 << 17, 2, 2, 1),
    (1 << 16, 8, 4, 4), (1 << 16, 16, 4, 4), (1 << 16, 8, 128, 5),
    (1 << 16, 8, 128, 128), (1 << 16, 10, 24, 24), (1 << 16, 12, 96, 96), (1 << 16, 16, 128, 128), (1 << 15, 3, 243, 243),
]
ROTATE = [  # N, L, max_rot, n_rot
    # digits and division by whole transforms
    (256, 1, 2, 2), (512, 3, 5, 5), (1024, 3, 3, 3), (1 << 12, 4, 4, 4), (2048, 10, 1, 1),
    (256, 2, 256, 256), (256, 2, 70, 70), (256, 2, 1, 1), (2048, 2, 1, 1),
    (1 << 13, 2, 64, 64),   # the division only
    # passes, c0 in natural order
    (1 << 13, 4, 7, 7), (1 << 14, 4, 9, 8), (1 << 15, 2, 3, 3), (1 << 16, 4, 1, 1),
    # and transposed
    (1 << 13, 2, 63, 63), (1 << 14, 4, 9, 9), (1 << 17, 2, 2, 2),
    (1 << 16, 8, 63, 63), (1 << 16, 10, 23, 23), (1 << 16, 10, 3, 3), (1 << 16, 12, 31, 31),
    (1 << 16, 16, 127, 127), (1 << 16, 16, 4, 4), (1 << 15, 8, 197, 197),
]


@pytest.mark.parametrize("N,L,max_ct,n_ct", RESCALE)
def test_rescale_accesses_in_bounds(N, L, max_ct, n_ct):
    rc, msg = fiona.check_ntt_offsets("rescale", N, L, synth.ntt_primes(N, L), max_ct, n_ct)
    assert rc == 0, msg


@pytest.mark.parametrize("N,L,max_rot,n_rot", ROTATE)
def test_rotate_accesses_in_bounds(N, L, max_rot, n_rot):
    rc, msg = fiona.check_ntt_offsets("rotate", N, L, synth.ntt_primes(N, L + 1), max_rot, n_rot)
    assert rc == 0, msg


@pytest.mark.parametrize("L", [1, 8, 16, 31, 32, 48, 63])
@pytest.mark.parametrize("n_rot", [1, 33, 63, 64, 127, 256])
def test_inner_product_lds_within_limit(L, n_rot):
    """The LDS of the rotations' inner product depends on the call's number of
    rotations (rounds of equal size, as few as fit): from L = 32 on fewer than 64
    rotations fit one round, and 63 then take more than half of 64."""
    rc, msg = fiona.check_ntt_offsets("rotate", 256, L, synth.ntt_primes(256, L + 1), 256, n_rot)
    assert rc == 0, msg


@pytest.mark.parametrize("op,N,L,cap,n", [("rescale", 256, 2, 3, 2), ("rescale", 1 << 16, 8, 128, 128),
                                           ("rotate", 256, 2, 2, 2), ("rotate", 1 << 16, 8, 63, 63)])
def test_replay_finds_an_overrun(op, N, L, cap, n):
    """The output buffer taken one word short: the replay reports the store
    that reaches past it (the last word of the output is written)."""
    mods = synth.ntt_primes(N, L if op == "rescale" else L + 1)
    rc, msg = fiona.check_ntt_offsets(op, N, L, mods, cap, n, out_shrink=8)
    assert rc == fiona.FIONA_ERR_BOUNDS and "out_cts" in msg and "bytes up to" in msg, msg
    if N == 256:   # whole transforms: found at the workgroup whose store it is, not as a range of the call
        assert "vector %d, modulus %d: output" % (2 * n - 1, L - (2 if op == "rescale" else 1)) in msg, msg


def test_replay_parameter_errors():
    q = synth.ntt_primes(256, 3)
    assert fiona.check_ntt_offsets("rescale", 256, 2, q, 2, 3)[0] == -1            # n_ct > max_ct
    assert fiona.check_ntt_offsets("rescale", 384, 2, q, 2, 1)[0] == -3            # N not a power of two
    assert fiona.check_ntt_offsets("rotate", 256, 2, q, 300, 1)[0] == -3           # max_rot > 256
