"""The split transforms (csrc/kernels_split.hip) at the primes nearest their bounds,
in batches on both sides of the step from one wave per block to shared twiddles
(3072 tensor blocks, 1536 of key switching), against the oracle word for word."""
import math

import numpy as np
import pytest

from oracle import bfv
from paper_2204_12201_amd import fhe, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fhe.lib()


def up(a):
    return fhe.from_numpy_u64(np.asarray(a, dtype=np.uint64), "cuda")


def primes(n, bits):
    """One prime per entry, distinct, the largest below each 2^bits."""
    out = []
    for b in bits:
        out.append(next(q for q in bfv.ntt_primes(n, b, len(bits) + 1) if q not in out))
    return out


def setup(n, qs, t):
    P = bfv.Params(n, qs, t, "coeff")
    km = inputs.key_material(n, qs, 5)
    _, rlk = bfv.keygen(P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    ctx = fhe.Context(n, qs, t, "coeff")
    return P, rlk, ctx, ctx.rlk_import(up(rlk))


def edge_cts(n, qs):
    """Every residue q - 1; (q - 1) / 2 and its successor alternating; uniform."""
    top = np.stack([np.full(n, q - 1, dtype=np.uint64) for q in qs])
    half = np.stack([np.where(np.arange(n) % 2, (q + 1) // 2, (q - 1) // 2).astype(np.uint64) for q in qs])
    rnd = inputs.uniform_ciphertexts(n, qs, 2, 3)
    return np.stack([np.stack([top, top]), np.stack([half, top]), rnd[0]]), \
        np.stack([np.stack([top, half]), rnd[1], rnd[1]])


@pytest.mark.parametrize("count", [3, 36])
def test_key_sums_of_eleven_digits(count):
    """Key switching in doubles modulo a prime next to 2^50 with more digits than
    eight, which one wave sums: a small prime per further digit, and the
    first squaring of the bridge, whose workspace holds the digits (t = 3: it is the
    only one)."""
    n, t = 4096, 3
    small = [i * 2 * n + 1 for i in range(1, 60)]
    small = [q for q in small if all(q % d for d in range(3, int(q ** 0.5) + 1, 2))]
    qs = primes(n, (50, 22)) + small[1:]
    k = len(qs)
    need = sum(map(math.log2, qs)) + math.log2(t) + math.log2(n) + 2
    assert k == 11 and 4 * 61 < need < 249  # five auxiliary primes, which may be below 2^50
    print(f"[gpu-split-edges] n={n} k={k} count={count}", flush=True)
    P, rlk, ctx, rlk_d = setup(n, qs, t)
    assert ctx.aux_primes == 5
    a, _ = edge_cts(n, qs)
    want = [bfv.bridge_to_bits(P, a[j], rlk, 2)[0] for j in range(3)]
    x = up(a).repeat(count // 3, 1, 1, 1)
    ctx.set_timing(True)
    got = fhe.to_numpy_u64(ctx.bridge_to_bits(rlk_d, x, 2))
    assert ctx.kernel_stats()["split_relin"][1] == 1
    for j in range(count):
        assert (got[j] == want[j % 3]).all(), j


# (n, bits of the primes of Q, t, items of the large batch)
SETS = [
    (4096, (47, 47, 47, 47, 45), 2, 80),    # doubles, the largest primes without extra reductions
    (4096, (49, 30), 17, 200),              # doubles, with them in Q and P
    (8192, (43,) * 5, 65537, 40),           # doubles, 50-bit auxiliary primes
    (16384, (50,), 17, 100),                # doubles, one prime next to 2^50
    (16384, (47, 47, 47, 47, 43), 2, 20),   # doubles, fourteen levels without extra reductions
    (16384, (55,) * 6, 65537, 17),          # integers: auxiliary primes too large for the lazy transforms
    (16384, (55,) * 7, 65537, 14),          # that Q takes, the digits straight from the scale
    (16384, (55,) * 8, 65537, 13),
]


@pytest.mark.parametrize("n,bits,t,many", SETS)
def test_few_and_many_blocks(n, bits, t, many):
    """Products and squares, in batches of three and of `many`, split and fused."""
    qs = primes(n, bits)
    k = len(qs)
    print(f"[gpu-split-edges] n={n} bits={bits}", flush=True)
    P, rlk, ctx, rlk_d = setup(n, qs, t)
    K, NB = k + ctx.aux_primes, n // 1024
    assert 3 * K * NB <= 3072 < many * K * NB and 3 * k * NB <= 1536 < many * k * NB
    a, b = edge_cts(n, qs)
    want_m = [bfv.mul_relin(P, a[j], b[j], rlk) for j in range(3)]
    want_s = [bfv.mul_relin(P, a[j], a[j], rlk) for j in range(3)]
    reps = (many + 2) // 3
    da, db = up(a), up(b)
    ba, bb = (x.repeat(reps, 1, 1, 1)[:many].contiguous() for x in (da, db))
    ctx.set_timing(True)
    for threshold in (2 ** 64 - 1, 0):  # never and always the fused kernels
        ctx.set_fused_threshold(False, threshold)
        ctx.set_fused_threshold(True, threshold)
        ctx.reset_kernel_stats()
        for x, y, want in ((da, db, want_m), (da, da, want_s), (ba, bb, want_m), (ba, ba, want_s)):
            got = fhe.to_numpy_u64(ctx.mul_relin(rlk_d, x, y))
            for j in range(got.shape[0]):
                assert (got[j] == want[j % 3]).all(), (threshold, x is y, got.shape[0], j)
        stats = ctx.kernel_stats()
        assert stats["split_tensor"][1] == (0 if threshold == 0 else 4), stats
        assert stats["split_relin"][1] == 4, stats
