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
    eight, whose products meet in one sum: a small prime per further digit, and the
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
