"""Encryption and decryption through the pinned staging: pieces of its halves,
errors of more than 16 bits, plaintext moduli at and above 2^32, more items than a
grid holds.  Word for word against the oracle at the edges of the pieces, and the
plaintexts back for every item."""
import numpy as np
import pytest

from oracle import bfv
from paper_2204_12201_amd import fhe, inputs

pytestmark = pytest.mark.gpu

N = 64


@pytest.fixture(scope="module", autouse=True)
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fhe.lib()


# One staging half holds 2^20 plaintext words, 2^21 error words, 2^22 of u: at
# n = 64 that is 16384, 16384 and 65536 items; a grid holds 65535 items.
@pytest.mark.parametrize("bits", [(40, 40), (58, 58), (61, 61)])  # lazy transforms up to 2^58, then not
@pytest.mark.parametrize("t,count,big", [
    (65537, 1, False),
    (65537, 16384, True),
    (65537, 16385, False),
    (65537, 65541, True),
    (1 << 32, 33, False),
    ((1 << 32) + 15, 33, True),
])
def test_pieces(bits, t, count, big):
    print(f"[gpu-client] bits={bits} t={t} count={count}", flush=True)
    qs = bfv.ntt_primes(N, bits[0], 2)
    P = bfv.Params(N, qs, t, "coeff")
    km = inputs.key_material(N, qs, 5)
    pk, _ = bfv.keygen(P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    ctx = fhe.Context(N, qs, t, "coeff")
    rng = np.random.default_rng(count + t)
    pts = rng.integers(0, t, (count, N), dtype=np.uint64)
    pts[0, :2] = t - 1, 0
    u = rng.integers(-1, 2, (count, N), dtype=np.int8)
    e = rng.integers(-19, 20, (count, 2, N), dtype=np.int32)
    e[-1, 1, -2:] = -32768, 32767
    if big:
        e[0, 0, :2] = -32769, 70000
    ct = ctx.encrypt(fhe.from_numpy_u64(pk, "cuda"), pts, u, e)
    back = ctx.decrypt(km["s"], ct)
    assert np.array_equal(back, pts)
    got = ct.cpu().numpy().view(np.uint64)
    for j in sorted({0, count // 2, count - 1, *(i for i in (16383, 16384, 65534, 65535, 65536) if i < count)}):
        assert np.array_equal(got[j], bfv.encrypt(P, pk, pts[j], u[j], e[j])), j
    bad = pts.copy()
    bad[-1, -1] = t
    with pytest.raises(fhe.FheError):
        ctx.encrypt(fhe.from_numpy_u64(pk, "cuda"), bad, u, e)
