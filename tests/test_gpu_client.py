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


@pytest.mark.parametrize("t,count", [(65537, 1), (65537, 37), ((1 << 32) + 15, 37)])
def test_workspace_is_used_and_held_to(t, count):
    """The workspaces hold the rows that the calls keep (key and u, or s and c0 + c1 s)
    and the client's words, nothing else, and nothing beyond them is written."""
    import ctypes
    import torch
    qs = bfv.ntt_primes(N, 40, 2)
    k = len(qs)
    P = bfv.Params(N, qs, t, "coeff")
    km = inputs.key_material(N, qs, 5)
    pk, _ = bfv.keygen(P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    ctx = fhe.Context(N, qs, t, "coeff")
    L = fhe.lib()
    rows = 8 * N
    enc, dec = (L.fhe_workspace_bytes(ctx._h, op, count) for op in (fhe.OP_ENCRYPT, fhe.OP_DECRYPT))
    assert enc <= rows * (2 * k + count * k + count) + 9 * N * count + 256
    assert dec <= rows * (k + count * k + count) + N + 256
    rng = np.random.default_rng(count)
    pts = rng.integers(0, t, (count, N), dtype=np.uint64)
    u = rng.integers(-1, 2, (count, N), dtype=np.int8)
    e = rng.integers(-19, 20, (count, 2, N), dtype=np.int32)
    pk_d = fhe.from_numpy_u64(pk, "cuda")
    ct = torch.empty((count, 2, k, N), dtype=torch.int64, device="cuda")
    back = np.empty_like(pts)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    guard = 4096
    ws = torch.full((enc + guard,), 77, dtype=torch.uint8, device="cuda")
    cast = lambda a, f, i: ctypes.cast(ptr(a), f.argtypes[i])  # noqa: E731
    f = L.fhe_encrypt
    assert f(ctx._h, pk_d.data_ptr(), cast(pts, f, 2), cast(u, f, 3), cast(e, f, 4), ct.data_ptr(), count,
             ws.data_ptr(), enc, stream) == 0
    assert (ws[enc:] == 77).all()
    ws = torch.full((dec + guard,), 77, dtype=torch.uint8, device="cuda")
    f = L.fhe_decrypt
    s = np.ascontiguousarray(km["s"], dtype=np.int8)
    assert f(ctx._h, cast(s, f, 1), ct.data_ptr(), cast(back, f, 3), count, ws.data_ptr(), dec, stream) == 0
    assert (ws[dec:] == 77).all()
    assert np.array_equal(back, pts)
    got = ct.cpu().numpy().view(np.uint64)
    for j in {0, count - 1}:
        assert np.array_equal(got[j], bfv.encrypt(P, pk, pts[j], u[j], e[j])), j
    assert f(ctx._h, cast(s, f, 1), ct.data_ptr(), cast(back, f, 3), count, ws.data_ptr(), dec - 1, stream) == -8
