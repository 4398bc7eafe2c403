"""The split transforms of the product pipeline (csrc/kernels_split.hip) against
the oracle, word for word: integer and floating-point fields, primes on both
sides of their bounds, residues at the ends of their range, batches small
enough for one wave per block and large enough for the shared-twiddle kernels,
products and squares."""
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


# (n, bits of the primes of Q, t, items of the large batch): the field they run
SETS = [
    (4096, (36, 36, 36), 65537, 90),    # floating point, all primes below 2^47
    (4096, (49, 30), 17, 90),           # floating point, 49-bit primes in Q and P, uneven digits
    (4096, (55, 40), 17, 130),          # integers, digits above four times the smallest prime
    (4096, (30,) * 10, 17, 30),         # key switching scratch does not fit: fused kernel
    (8192, (43,) * 5, 65537, 30),       # floating point, 50-bit auxiliary primes
    (8192, (55, 55, 55), 17, 50),       # integers, lazy
    (16384, (29,), 17, 30),             # floating point, one prime, 50-bit auxiliary prime
    (16384, (38, 38, 38), 17, 12),      # floating point, fourteen levels
    (16384, (60, 60), 17, 12),          # integers, primes too large for the lazy transforms
]


@pytest.mark.parametrize("n,bits,t,many", SETS)
def test_products_and_squares(n, bits, t, many):
    qs = primes(n, bits)
    k = len(qs)
    print(f"[gpu-split] n={n} bits={bits}", flush=True)
    P = bfv.Params(n, qs, t, "coeff")
    km = inputs.key_material(n, qs, 5)
    _, rlk = bfv.keygen(P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    ctx = fhe.Context(n, qs, t, "coeff")
    rlk_d = ctx.rlk_import(up(rlk))
    # every residue q - 1; (q - 1) / 2 and its successor alternating; uniform
    top = np.stack([np.full(n, q - 1, dtype=np.uint64) for q in qs])
    half = np.stack([np.where(np.arange(n) % 2, (q + 1) // 2, (q - 1) // 2).astype(np.uint64) for q in qs])
    rnd = inputs.uniform_ciphertexts(n, qs, 2, 3)
    a = np.stack([np.stack([top, top]), np.stack([half, top]), rnd[0]])
    b = np.stack([np.stack([top, half]), rnd[1], rnd[1]])
    want_m = [bfv.mul_relin(P, a[j], b[j], rlk) for j in range(3)]
    want_s = [bfv.mul_relin(P, a[j], a[j], rlk) for j in range(3)]
    da, db = up(a), up(b)
    reps = (many + 2) // 3
    ba, bb = da.repeat(reps, 1, 1, 1), db.repeat(reps, 1, 1, 1)
    for fused in (False, True):  # the fused kernels give the same words
        if fused:
            ctx.set_fused_threshold(False, 0)
            ctx.set_fused_threshold(True, 0)
        for got, want in ((ctx.mul_relin(rlk_d, da, db), want_m), (ctx.mul_relin(rlk_d, da, da), want_s),
                          (ctx.mul_relin(rlk_d, ba, bb), want_m), (ctx.mul_relin(rlk_d, ba, ba), want_s)):
            g = fhe.to_numpy_u64(got)
            for j in range(g.shape[0]):
                assert (g[j] == want[j % 3]).all(), (fused, g.shape[0], j)


@pytest.mark.parametrize("n,bits,ncls,count,nbits", [(256, (55, 55), 4, 2, 3), (4096, (36, 36, 36), 3, 5, 2),
                                                     (256, (40, 40, 40), 2, 3, 1), (256, (30,), 5, 1, 4)])
def test_comparisons_batched_or_in_turn(n, bits, ncls, count, nbits):
    """fhe_argmax and fhe_less_than give the same words with the bits and pairs
    side by side as one after the other (a workspace that only holds that), and
    with room for some of the pairs; sampled items equal the oracle."""
    import ctypes
    import torch
    qs = primes(n, bits)
    k = len(qs)
    print(f"[gpu-split] argmax n={n} ncls={ncls} count={count} nbits={nbits}", flush=True)
    P = bfv.Params(n, qs, 17, "coeff")
    km = inputs.key_material(n, qs, 6)
    _, rlk = bfv.keygen(P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    ctx = fhe.Context(n, qs, 17, "coeff")
    rlk_d = ctx.rlk_import(up(rlk))
    sc = inputs.uniform_ciphertexts(n, qs, ncls * count * nbits, 8).reshape(ncls, count, nbits, 2, k, n)
    d = up(sc)
    L = fhe.lib()
    ctb = 2 * k * n * 8
    mul = L.fhe_workspace_bytes(ctx._h, fhe.OP_MUL_RELIN, count)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def argmax(bytes_):
        ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        out = torch.empty((ncls, count, 2, k, n), dtype=torch.int64, device="cuda")
        st = L.fhe_argmax(ctx._h, rlk_d.data_ptr(), d.data_ptr(), ncls, nbits, out.data_ptr(), count, ws.data_ptr(),
                          bytes_, stream)
        return st, fhe.to_numpy_u64(out)

    whole = fhe.to_numpy_u64(ctx.argmax(rlk_d, d))
    in_turn = 8 * count * ctb + mul  # the least that was ever asked for
    need = L.fhe_workspace_bytes(ctx._h, fhe.OP_ARGMAX, count)
    assert in_turn <= need
    for b in (in_turn, (in_turn + need) // 2 // 256 * 256, need, 4 * need):
        st, got = argmax(b)
        assert st == 0 and (got == whole).all(), b
    assert argmax(in_turn - 256)[0] == -8
    lt = fhe.to_numpy_u64(ctx.less_than(rlk_d, d[0].contiguous(), d[1].contiguous()))
    for j in {0, count - 1}:
        assert (lt[j] == bfv.less_than(P, rlk, list(sc[0, j]), list(sc[1, j]))).all(), j
        want = bfv.argmax(P, rlk, [list(sc[c, j]) for c in range(ncls)])
        for c in range(ncls):
            assert (whole[c, j] == want[c]).all(), (j, c)
