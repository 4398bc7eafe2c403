"""Which kernels integer bases take, on both sides of the measured lines between split
and fused kernels (number of primes, fill of the last round, ring), and that the words
are the same on the other route."""
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


def setup(n, bits, k, t, items):
    qs = bfv.ntt_primes(n, bits, k)
    ctx = fhe.Context(n, qs, t, "coeff")
    km = inputs.key_material(n, qs, 3)
    _, rlk = ctx.keygen(km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    a = fhe.from_numpy_u64(inputs.uniform_ciphertexts(n, qs, items, 3, "a"), "cuda")
    b = fhe.from_numpy_u64(inputs.uniform_ciphertexts(n, qs, items, 3, "b"), "cuda")
    return ctx, rlk, a, b


def launches(ctx, call):
    ctx.set_timing(True)
    ctx.reset_kernel_stats()
    out = call()
    stats = {name: count for name, (_, count) in ctx.kernel_stats().items()}
    ctx.set_timing(False)
    return out, stats


@pytest.mark.parametrize("n,k,items,square,fused,relin_split", [
    (16384, 4, 16, False, False, True),   # few rows
    (16384, 4, 24, False, True, True),    # K = 9
    (16384, 4, 32, False, False, True),   # a round and an eighth
    (16384, 4, 56, False, True, False),
    (16384, 6, 32, True, True, False),    # K = 12
    (16384, 6, 48, False, False, True),
    (16384, 8, 24, True, False, True),    # K = 16
    (16384, 8, 32, True, True, False),
    (16384, 8, 32, False, False, False),
    (16384, 3, 32, True, False, True),    # at most four primes a side
    (8192, 5, 64, True, True, True),      # K = 11
    (8192, 5, 64, False, False, True),
    (8192, 8, 64, True, False, False),
    (4096, 5, 96, True, True, False),
    (4096, 5, 32, True, False, True),
    (8192, 10, 24, True, True, False),    # more than eight primes
    (8192, 10, 8, False, False, True),
])
def test_products(n, k, items, square, fused, relin_split):
    import torch
    print(f"[gpu-routes] n={n} k={k} items={items} square={square}", flush=True)
    ctx, rlk, a, b = setup(n, 55, k, 65537, items)
    y = a if square else b
    got, st = launches(ctx, lambda: ctx.mul_relin(rlk, a, y))
    assert (st["square_tensor" if square else "mul_tensor"] == 1) == fused, st
    assert (st["split_tensor"] == 1) == (not fused), st
    assert (st["split_relin"] == 1, st["relin_fused"] == 1) == (relin_split, not relin_split), st
    ctx.set_fused_threshold(square, 2 ** 64 - 1 if fused else 0)
    other, st = launches(ctx, lambda: ctx.mul_relin(rlk, a, y))
    assert (st["split_tensor"] == 1) == fused, st
    assert torch.equal(got, other)


@pytest.mark.parametrize("n,bits,k,count,split", [
    (8192, 43, 5, 4, True), (8192, 43, 5, 16, False), (8192, 43, 4, 16, True),
    (16384, 55, 6, 8, False), (16384, 55, 6, 4, True), (16384, 55, 8, 8, True), (4096, 55, 5, 32, True),
])
def test_powers(n, bits, k, count, split):
    import torch
    print(f"[gpu-routes] powers n={n} k={k} count={count}", flush=True)
    ctx, rlk, a, _ = setup(n, bits, k, 17, count)
    got, st = launches(ctx, lambda: ctx.bridge_to_bits_powers(rlk, a, 5))
    assert (st["split_tensor"] > 0) == split and (st["mul_tensor"] > 0) == (not split), st
    one, st = launches(ctx, lambda: torch.cat([ctx.bridge_to_bits_powers(rlk, a[j:j + 1], 5) for j in range(2)]))
    assert st["split_tensor"] > 0, st
    assert torch.equal(got[:2], one)
