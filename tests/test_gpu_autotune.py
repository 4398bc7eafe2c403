"""What the autotuner keeps: the choice for the chunks it timed.  Batches of other
sizes are chosen for by the library as before, and FHE_FUSED_AUTO restores its
choice altogether."""
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


def setup(n, bits, k):
    qs = bfv.ntt_primes(n, bits, k)
    ctx = fhe.Context(n, qs, 17, "coeff")
    km = inputs.key_material(n, qs, 3)
    _, rlk = ctx.keygen(km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
    a = fhe.from_numpy_u64(inputs.uniform_ciphertexts(n, qs, 64, 3, "a"), "cuda")
    b = fhe.from_numpy_u64(inputs.uniform_ciphertexts(n, qs, 64, 3, "b"), "cuda")
    return ctx, rlk, a, b


def fused(ctx, rlk, a, b, items):
    """Whether a batch of `items` takes the fused kernels."""
    ctx.set_timing(True)
    ctx.reset_kernel_stats()
    ctx.mul_relin(rlk, a[:items], b[:items])
    stats = ctx.kernel_stats()
    ctx.set_timing(False)
    n = stats["square_tensor" if a.data_ptr() == b.data_ptr() else "mul_tensor"][1]
    assert n in (0, 1)
    return n == 1


@pytest.mark.parametrize("square", [False, True])
@pytest.mark.parametrize("n,bits,k", [(4096, 36, 3), (16384, 55, 4)])
def test_other_sizes_keep_the_librarys_choice(n, bits, k, square):
    ctx, rlk, a, b = setup(n, bits, k)
    b = a if square else b
    print(f"[gpu-autotune] n={n} square={square}", flush=True)
    sizes = (1, 3, 29, 31, 60, 64)
    before = [fused(ctx, rlk, a, b, m) for m in sizes]
    chunk, kept = ctx.autotune_mul_relin(rlk, a[:2], b[:2])
    ctx.set_batch_limit(0)
    assert fused(ctx, rlk, a, b, chunk) == kept
    assert [fused(ctx, rlk, a, b, m) for m in sizes if m != chunk] == \
        [f for m, f in zip(sizes, before) if m != chunk]
    ctx.set_fused_threshold(square, 0)
    assert all(fused(ctx, rlk, a, b, m) for m in sizes)
    ctx.set_fused_threshold(square, fhe.FUSED_AUTO)
    assert [fused(ctx, rlk, a, b, m) for m in sizes] == before


def test_threshold_of_rings_without_split_transforms():
    """n = 1024: tuned on a large batch, smaller ones from 128 rows on stay fused as
    the library's threshold says, unless the unfused kernels were kept."""
    ctx, rlk, a, b = setup(1024, 36, 3)
    K = 3 + ctx.aux_primes
    m = -(-128 // K)
    assert not fused(ctx, rlk, a, b, m - 1) and fused(ctx, rlk, a, b, m)
    chunk, kept = ctx.autotune_mul_relin(rlk, a, b)
    ctx.set_batch_limit(0)
    assert fused(ctx, rlk, a, b, m) == (kept or m > chunk)
    ctx.set_fused_threshold(False, fhe.FUSED_AUTO)
    assert not fused(ctx, rlk, a, b, m - 1) and fused(ctx, rlk, a, b, m)
    assert fused(ctx, rlk, a, a, 1)
