"""Comparisons and argmax of many rows of small rings: more rows than a grid holds
(65535), with the bits of all items side by side, give the words of the same calls
in turn or in parts, and of the oracle; the workspace sizes ask for more than one
comparison at a time needs only where the call uses it."""
import ctypes

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


class Setup:
    def __init__(self, n, qs, t=17):
        self.n, self.qs, self.k = n, qs, len(qs)
        self.P = bfv.Params(n, qs, t, "coeff")
        km = inputs.key_material(n, qs, 6)
        _, self.rlk = bfv.keygen(self.P, km["s"], km["pk_a"], km["pk_e"], km["rlk_a"], km["rlk_e"])
        self.ctx = fhe.Context(n, qs, t, "coeff")
        self.rlk_d = self.ctx.rlk_import(up(self.rlk))
        self.ctb = 2 * self.k * n * 8

    def bytes(self, op, count):
        return fhe.lib().fhe_workspace_bytes(self.ctx._h, op, count)

    def argmax(self, d, nbytes):
        import torch
        ncls, count, nbits = d.shape[:3]
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = torch.empty((ncls, count, 2, self.k, self.n), dtype=torch.int64, device="cuda")
        self.ctx.set_timing(True)
        self.ctx.reset_kernel_stats()
        st = fhe.lib().fhe_argmax(self.ctx._h, self.rlk_d.data_ptr(), d.data_ptr(), ncls, nbits, out.data_ptr(), count,
                                  ws.data_ptr(), nbytes, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        steps = self.ctx.kernel_stats()["elementwise"][1]
        self.ctx.set_timing(False)
        return out, steps

    def less_than(self, a, b, nbytes):
        import torch
        count, nbits = a.shape[:2]
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = torch.empty((count, 2, self.k, self.n), dtype=torch.int64, device="cuda")
        self.ctx.set_timing(True)
        self.ctx.reset_kernel_stats()
        st = fhe.lib().fhe_less_than(self.ctx._h, self.rlk_d.data_ptr(), a.data_ptr(), b.data_ptr(), nbits,
                                     out.data_ptr(), count, ws.data_ptr(), nbytes,
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        steps = self.ctx.kernel_stats()["elementwise"][1]
        self.ctx.set_timing(False)
        return out, steps


def test_more_factor_rows_than_a_grid():
    import torch
    n, ncls, count, nbits = 64, 5, 14000, 2  # 70000 rows of factors
    s = Setup(n, bfv.ntt_primes(n, 40, 1))
    print(f"[gpu-comparisons] argmax n={n} ncls={ncls} count={count}", flush=True)
    sc = inputs.uniform_ciphertexts(n, s.qs, ncls * count * nbits, 8).reshape(ncls, count, nbits, 2, s.k, n)
    d = up(sc)
    in_turn, steps = s.argmax(d, 8 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, count))
    room = 15 * count * s.ctb + 12 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, ncls * count)
    got, grouped = s.argmax(d, room)
    assert grouped == 10 * nbits + ncls - 1 < steps  # one pair at a time, then the factors
    assert torch.equal(got, in_turn)
    for j in (0, 9534, 9535, count - 1):  # row 65535 is item 9535 of the last class
        want = bfv.argmax(s.P, s.rlk, [list(sc[c, j]) for c in range(ncls)])
        for c in range(ncls):
            assert (fhe.to_numpy_u64(got[c, j]) == want[c]).all(), (j, c)


def test_more_comparison_rows_than_a_grid():
    import torch
    n, count, nbits = 16, 65536, 2
    s = Setup(n, bfv.ntt_primes(n, 40, 1))
    print(f"[gpu-comparisons] less_than n={n} count={count}", flush=True)
    ab = inputs.uniform_ciphertexts(n, s.qs, 2 * count * nbits, 8).reshape(2, count, nbits, 2, s.k, n)
    a, b = up(ab[0]), up(ab[1])
    room = 6 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, 2 * count)
    got, grouped = s.less_than(a, b, room)
    assert grouped == nbits  # one step a bit: side by side
    h = count // 2
    halves = [s.less_than(a[i:i + h], b[i:i + h], room)[0] for i in (0, h)]
    assert torch.equal(got, torch.cat(halves))
    for j in (0, 65534, 65535):
        want = bfv.less_than(s.P, s.rlk, list(ab[0, j]), list(ab[1, j]))
        assert (fhe.to_numpy_u64(got[j]) == want).all(), j


@pytest.mark.parametrize("n,bits", [(256, (40,)), (256, (40,) * 3), (4096, (36,) * 3)])
def test_room_only_where_it_is_used(n, bits):
    """Argmax of three classes of two bits, items on both sides of every step of the
    size: side by side in the default workspace where that is larger than one
    comparison at a time needs, and the sequential size elsewhere."""
    s = Setup(n, bfv.ntt_primes(n, bits[0], len(bits)))
    most = (128 << 14) // n  # bit products that share a batch
    print(f"[gpu-comparisons] sizes n={n} k={s.k}", flush=True)
    for count in (1, 3, most // 6, most // 6 + 1, most // 4, most // 4 + 1, most // 2, most // 2 + 1, most):
        seq = 8 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, count)
        need = s.bytes(fhe.OP_ARGMAX, count)
        side = 2 * count <= most
        assert (need > seq) == side, (count, need, seq)
        assert s.bytes(fhe.OP_COMPARE, count) >= seq - 2 * count * s.ctb
        if not side:
            assert s.bytes(fhe.OP_COMPARE, count) == seq - 2 * count * s.ctb
        if need > 1 << 33:
            continue
        sc = fhe.from_numpy_u64(np.zeros((3, count, 2, 2, s.k, n), dtype=np.uint64), "cuda")
        steps = s.argmax(sc, need)[1]
        groups = -(-3 // min(3, max(1, most // (2 * count))))
        assert steps == groups * 2 + 2 if side else steps > 8, (count, steps)
        if side:  # four classes
            sc = fhe.from_numpy_u64(np.zeros((4, count, 2, 2, s.k, n), dtype=np.uint64), "cuda")
            assert s.argmax(sc, need)[1] < 24, count


def test_factors_in_parts():
    """Four classes where the workspace holds the factors' products of two at a time."""
    import torch
    n, ncls, count, nbits = 256, 4, 4000, 2
    s = Setup(n, bfv.ntt_primes(n, 40, 3))
    print(f"[gpu-comparisons] argmax n={n} ncls={ncls} count={count}", flush=True)
    sc = inputs.uniform_ciphertexts(n, s.qs, ncls * count * nbits, 9).reshape(ncls, count, nbits, 2, s.k, n)
    d = up(sc)
    need = s.bytes(fhe.OP_ARGMAX, count)
    assert need < 10 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, 3 * count)
    got, steps = s.argmax(d, need)
    assert steps == 6 * nbits + 3
    in_turn, _ = s.argmax(d, 8 * count * s.ctb + s.bytes(fhe.OP_MUL_RELIN, count))
    assert torch.equal(got, in_turn)
    want = bfv.argmax(s.P, s.rlk, [list(sc[c, 1]) for c in range(ncls)])
    for c in range(ncls):
        assert (fhe.to_numpy_u64(got[c, 1]) == want[c]).all(), c


def test_sizes_of_many_items():
    """At the largest ring: thousands of items need what one comparison at a time
    needs (3000: 59 GB, where room for groups that never run would take 222)."""
    s = Setup(16384, inputs.PRIMES[(16384, 55)])
    for count in (65, 256, 1000, 3000):
        mul = s.bytes(fhe.OP_MUL_RELIN, count)
        assert s.bytes(fhe.OP_ARGMAX, count) == 8 * count * s.ctb + mul
        assert s.bytes(fhe.OP_COMPARE, count) == 6 * count * s.ctb + mul
    assert s.bytes(fhe.OP_ARGMAX, 32) < 4 << 30
