"""Comparisons and argmax of many rows of small rings: more rows than a grid holds
(65535), with the bits of all items side by side, give the words of the same calls
in turn or in parts, and of the oracle."""
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
