// Every launch of the split transforms must report its error.  The launch functions
// of the runtime are replaced here, ahead of the library's: nothing reaches a device,
// and of the launches of a call the one that `fail_at` names fails.  Their shapes tell
// which kernel sums the keys: one wave an item where several could overflow a double.
#include "kernels.hpp"

#include <cstdio>

static hipError_t last = hipSuccess;
static int launches = 0, fail_at = 0;
static unsigned first_block = 0;  // threads of a workgroup of a call's first launch

extern "C" {
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
    if (launches++ != fail_at) return hipSuccess;
    return last = hipErrorInvalidConfiguration;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t __hipPushCallConfiguration(dim3, dim3 block, size_t, hipStream_t) {
    if (launches == 0) first_block = block.x;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
}

int main() {
    int bad = 0;
    for (int L = 12; L <= 14; L++)
        for (int kind = 0; kind < 4; kind++) {  // doubles, lazy integers with raw digits and without, mixed
            const SplitOps &o = *split_ops(L);
            DevCtx c = {};
            c.n = 1 << L;
            c.L = L;
            c.k = 2;
            c.kp = 3;
            c.K = 5;
            c.f64 = kind == 0;
            c.lazy_all = kind == 1 || kind == 2;
            c.digit_raw = kind == 1;
            uint64_t *p = nullptr;
            auto report = [&](const char *what, auto call) {
                int count = 1;
                for (fail_at = 0; fail_at < count; fail_at++) {
                    launches = 0;
                    const hipError_t e = call();
                    count = launches;
                    last = hipSuccess;
                    if (launches == 0 || e == hipSuccess) {
                        printf("no error: %s L=%d kind=%d, launch %d of %d failed\n", what, L, kind, fail_at, count);
                        bad++;
                    }
                }
            };
            report("lift_fwd", [&] { return o.lift_fwd(c, p, p, p, 2, 1, nullptr); });
            report("fwd", [&] { return o.fwd(c, p, p, p, p, 2, 1, nullptr); });
            report("fwd_blocks", [&] { return o.fwd_blocks(c, p, 1, nullptr); });
            report("inv", [&] { return o.inv(c, p, 1, nullptr); });
            for (size_t items : {1, 1000}) {
                report("blocks", [&] { return o.blocks(c, p, p, items == 1, items, nullptr); });
                report("pre2", [&] { return o.pre2(c, p, 1, 0, p, p, items, nullptr); });
                report("inv_scale", [&] { return o.inv_scale(c, p, p, p, items == 1 ? p : nullptr, items, nullptr); });
                report("digits", [&] { return o.digits(c, p, p, items, nullptr); });
                report("relin", [&] { return o.relin(c, p, p, p, p, items, nullptr); });
            }
        }
    for (int L = 12; L <= 14; L++)
        for (int k = 1; k <= 16; k++)
            for (int big = 0; big < 3; big++) {  // no prime of 2^47 or more, one in Q, one in P
                DevCtx c = {};
                c.n = 1 << L;
                c.L = L;
                c.k = k;
                c.kp = k;
                c.K = 2 * k;
                c.f64 = 1;
                c.big_limbs = big ? 1ull << (big == 1 ? k - 1 : k) : 0;
                launches = 0;
                fail_at = -1;
                split_ops(L)->relin(c, nullptr, nullptr, nullptr, nullptr, 1, nullptr);
                const unsigned waves = k > 8 ? (big == 1 ? 1 : 8) : k < 2 ? 2 : k;
                if (first_block != 64 * waves) {
                    printf("key sums of %d digits: %u threads, L=%d big=%d\n", k, first_block, L, big);
                    bad++;
                }
            }
    if (bad) return 1;
    printf("ok\n");
    return 0;
}
