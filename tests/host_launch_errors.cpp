// Every launch of the split transforms must report its error.  The launch functions
// of the runtime are replaced here, ahead of the library's: nothing reaches a device,
// and of the launches of a call the one that `fail_at` names fails.
#include "kernels.hpp"

#include <cstdio>

static hipError_t last = hipSuccess;
static int launches = 0, fail_at = 0;

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
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
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
    if (bad) return 1;
    printf("ok\n");
    return 0;
}
