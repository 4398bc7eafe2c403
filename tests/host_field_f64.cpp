// Host build of the floating-point field of the split transforms
// (csrc/ntt_field.hpp): its own passes, reductions, products and key sums, run
// thread by thread on the CPU, against the same transforms modulo p in integers.
// Values are congruent representatives pushed to the ends of the ranges that the
// header states, so that a sum leaving the doubles' 53 bits changes a residue.
//
//   host_field_f64 p...     the largest primes of both classes, 1 mod 2^15
//
// Prints "ok <count>" or the first failure.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

// every device function of the headers below also for the host
#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)(x))
#define __longlong_as_double bits_to_double
#define __double_as_longlong double_to_bits
inline double bits_to_double(long long v) {
    double d;
    memcpy(&d, &v, 8);
    return d;
}
inline long long double_to_bits(double d) {
    long long v;
    memcpy(&v, &d, 8);
    return v;
}
#include "ntt_field.hpp"

static uint64_t seed = 1;
static uint64_t rnd() {
    uint64_t z = (seed += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static uint64_t mulm(uint64_t a, uint64_t b, uint64_t p) { return (uint64_t)((u128)a * b % p); }
static uint64_t powm(uint64_t a, uint64_t e, uint64_t p) {
    uint64_t r = 1;
    for (; e; e >>= 1, a = mulm(a, a, p))
        if (e & 1) r = mulm(r, a, p);
    return r;
}
static uint64_t residue(double x, uint64_t p) {
    const int64_t v = (int64_t)x % (int64_t)p;
    return (uint64_t)(v < 0 ? v + (int64_t)p : v);
}
static TwF centred(uint64_t w, uint64_t p) {
    const double v = w > p / 2 ? -(double)(p - w) : (double)w, pinv = 1.0 / (double)p, e = v * pinv;
    return TwF{v, std::fma(std::fma(-e, (double)p, v), pinv, e)};
}

static const double LIMIT = 9007199254740992.0;  // 2^53
static int fails = 0;
static long checks = 0;
static void expect(bool ok, const char *what, int L, uint64_t p, int where) {
    checks++;
    if (!ok && fails++ < 8) printf("fail %s L=%d p=%llu at %d\n", what, L, (unsigned long long)p, where);
}

template <int L, bool BIG>
struct Check {
    typedef FieldF<BIG> F;
    typedef std::vector<double> Row;
    typedef std::vector<uint64_t> Ints;
    static constexpr int n = 1 << L, T = n / 16, NPASS = Geo<L>::NPASS;
    uint64_t p, ninv;
    Ints w, iw;
    std::vector<TwF> tw, itw;
    PrimeConst pc;
    DevCtx c;

    explicit Check(uint64_t p_) : p(p_), w(n), iw(n), tw(n), itw(n), pc(), c() {
        uint64_t psi = 0;
        for (uint64_t x = 2; !psi; x++) {
            const uint64_t v = powm(x, (p - 1) / (2 * n), p);
            if (powm(v, n, p) == p - 1) psi = v;
        }
        const uint64_t ipsi = powm(psi, p - 2, p);
        uint64_t a = 1, b = 1;
        for (int i = 0; i < n; i++, a = mulm(a, psi, p), b = mulm(b, ipsi, p)) {
            int r = 0;
            for (int j = 0; j < L; j++) r |= ((i >> j) & 1) << (L - 1 - j);
            w[r] = a;
            iw[r] = b;
        }
        for (int i = 0; i < n; i++) {
            tw[i] = centred(w[i], p);
            itw[i] = centred(iw[i], p);
        }
        ninv = powm(n, p - 2, p);
        pc.pf = (double)p;
        pc.pinvf = 1.0 / (double)p;
        pc.ninvf = centred(ninv, p).w;
        pc.ninvf_i = centred(ninv, p).wi;
        c.n = n;
        c.L = L;
        c.pc = &pc;
        c.twf = tw.data();
        c.itwf = itw.data();
    }

    // The transforms of the kernels' pass structure, one thread after the other
    template <int P, class Fn>
    void pass(Row &x, const Fn &fn) const {
        constexpr int R = 1 << Geo<L>::R(P), G = 16 / R;
        for (int t = 0; t < T; t++) {
            double v[1][16];
            for (int g = 0; g < G; g++)
                for (int e = 0; e < R; e++) v[0][g * R + e] = x[elem_index<L, 4, P>(t, g, e)];
            fn(v, t);
            for (int g = 0; g < G; g++)
                for (int e = 0; e < R; e++) x[elem_index<L, 4, P>(t, g, e)] = v[0][g * R + e];
        }
    }
    template <int P>
    void fwd_from(Row &x, const F &f) const {
        pass<P>(x, [&](double(&v)[1][16], int t) {
            if (P == 1) f.enter_block(v);
            if (P == 3) f.mid_block(v);
            fwd_pass_t<L, P, 1>(v, t, f, TwGlobal<TwF>{f.tw});
        });
        if constexpr (P + 1 < NPASS) fwd_from<P + 1>(x, f);
    }
    template <int P>
    void inv_from(Row &x, const F &f) const {
        pass<P>(x, [&](double(&v)[1][16], int t) { inv_pass_t<L, P, 1>(v, t, f, TwGlobal<TwF>{f.itw}); });
        if constexpr (P > 0) inv_from<P - 1>(x, f);
    }
    void operands(Row &x, const F &f) const {
        for (int i = 0; i < n; i += 16) {
            double v[1][16];
            for (int s = 0; s < 16; s++) v[0][s] = x[i + s];
            f.operands(v);
            for (int s = 0; s < 16; s++) x[i + s] = v[0][s];
        }
    }
    void ref(Ints &x, bool inverse) const {
        for (int l = inverse ? L - 1 : 0; inverse ? l >= 0 : l < L; l += inverse ? -1 : 1) {
            const int half = n >> (l + 1);
            for (int i = 0; i < n; i++) {
                if (i & half) continue;
                const uint64_t W = (inverse ? iw : w)[(1 << l) + (i >> (L - l))], a = x[i];
                const uint64_t b = inverse ? x[i + half] : mulm(x[i + half], W, p);
                x[i] = (a + b) % p;
                x[i + half] = inverse ? mulm((a + p - b) % p, W, p) : (a + p - b) % p;
            }
        }
    }
    void same(const Row &x, const Ints &r, const char *what) const {
        for (int i = 0; i < n; i++) expect(residue(x[i], p) == r[i], what, L, p, i);
    }
    // Congruent to r, as close to +-top as multiples of p bring it: sign 0 mixed
    double push(uint64_t r, double top, int sign) const {
        const double pf = (double)p;
        double v = (double)r;
        const double m = std::floor((top - v) / pf);
        const double hi = v + m * pf, lo = v - std::floor((top + v) / pf) * pf;
        return sign > 0 ? hi : sign < 0 ? lo : (rnd() & 1 ? hi : lo);
    }

    // Products of worst representatives: |operand| up to `b` (units of p), each
    // within the stated bound of a product, and their inverse transform.
    void tensor(double b, double prod) const {
        const F f(c, 0);
        for (int kind = 0; kind < 4; kind++) {
            Row x[2], z(n);
            Ints r[2], want(n);
            for (int m = 0; m < 2; m++) {
                r[m].resize(n);
                x[m].resize(n);
                for (int i = 0; i < n; i++) {
                    r[m][i] = kind == 0 ? p - 1 : kind == 1 ? (i & 1 ? p - 1 : 0) : rnd() % p;
                    x[m][i] = f.in(r[m][i]);
                }
                fwd_from<0>(x[m], f);
                ref(r[m], false);
                same(x[m], r[m], "forward");
                double most = 0;
                for (double v : x[m]) most = std::fmax(most, std::fabs(v));
                expect(most <= (BIG ? 7.6 : 9.1) * (double)p, "forward bound", L, p, kind);
                operands(x[m], f);
                same(x[m], r[m], "operands");
                for (int i = 0; i < n; i++) {
                    expect(std::fabs(x[m][i]) <= b * (double)p + 2.0, "operand bound", L, p, i);
                    if (kind) x[m][i] = push(r[m][i], b * (double)p, kind == 3 ? 1 : 0);
                }
            }
            for (int i = 0; i < n; i++) {
                z[i] = f.mul(x[0][i], x[1][i]);
                want[i] = mulm(r[0][i], r[1][i], p);
                expect(std::fabs(z[i]) <= prod * (double)p, "product bound", L, p, i);
            }
            same(z, want, "product");
            for (int sign = -1; sign <= 1; sign++) {
                Row y = z;
                Ints out = want;
                if (kind)
                    for (int i = 0; i < n; i++) y[i] = push(want[i], prod * (double)p, sign);
                inv_from<NPASS - 1>(y, f);
                ref(out, true);
                same(y, out, "inverse");
                for (int i = 0; i < n; i++)
                    expect(f.tensor_out(y[i]) == mulm(out[i], ninv, p), "tensor_out", L, p, i);
            }
        }
    }

    // The key sums of k digits: few items (waves w, w + W, ... meet in one sum) and
    // many (one wave takes all), every product at `prod` (units of p).
    void keys(double prod) const {
        const F f(c, 0);
        for (int k = 1; k <= 16; k++)
            for (int sign = -1; sign <= 1; sign += 2)
                for (int few = 0; few < (BIG && k > 8 ? 1 : 2); few++) {  // as the launch picks the kernel
                    const int W = !few ? 1 : k < 8 ? (k < 2 ? 2 : k) : 8;
                    const double v = sign * (2.0 * std::floor(prod * (double)p / 2) - 1);  // odd
                    double sum = 0.0;
                    for (int wave = 0; wave < W; wave++) {
                        double acc[2][16] = {};
                        int cnt = 0;
                        for (int i = wave; i < k; i += W, cnt++) {
                            f.acc_mid(acc, cnt);
                            for (auto &row : acc)
                                for (double &a : row) a += v;
                        }
                        sum += acc[1][7];
                        expect(std::fabs(sum) < LIMIT, "key sum bound", k, p, W);
                    }
                    const double out = f.acc_out(sum);
                    expect(residue(out, p) == residue(v, p) * (u128)k % p, "key sum", k, p, W);
                    expect(std::fabs(out) <= (double)p / 2 + 2.0, "reduced key sum", k, p, W);
                }
    }
};

// The bounds of the header in units of p: LIM = 2^53 / p.
template <int L, bool BIG>
static void check(uint64_t p) {
    Check<L, BIG> t(p);
    const double lim = LIMIT / (double)p;
    double b = 1.0;  // a forward level: b + 1/2 + b / LIM
    for (int l = 0; l < L; l++) b += 0.5 + b / lim;
    if (BIG) b = 0.5;
    t.tensor(b, 0.5 + 3.0 * b * b / lim);  // b^2 p and three roundings of the quotient
    t.keys(0.5 + 3.0 * b / lim);           // b p and the same
}

int main(int argc, char **argv) {
    for (int i = 1; i < argc; i++) {
        const uint64_t p = strtoull(argv[i], nullptr, 10);
        if (p >> 47) {
            check<12, true>(p);
            check<13, true>(p);
            check<14, true>(p);
        } else {
            check<12, false>(p);
            check<13, false>(p);
            check<14, false>(p);
        }
    }
    if (fails) return 1;
    printf("ok %ld\n", checks);
    return 0;
}
