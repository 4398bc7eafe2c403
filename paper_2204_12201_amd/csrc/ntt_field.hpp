// Transforms split at the first radix-16 pass, over two representations of the
// residues.
//
// With 16 residues per thread (ntt_core.hpp) only the exchange next to pass 0
// crosses waves.  The split transforms cut the transform there: a "column"
// kernel runs pass 0 alone (16 residues n/16 apart, no LDS), a "block" kernel
// runs the remaining passes, where one wave owns 1024 consecutive residues and
// exchanges them through its own LDS block, with no workgroup barrier.  A row
// is then n/1024 independent waves instead of one workgroup of n/16 threads,
// so that a single product already spreads over the chip.
//
// Field types:
//  FieldU<LZ>  64-bit integers, the lazy butterflies of ntt_core.hpp.
//  FieldF<BIG> signed integers held in doubles, for primes below 2^50.  A
//              product y w mod p is computed exactly (the floating-point modular
//              product with fused multiply-add of van der Hoeven, Lecerf and
//              Quintin, "Modular SIMD arithmetic in Mathemagix", 2016) as
//                g = rint(y w/p), h = y w, l = fma(y, w, -h), (h - g p) + l,
//              where h + l = y w exactly, h - g p is an integer below 2^53 (one
//              fma, exact) and |y w - g p| <= p (1/2 + |y| 2^-53) for |w| <= p/2:
//              six FP64 instructions for the product where the integer form
//              takes nine half-rate multiplies and about ten more
//              (in registers: 4.7 against 2.4 T butterflies/s).
//
// Bounds of FieldF in units of p (LIM = 2^53 / p >= 8 is the most a value may
// reach): a forward level takes the bound b to b + 1/2 + b/LIM.  Primes below
// 2^47 (LIM >= 64) run the levels from a canonical input without any reduction,
// to 7.8, 8.4 and 9.1 for 12, 13 and 14 of them, and multiply these values as they
// are: a product of two of them is at most 1/2 + 3 b^2/LIM (mulvar_f), 3.4, 3.9
// and 4.4.  Larger ones (BIG, LIM >= 8) go 1 -> 4.1 over pass 0, are
// reduced to 1/2 on entry of the block part, again before its third pass
// (1/2 -> 7.6 in eight levels) and before a product (0.6).  An inverse level
// doubles sums and brings differences to 1/2 + b/LIM: before_last and pass_end
// state where sums are reduced.
#pragma once
#include "kernels.hpp"
#include "modarith.hpp"
#include "ntt_core.hpp"

#pragma clang fp contract(off)

__device__ __forceinline__ double mulmod_f(double y, double w, double wi, double p) {
    const double g = __builtin_rint(y * wi);
    const double h = y * w;
    const double l = __builtin_fma(y, w, -h);
    return __builtin_fma(-g, p, h) + l;
}

// a b mod p for two variables: |result| <= p/2 + 3 |a b| 2^-53 (the roundings of
// a b, 1/p and their product), and a b - g p exactly while that is below 2^52.
__device__ __forceinline__ double mulvar_f(double a, double b, double p, double pinv) {
    const double h = a * b;
    const double g = __builtin_rint(h * pinv);
    const double l = __builtin_fma(a, b, -h);
    return __builtin_fma(-g, p, h) + l;
}

// x - rint(x / p) p: |result| <= p/2 + 2 for |x| <= 2^53.
__device__ __forceinline__ double red_f(double x, double p, double pinv) {
    return __builtin_fma(-__builtin_rint(x * pinv), p, x);
}

// Whole numbers below 2^52 to doubles and back, by the bits of 2^52 + x.
__device__ __forceinline__ double u52_to_f(uint64_t x) {
    return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
}
__device__ __forceinline__ uint64_t f_to_u52(double x) {  // 0 <= x < 2^52
    return (uint64_t)__double_as_longlong(x + 4503599627370496.0) & 0xFFFFFFFFFFFFFull;
}

// ---- twiddle sources -------------------------------------------------------
// The pass P twiddle (u, v) of index H (level 4P + u, entry (H << u) + v).

// Whole-wave uniform index of pass P (scalar loads).
template <int L, int P>
constexpr bool tw_uniform() {
    return Geo<L>::LO(P) >= 6 || Geo<L>::LT <= Geo<L>::LO(P);
}

// From the global table.
template <class T>
struct TwGlobal {
    static constexpr bool SHARED = false;
    const T *__restrict__ tab;
    template <int L, int P>
    __device__ __forceinline__ T get(int u, int v, uint32_t H) const {
        const uint32_t i = (1u << (4 * P + u)) + (H << u) + v;
        if constexpr (tw_uniform<L, P>()) {
            typedef decltype(T::w) S;
            typedef const __attribute__((address_space(4))) S *cptr;
            const cptr p = (cptr)tab + 2u * i;
            return T{p[0], p[1]};
        } else {
            return tab[i];
        }
    }
};

// From a table of one block's per-lane twiddles in LDS (tw_stage), the entries
// of one (P, u, v) side by side: consecutive lanes read consecutive words.
template <int L, int P>
constexpr int tw_nh() {  // values of H in a block
    return ((64 * (16 >> Geo<L>::R(P))) >> Geo<L>::LO(P));
}
template <int L, int P>
constexpr int tw_base() {
    if constexpr (P <= 1) return 0;
    else return tw_base<L, P - 1>() + (tw_uniform<L, P - 1>() ? 0 : tw_nh<L, P - 1>() * ((1 << Geo<L>::R(P - 1)) - 1));
}
template <int L>
constexpr int tw_block_entries() {
    constexpr int P = Geo<L>::NPASS - 1;
    return tw_base<L, P>() + tw_nh<L, P>() * ((1 << Geo<L>::R(P)) - 1);
}
template <class T>
struct TwBlock {
    static constexpr bool SHARED = true;
    const T *__restrict__ tab;   // the global table (uniform passes)
    const T *lds;
    uint32_t blk;
    template <int L, int P>
    __device__ __forceinline__ T get(int u, int v, uint32_t H) const {
        if constexpr (tw_uniform<L, P>()) return TwGlobal<T>{tab}.template get<L, P>(u, v, H);
        else return lds[tw_base<L, P>() + ((1 << u) - 1 + v) * tw_nh<L, P>() + (H - blk * tw_nh<L, P>())];
    }
};
// Copies block blk's entries of pass P and the later ones (all threads of the workgroup).
template <int L, int P, class T>
__device__ __forceinline__ void tw_stage(T *lds, const T *__restrict__ tab, uint32_t blk) {
    if constexpr (!tw_uniform<L, P>()) {
        constexpr int NH = tw_nh<L, P>(), CNT = NH * ((1 << Geo<L>::R(P)) - 1);
        for (int e = threadIdx.x; e < CNT; e += blockDim.x) {
            const uint32_t uv1 = (uint32_t)e / NH + 1, H = blk * NH + (uint32_t)e % NH;
            const uint32_t u = 31 - __builtin_clz(uv1), v = uv1 - (1u << u);
            lds[tw_base<L, P>() + e] = tab[(1u << (4 * P + u)) + (H << u) + v];
        }
    }
    if constexpr (P + 1 < Geo<L>::NPASS) tw_stage<L, P + 1, T>(lds, tab, blk);
}

// Where registers are short (many waves per CU, twiddles in LDS) the FP64
// kernels take one row at a time and schedule level by level: left alone, the
// scheduler spreads the long chains of two rows over more registers than three
// waves per SIMD have (38 to 162 spilled in the tensor kernels).  With few waves
// two rows side by side hide each other's latency.
template <class F, class TW>
constexpr bool serial() {
    return F::FLOAT && TW::SHARED;
}

// ---- passes -----------------------------------------------------------------

// Pass P of the forward transform on NR rows of one prime (one twiddle load for all).
template <int L, int P, int NR, class F, class TW>
__device__ __forceinline__ void fwd_pass_t(typename F::V (&x)[NR][16], int tid, const F &f, const TW &tw) {
    constexpr int r = Geo<L>::R(P), lo = Geo<L>::LO(P);
    constexpr int R = 1 << r, G = 16 >> r;
#pragma unroll
    for (int g = 0; g < G; g++) {
        uint32_t H = fixed_bits<L, 4, P>((uint32_t)tid, (uint32_t)g) >> lo;
        if constexpr (tw_uniform<L, P>()) H = __builtin_amdgcn_readfirstlane(H);
#pragma unroll
        for (int u = 0; u < r; u++) {
            const int half = R >> (u + 1);
#pragma unroll
            for (int v = 0; v < (1 << u); v++) {
                const typename F::T W = tw.template get<L, P>(u, v, H);
#pragma unroll
                for (int w = 0; w < half; w++) {
                    const int e0 = g * R + ((v << (r - u)) | w);
#pragma unroll
                    for (int m = 0; m < NR; m++) f.ct(x[m][e0], x[m][e0 + half], W);
                }
            }
            if constexpr (serial<F, TW>()) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Pass P of the inverse transform on NR rows (bounds: gs, before_last and
// pass_end of the field).
template <int L, int P, int NR, class F, class TW>
__device__ __forceinline__ void inv_pass_t(typename F::V (&x)[NR][16], int tid, const F &f, const TW &tw) {
    constexpr int r = Geo<L>::R(P), lo = Geo<L>::LO(P);
    constexpr int R = 1 << r, G = 16 >> r;
    constexpr bool FIRST = P == Geo<L>::NPASS - 1;
#pragma unroll
    for (int g = 0; g < G; g++) {
        uint32_t H = fixed_bits<L, 4, P>((uint32_t)tid, (uint32_t)g) >> lo;
        if constexpr (tw_uniform<L, P>()) H = __builtin_amdgcn_readfirstlane(H);
#pragma unroll
        for (int u = r - 1; u >= 0; u--) {
            const int half = R >> (u + 1);
            if constexpr (r == 4)
                if (u == 0) f.template before_last<NR>(x);
#pragma unroll
            for (int v = 0; v < (1 << u); v++) {
                const typename F::T W = tw.template get<L, P>(u, v, H);
#pragma unroll
                for (int w = 0; w < half; w++) {
                    const int e0 = g * R + ((v << (r - u)) | w);
                    const bool sums = u == r - 1 ? !FIRST : ((w >> (r - 2 - u)) & 1) == 0;
#pragma unroll
                    for (int m = 0; m < NR; m++) f.gs(x[m][e0], x[m][e0 + half], W, sums);
                }
            }
            if constexpr (serial<F, TW>()) __builtin_amdgcn_sched_barrier(0);
        }
    }
    f.template pass_end<r, NR>(x);
}

// UNI: the prime is the same in the whole wave (its constants then live in
// scalar registers).
template <bool LZ, bool UNI = true>
struct FieldU {
    typedef uint64_t V;
    typedef Tw T;
    static constexpr bool FLOAT = false;
    uint64_t q, qi, one_p, nq;
    const Tw *tw, *itw;
    const PrimeConst *P;

    __device__ __forceinline__ FieldU(const DevCtx &c, int limb) {
        P = c.pc + limb;
        q = P->q;
        qi = P->qinv_neg;
        one_p = P->one_p;
        if constexpr (UNI) {
            nq = neg_opaque(q);
        } else {
            nq = 0 - q;
            asm("" : "+v"(nq));
        }
        tw = c.tw + (size_t)limb * c.n;
        itw = c.itw + (size_t)limb * c.n;
    }
    __device__ __forceinline__ V in(uint64_t v) const { return v; }
    // a residue of another prime: any 64-bit word to [0, 4q)
    template <bool RAW>
    __device__ __forceinline__ V digit(uint64_t v) const {
        return RAW ? v : mul_shoup_lazy4n(v, 1, one_p, nq);
    }
    static __device__ __forceinline__ V from_bits(uint64_t v) { return v; }
    static __device__ __forceinline__ uint64_t to_bits(V v) { return v; }
    __device__ __forceinline__ void ct(V &X, V &Y, const T &W) const { ct_bfly<!LZ>(X, Y, W.w, W.wp, nq, q << 2); }
    // LZ: sums says that both inputs were sums of the level before (ntt_core.hpp)
    __device__ __forceinline__ void gs(V &X, V &Y, const T &W, bool sums) const {
        if constexpr (!LZ) gs_bfly(X, Y, W.w, W.wp, nq, q << 2);
        else if (sums) gs_bfly_semi<true>(X, Y, W.w, W.wp, nq, q << 3);
        else gs_bfly_semi<false>(X, Y, W.w, W.wp, nq, q << 2);
    }
    template <int NR>
    __device__ __forceinline__ void before_last(V (&)[NR][16]) const {}
    template <int r, int NR>
    __device__ __forceinline__ void pass_end(V (&)[NR][16]) const {}
    template <int NR>
    __device__ __forceinline__ void enter_block(V (&)[NR][16]) const {}
    template <int NR>
    __device__ __forceinline__ void mid_block(V (&)[NR][16]) const {}
    // forward output -> operand of mul(), mul(): Montgomery, below 2q
    __device__ __forceinline__ V operand(V v) const {
        if constexpr (LZ) return mul_shoup_lazy4n(v, 1, one_p, nq);
        else return csub(csub(v, q << 2), q << 1);
    }
    template <int NR>
    __device__ __forceinline__ void operands(V (&x)[NR][16]) const {
#pragma unroll
        for (int m = 0; m < NR; m++)
#pragma unroll
            for (int s = 0; s < 16; s++) x[m][s] = operand(x[m][s]);
    }
    __device__ __forceinline__ V mul(V a, V b) const { return mont_mul_lazy_u(a, b, q, qi); }
    __device__ __forceinline__ V add2(V a, V b) const { return a + b; }  // two products: below 4q
    // key switching (LZ only): sums of at most 16 products below 2q
    template <int NR>
    __device__ __forceinline__ void key_operands(V (&)[NR][16]) const {}
    __device__ __forceinline__ void acc_mid(V (&)[2][16], int) const {}
    __device__ __forceinline__ V key(uint64_t w) const { return w; }
    __device__ __forceinline__ V acc(V a, V x, V key) const { return a + mont_mul_lazy_u(x, key, q, qi); }
    __device__ __forceinline__ V acc_out(V a) const { return csub(csub(csub(a, q << 4), q << 3), q << 2); }
    // tensor output: times n^-1 (and the Montgomery factor), canonical
    __device__ __forceinline__ uint64_t tensor_out(V v) const {
        return csub(v * P->ninvm + mulhi64(v, P->ninvm_p) * nq, q);
    }
    // key switching output: the key carries n^-1 2^64, canonical from [0, 8q)
    __device__ __forceinline__ uint64_t relin_out(V v) const { return csub(csub(csub(v, q << 2), q << 1), q); }
};

template <bool BIG>
struct FieldF {
    typedef double V;
    typedef TwF T;
    static constexpr bool FLOAT = true;
    double p, pinv;
    const TwF *tw, *itw;
    const PrimeConst *P;

    __device__ __forceinline__ FieldF(const DevCtx &c, int limb) {
        P = c.pc + limb;
        p = P->pf;
        pinv = P->pinvf;
        tw = c.twf + (size_t)limb * c.n;
        itw = c.itwf + (size_t)limb * c.n;
    }
    __device__ __forceinline__ V in(uint64_t v) const { return u52_to_f(v); }
    template <bool RAW>
    __device__ __forceinline__ V digit(uint64_t v) const {
        return red_f(u52_to_f(v), p, pinv);
    }
    static __device__ __forceinline__ V from_bits(uint64_t v) { return __longlong_as_double((long long)v); }
    static __device__ __forceinline__ uint64_t to_bits(V v) { return (uint64_t)__double_as_longlong(v); }
    template <int NR>
    __device__ __forceinline__ void reduce_all(V (&x)[NR][16]) const {
        if constexpr (BIG) {
#pragma unroll
            for (int m = 0; m < NR; m++)
#pragma unroll
                for (int s = 0; s < 16; s++) x[m][s] = red_f(x[m][s], p, pinv);
        }
    }
    __device__ __forceinline__ void ct(V &X, V &Y, const T &W) const {
        const V x = X, t = mulmod_f(Y, W.w, W.wi, p);
        X = x + t;
        Y = x - t;
    }
    __device__ __forceinline__ void gs(V &X, V &Y, const T &W, bool) const {
        const V x = X, y = Y;
        X = x + y;
        Y = mulmod_f(x - y, W.w, W.wi, p);
    }
    // Slots of a radix-16 inverse pass (low slot bit first): slot s ends as a sum
    // of 2^z values of its last product, z the number of zero bits above its
    // highest one bit (16 input sums for slot 0).  BIG (LIM >= 8, inputs at most
    // p): after three levels the slots whose low three bits are 0 or 1 hold up
    // to 8 or 4 p and are reduced before the last level (every sum and
    // difference then stays below 8p, every product below 1.02 p), the sums
    // (slots 0..7) at the end.  Otherwise (LIM >= 64): slots 0..3 at the end, which
    // leaves the others below 2p; inputs are at most 3.4 p in the first pass of
    // n = 4096 (unreduced products: slot 0 reaches 55p) and 2p in the others (32p).
    // Shorter passes, the first of n = 8192 and 16384 (inputs at most 4.4 p, BIG 0.6
    // p): the sums, at most 18p (BIG 2.4 p), at the end, products stay below 0.8 p.
    template <int NR>
    __device__ __forceinline__ void before_last(V (&x)[NR][16]) const {
        if constexpr (BIG) {
#pragma unroll
            for (int m = 0; m < NR; m++) {
                x[m][0] = red_f(x[m][0], p, pinv);
                x[m][1] = red_f(x[m][1], p, pinv);
                x[m][8] = red_f(x[m][8], p, pinv);
                x[m][9] = red_f(x[m][9], p, pinv);
            }
        }
    }
    template <int r, int NR>
    __device__ __forceinline__ void pass_end(V (&x)[NR][16]) const {
        static_assert(r == 4 || r <= 2, "the reduction rules cover radix 16, 4 and 2");
        if constexpr (r == 4) {
#pragma unroll
            for (int m = 0; m < NR; m++)
#pragma unroll
                for (int s = 0; s < 4; s++) x[m][s] = red_f(x[m][s], p, pinv);
            if constexpr (BIG) {
#pragma unroll
                for (int m = 0; m < NR; m++)
#pragma unroll
                    for (int s = 4; s < 8; s++) x[m][s] = red_f(x[m][s], p, pinv);
            }
        } else {
            constexpr int R = 1 << r;
#pragma unroll
            for (int m = 0; m < NR; m++)
#pragma unroll
                for (int s = 0; s < 16; s++)
                    if (s % R < R / 2) x[m][s] = red_f(x[m][s], p, pinv);
        }
    }
    template <int NR>
    __device__ __forceinline__ void enter_block(V (&x)[NR][16]) const { reduce_all(x); }
    template <int NR>
    __device__ __forceinline__ void mid_block(V (&x)[NR][16]) const { reduce_all(x); }
    template <int NR>
    __device__ __forceinline__ void operands(V (&x)[NR][16]) const { reduce_all(x); }
    __device__ __forceinline__ V mul(V a, V b) const { return mulvar_f(a, b, p, pinv); }
    __device__ __forceinline__ V add2(V a, V b) const { return red_f(a + b, p, pinv); }
    template <int NR>
    __device__ __forceinline__ void key_operands(V (&x)[NR][16]) const { reduce_all(x); }
    // Key sums.  BIG (operands reduced to p/2, keys below p): a product is at most
    // p (1/2 + 3/16), 3/(2 LIM) for the quotient's three roundings (mulvar_f);
    // eight of them, or eight and a reduced sum, stay below 8p.  Otherwise the
    // forward values reach 9.1p and a product 0.93p: 16 of them stay below 64p.
    // acc_mid: before product number cnt of one wave's sum.  (Sums of several waves
    // are of at most eight products: SplitL::relin.)
    __device__ __forceinline__ void acc_mid(V (&a)[2][16], int cnt) const {
        if ((cnt & 7) == 7) reduce_all(a);
    }
    __device__ __forceinline__ V key(uint64_t w) const { return u52_to_f(w); }
    __device__ __forceinline__ V acc(V a, V x, V key) const { return a + mulvar_f(x, key, p, pinv); }
    __device__ __forceinline__ V acc_out(V a) const { return red_f(a, p, pinv); }
    __device__ __forceinline__ uint64_t canon(V v) const { return f_to_u52(v < 0.0 ? v + p : v); }
    __device__ __forceinline__ uint64_t tensor_out(V v) const {
        return canon(mulmod_f(v, P->ninvf, P->ninvf_i, p));
    }
    // the key carries n^-1 2^64: times 2^-64
    __device__ __forceinline__ uint64_t relin_out(V v) const { return canon(mulmod_f(v, P->m64f, P->m64f_i, p)); }
};

// The fields of a context's primes: fn(field of prime `limb`).  A kernel runs
// one body per field behind a branch on the prime (the same in the whole
// workgroup): as a run-time flag inside one body the large primes' reductions
// cost 30 to 340 spilled registers in the tensor kernels.
template <bool LZ>
struct FamU {
    typedef uint64_t V;
    typedef Tw T;
    template <class Fn>
    static __device__ __forceinline__ void with(const DevCtx &c, int limb, const Fn &fn) {
        fn(FieldU<LZ>(c, limb));
    }
    // the same with a prime per lane
    template <class Fn>
    static __device__ __forceinline__ void with_lanes(const DevCtx &c, int limb, const Fn &fn) {
        fn(FieldU<LZ, false>(c, limb));
    }
};
// Integer primes of both kinds: the lazy butterflies where the prime allows
// them (the primes of Q do where P needs primes too large).
struct FamM {
    typedef uint64_t V;
    typedef Tw T;
    template <class Fn>
    static __device__ __forceinline__ void with(const DevCtx &c, int limb, const Fn &fn) {
        if ((c.lazy_limbs >> limb) & 1) fn(FieldU<true>(c, limb));
        else fn(FieldU<false>(c, limb));
    }
    template <class Fn>
    static __device__ __forceinline__ void with_lanes(const DevCtx &c, int limb, const Fn &fn) {
        if ((c.lazy_limbs >> limb) & 1) fn(FieldU<true, false>(c, limb));
        else fn(FieldU<false, false>(c, limb));
    }
};
struct FamF {
    typedef double V;
    typedef TwF T;
    template <class Fn>
    static __device__ __forceinline__ void with(const DevCtx &c, int limb, const Fn &fn) {
        if ((c.big_limbs >> limb) & 1) fn(FieldF<true>(c, limb));
        else fn(FieldF<false>(c, limb));
    }
    template <class Fn>
    static __device__ __forceinline__ void with_lanes(const DevCtx &c, int limb, const Fn &fn) {
        with(c, limb, fn);
    }
};

// Passes P.. (P >= 1) of the forward transform of NR rows, one wave per block
// of 1024 residues: tid = 64 block + lane picks the twiddles, the exchanges use
// the wave's own LDS block of 1088 words.
template <int L, int P, int NR, class F, class TW>
__device__ __forceinline__ void fwd_block(typename F::V (&x)[NR][16], typename F::V *lds, int lane, int tid, const F &f,
                                          const TW &tw) {
    fwd_pass_t<L, P, NR>(x, (int)fresh((uint32_t)tid), f, tw);
    if constexpr (P + 1 < Geo<L>::NPASS) {
#pragma unroll
        for (int m = 0; m < NR; m++) exchange<L, 4, P, P + 1>(lds, x[m], (int)fresh((uint32_t)lane));
        if constexpr (P == 2) f.mid_block(x);
        fwd_block<L, P + 1, NR>(x, lds, lane, tid, f, tw);
    }
}

// Passes NPASS-1 .. 1 of the inverse transform.
template <int L, int P, int NR, class F, class TW>
__device__ __forceinline__ void inv_block(typename F::V (&x)[NR][16], typename F::V *lds, int lane, int tid, const F &f,
                                          const TW &tw) {
    inv_pass_t<L, P, NR>(x, (int)fresh((uint32_t)tid), f, tw);
    if constexpr (P > 1) {
#pragma unroll
        for (int m = 0; m < NR; m++) exchange<L, 4, P, P - 1>(lds, x[m], (int)fresh((uint32_t)lane));
        inv_block<L, P - 1, NR>(x, lds, lane, tid, f, tw);
    }
}

// The block parts of two rows, side by side or one after the other.
template <int L, class F, class TW>
__device__ __forceinline__ void fwd_block_pair(typename F::V (&x)[2][16], typename F::V *lds, int lane, int tid,
                                               const F &f, const TW &tw) {
    typedef typename F::V row_t[1][16];
    if constexpr (!serial<F, TW>()) {
        fwd_block<L, 1, 2>(x, lds, lane, tid, f, tw);
    } else {
        fwd_block<L, 1, 1>(reinterpret_cast<row_t &>(x[0]), lds, lane, tid, f, tw);
        asm volatile("" ::: "memory");
        fwd_block<L, 1, 1>(reinterpret_cast<row_t &>(x[1]), lds, lane, tid, f, tw);
        asm volatile("" ::: "memory");
    }
}

template <int L, class F, class TW>
__device__ __forceinline__ void inv_block_pair(typename F::V (&x)[2][16], typename F::V *lds, int lane, int tid,
                                               const F &f, const TW &tw) {
    typedef typename F::V row_t[1][16];
    constexpr int LAST = Geo<L>::NPASS - 1;
    if constexpr (!serial<F, TW>()) {
        inv_block<L, LAST, 2>(x, lds, lane, tid, f, tw);
    } else {
        inv_block<L, LAST, 1>(reinterpret_cast<row_t &>(x[0]), lds, lane, tid, f, tw);
        asm volatile("" ::: "memory");
        inv_block<L, LAST, 1>(reinterpret_cast<row_t &>(x[1]), lds, lane, tid, f, tw);
        asm volatile("" ::: "memory");
    }
}
