// Device code of the base conversions shared by the conversion kernels
// (kernels_conv.hip) and the column kernels that fuse them with the first
// transform pass (kernels_split.hip): the exact mixed-radix path and the tiles
// of the int8 matrix cores.
#pragma once
#include "kernels.hpp"
#include "modarith.hpp"

namespace {

// A table word read through the constant address space: the tables do not
// change while a kernel runs, and wave-uniform reads then become scalar loads
// (the multiply-add asm takes its constant operand from SGPRs).
__device__ __forceinline__ uint64_t ldc(const uint64_t *p) {
    return *(const __attribute__((address_space(4))) uint64_t *)p;
}

// ---------------------------------------------------------------- exact path --

// The exact path runs for a tiny fraction of the coefficients: its loops stay
// rolled so that it does not raise the register count (and so the occupancy)
// of the fast path that shares the kernel.

// Garner digits d of X (residues r in basis M): X = sum_b d_b prod_{a<b} m_a.
template <int MB>
__device__ __forceinline__ void mrc_digits(const MrcConst &M, const uint64_t (&r)[MB],
                                           uint64_t (&d)[MB]) {
    const int K = (int)M.K;
#pragma unroll 1
    for (int b = 0; b < MB; b++) {
        d[b] = 0;
        if (b < K) {
            const uint64_t mb = M.m[b];
            uint64_t v = r[b];
#pragma unroll 1
            for (int a = 0; a < MB; a++) {
                if (a < b) {
                    const uint64_t da = mul_shoup(d[a], 1, M.one_p[b], mb);
                    v = sub_mod(v, da, mb);
                    v = mul_shoup(v, M.inv[a][b], M.inv_p[a][b], mb);
                }
            }
            d[b] = v;
        }
    }
}

// X > (M - 1) / 2 ?  (lexicographic on the digits, most significant first)
template <int MB>
__device__ __forceinline__ bool mrc_gt_half(const MrcConst &M, const uint64_t (&d)[MB]) {
    int res = 0;
#pragma unroll 1
    for (int b = MB - 1; b >= 0; b--) {
        if (b < (int)M.K && res == 0) {
            const uint64_t h = M.half_digit[b];
            res = d[b] > h ? 1 : (d[b] < h ? -1 : 0);
        }
    }
    return res == 1;
}

// X mod target j by Horner on the digits: acc = acc * m_b + d_b, b = K-1 .. 0.
template <int MB>
__device__ __forceinline__ uint64_t mrc_eval(const MrcConst &M, const uint64_t (&d)[MB], int j) {
    const uint64_t p = M.target[j], op = M.tgt_one_p[j];
    uint64_t acc = 0;
#pragma unroll 1
    for (int b = MB - 1; b >= 0; b--) {
        if (b < (int)M.K) {
            acc = mul_shoup(acc, M.m_mod_t[b][j], M.m_mod_t_p[b][j], p);
            acc = add_mod(acc, mul_shoup(d[b], 1, op, p), p);
        }
    }
    return acc;
}

// ---- exact conversions of one coefficient ----

// Exact centred lift of one coefficient (residues x in Q) by mixed-radix
// conversion; put(j, r) receives r = x~ mod p_j.  Counts the coefficient in
// the fallback counter.
template <int MK, int MKP, bool EX, class Put>
__device__ __forceinline__ void lift_exact(const DevCtx &c, const uint64_t (&x)[MK], Put put) {
    const int kp = EX ? MKP : c.kp;
    const ConvConst &cc = *c.cc;
    atomicAdd(c.fallback, 1ull);
    const MrcConst &M = *c.mrc_q;
    uint64_t dg[MK];
    mrc_digits<MK>(M, x, dg);
    const bool gt = mrc_gt_half<MK>(M, dg);
#pragma unroll 1
    for (int j = 0; j < MKP; j++) {
        if (j < kp) {
            uint64_t r = mrc_eval<MK>(M, dg, j);
            if (gt) r = sub_mod(r, M.M_mod_t[j], cc.p[j]);
            put(j, r);
        }
    }
}

// Exact scale-and-round of one coefficient: Y = t D + h; [Y]_q by Garner over
// Q; C_p = (Y_p - [Y]_q) q^-1; then the centred value of C by Garner over P.
// Counts the coefficient in the fallback counter.
template <int MK, int MKP, bool EX, class Put>
__device__ __forceinline__ void scale_exact(const DevCtx &c, const uint64_t (&dq)[MK], const uint64_t (&dp)[MKP],
                                            Put put) {
    const int k = EX ? MK : c.k, kp = EX ? MKP : c.kp;
    const ConvConst &cc = *c.cc;
    atomicAdd(c.fallback, 1ull);
    const MrcConst &MQ = *c.mrc_q;
    const MrcConst &MP = *c.mrc_p;
    uint64_t yq[MK], dgq[MK];
#pragma unroll
    for (int i = 0; i < MK; i++) {
        yq[i] = 0;
        if (i < k) yq[i] = add_mod(mul_shoup(dq[i], cc.t_q[i], cc.t_qs[i], cc.q[i]), cc.h_q[i], cc.q[i]);
    }
    mrc_digits<MK>(MQ, yq, dgq);
    uint64_t cp[MKP], dgp[MKP];
#pragma unroll 1
    for (int j = 0; j < MKP; j++) {
        cp[j] = 0;
        if (j < kp) {
            const uint64_t pj = cc.p[j];
            const uint64_t ypj = add_mod(mul_shoup(dp[j], cc.t_p[j], cc.t_ps[j], pj), cc.h_p[j], pj);
            const uint64_t xpj = mrc_eval<MK>(MQ, dgq, j);
            cp[j] = mul_shoup(sub_mod(ypj, xpj, pj), cc.qinv_p[j], cc.qinv_ps[j], pj);
        }
    }
    mrc_digits<MKP>(MP, cp, dgp);
    const bool gt = mrc_gt_half<MKP>(MP, dgp);
#pragma unroll 1
    for (int i = 0; i < MK; i++) {
        if (i < k) {
            uint64_t r = mrc_eval<MKP>(MP, dgp, i);
            if (gt) r = sub_mod(r, MP.M_mod_t[i], cc.q[i]);
            put(i, r);
        }
    }
}

// ------------------------------------------ conversions on the matrix cores --
//
// The base conversions of the lift and of the scale-and-round are dense
// contractions (coefficients x sources against a sources x targets matrix of
// constants), so for bases of at most 8 primes on each side they run on the
// int8 matrix cores, exactly, with the operand tables of ConvMx.  Per tile of
// 16 coefficients and per conversion: four v_mfma_i32_16x16x64_i8 give every
// target's eight partial sums (eight in the scale's first conversion, whose
// D_p term is a second, block-diagonal block chained onto the first); each
// lane recombines the sums of its two targets, adds the conversion's extra
// terms and reduces once (Montgomery).
// The floating estimates are summed over the four lanes of a column.  A
// coefficient whose estimate falls within FHE_EST_MARGIN of a decision
// boundary is queued in LDS and converted exactly (mixed radix) by one thread
// after the tiles; every output word is therefore the exact one, as on the
// vector ALU path.  The operand tables and the constants of every slot (prime
// s of the source and target bases) are staged in LDS and read per tile,
// which keeps the register count of a wave low.

typedef int mx_v4i __attribute__((ext_vector_type(4)));

// Coefficients per workgroup (four waves, tiles of 16).
constexpr int kMxSpan = 1024;

// Balanced base-256 digits of x as eight signed bytes: the bytes of x + B
// (B = 0x80 in every byte) are d_u + 128, and xor 0x80 turns each into d_u in
// two's complement.  Valid while x + B < 2^64 (x <= 0x7F7F7F7F7F7F7F7F, about
// 2^63 - 2^55); every value decomposed here is below 2^62.
__device__ __forceinline__ uint64_t mx_digits(uint64_t x) {
    constexpr uint64_t B = 0x8080808080808080ull;
    return (x + B) ^ B;
}

// B operand of a lane: the digits of its two sources (bytes 0..7, 8..15).
__device__ __forceinline__ mx_v4i mx_operand(uint64_t x0, uint64_t x1) {
    const uint64_t a = mx_digits(x0), b = mx_digits(x1);
    return mx_v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)(uint32_t)b, (int)(uint32_t)(b >> 32)};
}

// LDS of a workgroup: the operand tables of its NT conversions, the constants
// of each slot on the Q side and on the P side, and the exact-path queue
// (offsets of coefficients within the workgroup's SPAN).
template <int NT, int SPAN>
struct MxSharedT {
    mx_v4i a[NT][4][64];
    uint64_t cq[FHE_MX_MAXB][10];
    uint64_t cp[FHE_MX_MAXB][8];
    int item[SPAN];
    int count;
};
typedef MxSharedT<3, kMxSpan> MxShared;

// acc[mm] = FHE_MX_BIAS + A[mm] B, mm = 0..3 (A = table `t` of the LDS): lane
// gets P' of target l/16 (acc[0]: digits 0..3, acc[1]: 4..7) and of target
// l/16 + 4 (acc[2], acc[3]).
template <int H = 2, class Sh>
__device__ __forceinline__ void mx_products(const Sh &sh, int t, uint32_t lane, const mx_v4i B,
                                            mx_v4i (&acc)[4]) {
    const mx_v4i bias = {FHE_MX_BIAS, FHE_MX_BIAS, FHE_MX_BIAS, FHE_MX_BIAS};
#pragma unroll
    for (int mm = 0; mm < 2 * H; mm++) acc[mm] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sh.a[t][mm][lane], B, bias, 0, 0, 0);
}

// acc[mm] += A[mm] B (table `t`): a second block of 64 (source, digit) pairs.
template <int H = 2, class Sh>
__device__ __forceinline__ void mx_products_add(const Sh &sh, int t, uint32_t lane, const mx_v4i B,
                                                mx_v4i (&acc)[4]) {
#pragma unroll
    for (int mm = 0; mm < 2 * H; mm++)
        acc[mm] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sh.a[t][mm][lane], B, acc[mm], 0, 0, 0);
}

// hi:lo = sum_v 256^v P'_v with P'_v = a[v] (v < 4), b[v - 4] (v >= 4), each in
// [0, 2^22]: pairs within 32 bits (< 2^31), then x = a01 + a23 2^16 and
// w = a45 + a67 2^16 (< 2^47), and the sum x + w 2^32 (< 2^79).
__device__ __forceinline__ void mx_recombine(const mx_v4i a, const mx_v4i b, uint64_t &lo, uint64_t &hi) {
    const uint32_t a01 = (uint32_t)a[0] + ((uint32_t)a[1] << 8);
    const uint32_t a23 = (uint32_t)a[2] + ((uint32_t)a[3] << 8);
    const uint32_t a45 = (uint32_t)b[0] + ((uint32_t)b[1] << 8);
    const uint32_t a67 = (uint32_t)b[2] + ((uint32_t)b[3] << 8);
    const uint64_t x = (uint64_t)a01 + ((uint64_t)a23 << 16);
    const uint64_t w = (uint64_t)a45 + ((uint64_t)a67 << 16);
    lo = x + (w << 32);
    hi = (w >> 32) + (lo < x ? 1u : 0u);
}

// (hi:lo) 2^-64 mod m in [0, m) for the sums of the matrix-core tiles: below
// 2^79 plus two 64-bit constants, so hi < 2^16 < m - 1 (every prime here is at
// least 2^20) and the Montgomery reduction hi + floor(m' m / 2^64) + [lo != 0]
// (m' = lo (-m^-1) mod 2^64) is already below 2m: one conditional subtraction.
__device__ __forceinline__ uint64_t mx_reduce(uint64_t lo, uint64_t hi, uint64_t m, uint64_t minv_neg) {
    return csub(redc_lazy(hi, lo, m, minv_neg), m);
}

__device__ __forceinline__ void mx_add(uint64_t &lo, uint64_t &hi, uint64_t alo, uint64_t ahi) {
    lo += alo;
    hi += ahi + (lo < alo ? 1u : 0u);
}

// Sum over the four lanes of a column (l, l ^ 16, l ^ 32, l ^ 48); every one
// of them gets the same value (each addition pairs the same two operands).
// a16, a32: byte addresses (l ^ 16) 4 and (l ^ 32) 4 of the lane exchange.
__device__ __forceinline__ double mx_swap(double x, int a) {
    const int lo = __builtin_amdgcn_ds_bpermute(a, __double2loint(x));
    const int hi = __builtin_amdgcn_ds_bpermute(a, __double2hiint(x));
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double mx_colsum(double x, int a16, int a32) {
    x += mx_swap(x, a16);
    x += mx_swap(x, a32);
    return x;
}

// Tiles w, w + 4, ... (< ntiles) of wave w with their inputs loaded one tile
// ahead: load(R, tile) fills R, body(R, tile) uses it.
template <class Regs, class Load, class Body>
__device__ __forceinline__ void mx_tiles1(int wave, int ntiles, Load load, Body body) {
    Regs r;
    if (wave < ntiles) load(r, wave);
    for (int tile = wave; tile < ntiles; tile += 4) {
        asm volatile("" ::: "memory");  // read the LDS constants per tile
        const Regs cur = r;
        if (tile + 4 < ntiles) load(r, tile + 4);
        body(cur, tile);
    }
}

// The same with the inputs loaded two tiles ahead into two register sets.
template <class Regs, class Load, class Body>
__device__ __forceinline__ void mx_tiles(int wave, int ntiles, Load load, Body body) {
    Regs r0, r1;
    if (wave < ntiles) load(r0, wave);
    if (wave + 4 < ntiles) load(r1, wave + 4);
    for (int tile = wave; tile < ntiles; tile += 8) {
        asm volatile("" ::: "memory");  // read the LDS constants per tile
        {
            const Regs cur = r0;
            if (tile + 8 < ntiles) load(r0, tile + 8);
            body(cur, tile);
        }
        if (tile + 4 < ntiles) {
            asm volatile("" ::: "memory");
            const Regs cur = r1;
            if (tile + 12 < ntiles) load(r1, tile + 12);
            body(cur, tile + 4);
        }
    }
}

__device__ __forceinline__ double mx_f64(uint64_t bits) { return __longlong_as_double((long long)bits); }

// Table t of the LDS := operand table `src` (256 entries of 16 bytes; one per
// thread of the first 256).
template <class Sh>
__device__ __forceinline__ void mx_stage_table(Sh &sh, int t, const int32_t (*src)[64][4]) {
    const int e = (int)threadIdx.x;
    if (e < 256) sh.a[t][e >> 6][e & 63] = reinterpret_cast<const mx_v4i *>(&src[0][0][0])[e];
}

// Scale slot constants.  Q side of slot s: q, -q^-1 mod 2^64, [t qhat^-1]
// (Shoup pair), [h qhat^-1], [-P] 2^64, bias removal, 1/q; P side: p,
// -p^-1 mod 2^64, (word 2 unused), the v multiplier, bias removal plus
// constant, 1/p.  Absent primes: zeros.
template <class Sh>
__device__ __forceinline__ void mx_stage_scale_slots(Sh &sh, const DevCtx &c) {
    const ConvConst &cc = *c.cc;
    const ConvMx &mx = *c.mx;
    const int t = (int)threadIdx.x;
    if (t < FHE_MX_MAXB) {
        uint64_t *w = sh.cq[t];
        const bool ok = t < c.k;
        w[0] = ok ? cc.q[t] : 0;
        w[1] = ok ? cc.q_qinv[t] : 0;
        w[2] = ok ? cc.tqhinv[t] : 0;
        w[3] = ok ? cc.tqhinv_p[t] : 0;
        w[4] = ok ? cc.hqhinv[t] : 0;
        w[5] = ok ? mx.p_beta[t] : 0;
        w[6] = ok ? mx.e_p2q[t] : 0;
        w[7] = ok ? (uint64_t)__double_as_longlong(cc.inv_q[t]) : 0;
    } else if (t < 2 * FHE_MX_MAXB) {
        const int s = t - FHE_MX_MAXB;
        uint64_t *w = sh.cp[s];
        const bool ok = s < c.kp;
        w[0] = ok ? cc.p[s] : 0;
        w[1] = ok ? cc.p_qinv[s] : 0;
        w[3] = ok ? mx.s_v[s] : 0;
        w[4] = ok ? mx.e_scale[s] : 0;
        w[5] = ok ? (uint64_t)__double_as_longlong(cc.inv_p[s]) : 0;
    }
}

// H: slots per lane (1 where both bases have at most 4 primes: half the products
// and half the lanes' arithmetic; slots g + 4h, h < H).
//
// Scale-and-round of one tile column on the matrix cores (tables 0: scale in
// P from the y_i, 1: P -> Q, 2: scale in P from D_p, block-diagonal).  dq,
// dp: the lane's two Q and two P residues of D, any representatives below
// 2^62 (absent primes read a present row; their constants and weights are
// zero); jv[h]: slot g + 4h is a P prime.  Returns false when the coefficient must take the exact path, else
// the lane's two outputs C mod q_s in out.
template <int H = 2, class Sh>
__device__ __forceinline__ bool mx_scale_tile(const Sh &sh, uint32_t lane, int a16, int a32,
                                              const uint64_t (&dq)[H], const uint64_t (&dp)[H], const bool (&jv)[H],
                                              uint64_t (&out)[H]) {
    const uint32_t g = lane >> 4;
    uint64_t y[H];
    double e = 0.0;
#pragma unroll
    for (int h = 0; h < H; h++) {
        const uint64_t *Q = sh.cq[g + 4 * h];
        y[h] = add_mod(mul_shoup(dq[h], Q[2], Q[3], Q[0]), Q[4], Q[0]);
        e = fma((double)y[h], mx_f64(Q[7]), e);
    }
    e = mx_colsum(e, a16, a32);
    const double fl = floor(e), d = e - fl;
    bool exact = (d < FHE_EST_MARGIN) || (d > 1.0 - FHE_EST_MARGIN);
    const uint64_t v = (uint32_t)fl;  // < k
    mx_v4i acc[4];
    mx_products<H>(sh, 0, lane, mx_operand(y[0], H == 2 ? y[H - 1] : 0), acc);
    mx_products_add<H>(sh, 2, lane, mx_operand(dp[0], H == 2 ? dp[H - 1] : 0), acc);
    uint64_t z[H];
    double e2 = 0.0;
#pragma unroll
    for (int h = 0; h < H; h++) {
        const uint64_t *Pc = sh.cp[g + 4 * h];
        uint64_t lo, hi;
        mx_recombine(acc[2 * h], acc[2 * h + 1], lo, hi);
        mx_add(lo, hi, v * Pc[3], 0);
        mx_add(lo, hi, Pc[4], 0);
        // z_j = C_{p_j} phat_j^-1 mod p_j (the factor is folded into the table)
        z[h] = jv[h] ? mx_reduce(lo, hi, Pc[0], Pc[1]) : 0;
        e2 = fma((double)z[h], mx_f64(Pc[5]), e2);
    }
    e2 = mx_colsum(e2, a16, a32);
    const double fl2 = floor(e2), d2 = e2 - fl2;
    exact = exact || (fabs(d2 - 0.5) < FHE_EST_MARGIN);
    const uint64_t beta = (uint32_t)fl2 + (d2 > 0.5 ? 1u : 0u);  // <= k'
    mx_products<H>(sh, 1, lane, mx_operand(z[0], H == 2 ? z[H - 1] : 0), acc);
#pragma unroll
    for (int h = 0; h < H; h++) {
        const uint64_t *Q = sh.cq[g + 4 * h];
        uint64_t lo, hi;
        mx_recombine(acc[2 * h], acc[2 * h + 1], lo, hi);
        mx_add(lo, hi, beta * Q[5], 0);
        mx_add(lo, hi, Q[6], 0);
        out[h] = mx_reduce(lo, hi, Q[0], Q[1]);
    }
    return !exact;
}

// Row offsets (in words) of the lane's two slots: slot s = l/16 + 4h, clamped
// to the basis (an absent prime reads a present row; its constants are zero,
// so the words read there do not enter any output).
__device__ __forceinline__ uint32_t mx_row(int s, int nb, int first, int n) {
    return (uint32_t)((first + (s < nb ? s : nb - 1)) * n);
}

// Lift slot constants.  Q side: q, [qhat^-1] (Shoup pair), 1/q; P side: p,
// -p^-1 mod 2^64, [-q] 2^64, bias removal.  Absent primes: zeros.
template <class Sh>
__device__ __forceinline__ void mx_stage_lift_slots(Sh &sh, const DevCtx &c) {
    const ConvConst &cc = *c.cc;
    const ConvMx &mx = *c.mx;
    const int t = (int)threadIdx.x;
    if (t < FHE_MX_MAXB) {
        const bool ok = t < c.k;
        sh.cq[t][0] = ok ? cc.q[t] : 0;
        sh.cq[t][1] = ok ? cc.qhinv[t] : 0;
        sh.cq[t][2] = ok ? cc.qhinv_p[t] : 0;
        sh.cq[t][3] = ok ? (uint64_t)__double_as_longlong(cc.inv_q[t]) : 0;
    } else if (t < 2 * FHE_MX_MAXB) {
        const int s = t - FHE_MX_MAXB;
        const bool ok = s < c.kp;
        sh.cp[s][0] = ok ? cc.p[s] : 0;
        sh.cp[s][1] = ok ? cc.p_qinv[s] : 0;
        sh.cp[s][2] = ok ? mx.l_beta[s] : 0;
        sh.cp[s][3] = ok ? mx.e_lift[s] : 0;
    }
}

// Centred lift of one tile column on the matrix cores (table 0): x the lane's
// two Q residues.  Returns false when the coefficient must take the exact
// path, else the lane's two residues modulo P in out.
template <int H = 2, class Sh>
__device__ __forceinline__ bool mx_lift_tile(const Sh &sh, uint32_t lane, int a16, int a32,
                                             const uint64_t (&x)[H], uint64_t (&out)[H]) {
    const uint32_t g = lane >> 4;
    uint64_t yv[H];
    double e = 0.0;
#pragma unroll
    for (int h = 0; h < H; h++) {
        const uint64_t *Q = sh.cq[g + 4 * h];
        yv[h] = mul_shoup(x[h], Q[1], Q[2], Q[0]);
        e = fma((double)yv[h], mx_f64(Q[3]), e);
    }
    e = mx_colsum(e, a16, a32);
    const double fl = floor(e), d = e - fl;
    const uint64_t beta = (uint32_t)fl + (d > 0.5 ? 1u : 0u);  // <= k
    mx_v4i acc[4];
    mx_products<H>(sh, 0, lane, mx_operand(yv[0], H == 2 ? yv[H - 1] : 0), acc);
    if (fabs(d - 0.5) < FHE_EST_MARGIN) return false;
#pragma unroll
    for (int h = 0; h < H; h++) {
        const uint64_t *Pc = sh.cp[g + 4 * h];
        uint64_t lo, hi;
        mx_recombine(acc[2 * h], acc[2 * h + 1], lo, hi);
        mx_add(lo, hi, beta * Pc[2], 0);
        mx_add(lo, hi, Pc[3], 0);
        out[h] = mx_reduce(lo, hi, Pc[0], Pc[1]);
    }
    return true;
}

}  // namespace
