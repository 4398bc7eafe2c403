// Product pipeline on the split transforms (ntt_field.hpp): column kernels run
// radix-16 pass 0 of rows (one thread per 16 residues n/16 apart), block
// kernels run the other passes of 1024 consecutive residues in one wave.
// Rows between the two halves hold field values (lazy integers or doubles).
//
//  k_col_lift      lift of the inputs and pass 0 of their forward transforms
//  k_col_scale     pass 0 of the inverse of the tensor rows, scale-and-round, and
//                  pass 0 of the digits
//  k_split_fwd     pass 0 of the extended inputs
//  k_split_tensor  blocks: forward, tensor product, inverse
//  k_split_inv     pass 0 of the inverse of the tensor rows, canonical
//  k_split_digits  pass 0 of every digit modulo every prime of Q
//  k_split_relin   blocks: forward of the digits, inner product with the key,
//                  inverse
//  k_split_fin     pass 0 of the inverse of the key-switching rows, added to out
//
// One object per ring degree 2^FHE_NTT_L.
#include <type_traits>

#include "conv_mx.hpp"
#include "kernels.hpp"
#include "modarith.hpp"
#include "ntt_core.hpp"
#include "ntt_field.hpp"

namespace {

constexpr int kColThreads = 256;
constexpr int kBlkWords = 1088;  // LDS words of one wave's block (1024 plus padding)

template <int L>
constexpr int col_groups() {
    return Geo<L>::T / kColThreads;
}

// ---- column kernels fused with the base conversions ----------------------------
// A workgroup of W waves owns C columns: the 16 C coefficients c0 + [0, C) + e
// n/16, e = 0..15.  The conversions need every residue of a coefficient, pass 0
// the 16 residues of a column modulo one prime: they meet in LDS
// (rows[limb][e][C]), so the lifted and the inverse transformed rows never go
// through memory.  Bases of at most 8 primes a side (ConvMx).

template <int C, int NT>
struct ColShared {
    MxSharedT<NT, 16 * C> mx;
    uint64_t rows[1][16][C];  // [limbs], dynamic
};

// Calls fn(unit, column, field) for the units 0 .. count - 1 of the workgroup's
// waves: 64 / C units side by side in the lanes of a wave, unit u with the
// field of prime limb(u).
template <class F, int C, int W, class Limb, class Fn>
__device__ __forceinline__ void col_units(const DevCtx &c, int first, int step, int count, const Limb &limb,
                                          const Fn &fn) {
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (C == 64) {
        for (int u = first + step * w; u < count; u += step * W)
            F::with(c, limb(u), [&](const auto &f) { fn(u, lane, f); });
    } else {
        constexpr int S = 64 / C;
        for (int u = first + step * (w * S + lane / C); u < count; u += step * W * S)
            F::with_lanes(c, limb(u), [&](const auto &f) { fn(u, lane % C, f); });
    }
}

// Lift of the inputs and pass 0 of their forward transforms: grid (n/16/C,
// npoly, items).  The Q rows go straight through pass 0, the lifted P rows
// through LDS.
template <int L, class F, int C, int W, int H>
__global__ __launch_bounds__(64 * W) void k_col_lift(DevCtx c, const uint64_t *__restrict__ a,
                                                     const uint64_t *__restrict__ b, uint64_t *__restrict__ X,
                                                     int npoly) {
    constexpr int n = Geo<L>::N, T = Geo<L>::T;
    extern __shared__ uint64_t shared_words[];
    ColShared<C, 1> &sh = *(ColShared<C, 1> *)shared_words;
    const int k = c.k, kp = c.kp, K = c.K, poly = (int)blockIdx.y, c0 = (int)blockIdx.x * C;
    const size_t item = blockIdx.z;
    const uint64_t *src = poly < 2 ? a + (item * 2 + poly) * (size_t)k * n : b + (item * 2 + poly - 2) * (size_t)k * n;
    uint64_t *dst = X + (item * npoly + poly) * (size_t)K * n;
    const uint32_t lane = threadIdx.x & 63u, col = lane & 15u, g = lane >> 4;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    mx_stage_table(sh.mx, 0, c.mx->a_lift);
    mx_stage_lift_slots(sh.mx, c);
    if (threadIdx.x == 0) sh.mx.count = 0;
    __syncthreads();
    const int a16 = (int)((lane ^ 16u) << 2), a32 = (int)((lane ^ 32u) << 2);
    uint32_t rq[H];
    bool jv[H];
#pragma unroll
    for (int h = 0; h < H; h++) {
        rq[h] = mx_row((int)g + 4 * h, k, 0, n);
        jv[h] = (int)g + 4 * h < kp;
    }
    for (int t = w; t < C; t += W) {  // tile: stride e, 16 columns
        const int e = t / (C / 16), cc = t % (C / 16) * 16 + (int)col;
        const uint64_t *s0 = src + e * T + c0 + cc;
        uint64_t x[H], r[H];
#pragma unroll
        for (int h = 0; h < H; h++) x[h] = s0[rq[h]];
        if (mx_lift_tile<H>(sh.mx, lane, a16, a32, x, r)) {
#pragma unroll
            for (int h = 0; h < H; h++)
                if (jv[h]) sh.rows[g + 4 * h][e][cc] = r[h];
        } else if (g == 0) {
            sh.mx.item[atomicAdd(&sh.mx.count, 1)] = e * C + cc;
        }
    }
    auto limb_q = [](int l) { return l; };
    col_units<F, C, W>(c, 0, 1, k, limb_q, [&](int l, int cl, const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
        const uint64_t *row = src + (size_t)l * n + c0 + cl;
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = f.in(row[s * T]);
        fwd_pass_t<L, 0, 1>(x, 0, f, TwGlobal<typename Fd::T>{f.tw});
        uint64_t *o = dst + (size_t)l * n + c0 + cl;
#pragma unroll
        for (int s = 0; s < 16; s++) o[s * T] = Fd::to_bits(x[0][s]);
    });
    __syncthreads();
    const int cnt = sh.mx.count;
    if (cnt) {  // the same in the whole workgroup
        for (int i = (int)threadIdx.x; i < cnt; i += 64 * W) {
            const int e = sh.mx.item[i] / C, cc = sh.mx.item[i] % C;
            uint64_t xa[FHE_MX_MAXB];
#pragma unroll
            for (int l = 0; l < FHE_MX_MAXB; l++) xa[l] = l < k ? src[(size_t)l * n + e * T + c0 + cc] : 0;
            lift_exact<FHE_MX_MAXB, FHE_MX_MAXB, false>(c, xa, [&](int j, uint64_t r) { sh.rows[j][e][cc] = r; });
        }
        __syncthreads();
    }
    auto limb_p = [k](int l) { return k + l; };
    col_units<F, C, W>(c, 0, 1, kp, limb_p, [&](int l, int cl, const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = f.in(sh.rows[l][s][cl]);
        fwd_pass_t<L, 0, 1>(x, 0, f, TwGlobal<typename Fd::T>{f.tw});
        uint64_t *o = dst + (size_t)(k + l) * n + c0 + cl;
#pragma unroll
        for (int s = 0; s < 16; s++) o[s * T] = Fd::to_bits(x[0][s]);
    });
}

// Pass 0 of the inverse transforms of the tensor rows, scale-and-round, and
// pass 0 of the digits: grid (n/16/C, 2 + J, items).  blockIdx.y 0, 1:
// components 0, 1 into out.  2 + p: component 2 (computed by each of the J
// parts), whose digits p, p + J, ... of the k^2 (digit, prime) pairs go to D
// [item][digit][prime] (field DF of the key switching); D null: the component itself to C2 (J = 1).
template <int L, class F, class DF, bool RAW, int C, int W, int H>
__global__ __launch_bounds__(64 * W) void k_col_scale(DevCtx c, const uint64_t *__restrict__ Dt,
                                                      uint64_t *__restrict__ out, uint64_t *__restrict__ C2,
                                                      uint64_t *__restrict__ D, int J) {
    constexpr int n = Geo<L>::N, T = Geo<L>::T;
    extern __shared__ uint64_t shared_words[];
    ColShared<C, 3> &sh = *(ColShared<C, 3> *)shared_words;
    const int k = c.k, kp = c.kp, K = c.K, c0 = (int)blockIdx.x * C;
    const int comp = blockIdx.y < 2 ? (int)blockIdx.y : 2, part = (int)blockIdx.y - 2;
    const size_t item = blockIdx.z;
    const uint64_t *src = Dt + (item * 3 + comp) * (size_t)K * n + c0;
    uint64_t *dst = (comp < 2 ? out + (item * 2 + comp) * (size_t)k * n : C2 + item * (size_t)k * n) + c0;
    const bool digits = comp == 2 && D;
    const uint32_t lane = threadIdx.x & 63u, col = lane & 15u, g = lane >> 4;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    mx_stage_table(sh.mx, 0, c.mx->a_scale);
    mx_stage_table(sh.mx, 1, c.mx->a_p2q);
    mx_stage_table(sh.mx, 2, c.mx->a_sdp);
    mx_stage_scale_slots(sh.mx, c);
    if (threadIdx.x == 0) sh.mx.count = 0;
    col_units<F, C, W>(c, 0, 1, K, [](int l) { return l; }, [&](int l, int cl, const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
        const uint64_t *row = src + (size_t)l * n + cl;
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(row[s * T]);
        inv_pass_t<L, 0, 1>(x, 0, f, TwGlobal<typename Fd::T>{f.itw});
#pragma unroll
        for (int s = 0; s < 16; s++) sh.rows[l][s][cl] = f.tensor_out(x[0][s]);
    });
    __syncthreads();
    const int a16 = (int)((lane ^ 16u) << 2), a32 = (int)((lane ^ 32u) << 2);
    int sq[H], sp[H];
    bool iv[H], jv[H];
#pragma unroll
    for (int h = 0; h < H; h++) {
        const int s = (int)g + 4 * h;
        iv[h] = s < k;
        jv[h] = s < kp;
        sq[h] = s < k ? s : k - 1;  // absent primes read a present row (their constants are zero)
        sp[h] = k + (s < kp ? s : kp - 1);
    }
    for (int t = w; t < C; t += W) {
        const int e = t / (C / 16), cc = t % (C / 16) * 16 + (int)col;
        uint64_t dq[H], dp[H], r[H];
#pragma unroll
        for (int h = 0; h < H; h++) {
            dq[h] = sh.rows[sq[h]][e][cc];
            dp[h] = sh.rows[sp[h]][e][cc];
        }
        if (mx_scale_tile<H>(sh.mx, lane, a16, a32, dq, dp, jv, r)) {
#pragma unroll
            for (int h = 0; h < H; h++) {
                if (iv[h]) {
                    // a tile's words are read by this wave alone, before it writes them
                    if (digits) sh.rows[g + 4 * h][e][cc] = r[h];
                    else dst[(size_t)(g + 4 * h) * n + e * T + cc] = r[h];
                }
            }
        } else if (g == 0) {
            sh.mx.item[atomicAdd(&sh.mx.count, 1)] = e * C + cc;
        }
    }
    __syncthreads();
    const int cnt = sh.mx.count;
    if (cnt) {
        for (int i = (int)threadIdx.x; i < cnt; i += 64 * W) {
            const int e = sh.mx.item[i] / C, cc = sh.mx.item[i] % C;
            uint64_t dqa[FHE_MX_MAXB], dpa[FHE_MX_MAXB];
#pragma unroll
            for (int l = 0; l < FHE_MX_MAXB; l++) {
                dqa[l] = l < k ? sh.rows[l][e][cc] : 0;
                dpa[l] = l < kp ? sh.rows[k + l][e][cc] : 0;
            }
            scale_exact<FHE_MX_MAXB, FHE_MX_MAXB, false>(c, dqa, dpa, [&](int l, uint64_t r) {
                if (digits) sh.rows[l][e][cc] = r;
                else dst[(size_t)l * n + e * T + cc] = r;
            });
        }
        __syncthreads();
    }
    if (!digits) return;
    col_units<DF, C, W>(c, part, J, k * k, [k](int u) { return u % k; }, [&](int u, int cl, const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = f.template digit<RAW>(sh.rows[u / k][s][cl]);
        fwd_pass_t<L, 0, 1>(x, 0, f, TwGlobal<typename Fd::T>{f.tw});
        uint64_t *o = D + (item * k * k + u) * (size_t)n + c0 + cl;
#pragma unroll
        for (int s = 0; s < 16; s++) o[s * T] = Fd::to_bits(x[0][s]);
    });
}

// grid (column groups, K npoly, items)
template <int L, class F>
__global__ __launch_bounds__(kColThreads) void k_split_fwd(DevCtx c, const uint64_t *__restrict__ a,
                                                           const uint64_t *__restrict__ b, const uint64_t *E,
                                                           uint64_t *X, int npoly) {
    constexpr int n = Geo<L>::N;
    const uint32_t tid = blockIdx.x * kColThreads + threadIdx.x;
    const int k = c.k, K = c.K;
    const int poly = (int)blockIdx.y / K, limb = (int)blockIdx.y % K;
    const size_t item = blockIdx.z;
    const size_t row = ((item * npoly + poly) * K + limb) * (size_t)n;
    uint64_t *dst = X + row;
    const uint64_t *src = limb < k ? (poly < 2 ? a + ((item * 2 + poly) * k + limb) * (size_t)n
                                               : b + ((item * 2 + poly - 2) * k + limb) * (size_t)n)
                                   : E + row;
    uint64_t v[16];  // in flight while the prime's constants are fetched
#pragma unroll
    for (int s = 0; s < 16; s++) v[s] = src[natural_index<L>(tid, s)];
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = f.in(v[s]);
        fwd_pass_t<L, 0, 1>(x, (int)tid, f, TwGlobal<typename Fd::T>{f.tw});
#pragma unroll
        for (int s = 0; s < 16; s++) dst[natural_index<L>(tid, s)] = Fd::to_bits(x[0][s]);
    });
}

// Loads / stores a block's residues in the pass-1 layout.
template <int L, class F>
__device__ __forceinline__ void load_block(typename F::V (&x)[16], const uint64_t *__restrict__ row, uint32_t tid) {
    const uint32_t t = fresh(tid);
#pragma unroll
    for (int s = 0; s < 16; s++) x[s] = F::from_bits(row[elem_index<L, 4, 1>(t, 0, s)]);
}
template <int L, class F>
__device__ __forceinline__ void store_block(uint64_t *__restrict__ row, const typename F::V (&x)[16], uint32_t tid) {
    const uint32_t t = fresh(tid);
#pragma unroll
    for (int s = 0; s < 16; s++) row[elem_index<L, 4, 1>(t, 0, s)] = F::to_bits(x[s]);
}

// Blocks of one item and limb in one wave: forward transforms of the operands'
// rows (src, row stride rs), tensor product, inverse transforms into dst.
template <int L, class F, bool SQ, class TW>
__device__ __forceinline__ void tensor_block(const F &f, const uint64_t *__restrict__ src, uint64_t *__restrict__ dst,
                                             size_t rs, typename F::V *lds, int lane, uint32_t tid, const TW &tw,
                                             const TW &itw) {
    typedef typename F::V V;
    constexpr int LAST = Geo<L>::NPASS - 1;
    V x[2][16], z[1][16];
    load_block<L, F>(x[0], src, tid);
    load_block<L, F>(x[1], src + rs, tid);
    f.enter_block(x);
    fwd_block_pair<L>(x, lds, lane, (int)tid, f, tw);
    if constexpr (SQ) {
        f.operands(x);
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const V a0 = x[0][s], a1 = x[1][s];
            const V m = f.mul(a0, a1);
            x[0][s] = f.mul(a0, a0);
            x[1][s] = f.mul(a1, a1);
            z[0][s] = f.add2(m, m);
            if constexpr (serial<F, TW>()) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        V y[2][16];
        asm volatile("" ::: "memory");
        load_block<L, F>(y[0], src + 2 * rs, tid);
        load_block<L, F>(y[1], src + 3 * rs, tid);
        f.enter_block(y);
        fwd_block_pair<L>(y, lds, lane, (int)tid, f, tw);
        f.operands(x);
        f.operands(y);
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const V a0 = x[0][s], a1 = x[1][s], b0 = y[0][s], b1 = y[1][s];
            x[0][s] = f.mul(a0, b0);
            z[0][s] = f.add2(f.mul(a0, b1), f.mul(a1, b0));
            x[1][s] = f.mul(a1, b1);
            if constexpr (serial<F, TW>()) __builtin_amdgcn_sched_barrier(0);
        }
    }
    asm volatile("" ::: "memory");
    inv_block_pair<L>(x, lds, lane, (int)tid, f, itw);
    store_block<L, F>(dst, x[0], tid);
    store_block<L, F>(dst + 2 * rs, x[1], tid);
    asm volatile("" ::: "memory");
    inv_block<L, LAST, 1>(z, lds, lane, (int)tid, f, itw);
    store_block<L, F>(dst + rs, z[0], tid);
}

// Few items: grid (K n/1024, items), a workgroup of four waves (three for a
// square) per (limb, block, item): one forward transform per wave, the rows
// meet in LDS, one tensor component and its inverse transform per wave.  A
// single product is bound by latency and instruction fetch: the chain of one
// wave is two transforms instead of seven, over code a third as long (one
// product at n = 16384: 43.9 us with all seven in one wave, 22.2 so).
template <int L, class F, bool SQ>
__global__ __launch_bounds__(256) void k_split_tensor(DevCtx c, const uint64_t *__restrict__ X,
                                                      uint64_t *__restrict__ Dt) {
    typedef typename F::V V;
    typedef TwGlobal<typename F::T> TW;
    constexpr int n = Geo<L>::N, NB = n / 1024, LAST = Geo<L>::NPASS - 1, NP = SQ ? 2 : 4;
    __shared__ V lds[SQ ? 3 : 4][kBlkWords];
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int limb = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, K = c.K;
    const uint32_t tid = 64u * blk + lane;
    const size_t item = blockIdx.y;
    uint64_t raw[16];  // in flight while the prime's constants are fetched
    if (w < NP) {
        const uint64_t *row = X + ((item * NP + w) * K + limb) * (size_t)n;
#pragma unroll
        for (int s = 0; s < 16; s++) raw[s] = row[elem_index<L, 4, 1>(tid, 0, s)];
    }
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        V x[1][16];
        if (w < NP) {
#pragma unroll
            for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(raw[s]);
            f.enter_block(x);
            fwd_block<L, 1, 1>(x, lds[w], lane, (int)tid, f, TW{f.tw});
            f.operands(x);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < 16; s++) lds[w][s * 64 + lane] = x[0][s];
        }
        __syncthreads();
        // rows a0, a1 (, b0, b1): component 0 = a0 b0, 1 = a0 b1 + a1 b0, 2 = a1 b1
        const V *a0 = lds[0], *a1 = lds[1], *b0 = SQ ? lds[0] : lds[2], *b1 = SQ ? lds[1] : lds[3];
        if (w == 1) {
#pragma unroll
            for (int s = 0; s < 16; s++) {
                const int o = s * 64 + lane;
                const V m = f.mul(a0[o], b1[o]);
                x[0][s] = f.add2(m, SQ ? m : f.mul(a1[o], b0[o]));
            }
        } else if (w < 3) {
            const V *u = w ? a1 : a0, *v = w ? b1 : b0;
#pragma unroll
            for (int s = 0; s < 16; s++) x[0][s] = f.mul(u[s * 64 + lane], v[s * 64 + lane]);
        }
        __syncthreads();
        if (w < 3) {
            inv_block<L, LAST, 1>(x, lds[w], lane, (int)tid, f, TW{f.itw});
            store_block<L, Fd>(Dt + ((item * 3 + w) * K + limb) * (size_t)n, x[0], tid);
        }
    });
}

// Many items: grid (K n/1024, item groups) of W waves; the waves of a workgroup
// share one block and limb, whose twiddles they read from LDS, and take the
// items group, group + gridDim.y, ... W at a time.
template <int L, class F, bool SQ, int W>
__global__ __launch_bounds__(64 * W) void k_split_tensor_many(DevCtx c, const uint64_t *__restrict__ X,
                                                              uint64_t *__restrict__ Dt, size_t items) {
    typedef TwBlock<typename F::T> TW;
    constexpr int n = Geo<L>::N, NB = n / 1024, TE = tw_block_entries<L>();
    __shared__ typename F::T tws[2][TE];
    __shared__ typename F::V lds[W][kBlkWords];
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t wpg = blockDim.x >> 6;  // waves: W or fewer
    const int limb = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, K = c.K;
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws[0], f.tw, blk);
        tw_stage<L, 1>(tws[1], f.itw, blk);
        __syncthreads();
        for (size_t item = blockIdx.y * wpg + w; item < items; item += gridDim.y * wpg)
            tensor_block<L, Fd, SQ>(f, X + (item * (SQ ? 2 : 4) * K + limb) * (size_t)n,
                                    Dt + (item * 3 * K + limb) * (size_t)n, (size_t)K * n, lds[w], lane,
                                    64u * blk + fresh(lane), TW{f.tw, tws[0], (uint32_t)blk},
                                    TW{f.itw, tws[1], (uint32_t)blk});
    });
}

// Operands kept transformed (the powers of the bridge): k_split_ops finishes
// the forward transforms in place, operands' values ready for products;
// k_split_pre2 multiplies two of them and runs the inverse's block part.  Grids
// (K n/1024, item groups) of W waves as for k_split_tensor_many.
template <int L, class F, int W>
__global__ __launch_bounds__(64 * W) void k_split_ops(DevCtx c, uint64_t *__restrict__ X, size_t items) {
    typedef typename F::V V;
    typedef TwBlock<typename F::T> TW;
    constexpr int n = Geo<L>::N, NB = n / 1024, TE = tw_block_entries<L>();
    __shared__ typename F::T tws[TE];
    __shared__ V lds[W][kBlkWords];
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t wpg = blockDim.x >> 6;  // waves: W or fewer
    const int limb = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, K = c.K;
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws, f.tw, blk);
        __syncthreads();
        const TW tw{f.tw, tws, (uint32_t)blk};
        for (size_t item = blockIdx.y * wpg + w; item < items; item += gridDim.y * wpg) {
            const uint32_t tid = 64u * blk + fresh(lane);
            uint64_t *row = X + (item * 2 * K + limb) * (size_t)n;
            V x[2][16];
            load_block<L, Fd>(x[0], row, tid);
            load_block<L, Fd>(x[1], row + (size_t)K * n, tid);
            f.enter_block(x);
            fwd_block_pair<L>(x, lds[w], lane, (int)tid, f, tw);
            f.operands(x);
            // lane order: only k_split_pre2 reads these
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int s = 0; s < 16; s++)
                    row[(size_t)p * K * n + blk * 1024u + s * 64u + lane] = Fd::to_bits(x[p][s]);
        }
    });
}

template <int L, class F, int W>
__global__ __launch_bounds__(64 * W) void k_split_pre2(DevCtx c, const uint64_t *__restrict__ Ahat, size_t na,
                                                       size_t item0, const uint64_t *__restrict__ Bhat,
                                                       uint64_t *__restrict__ Dt, size_t items) {
    typedef typename F::V V;
    typedef TwBlock<typename F::T> TW;
    constexpr int n = Geo<L>::N, NB = n / 1024, TE = tw_block_entries<L>(), LAST = Geo<L>::NPASS - 1;
    __shared__ typename F::T tws[TE];
    __shared__ V lds[W][kBlkWords];
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t wpg = blockDim.x >> 6;  // waves: W or fewer
    const int limb = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, K = c.K;
    const size_t rs = (size_t)K * n;
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws, f.itw, blk);
        __syncthreads();
        const TW itw{f.itw, tws, (uint32_t)blk};
        for (size_t item = blockIdx.y * wpg + w; item < items; item += gridDim.y * wpg) {
            const uint32_t tid = 64u * blk + fresh(lane);
            const size_t o = (size_t)limb * n + blk * 1024u + fresh(lane);
            const uint64_t *a = Ahat + ((item0 + item) % na) * 2 * rs + o, *b = Bhat + (item0 + item) * 2 * rs + o;
            V x[2][16], z[1][16];
#pragma unroll
            for (int s = 0; s < 16; s++) {
                const V a0 = Fd::from_bits(a[s * 64]), a1 = Fd::from_bits(a[rs + s * 64]);
                const V b0 = Fd::from_bits(b[s * 64]), b1 = Fd::from_bits(b[rs + s * 64]);
                x[0][s] = f.mul(a0, b0);
                z[0][s] = f.add2(f.mul(a0, b1), f.mul(a1, b0));
                x[1][s] = f.mul(a1, b1);
                if constexpr (serial<Fd, TW>()) __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("" ::: "memory");
            uint64_t *dst = Dt + (item * 3 * K + limb) * (size_t)n;
            inv_block_pair<L>(x, lds[w], lane, (int)tid, f, itw);
            store_block<L, Fd>(dst, x[0], tid);
            store_block<L, Fd>(dst + 2 * rs, x[1], tid);
            asm volatile("" ::: "memory");
            inv_block<L, LAST, 1>(z, lds[w], lane, (int)tid, f, itw);
            store_block<L, Fd>(dst + rs, z[0], tid);
        }
    });
}

// grid (column groups, 3 K, items): rows of Dt [item][comp][limb], in place.
template <int L, class F>
__global__ __launch_bounds__(kColThreads) void k_split_inv(DevCtx c, uint64_t *__restrict__ Dt) {
    constexpr int n = Geo<L>::N;
    const uint32_t tid = blockIdx.x * kColThreads + threadIdx.x;
    const int K = c.K, limb = (int)blockIdx.y % K;
    uint64_t *row = Dt + ((size_t)blockIdx.z * 3 * K + blockIdx.y) * (size_t)n;
    uint64_t v[16];
#pragma unroll
    for (int s = 0; s < 16; s++) v[s] = row[natural_index<L>(tid, s)];
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(v[s]);
        inv_pass_t<L, 0, 1>(x, (int)tid, f, TwGlobal<typename Fd::T>{f.itw});
#pragma unroll
        for (int s = 0; s < 16; s++) row[natural_index<L>(tid, s)] = f.tensor_out(x[0][s]);
    });
}

// grid (column groups, k, items): digit i = blockIdx.y modulo every prime j,
// into D[item][i][j].
template <int L, class F, bool RAW>
__global__ __launch_bounds__(kColThreads) void k_split_digits(DevCtx c, const uint64_t *__restrict__ C2,
                                                              uint64_t *__restrict__ D, int jper) {
    constexpr int n = Geo<L>::N;
    const uint32_t tid = blockIdx.x * kColThreads + threadIdx.x;
    const int k = c.k, parts = (k + jper - 1) / jper;
    const int i = (int)blockIdx.y / parts, j0 = (int)blockIdx.y % parts * jper;
    const int j1 = j0 + jper < k ? j0 + jper : k;
    const size_t item = blockIdx.z;
    const uint64_t *src = C2 + (item * k + i) * (size_t)n;
    uint64_t v[16];
#pragma unroll
    for (int s = 0; s < 16; s++) v[s] = src[natural_index<L>(tid, s)];
    for (int j = j0; j < j1; j++) {
        uint64_t *dst = D + ((item * k + i) * k + j) * (size_t)n;
        F::with(c, j, [&](const auto &f) {
            typedef std::decay_t<decltype(f)> Fd;
            typename Fd::V x[1][16];
#pragma unroll
            for (int s = 0; s < 16; s++) x[0][s] = f.template digit<RAW>(v[s]);
            fwd_pass_t<L, 0, 1>(x, (int)tid, f, TwGlobal<typename Fd::T>{f.tw});
#pragma unroll
            for (int s = 0; s < 16; s++) dst[natural_index<L>(tid, s)] = Fd::to_bits(x[0][s]);
        });
    }
}

__device__ __forceinline__ void lds_add(uint64_t *p, uint64_t v) {
    atomicAdd((unsigned long long *)p, (unsigned long long)v);
}
__device__ __forceinline__ void lds_add(double *p, double v) { unsafeAtomicAdd(p, v); }

// acc[l] += (block of digit row x) * key rows r0, r1.
template <int L, class F, class TW>
__device__ __forceinline__ void digit_block(const F &f, const uint64_t *__restrict__ row,
                                            const uint64_t *__restrict__ r0, const uint64_t *__restrict__ r1,
                                            typename F::V (&acc)[2][16], int cnt, typename F::V *lds, int lane,
                                            uint32_t tid, const TW &tw) {
    typedef typename F::V V;
    V x[1][16];
    load_block<L, F>(x[0], row, tid);
    f.enter_block(x);
    fwd_block<L, 1, 1>(x, lds, lane, (int)tid, f, tw);
    f.key_operands(x);
    f.acc_mid(acc, cnt);
    // the key words of slots s + 2, s + 3 in flight while s, s + 1 are multiplied
    const uint32_t t1 = fresh(tid);
    uint64_t ka[4], kb[4];
#pragma unroll
    for (int u = 0; u < 2; u++) {
        ka[u] = r0[bitrev_layout_index<L>(t1, u)];
        kb[u] = r1[bitrev_layout_index<L>(t1, u)];
    }
#pragma unroll
    for (int s = 0; s < 16; s += 2) {
        if (s + 2 < 16) {
#pragma unroll
            for (int u = 0; u < 2; u++) {
                ka[2 + u] = r0[bitrev_layout_index<L>(t1, s + 2 + u)];
                kb[2 + u] = r1[bitrev_layout_index<L>(t1, s + 2 + u)];
            }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const V v = x[0][s + u];
            acc[0][s + u] = f.acc(acc[0][s + u], v, f.key(ka[u]));
            acc[1][s + u] = f.acc(acc[1][s + u], v, f.key(kb[u]));
            ka[u] = ka[2 + u];
            kb[u] = kb[2 + u];
        }
    }
}

template <class V>
__device__ __forceinline__ void zero2(V (&acc)[2][16]) {
#pragma unroll
    for (int s = 0; s < 16; s++) {
        acc[0][s] = V(0);
        acc[1][s] = V(0);
    }
}

// Few items: grid (k n/1024, items), blockDim 64 W: prime j, block and item of
// the workgroup; wave w takes digits w, w + W, ...; the waves' sums meet in LDS
// (integers, or doubles holding integers below 2^53: any order gives the same
// sum) and waves 0 and 1 finish one component each.  Dynamic LDS: W blocks and
// 2048 words of sums.
template <int L, class F>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_split_relin(
    DevCtx c, const uint64_t *__restrict__ D, const uint64_t *__restrict__ rlk, uint64_t *__restrict__ R) {
    typedef typename F::V V;
    constexpr int n = Geo<L>::N, NB = n / 1024, LAST = Geo<L>::NPASS - 1;
    extern __shared__ uint64_t shared_words[];
    const int lane = threadIdx.x & 63;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = (int)(blockDim.x >> 6);
    V *lds = (V *)shared_words + w * kBlkWords;
    V *sums = (V *)shared_words + W * kBlkWords;
    const int j = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, k = c.k;
    const uint32_t tid = 64u * blk + lane;
    const size_t item = blockIdx.y;
    for (int s = threadIdx.x; s < 2048; s += blockDim.x) sums[s] = V(0);
    __syncthreads();
    F::with(c, j, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        const TwGlobal<typename Fd::T> tw{f.tw}, itw{f.itw};
        V acc[2][16];
        zero2(acc);
        int cnt = 0;
        for (int i = w; i < k; i += W, cnt++)
            digit_block<L, Fd>(f, D + ((item * k + i) * k + j) * (size_t)n, rlk + (((size_t)i * 2 + 0) * k + j) * n,
                               rlk + (((size_t)i * 2 + 1) * k + j) * n, acc, cnt, lds, lane, tid, tw);
#pragma unroll
        for (int s = 0; s < 16; s++) {
            lds_add(&sums[s * 64 + lane], acc[0][s]);
            lds_add(&sums[1024 + s * 64 + lane], acc[1][s]);
        }
        __syncthreads();
        if (w < 2) {
            V y[1][16];
#pragma unroll
            for (int s = 0; s < 16; s++) y[0][s] = f.acc_out(sums[w * 1024 + s * 64 + lane]);
            inv_block<L, LAST, 1>(y, lds, lane, (int)tid, f, itw);
            store_block<L, Fd>(R + ((item * 2 + w) * k + j) * (size_t)n, y[0], tid);
        }
    });
}

// Many items: grid (k n/1024, item groups) of W waves, each with items of its
// own; prime j and block of the workgroup, whose twiddles are read from LDS and
// whose key rows the waves share through the caches.
template <int L, class F, int W>
__global__ __launch_bounds__(64 * W) void k_split_relin_many(DevCtx c, const uint64_t *__restrict__ D,
                                                             const uint64_t *__restrict__ rlk, uint64_t *__restrict__ R,
                                                             size_t items) {
    typedef typename F::V V;
    typedef TwBlock<typename F::T> TW;
    constexpr int n = Geo<L>::N, NB = n / 1024, LAST = Geo<L>::NPASS - 1, TE = tw_block_entries<L>();
    __shared__ typename F::T tws[2][TE];
    __shared__ V lds[W][kBlkWords];
    const int lane = threadIdx.x & 63, w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t wpg = blockDim.x >> 6;  // waves: W or fewer
    const int j = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, k = c.k;
    F::with(c, j, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws[0], f.tw, blk);
        tw_stage<L, 1>(tws[1], f.itw, blk);
        __syncthreads();
        const TW tw{f.tw, tws[0], (uint32_t)blk}, itw{f.itw, tws[1], (uint32_t)blk};
        for (size_t item = blockIdx.y * wpg + w; item < items; item += gridDim.y * wpg) {
            const uint32_t tid = 64u * blk + fresh(lane);
            V acc[2][16];
            zero2(acc);
            for (int i = 0; i < k; i++)
                digit_block<L, Fd>(f, D + ((item * k + i) * k + j) * (size_t)n,
                                   rlk + (((size_t)i * 2 + 0) * k + j) * n, rlk + (((size_t)i * 2 + 1) * k + j) * n,
                                   acc, i, lds[w], lane, tid, tw);
#pragma unroll
            for (int s = 0; s < 16; s++) {
                acc[0][s] = f.acc_out(acc[0][s]);
                acc[1][s] = f.acc_out(acc[1][s]);
            }
            inv_block_pair<L>(acc, lds[w], lane, (int)tid, f, itw);
            uint64_t *row = R + (item * 2 * k + j) * (size_t)n;
            store_block<L, Fd>(row, acc[0], tid);
            store_block<L, Fd>(row + (size_t)k * n, acc[1], tid);
        }
    });
}

// grid (column groups, 2 k, items): out += rows of R [item][comp][limb].
template <int L, class F>
__global__ __launch_bounds__(kColThreads) void k_split_fin(DevCtx c, const uint64_t *__restrict__ R,
                                                           uint64_t *__restrict__ out) {
    constexpr int n = Geo<L>::N;
    const uint32_t tid = blockIdx.x * kColThreads + threadIdx.x;
    const int k = c.k, limb = (int)blockIdx.y % k;
    const size_t o = ((size_t)blockIdx.z * 2 * k + blockIdx.y) * (size_t)n;
    const uint64_t q = c.pc[limb].q;
    // both inputs in flight while the prime's constants are fetched
    uint64_t v[16], a[16];
#pragma unroll
    for (int s = 0; s < 16; s++) v[s] = R[o + natural_index<L>(tid, s)];
#pragma unroll
    for (int s = 0; s < 16; s++) a[s] = out[o + natural_index<L>(tid, s)];
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(v[s]);
        inv_pass_t<L, 0, 1>(x, (int)tid, f, TwGlobal<typename Fd::T>{f.itw});
#pragma unroll
        for (int s = 0; s < 16; s++)
            out[o + natural_index<L>(tid, s)] = add_mod(f.relin_out(x[0][s]), a[s], q);
    });
}

// A workgroup of W waves fills a CU (its LDS): item groups for about one
// workgroup per CU, which then keeps its twiddles and its waves until the end.
// Its waves: W, or as many as give every wave of every group the same number of
// items (16 items of key switching at n = 16384 on two groups: eight waves each,
// not twelve and four).
struct ManyShape {
    dim3 grid, block;
};
template <int W>
ManyShape many_shape(size_t cols, size_t items) {
    const size_t most = (items + W - 1) / W, fit = cols < 256 ? 256 / cols : 1, y = fit < most ? fit : most;
    const size_t per = (items + y - 1) / y, rounds = (per + W - 1) / W, waves = (per + rounds - 1) / rounds;
    return {dim3((unsigned)cols, (unsigned)y), dim3((unsigned)(64 * waves))};
}

// ---- launches --------------------------------------------------------------------

template <int L>
struct SplitL {
    static constexpr unsigned CG = col_groups<L>(), NB = Geo<L>::N / 1024;

    // fn(field family of the tensor rows)
    template <class Fn>
    static hipError_t tensor_field(const DevCtx &c, const Fn &fn) {
        if (c.f64) fn(FamF());
        else if (c.lazy_all) fn(FamU<true>());
        else fn(FamM());
        return hipGetLastError();
    }
    // fn(field family of key switching, digits enter as they are)
    template <class Fn>
    static hipError_t digit_field(const DevCtx &c, const Fn &fn) {
        if (c.f64) fn(FamF(), std::false_type());
        else if (c.digit_raw) fn(FamU<true>(), std::true_type());
        else fn(FamU<true>(), std::false_type());
        return hipGetLastError();
    }

    static hipError_t fwd(const DevCtx &c, const uint64_t *a, const uint64_t *b, const uint64_t *E, uint64_t *X,
                          int npoly, size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            hipLaunchKernelGGL((k_split_fwd<L, decltype(fam)>), dim3(CG, c.K * npoly, (unsigned)items),
                               dim3(kColThreads), 0, s, c, a, b, E, X, npoly);
        });
    }
    static hipError_t blocks(const DevCtx &c, const uint64_t *X, uint64_t *Dt, bool sq, size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            typedef decltype(fam) F;
            constexpr int W = 12;
            if (items * c.K * NB <= kFewBlocks) {
                const dim3 grid(c.K * NB, (unsigned)items);
                if (sq) hipLaunchKernelGGL((k_split_tensor<L, F, true>), grid, dim3(192), 0, s, c, X, Dt);
                else hipLaunchKernelGGL((k_split_tensor<L, F, false>), grid, dim3(256), 0, s, c, X, Dt);
            } else if (sq) {
                const ManyShape g = many_shape<W>(c.K * NB, items);
                hipLaunchKernelGGL((k_split_tensor_many<L, F, true, W>), g.grid, g.block, 0, s, c, X, Dt, items);
            } else {
                const ManyShape g = many_shape<W>(c.K * NB, items);
                hipLaunchKernelGGL((k_split_tensor_many<L, F, false, W>), g.grid, g.block, 0, s, c, X, Dt, items);
            }
        });
    }
    // W waves per workgroup: as many as share a CU where the blocks fill it,
    // fewer for small launches, which then spread over more CUs.
    static hipError_t fwd_blocks(const DevCtx &c, uint64_t *X, size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            typedef decltype(fam) F;
            if (items * c.K * NB <= kFewBlocks) {
                hipLaunchKernelGGL((k_split_ops<L, F, 4>), dim3(c.K * NB, (unsigned)((items + 3) / 4)), dim3(256), 0,
                                   s, c, X, items);
            } else {
                const ManyShape g = many_shape<12>(c.K * NB, items);
                hipLaunchKernelGGL((k_split_ops<L, F, 12>), g.grid, g.block, 0, s, c, X, items);
            }
        });
    }
    static hipError_t pre2(const DevCtx &c, const uint64_t *Ahat, size_t na, size_t item0, const uint64_t *Bhat,
                           uint64_t *Dt, size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            typedef decltype(fam) F;
            if (items * c.K * NB <= kFewBlocks) {
                hipLaunchKernelGGL((k_split_pre2<L, F, 4>), dim3(c.K * NB, (unsigned)((items + 3) / 4)), dim3(256), 0,
                                   s, c, Ahat, na, item0, Bhat, Dt, items);
            } else {
                const ManyShape g = many_shape<12>(c.K * NB, items);
                hipLaunchKernelGGL((k_split_pre2<L, F, 12>), g.grid, g.block, 0, s, c, Ahat, na, item0, Bhat, Dt,
                                   items);
            }
        });
    }
    static hipError_t inv(const DevCtx &c, uint64_t *Dt, size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            hipLaunchKernelGGL((k_split_inv<L, decltype(fam)>), dim3(CG, 3 * c.K, (unsigned)items), dim3(kColThreads),
                               0, s, c, Dt);
        });
    }
    static hipError_t digits(const DevCtx &c, const uint64_t *C2, uint64_t *D, size_t items, hipStream_t s) {
        // few items: one thread group per (digit, prime); many: one pass over C2
        const size_t k = c.k;
        const int jper = items * k * k * CG <= 1024 ? 1 : (int)k;
        const unsigned parts = (unsigned)((k + jper - 1) / jper);
        return digit_field(c, [&](auto fam, auto raw) {
            hipLaunchKernelGGL((k_split_digits<L, decltype(fam), decltype(raw)::value>),
                               dim3(CG, (unsigned)k * parts, (unsigned)items), dim3(kColThreads), 0, s, c, C2, D,
                               jper);
        });
    }
    static hipError_t relin(const DevCtx &c, const uint64_t *D, const uint64_t *rlk, uint64_t *R, uint64_t *out,
                            size_t items, hipStream_t s) {
        const size_t k = c.k;
        return digit_field(c, [&](auto fam, auto) {
            typedef decltype(fam) F;
            constexpr int WM = 12;
            // More than eight products modulo a prime of 2^47 or more can pass a
            // double's 53 bits: only one wave's sum, reduced on the way, takes them.
            // (Reducing the waves' sums first cost 64 products at n = 4096 1.5 %
            // as a branch, and one at n = 16384 1 % as a kernel of its own.)
            const bool sums_fit = !c.f64 || k <= 8 || !(c.big_limbs & ((1ull << k) - 1));
            if (sums_fit && items * k * NB <= kFewBlocks / 2) {
                const unsigned W = k < 8 ? (k < 2 ? 2 : (unsigned)k) : 8;
                hipLaunchKernelGGL((k_split_relin<L, F>), dim3((unsigned)k * NB, (unsigned)items), dim3(64 * W),
                                   (W * kBlkWords + 2048) * 8, s, c, D, rlk, R);
            } else {
                const ManyShape g = many_shape<WM>(k * NB, items);
                hipLaunchKernelGGL((k_split_relin_many<L, F, WM>), g.grid, g.block, 0, s, c, D, rlk, R, items);
            }
            hipLaunchKernelGGL((k_split_fin<L, F>), dim3(CG, 2 * (unsigned)k, (unsigned)items), dim3(kColThreads), 0,
                               s, c, R, out);
        });
    }

    // Columns per workgroup of the fused column kernels: 64 fill the lanes of
    // the pass-0 parts; 32 where 64 would leave one workgroup per CU (more than
    // 8 rows in LDS), which cannot overlap its loads with its arithmetic; 16 (and
    // 16 waves) for launches too small to fill the chip.
    template <int C, int W, int NT, class Kern, class... A>
    static void launch_col(Kern kern, const DevCtx &c, int limbs, unsigned y, size_t items, hipStream_t s, A... args) {
        const size_t lds = sizeof(ColShared<C, NT>) + (size_t)(limbs - 1) * 16 * C * 8;
        hipLaunchKernelGGL(kern, dim3(Geo<L>::T / C, y, (unsigned)items), dim3(64 * W), lds, s, c, args...);
    }
    template <class F, int H>
    static void lift_fwd_h(const DevCtx &c, const uint64_t *a, const uint64_t *b, uint64_t *X, int npoly, size_t items,
                           hipStream_t s) {
        if (npoly * items * (Geo<L>::T / 64) <= 128)
            launch_col<16, 8, 1>(k_col_lift<L, F, 16, 8, H>, c, c.kp, npoly, items, s, a, b, X, npoly);
        else
            launch_col<64, 8, 1>(k_col_lift<L, F, 64, 8, H>, c, c.kp, npoly, items, s, a, b, X, npoly);
    }
    static hipError_t lift_fwd(const DevCtx &c, const uint64_t *a, const uint64_t *b, uint64_t *X, int npoly,
                               size_t items, hipStream_t s) {
        return tensor_field(c, [&](auto fam) {
            if (c.k <= 4 && c.kp <= 4) lift_fwd_h<decltype(fam), 1>(c, a, b, X, npoly, items, s);
            else lift_fwd_h<decltype(fam), 2>(c, a, b, X, npoly, items, s);
        });
    }
    template <class F, class DF, bool RAW, int H>
    static void inv_scale_h(const DevCtx &c, const uint64_t *Dt, uint64_t *out, uint64_t *C2, uint64_t *D,
                            size_t items, hipStream_t s) {
        if (3 * items * (Geo<L>::T / 64) <= 128) {
            const int J = D && c.k > 3 ? 4 : 1;
            launch_col<16, 8, 3>(k_col_scale<L, F, DF, RAW, 16, 8, H>, c, c.K, 2 + J, items, s, Dt, out, C2, D, J);
        } else {
            constexpr int C = H == 1 ? 64 : 32;  // H = 1: at most 8 rows
            launch_col<C, 8, 3>(k_col_scale<L, F, DF, RAW, C, 8, H>, c, c.K, 3, items, s, Dt, out, C2, D, 1);
        }
    }
    static hipError_t inv_scale(const DevCtx &c, const uint64_t *Dt, uint64_t *out, uint64_t *C2, uint64_t *D,
                                size_t items, hipStream_t s) {
        hipError_t e = hipSuccess;  // of the launch, which digit_field takes from the runtime
        const hipError_t rest = tensor_field(c, [&](auto fam) {
            typedef decltype(fam) F;
            e = digit_field(c, [&](auto dfam, auto raw) {
                typedef decltype(dfam) DF;
                constexpr bool RAW = decltype(raw)::value;
                if constexpr (std::is_same<F, FamF>::value == std::is_same<DF, FamF>::value) {
                    if (c.k <= 4 && c.kp <= 4) inv_scale_h<F, DF, RAW, 1>(c, Dt, out, C2, D, items, s);
                    else inv_scale_h<F, DF, RAW, 2>(c, Dt, out, C2, D, items, s);
                }
            });
        });
        return e != hipSuccess ? e : rest;
    }
};

}  // namespace

#define FHE_CAT2(a, b) a##b
#define FHE_CAT(a, b) FHE_CAT2(a, b)
const SplitOps *FHE_CAT(split_ops_, FHE_NTT_L)() {
    typedef SplitL<FHE_NTT_L> S;
    static const SplitOps o = {S::lift_fwd, S::fwd,       S::blocks, S::fwd_blocks, S::pre2,
                               S::inv,      S::inv_scale, S::digits, S::relin};
    return &o;
}
