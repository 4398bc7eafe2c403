// Product pipeline on the split transforms (ntt_field.hpp): column kernels run
// radix-16 pass 0 of rows (one thread per 16 residues n/16 apart), block
// kernels run the other passes of 1024 consecutive residues in one wave.
// Rows between the two halves hold field values (lazy integers or doubles).
//
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
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = f.in(src[natural_index<L>(tid, s)]);
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
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        V x[1][16];
        if (w < NP) {
            load_block<L, Fd>(x[0], X + ((item * NP + w) * K + limb) * (size_t)n, tid);
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
    const int limb = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, K = c.K;
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws[0], f.tw, blk);
        tw_stage<L, 1>(tws[1], f.itw, blk);
        __syncthreads();
        for (size_t item = (size_t)blockIdx.y * W + w; item < items; item += (size_t)gridDim.y * W)
            tensor_block<L, Fd, SQ>(f, X + (item * (SQ ? 2 : 4) * K + limb) * (size_t)n,
                                    Dt + (item * 3 * K + limb) * (size_t)n, (size_t)K * n, lds[w], lane,
                                    64u * blk + fresh(lane), TW{f.tw, tws[0], (uint32_t)blk},
                                    TW{f.itw, tws[1], (uint32_t)blk});
    });
}

// grid (column groups, 3 K, items): rows of Dt [item][comp][limb], in place.
template <int L, class F>
__global__ __launch_bounds__(kColThreads) void k_split_inv(DevCtx c, uint64_t *__restrict__ Dt) {
    constexpr int n = Geo<L>::N;
    const uint32_t tid = blockIdx.x * kColThreads + threadIdx.x;
    const int K = c.K, limb = (int)blockIdx.y % K;
    uint64_t *row = Dt + ((size_t)blockIdx.z * 3 * K + blockIdx.y) * (size_t)n;
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(row[natural_index<L>(tid, s)]);
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
    const int j = (int)blockIdx.x / NB, blk = (int)blockIdx.x % NB, k = c.k;
    F::with(c, j, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        tw_stage<L, 1>(tws[0], f.tw, blk);
        tw_stage<L, 1>(tws[1], f.itw, blk);
        __syncthreads();
        const TW tw{f.tw, tws[0], (uint32_t)blk}, itw{f.itw, tws[1], (uint32_t)blk};
        for (size_t item = (size_t)blockIdx.y * W + w; item < items; item += (size_t)gridDim.y * W) {
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
    F::with(c, limb, [&](const auto &f) {
        typedef std::decay_t<decltype(f)> Fd;
        typename Fd::V x[1][16];
#pragma unroll
        for (int s = 0; s < 16; s++) x[0][s] = Fd::from_bits(R[o + natural_index<L>(tid, s)]);
        inv_pass_t<L, 0, 1>(x, (int)tid, f, TwGlobal<typename Fd::T>{f.itw});
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const size_t i = o + natural_index<L>(tid, s);
            out[i] = add_mod(f.relin_out(x[0][s]), out[i], q);
        }
    });
}

// Blocks of a launch up to which it is spread (one transform per wave) instead
// of sharing the twiddles: four workgroups of the spread tensor kernel fill a
// CU about three times over (products at n = 4096, 128 items: 268 against 272
// us; n = 8192, 32: 240 against 248, 64: 463 against 436; n = 16384, 12: 405
// against 419, 15: 516 against 493); key switching has half the blocks.
constexpr size_t kFewBlocks = 3072;

// A workgroup of W waves fills a CU (its LDS): item groups for about one
// workgroup per CU, which then keeps its twiddles and its waves until the end.
template <int W>
dim3 many_grid(size_t cols, size_t items) {
    const size_t most = (items + W - 1) / W, fit = cols < 256 ? 256 / cols : 1;
    return dim3((unsigned)cols, (unsigned)(fit < most ? fit : most));
}

template <int L, class F>
hipError_t split_tensor_f(const DevCtx &c, const uint64_t *a, const uint64_t *b, const uint64_t *E, uint64_t *X,
                          uint64_t *Dt, bool sq, size_t items, hipStream_t s) {
    constexpr unsigned CG = col_groups<L>(), NB = Geo<L>::N / 1024;
    const int npoly = sq ? 2 : 4;
    hipLaunchKernelGGL((k_split_fwd<L, F>), dim3(CG, c.K * npoly, (unsigned)items), dim3(kColThreads), 0, s, c, a, b, E,
                       X, npoly);
    if (items * c.K * NB <= kFewBlocks) {
        const dim3 grid(c.K * NB, (unsigned)items);
        if (sq) hipLaunchKernelGGL((k_split_tensor<L, F, true>), grid, dim3(192), 0, s, c, X, Dt);
        else hipLaunchKernelGGL((k_split_tensor<L, F, false>), grid, dim3(256), 0, s, c, X, Dt);
    } else if (sq) {
        constexpr int W = 12;
        hipLaunchKernelGGL((k_split_tensor_many<L, F, true, W>), many_grid<W>(c.K * NB, items), dim3(64 * W), 0, s, c,
                           X, Dt, items);
    } else {
        constexpr int W = 12;
        hipLaunchKernelGGL((k_split_tensor_many<L, F, false, W>), many_grid<W>(c.K * NB, items), dim3(64 * W), 0, s, c,
                           X, Dt, items);
    }
    hipLaunchKernelGGL((k_split_inv<L, F>), dim3(CG, 3 * c.K, (unsigned)items), dim3(kColThreads), 0, s, c, Dt);
    return hipGetLastError();
}

template <int L>
hipError_t split_tensor(const DevCtx &c, const uint64_t *a, const uint64_t *b, const uint64_t *E, uint64_t *X,
                        uint64_t *Dt, bool sq, size_t items, hipStream_t s) {
    if (c.f64) return split_tensor_f<L, FamF>(c, a, b, E, X, Dt, sq, items, s);
    if (c.lazy_all) return split_tensor_f<L, FamU<true>>(c, a, b, E, X, Dt, sq, items, s);
    return split_tensor_f<L, FamU<false>>(c, a, b, E, X, Dt, sq, items, s);
}

template <int L, class F, bool RAW>
hipError_t split_relin_f(const DevCtx &c, const uint64_t *C2, const uint64_t *rlk, uint64_t *ws, uint64_t *out,
                         size_t items, hipStream_t s) {
    constexpr unsigned CG = col_groups<L>(), NB = Geo<L>::N / 1024;
    const size_t k = c.k;
    uint64_t *D = ws, *R = ws + items * k * k * Geo<L>::N;
    // few items: one thread group per (digit, prime), and the digits of a block
    // spread over waves; many: one pass over C2, one wave per block
    const size_t waves = items * k * NB;
    const int jper = items * k * k * CG <= 1024 ? 1 : (int)k;
    const unsigned parts = (unsigned)((k + jper - 1) / jper);
    hipLaunchKernelGGL((k_split_digits<L, F, RAW>), dim3(CG, (unsigned)k * parts, (unsigned)items), dim3(kColThreads),
                       0, s, c, C2, D, jper);
    if (waves <= kFewBlocks / 2) {
        const unsigned W = k < 8 ? (k < 2 ? 2 : (unsigned)k) : 8;
        hipLaunchKernelGGL((k_split_relin<L, F>), dim3((unsigned)k * NB, (unsigned)items), dim3(64 * W),
                           (W * kBlkWords + 2048) * 8, s, c, D, rlk, R);
    } else {
        constexpr int W = 12;
        hipLaunchKernelGGL((k_split_relin_many<L, F, W>), many_grid<W>(k * NB, items), dim3(64 * W), 0, s, c, D, rlk,
                           R, items);
    }
    hipLaunchKernelGGL((k_split_fin<L, F>), dim3(CG, 2 * (unsigned)k, (unsigned)items), dim3(kColThreads), 0, s, c, R,
                       out);
    return hipGetLastError();
}

template <int L>
hipError_t split_relin(const DevCtx &c, const uint64_t *C2, const uint64_t *rlk, uint64_t *ws, uint64_t *out,
                       size_t items, hipStream_t s) {
    if (c.f64) return split_relin_f<L, FamF, false>(c, C2, rlk, ws, out, items, s);
    if (c.digit_raw) return split_relin_f<L, FamU<true>, true>(c, C2, rlk, ws, out, items, s);
    return split_relin_f<L, FamU<true>, false>(c, C2, rlk, ws, out, items, s);
}

}  // namespace

#define FHE_CAT2(a, b) a##b
#define FHE_CAT(a, b) FHE_CAT2(a, b)
const SplitOps *FHE_CAT(split_ops_, FHE_NTT_L)() {
    static const SplitOps o = {split_tensor<FHE_NTT_L>, split_relin<FHE_NTT_L>};
    return &o;
}
