// Exact top lists and 16-lane row rotations shared by the kernels that select
// a working set (k_select, one launch per outer iteration; k_resident, the
// whole loop in one launch).  All run on a block of kSelThreads threads.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "device.hpp"

namespace msvm {

// max of two values that are not NaN, in one instruction (fmax quiets each
// operand first)
__device__ __forceinline__ double max_f64(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ double min_f64(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// every lane of each 16-lane row receives the row maximum
__device__ __forceinline__ double rmax_f64(double v)
{
    v = max_f64(v, dpp_f64<kDppRor8>(v));
    v = max_f64(v, dpp_f64<kDppRor4>(v));
    v = max_f64(v, dpp_f64<kDppRor2>(v));
    v = max_f64(v, dpp_f64<kDppRor1>(v));
    return v;
}

// Survivor-list capacity per side of the threshold filter.
constexpr int kSurv = 1024;

// Top `half` of (k[0..M), i[0..M)) in the order of better(), by `half`
// rounds over one wave (entries are distinct (key, index) pairs); lane 0
// writes ok/oi.  The first 256 entries are held in registers.
__device__ inline void wave_top(const double* k, const int32_t* i, int M, int half,
                         double* ok, int32_t* oi, int tid)
{
    const int lane = tid & 63;
    double ck[4];
    int32_t ci[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int e = lane + 64 * j;
        ck[j] = e < M ? k[e] : -INFINITY;
        ci[j] = e < M ? i[e] : INT_MAX;
    }
    double pk = INFINITY;
    int32_t pi = -1;
    for (int r = 0; r < half; ++r) {
        double bk = -INFINITY;
        int32_t bi = INT_MAX;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (after(ck[j], ci[j], pk, pi) && better(ck[j], ci[j], bk, bi)) {
                bk = ck[j];
                bi = ci[j];
            }
        for (int e = lane + 256; e < M; e += 64) {
            const double ke = k[e];
            const int32_t ie = i[e];
            if (after(ke, ie, pk, pi) && better(ke, ie, bk, bi)) {
                bk = ke;
                bi = ie;
            }
        }
        wave_best_fast(bk, bi);
        if (lane == 0) {
            ok[r] = bk;
            oi[r] = bi;
        }
        pk = bk;
        pi = bi;
    }
}

// Largest list (per side) ranked by pairs in one pass.
constexpr int kPairSmall = 64;

// Top `half` of each side's entries (k[s][0..M_s), i[s][0..M_s)), M_s <=
// kSelThreads / LPE, by ranks computed all at once: LPE threads share one
// entry, each compares it with a slice of the others, and a sum over the
// LPE threads gives its rank (the number of entries before it in the order
// of better(); entries are distinct, so ranks are unique).  Run by the
// whole block.
template <int LPE>
__device__ __forceinline__ void pair_rank_top(const double (*k)[kSurv],
                                              const int32_t (*i)[kSurv],
                                              int M0, int M1, int half,
                                              double* ku, int32_t* iu,
                                              double* kl, int32_t* il,
                                              int tid)
{
    constexpr int E = kSelThreads / LPE;  // entries covered
    constexpr int F = E / LPE;            // comparisons per thread
    // thread (e, l) compares entry e with entries l, l + LPE, ...: the
    // LPE lanes of an entry read consecutive entries (no LDS bank
    // conflicts), and the count does not depend on the split
    const int e = tid / LPE, f0 = tid % LPE;
    // first entry of this wave: a wave whose entries are all past a side's
    // list skips that side
    const int e_wave = (tid & ~63) / LPE;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int M = side ? M1 : M0;
        if (e_wave >= M) continue;  // uniform over the wave
        const bool ve = e < M;
        const double ke = k[side][ve ? e : 0];
        const int32_t ie = i[side][ve ? e : 0];
        int c = 0;
#pragma unroll 8
        for (int j = 0; j < F; ++j) {
            const int f = f0 + LPE * j;
            const double kf = k[side][f];
            const int32_t iff = i[side][f];
            c += (f < M && better(kf, iff, ke, ie)) ? 1 : 0;
        }
        if (LPE == 16) {
            c = row_sum_i32(c);
        } else {
#pragma unroll
            for (int o = 1; o < LPE; o <<= 1) c += __shfl_xor(c, o);
        }
        if (ve && tid % LPE == 0 && c < half) {
            (side ? kl : ku)[c] = ke;
            (side ? il : iu)[c] = ie;
        }
    }
}

// the rank of every entry of both sides' lists among its side's, and the
// first `half` of each list into (ku, iu) and (kl, il), their places in the
// lists into pu and pl where given: waves 0 .. 7 take side 0, the others
// side 1, 16 lanes an entry
template <int CAP>
__device__ __forceinline__ void rank_lists(const double (*k)[CAP],
                                           const int32_t (*i)[CAP],
                                           int M0, int M1, int half,
                                           double* ku, int32_t* iu, double* kl,
                                           int32_t* il, int tid,
                                           int32_t* pu = nullptr,
                                           int32_t* pl = nullptr)
{
    const int side = tid >> 9, l = tid & 15;
    const int M = side ? M1 : M0;
    for (int e = (tid & 511) >> 4; e < M; e += 32) {
        const double ke = k[side][e];
        const int32_t ie = i[side][e];
        int c = 0;
#pragma unroll 4
        for (int f = l; f < M; f += 16)
            c += better(k[side][f], i[side][f], ke, ie) ? 1 : 0;
        c = row_sum_i32(c);
        if (l == 0 && c < half) {
            (side ? kl : ku)[c] = ke;
            (side ? il : iu)[c] = ie;
            if (pu) (side ? pl : pu)[c] = e;
        }
    }
}

// Exact top `half` of each side's entries (k[s][0..M_s), i[s][0..M_s)),
// M_s <= kSurv, into (ku, iu) and (kl, il).  A list longer than one pair
// pass ranks cheaply is cut first: the half-th best of its first 64
// entries bounds the half-th best of the whole list from below, so the
// entries at or above it (at least `half` of them) hold the top `half`;
// they are compacted in place and ranked.  Run by the whole block; k and i
// are overwritten.
__device__ __forceinline__ void top_half(double (*k)[kSurv], int32_t (*i)[kSurv], int M0,
                         int M1, int half, double* ku, int32_t* iu, double* kl,
                         int32_t* il, int32_t* shM, int tid)
{
    const int lane = tid & 63;
    if (M0 > kPairSmall || M1 > kPairSmall) {
        pair_rank_top<16>(k, i, min(M0, kPairSmall), min(M1, kPairSmall), half,
                          ku, iu, kl, il, tid);
        if (tid < 2) shM[tid] = 0;
        __syncthreads();
        double ke[2];
        int32_t ie[2];
        bool keep[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int M = side ? M1 : M0;
            const double bk = (side ? kl : ku)[half - 1];
            const int32_t bi = (side ? il : iu)[half - 1];
            const bool in = tid < M;
            ke[side] = in ? k[side][tid] : -INFINITY;
            ie[side] = in ? i[side][tid] : INT_MAX;
            keep[side] = in && (M <= kPairSmall || !after(ke[side], ie[side], bk, bi));
        }
        __syncthreads();  // every entry read before the in-place writes
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const unsigned long long m = __ballot(keep[side]);
            if (m == 0) continue;
            int base = 0;
            if (lane == 0) base = atomicAdd(&shM[side], __popcll(m));
            base = __builtin_amdgcn_readfirstlane(base);
            if (keep[side]) {
                const int pos = base + lanes_below(m);
                k[side][pos] = ke[side];
                i[side][pos] = ie[side];
            }
        }
        __syncthreads();
        M0 = shM[0];
        M1 = shM[1];
    }
    const int lm = max(M0, M1);
    if (lm <= kPairSmall) {
        rank_lists(k, i, M0, M1, half, ku, iu, kl, il, tid);
    } else if (lm <= 2 * kPairSmall) {
        pair_rank_top<8>(k, i, M0, M1, half, ku, iu, kl, il, tid);
    } else {
        const int wave = tid >> 6;
        if (wave == 0) wave_top(k[0], i[0], M0, half, ku, iu, tid);
        if (wave == 1) wave_top(k[1], i[1], M1, half, kl, il, tid);
    }
    __syncthreads();
}

// Exact top-`half` over `count` entries produced by get(e, key, index), by
// `half` block-wide rounds (each: the best entry after the previous winner).
// Up to kRoundRegs entries per thread are fetched once and kept in
// registers; larger counts fetch in every round.  All threads of the block
// take part; thread 0 writes ok/oi.
constexpr int kRoundRegs = 4;
template <class Get>
__device__ void block_rounds(int64_t count, Get get, int half, double* ok,
                             int32_t* oi, double (*rk)[kSelThreads / 64],
                             int32_t (*ri)[kSelThreads / 64])
{
    constexpr int NW = kSelThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool held = count <= (int64_t)kRoundRegs * kSelThreads;
    double hk[kRoundRegs];
    int32_t hi[kRoundRegs];
#pragma unroll
    for (int j = 0; j < kRoundRegs; ++j) {
        const int64_t e = tid + (int64_t)j * kSelThreads;
        hk[j] = -INFINITY;
        hi[j] = INT_MAX;
        if (held && e < count) get(e, hk[j], hi[j]);
    }
    double pk = INFINITY;
    int32_t pi = -1;
    for (int k = 0; k < half; ++k) {
        double bk = -INFINITY;
        int32_t bi = INT_MAX;
        if (held) {
#pragma unroll
            for (int j = 0; j < kRoundRegs; ++j)
                if (after(hk[j], hi[j], pk, pi) && better(hk[j], hi[j], bk, bi)) {
                    bk = hk[j];
                    bi = hi[j];
                }
        } else {
            for (int64_t e = tid; e < count; e += kSelThreads) {
                double key;
                int32_t t;
                get(e, key, t);
                if (after(key, t, pk, pi) && better(key, t, bk, bi)) {
                    bk = key;
                    bi = t;
                }
            }
        }
        wave_best_fast(bk, bi);
        if (lane == 0) {
            rk[k & 1][wave] = bk;
            ri[k & 1][wave] = bi;
        }
        __syncthreads();
        bk = rk[k & 1][0];
        bi = ri[k & 1][0];
        for (int w = 1; w < NW; ++w)
            if (better(rk[k & 1][w], ri[k & 1][w], bk, bi)) {
                bk = rk[k & 1][w];
                bi = ri[k & 1][w];
            }
        pk = bk;
        pi = bi;
        if (tid == 0) {
            ok[k] = bk;
            oi[k] = bi;
        }
    }
    __syncthreads();
}

// Value of the lane R places along this lane's 16-lane row (a row rotate:
// every lane has a source, so none keeps its old value); R = 1 .. 15 meet
// every other lane of the row once.  Needs the whole row active.
template <int R>
__device__ __forceinline__ int row_rot(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x120 + R, 0xF, 0xF, false);
}

template <int R = 1, class Fn>
__device__ __forceinline__ void for_row_rotations(Fn&& fn)
{
    if constexpr (R < 16) {
        fn(std::integral_constant<int, R>{});
        // one rotation at a time (hoisting them all would hold 15 values)
        __builtin_amdgcn_sched_barrier(0);
        for_row_rotations<R + 1>(fn);
    }
}

}  // namespace msvm
