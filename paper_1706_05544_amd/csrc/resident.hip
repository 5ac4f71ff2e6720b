// The solve loop resident on the GPU (gfx950), for training sets whose whole
// kernel matrix is held in HBM.
//
// k_gram computes every K(x_i, x_j) once, on the matrix cores.  k_resident
// then runs many outer iterations (Section 3: select 16 coefficients,
// optimise them, update the responses) in one launch.  What bounds a small
// solve is not work but the chain of dependent steps of an iteration: two
// launches of about 3 us of gap, the candidate records of a whole grid
// merged through memory, and working-set rows staged before the subproblem
// can start.  Here a problem's rows are dealt to R blocks that stay on their
// compute units: a thread keeps the responses of its rows in registers, the
// block selects from them directly, the 16 kernel rows of the working set
// are requested before the subproblem and arrive while one wave solves it.
// With R > 1 every block selects and solves for itself from the same
// candidates, so one exchange through memory is the only step between
// blocks.
//
// Measured (MI355X, us an outer iteration, two-launch loop -> this): eps-SVR
// 4000 x 50 24.0 -> 8.1 (3 blocks), 1501 x 50 24.6 -> 6.8 (1 block); C-SVC
// 20000 x 128 25.3 -> 13.3 with the 1 ms of k_gram in it (11 blocks).  Of
// the 8.1: update and keys 1.2, bound 0.4, candidates 0.6, rank and exchange
// 1.7, K_BB and alpha (with the working set built beside it) 1.1, curvature
// table 0.7, 6.8 subproblem steps 1.7, results 0.6.
//
// The working sets, the kernel values (the same matrix-core order), the
// subproblem and the fp64 order of the update are those of the two-launch
// loop, so every result has the same bits.
#include "common.hpp"
#include "device.hpp"
#include "resident.hpp"
#include "seltop.hpp"

namespace msvm {

// ---------------------------------------------------------------------------
// the kernel matrix
// ---------------------------------------------------------------------------

// One wave computes a 64 x 64 tile (4 x 4 matrix-core tiles) and a block of
// four waves a 128 x 128 one; only tiles on or above the diagonal are
// computed and each is stored twice (the products and their order are
// symmetric, so K is, bit for bit).  The operands are read straight from
// global memory in the matrix-core layout: a chunk of 16 features feeds 64
// matrix-core instructions (2048 cycles of a SIMD) per 8 KB, which the
// caches sustain without LDS.
constexpr int kGramTile = 128;

__global__ __launch_bounds__(256, 2) void k_gram(const float* X,
                                                 const float* sq, int64_t n,
                                                 int64_t ldp64, KernelFn kf,
                                                 float* K, int64_t ldc)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, nl = lane & 15;
    const int ldp = (int)ldp64;
    // tile (bi, bj), bi <= bj, of the upper triangle: blockIdx.x = bi + bj
    // (bj + 1) / 2
    const int64_t b = blockIdx.x;
    int64_t bj = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    while (bj * (bj + 1) / 2 > b) --bj;
    while ((bj + 1) * (bj + 2) / 2 <= b) ++bj;
    const int64_t bi = b - bj * (bj + 1) / 2;
    // row n: zeros (k_resident reads it for slots that are not used)
    if (bi == bj && tid < kGramTile && bj * kGramTile + tid < ldc)
        K[n * ldc + bj * kGramTile + tid] = 0.0f;
    const int64_t i0 = bi * kGramTile + 64 * (wave >> 1);
    const int64_t j0 = bj * kGramTile + 64 * (wave & 1);
    if (i0 >= n || j0 >= n) return;
    if (bi == bj && i0 > j0) return;  // its mirror image is computed
    const Rsrc rA = make_rsrc(X + i0 * ldp,
                              min((int64_t)64, n - i0) * ldp * 4);
    const Rsrc rB = make_rsrc(X + j0 * ldp,
                              min((int64_t)64, n - j0) * ldp * 4);
    floatx4 acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    float4 av[2][4], bv[2][4];
    auto fetch = [&](int ch, float4 (&x)[4], float4 (&y)[4]) {
        const int col = 16 * ch + 4 * g;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t o = col < ldp
                                   ? (uint32_t)(((16 * t + nl) * ldp + col) * 4)
                                   : kOob;
            x[t] = bld_f4(rA, o);
            y[t] = bld_f4(rB, o);
        }
    };
    const int nch = (ldp + 15) >> 4;
    auto step = [&](const float4 (&x)[4], const float4 (&y)[4]) {
        // (the four features of a chunk in order, 16 independent tiles each)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[r][c] = mfma_chunk(acc[r][c], x[r], y[c]);
    };
    fetch(0, av[0], bv[0]);
    for (int ch = 0; ch < nch; ch += 2) {
        fetch(ch + 1, av[1], bv[1]);  // (zeros past the last chunk)
        step(av[0], bv[0]);
        fetch(ch + 2, av[0], bv[0]);
        if (ch + 1 < nch) step(av[1], bv[1]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int64_t j = j0 + 16 * c + nl;
        const float sj = j < n ? sq[j] : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + 16 * r + 4 * g;
            float kv[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float si = i + v < n ? sq[i + v] : 0.0f;
                kv[v] = (i + v == j && kernel_self_is_one(kf))
                            ? 1.0f
                            : kernel_from_dot(kf, si, sj, acc[r][c][v]);
            }
            // rows are padded to ldc (a multiple of 4): row j, columns i ..
            // i + 3 are inside when i is
            if (j < n && i < n)
                *reinterpret_cast<float4*>(K + j * ldc + i) =
                    make_float4(kv[0], kv[1], kv[2], kv[3]);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (i + v < n && j < n) K[(i + v) * ldc + j] = kv[v];
        }
    }
}

void launch_gram(const float* X, const float* sq, int64_t n, int64_t ldp,
                 const KernelFn& kf, float* K, int64_t ldc, hipStream_t s)
{
    // (byte offsets inside a tile's rows stay below 2^31)
    if (n <= 0) return;
    if (64 * ldp * 4 >= ((int64_t)1 << 31))
        throw Error{SVM_E_INTERNAL, "rows too long for the kernel matrix"};
    const int64_t nt = (n + kGramTile - 1) / kGramTile;
    k_gram<<<(uint32_t)(nt * (nt + 1) / 2), 256, 0, s>>>(X, sq, n, ldp, kf, K,
                                                         ldc);
}

// ---------------------------------------------------------------------------
// the loop
// ---------------------------------------------------------------------------

namespace {

constexpr int kWaves = kSelThreads / 64;
constexpr int kRowWavesRes = kWaves - 1;  // waves that hold rows
// Fields of an exchanged candidate: the two halves of its key, its variable,
// the two halves of its alpha, each the low half of a 64-bit word whose high
// half is the iteration it belongs to.  A block's words: field by field, 16
// lanes each (up winners, then low winners).
constexpr int kXchFields = 5;
constexpr int kXchBlock = kXchFields * 16;
static_assert(kResBlocks * 16 <= kSelThreads, "a thread a candidate");
// candidates per side ranked by pairs (more: rounds over the block)
constexpr int kResCand = 256;

// pointers read from memory, said to be global memory (else they are
// accessed through the flat path, whose loads every LDS wait waits for)
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p)
{
    return (__attribute__((address_space(1))) T*)p;
}
template <class T>
using Glob = __attribute__((address_space(1))) T*;

__device__ __forceinline__ uint64_t agent_load(Glob<const uint64_t> p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void agent_store(Glob<uint64_t> p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Blocks of a problem that start one launch must all be on the chip before
// any of them waits for another: they count themselves in and go on only
// when the last one has said so.  If they do not all arrive in time (other
// work holds the compute units), the launch is called off: one atomic
// decides between the two, so every block of the problem does the same.
// (No time at all: it is called off without being tried.)
__device__ bool resident_start(uint32_t* hs, int R, uint64_t wait)
{
    if (wait == 0) return false;
    const uint32_t old = __hip_atomic_fetch_add(
        &hs[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == (uint32_t)R) {
        uint32_t z = 0;
        __hip_atomic_compare_exchange_strong(&hs[1], &z, 1u, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint64_t t0 = wall_clock64();
    for (;;) {
        const uint32_t st = __hip_atomic_load(&hs[1], __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
        if (st != 0) return st == 1;
        if (wall_clock64() - t0 > wait) {
            uint32_t z = 0;
            __hip_atomic_compare_exchange_strong(
                &hs[1], &z, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

}  // namespace

// Dynamic LDS: the state byte of each of the block's variables (copy (i,-)
// of eps-SVR kResRows bytes later), then the responses of its rows, then the
// alpha of its variables (copies as the state bytes).
//
// Alpha in memory is read before the first iteration and written after the
// last, by the block that holds the variable.  In between a candidate's alpha
// travels with it through the exchange: the words of iteration t hold the
// value before t, and they are not written again before t + 2, so a block
// that is late finds it as it was, however far the owner of the variable has
// got with its own iteration t.  (Read from memory, nothing would order it
// before the owner's store at the end of t.)
//
// Waves 1 .. 15 hold the rows, two consecutive ones a thread, dealt evenly to
// the waves (four rows a thread took 3.1 us for the update and the keys of
// an iteration against 1.2: the instructions of the four waves of a SIMD
// follow one another); wave 0 builds the working set and solves.  While wave
// 0 builds, other waves fetch what the subproblem needs (K_BB, alpha) by
// candidate, so that its memory latency is not on the chain; the 16 kernel
// rows of the update are requested when the working set is known and arrive
// while wave 0 solves.
template <bool SVR>
__global__ __launch_bounds__(kSelThreads) void k_resident(ResidentArgs a)
{
    __shared__ __align__(16) double rmax[2][64];
    __shared__ double theta[2];
    __shared__ double upk[8], lok[8];
    __shared__ int32_t upi[8], loi[8];
    __shared__ double svk[2][kResCand];
    __shared__ int32_t svi[2][kResCand];
    __shared__ int32_t src[2][8];  // R > 1: the winners' places there
    __shared__ int32_t nsv[2];
    __shared__ double rk[2][kWaves];
    __shared__ int32_t ri[2][kWaves];
    __shared__ float kbb[16][17];   // K of candidates a and b
    __shared__ double shAl[16];     // by candidate: alpha, label, used before
    __shared__ float shY[16];
    __shared__ int32_t shSeen[16];
    __shared__ __align__(16) int32_t shCand[16];  // candidate of rank p in B
    __shared__ int32_t shSlot[16];  // by candidate
    __shared__ int32_t shS[16];     // sample of each slot
    __shared__ double2 shCur[16][16];  // curvature of a pair of ranks, 1 / it
    __shared__ double shDc[16];
    __shared__ __align__(16) double shCoef[16];  // slot s at 4 (s % 4) + s / 4
    __shared__ int32_t shNS, shGo;
    __shared__ double shC, shTol, shRatio;
    extern __shared__ __align__(16) uint8_t stl[];
    constexpr int NC = SVR ? 2 : 1;

    const int R = a.R;
    const int prob = blockIdx.x / R, blk = blockIdx.x - prob * R;
    const ResidentProblem& P = a.p[prob];
    WorkingSet* ws = P.ws;
    if (ws->done) return;  // (uniform over the problem's blocks)
    int tid = threadIdx.x, lane = tid & 63;
    int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (R > 1) {
        if (tid == 0) shGo = resident_start(a.hs + 2 * prob, R, a.wait) ? 1 : 0;
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(shGo)) {
            if (blk == 0 && tid == 0) ws->called_off += 1;
            return;
        }
    }
    const int half = a.half;
    const int n = (int)a.n;
    const int64_t ldc = a.ldc;
    const Glob<const float> K = as_global(P.K);
    const double eps = P.eps;
    const int max_inner = P.max_inner;
    const int64_t iter0 = ws->iter;
    // iterations this launch may still do (max_iter)
    const int64_t left = P.max_iter - iter0;
    if (tid == 0) {
        shC = P.C;
        shTol = P.tol;
        shRatio = P.inner_ratio;
    }

    // rows of this block: whole units of two, upw of them a wave
    const int U = (n + 1) >> 1;
    const int u0 = (int)((int64_t)blk * U / R);
    const int r0 = 2 * u0;
    const int nu = (int)(((int64_t)blk + 1) * U / R) - u0;
    const int upw = (nu + kRowWavesRes - 1) / kRowWavesRes;  // at most 64
    const int unit = (wave - 1) * upw + lane;
    const bool holds = wave > 0 && lane < upw && unit < nu;
    const int lr = holds ? 2 * unit : 0;  // first row of the thread, local
    const int row = r0 + lr;
    const int nr = holds ? min(2, n - row) : 0;  // its rows

    float z[2] = {};
    if (SVR) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (j < nr) z[j] = P.z[row + j];
    }
    double* Fl = reinterpret_cast<double*>(stl + NC * kResRows);
    double* All = Fl + kResRows;
    for (int e = tid; e < kResRows; e += kSelThreads) {
        const bool in = e < 2 * nu && r0 + e < n;
        Fl[e] = in ? P.F[r0 + e] : 0.0;
        stl[e] = in ? P.st[r0 + e] : (uint8_t)0;
        All[e] = in ? P.alpha[r0 + e] : 0.0;
        if (SVR) {
            stl[kResRows + e] = in ? P.st[n + r0 + e] : (uint8_t)0;
            All[kResRows + e] = in ? P.alpha[n + r0 + e] : 0.0;
        }
    }
    if (tid < 128) (&rmax[0][0])[tid] = -INFINITY;  // (wave 0 holds no rows)
    __syncthreads();

    // candidate c of the working set: up winner c (c < half), then the low
    // winners
    auto cand = [&](int c, double& key, int32_t& idx) {
        key = c < half ? upk[c] : (c < 2 * half ? lok[c - half] : -INFINITY);
        idx = c < half ? upi[c] : (c < 2 * half ? loi[c - half] : INT_MAX);
    };
    // place of variable t of this block in stl and All
    auto local = [&](int32_t t) {
        return SVR && t >= n ? t - n - r0 + kResRows : t - r0;
    };
    // The steps every wave takes part in: the candidates at or above the
    // bound ranked, and with R > 1 the blocks' lists exchanged through
    // memory and ranked again.  best(side, pk, pi, k, i): the caller's best
    // variable of a side after (pk, pi).
    auto winners = [&](int it, auto best) {
        const int M0 = __builtin_amdgcn_readfirstlane(nsv[0]);
        const int M1 = __builtin_amdgcn_readfirstlane(nsv[1]);
        if (M0 <= kResCand && M1 <= kResCand) {
            rank_lists(svk, svi, M0, M1, half, upk, upi, lok, loi, tid);
        } else {
            // too many ties at the bound (alpha = 0): rounds over the block,
            // each the best variable after the previous winner
            for (int side = 0; side < 2; ++side) {
                double pk = INFINITY;
                int32_t pi = -1;
                for (int k = 0; k < half; ++k) {
                    double bk = -INFINITY;
                    int32_t bi = INT_MAX;
                    best(side, pk, pi, bk, bi);
                    wave_best_fast(bk, bi);
                    if (lane == 0) {
                        rk[k & 1][wave] = bk;
                        ri[k & 1][wave] = bi;
                    }
                    __syncthreads();
                    bk = rk[k & 1][0];
                    bi = ri[k & 1][0];
                    for (int w = 1; w < kWaves; ++w)
                        if (better(rk[k & 1][w], ri[k & 1][w], bk, bi)) {
                            bk = rk[k & 1][w];
                            bi = ri[k & 1][w];
                        }
                    pk = bk;
                    pi = bi;
                    if (tid == 0) {
                        (side ? lok : upk)[k] = bk;
                        (side ? loi : upi)[k] = bi;
                    }
                }
                __syncthreads();
            }
        }
        __syncthreads();
        // A word of the exchange carries the iteration it belongs to, so a
        // reader needs no flag and no second round trip; two sets of words
        // by the iteration's parity are enough, as no block can be two
        // iterations ahead of another.
        if (R > 1) {
            const uint32_t tag = (uint32_t)(iter0 + it + 1);
            const Glob<uint64_t> xb =
                as_global(P.xch) + (size_t)(tag & 1u) * R * kXchBlock;
            if (wave == 0 && lane < 2 * half) {
                const bool lo = lane >= half;
                const int k = lo ? lane - half : lane;
                const double key = lo ? lok[k] : upk[k];
                const int32_t idx = lo ? loi[k] : upi[k];
                const double al =
                    key == -INFINITY ? 0.0 : All[local(idx)];
                const uint64_t kb = __builtin_bit_cast(uint64_t, key);
                const uint64_t ab = __builtin_bit_cast(uint64_t, al);
                const uint64_t tg = (uint64_t)tag << 32;
                const Glob<uint64_t> w = xb + (size_t)blk * kXchBlock + lane;
                agent_store(w, tg | (uint32_t)kb);
                agent_store(w + 16, tg | (uint32_t)(kb >> 32));
                agent_store(w + 32, tg | (uint32_t)idx);
                agent_store(w + 48, tg | (uint32_t)ab);
                agent_store(w + 64, tg | (uint32_t)(ab >> 32));
            }
            // A thread a candidate; alpha is read for the winners only,
            // beside K_BB (with all of it here, by 5 words a candidate, an
            // iteration took 8.2 us with 3 blocks, 10.9 with 11, 12.4 with 16
            // and 23.0 with 32; now 8.1, 10.3, 11.7 and 21.8)
            const int b = tid >> 4, l = tid & 15;
            if (b < R && l < 2 * half) {
                const Glob<const uint64_t> w = xb + tid + b * (kXchBlock - 16);
                uint64_t w0, w1, w2;
                do {
                    w0 = agent_load(w);
                    w1 = agent_load(w + 16);
                    w2 = agent_load(w + 32);
                } while ((uint32_t)(w0 >> 32) != tag ||
                         (uint32_t)(w1 >> 32) != tag ||
                         (uint32_t)(w2 >> 32) != tag);
                const int side = l >= half ? 1 : 0;
                const int pos = b * half + (side ? l - half : l);
                svk[side][pos] = __builtin_bit_cast(
                    double, (w1 << 32) | (uint64_t)(uint32_t)w0);
                svi[side][pos] = (int32_t)(uint32_t)w2;
            }
            if (a.lag && blk == R - 1) {  // (developer override)
                const uint64_t t0 = wall_clock64();
                while (wall_clock64() - t0 < a.lag) __builtin_amdgcn_s_sleep(1);
            }
            __syncthreads();
            rank_lists(svk, svi, R * half, R * half, half, upk, upi, lok, loi,
                       tid, src[0], src[1]);
            __syncthreads();
        }
        return M0 <= kResCand && M1 <= kResCand;
    };

    // The two roles run loops of their own (the same barriers in both), so
    // that neither's registers are held through the other's code.
    // (the thread index is made new in every iteration: the many LDS
    // addresses formed from it are then computed where they are used, not
    // before the loop and kept in scratch memory)
    auto renew = [&]() {
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
    };
    if (wave != 0) {
        for (int it = 0; it < a.iters; ++it) {
            renew();
            // (1) this thread's scores on each side (up v, low -v, exactly
            // as the row kernel computes them; copy c of row j: 0 the sample
            // or its (i,+), 1 its (i,-)), and the maxima of the 16-lane rows
            double su[2 * NC], sl_[2 * NC];
            double mu = -INFINITY, ml = -INFINITY;
            {
                const double2 F = *reinterpret_cast<const double2*>(Fl + lr);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint32_t st2 =
                        holds ? *reinterpret_cast<const uint16_t*>(
                                    stl + c * kResRows + lr)
                              : 0u;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t s = st2 >> (8 * j);
                        const double r =
                            SVR ? (c ? (double)z[j] + eps : (double)z[j] - eps)
                                : ((s & ST_YPOS) ? 1.0 : -1.0);
                        const double v = r - (j ? F.y : F.x);
                        su[2 * c + j] = (s & ST_UP) ? v : -INFINITY;
                        sl_[2 * c + j] = (s & ST_LOW) ? -v : -INFINITY;
                        mu = max_f64(mu, su[2 * c + j]);
                        ml = max_f64(ml, sl_[2 * c + j]);
                    }
                }
                const double xu = rmax_f64(mu), xl = rmax_f64(ml);
                if ((lane & 15) == 0) {
                    rmax[0][wave * 4 + (lane >> 4)] = xu;
                    rmax[1][wave * 4 + (lane >> 4)] = xl;
                }
            }
            __syncthreads();
            __syncthreads();
            // (3) every variable at or above the bound
            {
                const double th0 = theta[0], th1 = theta[1];
                if (mu != -INFINITY && mu >= th0) {
#pragma unroll
                    for (int j = 0; j < 2 * NC; ++j)
                        if (su[j] != -INFINITY && su[j] >= th0) {
                            const int pos = atomicAdd(&nsv[0], 1);
                            if (pos < kResCand) {
                                svk[0][pos] = su[j];
                                svi[0][pos] = (j >> 1) * n + row + (j & 1);
                            }
                        }
                }
                if (ml != -INFINITY && ml >= th1) {
#pragma unroll
                    for (int j = 0; j < 2 * NC; ++j)
                        if (sl_[j] != -INFINITY && sl_[j] >= th1) {
                            const int pos = atomicAdd(&nsv[1], 1);
                            if (pos < kResCand) {
                                svk[1][pos] = sl_[j];
                                svi[1][pos] = (j >> 1) * n + row + (j & 1);
                            }
                        }
                }
            }
            __syncthreads();
            winners(it, [&](int side, double pk, int32_t pi, double& bk,
                            int32_t& bi) {
#pragma unroll
                for (int j = 0; j < 2 * NC; ++j) {
                    const double kk = side ? sl_[j] : su[j];
                    const int32_t ii = (j >> 1) * n + row + (j & 1);
                    if (kk != -INFINITY && after(kk, ii, pk, pi) &&
                        better(kk, ii, bk, bi)) {
                        bk = kk;
                        bi = ii;
                    }
                }
            });
            if (wave >= 8 && wave < 12) {
                    // (5) K of every pair of candidates, one a thread
                    const int e = tid - 512, ca = e >> 4, cb = e & 15;
                    double ka, kb;
                    int32_t ia, ib;
                    cand(ca, ka, ia);
                    cand(cb, kb, ib);
                    const int32_t sa =
                        ka == -INFINITY ? 0 : (SVR && ia >= n ? ia - n : ia);
                    const int32_t sb =
                        kb == -INFINITY ? 0 : (SVR && ib >= n ? ib - n : ib);
                    kbb[ca][cb] = K[(int64_t)sa * ldc + sb];
                } else if (wave == 12 && lane < 16) {
                    // their alpha, labels and first use
                    double key;
                    int32_t idx;
                    cand(lane, key, idx);
                    const bool ok = key != -INFINITY;
                    const int32_t t = ok ? idx : 0;
                    const int32_t smp = SVR && t >= n ? t - n : t;
                    const float zb = as_global(P.z)[smp];
                    int32_t seen = 0;
                    if (blk == 0) seen = as_global(P.seen)[smp];
                    double al = 0.0;
                    if (ok && R == 1) {
                        al = All[local(t)];
                    } else if (ok) {
                        // the words that its block published with it
                        const uint32_t tag = (uint32_t)(iter0 + it + 1);
                        const int low = lane >= half ? 1 : 0;
                        const int e = src[low][low ? lane - half : lane];
                        const int b = e / half, k = e - b * half;
                        const Glob<const uint64_t> w =
                            as_global(P.xch) +
                            ((size_t)(tag & 1u) * R + b) * kXchBlock + 48 +
                            (low ? half + k : k);
                        uint64_t w0, w1;
                        do {
                            w0 = agent_load(w);
                            w1 = agent_load(w + 16);
                        } while ((uint32_t)(w0 >> 32) != tag ||
                                 (uint32_t)(w1 >> 32) != tag);
                        al = __builtin_bit_cast(
                            double, (w1 << 32) | (uint64_t)(uint32_t)w0);
                    }
                    shAl[lane] = al;
                    const bool yp = SVR ? t < n : zb > 0.0f;
                    shY[lane] = yp ? 1.0f : -1.0f;
                    shSeen[lane] = seen;
                }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(shGo) == 0) break;
            // (7) the kernel values of this thread's rows, in flight while
            // wave 0 solves (slots past nS: the row of zeros, as the change
            // is 0 and a sample's row may hold an infinity)
            // (already as fp64: converting them is then not on the chain)
            typedef float floatx2 __attribute__((ext_vector_type(2)));
            double kd[16][2];
            {
                const int32_t smps = shS[lane & 15];
                const uint32_t off = 4u * (uint32_t)row;
                floatx2 kv[16];
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const uint64_t ro =
                        (uint64_t)(uint32_t)rl_i32(smps, s) * (uint32_t)ldc;
                    const Glob<const char> kr = (Glob<const char>)(K + ro);
                    kv[s] = *(Glob<const floatx2>)(kr + off);
                }
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    kd[s][0] = (double)kv[s][0];
                    kd[s][1] = (double)kv[s][1];
                    asm volatile("" : "+v"(kd[s][0]), "+v"(kd[s][1]));
                }
            }
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            // (8) F_i += sum_s dc_s K_is in the order of the row kernel's
            // 16-lane sum: ((t_s + t_s+8) + (t_s+4 + t_s+12)) pairwise
            auto quad = [&](int s, int j) -> double {
                const double2 c04 =
                    *reinterpret_cast<const double2*>(shCoef + 4 * s);
                const double2 c8c =
                    *reinterpret_cast<const double2*>(shCoef + 4 * s + 2);
                return (fma(c04.x, kd[s][j], 0.0) +
                        fma(c8c.x, kd[s + 8][j], 0.0)) +
                       (fma(c04.y, kd[s + 4][j], 0.0) +
                        fma(c8c.y, kd[s + 12][j], 0.0));
            };
            if (holds) {
                double2* Fp = reinterpret_cast<double2*>(Fl + lr);
                double2 f = *Fp;
                f.x += (quad(0, 0) + quad(2, 0)) + (quad(1, 0) + quad(3, 0));
                f.y += (quad(0, 1) + quad(2, 1)) + (quad(1, 1) + quad(3, 1));
                *Fp = f;
            }
        }
    } else {
        // this launch's counts, and the state of the gap test
        int d_iter = 0, d_rows = 0, d_inner = 0, d_served = 0, d_filled = 0;
        int d_slow = 0, done = 0, last_steps = 0;
        double gap_out = 0.0, m_out = 0.0, M_out = 0.0;
        for (int it = 0; it < a.iters; ++it) {
            renew();
            __syncthreads();
            // (2) a bound from below on the half-th best key of each side:
            // the half-th largest of the waves' maxima (distinct variables).
            // Row 0 takes the up side, row 1 the low side, a lane a wave.
            // (the first uses stored in the last iteration are out before
            // they are read again)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(kVmcnt0);
            asm volatile("" ::: "memory");
            const double* rm = rmax[(lane >> 4) & 1] + 4 * (lane & 15);
            const double2 x01 = *reinterpret_cast<const double2*>(rm);
            const double2 x23 = *reinterpret_cast<const double2*>(rm + 2);
            const double x = max_f64(max_f64(x01.x, x01.y),
                                     max_f64(x23.x, x23.y));
            int c = 1;
            const int xlo = __double2loint(x), xhi = __double2hiint(x);
            for_row_rotations([&](auto r) {
                constexpr int RR = decltype(r)::value;
                const double o =
                    __hiloint2double(row_rot<RR>(xhi), row_rot<RR>(xlo));
                c += o >= x ? 1 : 0;
            });
            double th = c >= half ? x : -INFINITY;
            th = rmax_f64(th);
            if ((lane & 15) == 0 && lane < 32) theta[lane >> 4] = th;
            if (lane < 8) {
                upk[lane] = lok[lane] = -INFINITY;
                upi[lane] = loi[lane] = INT_MAX;
            }
            if (lane < 2) nsv[lane] = 0;
            __syncthreads();
            __syncthreads();
            if (!winners(it, [](int, double, int32_t, double&, int32_t&) {}))
                d_slow += 1;
            // (6) gap test, working set (U0 L0 U1 L1 ..., repeats dropped),
            // distinct samples, order by index.  A candidate stays in its
            // lane; the 15 row rotations meet every other candidate.
            uint32_t keepm = 0, firstm = 0;
            double key;
            int32_t idx;
            cand(lane & 15, key, idx);
            const bool ent = key != -INFINITY;
            const double m = rl_f64(key, 0), Ml = rl_f64(key, half);
            const bool valid = m != -INFINITY && Ml != -INFINITY;
            gap_out = valid ? m + Ml : 0.0;  // m - M with M = -Ml
            m_out = valid ? m : 0.0;
            M_out = valid ? -Ml : 0.0;
            int nB = 0;
            if (!valid || gap_out <= uniform_f64(shTol)) {
                done = 1;
            } else if (it >= left) {
                done = 2;
            } else {
                const int c = lane & 15;
                const bool isU = c < half;
                const int k = isU ? c : c - half;
                // a variable already placed earlier: up entry k follows low
                // entries 0 .. k - 1, low entry k up entries 0 .. k
                const uint32_t before =
                    isU ? ((1u << k) - 1u) << half : (2u << k) - 1u;
                uint32_t eqm = 0, ltm = 0, twm = 0;
                const int32_t smp = SVR && idx >= n ? idx - n : idx;
                for_row_rotations([&](auto r) {
                    constexpr int RR = decltype(r)::value;
                    const int32_t im = row_rot<RR>(idx);
                    const uint32_t bit = 1u << ((c - RR) & 15);
                    eqm |= im == idx ? bit : 0u;
                    ltm |= im < idx ? bit : 0u;
                    if (SVR) {
                        const int32_t sm = im >= n ? im - n : im;
                        twm |= sm == smp ? bit : 0u;
                    }
                });
                const bool keep = ent && c < 2 * half && !(eqm & before);
                keepm = (uint32_t)__ballot(keep) & 0xffffu;
                const uint32_t ku = keepm & ((1u << half) - 1u);
                const uint32_t kl = keepm >> half;
                const uint32_t below = (1u << k) - 1u;
                int pos = __popc(ku & below) + __popc(kl & below);
                if (!isU) pos += (int)((ku >> k) & 1u);
                nB = __popc(keepm);
                const int p = __popc(ltm & keepm);
                // slot: the samples in the order of B; the second of two
                // copies of a sample shares the slot of the first
                int slot = pos;
                firstm = keepm;
                if (SVR) {
                    const uint32_t tw = twm & keepm;  // its twin, if any
                    const int tc = tw ? __builtin_ctz(tw) : c;
                    const int tpos = __shfl(pos, tc);
                    const bool second = keep && tw && tpos < pos;
                    uint32_t sm = (uint32_t)__ballot(second) & 0xffffu;
                    firstm = keepm & ~sm;
                    if (second) slot = tpos;
                    int drop = 0;  // seconds placed before the slot's first
                    while (sm) {
                        const int o = __builtin_ctz(sm);
                        sm &= sm - 1;
                        drop += rl_i32(pos, o) < slot ? 1 : 0;
                    }
                    slot -= drop;
                }
                if (lane < 16) {
                    if (keep) {
                        shCand[p] = c;
                        shSlot[c] = slot;
                        shS[slot] = smp;
                    }
                    // ranks past nB: any (not used); slots past theirs: the
                    // row of zeros
                    if (lane >= nB) shCand[lane] = 0;
                    if (lane >= __popc(firstm)) shS[lane] = n;
                }
            }
            if (lane == 0) {
                shGo = nB;
                shNS = __popc(firstm);
            }
            __syncthreads();
            if (nB == 0) break;  // uniform over the problem's blocks
            const int nS = __popc(firstm);
            // (9) the subproblem: maximal-violating-pair steps.  The
            // variable of rank p by index sits in lane p of row 0 (its up
            // side: w = v) and of row 1 (its low side: w = -v), so that one
            // row maximum serves both sides of a step.
            const int p = lane & 15, prow = lane >> 4;
            const bool act = p < nB;
            const int cp = shCand[p];
            const bool low = prow == 1;
            double kc;
            int32_t t;
            cand(cp, kc, t);
            const double C = act ? shC : 0.0;
            double al = act ? shAl[cp] : 0.0;
            const float yf = shY[cp];
            const bool pos = yf > 0.0f;
            const double yv = (double)yf;
            const double a0 = al;
            const int slot = shSlot[cp];
            // the key of a candidate: v of an up winner, -v of a low one
            const double v0 = cp < half ? kc : -kc;
            double w = act ? (low ? -v0 : v0) : 0.0;
            // K of the lane's variable with the variable of rank c (negated
            // in row 1: w moves by s (K_pi - K_pj) with the sign of its side)
            float krow[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const float k = kbb[cp][rl_i32(cp, c)];
                krow[c] = low ? -k : k;
            }
            // the pairs' curvatures and their reciprocals (refined twice, as
            // a division does it), lane (r, p) those of p with ranks 4 r ..
            // 4 r + 3; a step reads its pair's
            {
                const float kpp = kbb[cp][cp];
                const int4 cc =
                    *reinterpret_cast<const int4*>(shCand + 4 * prow);
                const int cx[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double kii = (double)kpp;
                    const double kjj = (double)kbb[cx[i]][cx[i]];
                    double a2 =
                        fma(-2.0, (double)kbb[cp][cx[i]], kii + kjj);
                    if (a2 <= 0.0) a2 = kTau;
                    double y = __builtin_amdgcn_rcp(a2);
                    y = fma(y, fma(-a2, y, 1.0), y);
                    y = fma(y, fma(-a2, y, 1.0), y);
                    shCur[p][4 * prow + i] = make_double2(a2, y);
                }
            }
            const double itol =
                uniform_f64(fmax(shRatio * gap_out, 0.5 * shTol));
            // room of the lane's side: C - alpha (an up variable with y = +1
            // or a low one with y = -1), else alpha
            const bool fromC = pos != low;
            int steps = 0;
            for (;;) {
                const double cap = fromC ? C - al : al;
                const bool has = cap > 0.0;
                const double kx = has ? w : -INFINITY;
                const double Mx = rmax_f64(kx);
                const unsigned long long hit = __ballot(has && kx == Mx);
                const double diff = rl_f64(Mx, 0) + rl_f64(Mx, 16);
                if (!(diff > itol)) break;  // (-inf: a side has no variable)
                const int Li = __builtin_ctzll(hit);  // lowest lane = index
                const int Lj = __builtin_ctzll(hit >> 16) & 15;
                const double2 cur = shCur[Li][Lj];
                const double Ui = rl_f64(cap, Li), Lb = rl_f64(cap, 16 + Lj);
                const double dk = (double)krow[Li] - (double)krow[Lj];
                // diff / a2, the last steps of the division; clipped at the
                // rooms of both (a variable whose room is used up lands on
                // its bound exactly)
                const double q0 = diff * cur.y;
                double st = fma(fma(-cur.x, q0, diff), cur.y, q0);
                st = min_f64(min_f64(st, Ui), Lb);
                w = fma(-dk, st, w);
                const bool isI = p == Li;
                const double an = fma(isI ? yv : -yv, st, al);
                const bool clip = (isI ? Ui : Lb) == st;
                const double bound = isI == pos ? C : 0.0;
                if (isI || p == Lj) al = clip ? bound : an;
                if (++steps >= max_inner) break;
            }
            // (10) results: alpha and the state byte (the block that holds
            // the row), the change of each slot's coefficient
            const bool own = act && prow == 0;
            const double dc = own ? yv * (al - a0) : 0.0;
            const int32_t sm = SVR && t >= n ? t - n : t;
            const int o = sm - r0;  // local row
            if (lane < 16) {
                shDc[p] = 0.0;
                shCoef[p] = 0.0;
            }
            __builtin_amdgcn_wave_barrier();
            if (own) {
                if (o >= 0 && o < 2 * nu) {
                    All[local(t)] = al;
                    stl[local(t)] = state_bits(yv, al, C);
                }
                if (SVR) shDc[p] = dc;
            }
            double dsum = dc;
            if (SVR) {
                // the twin of a sample's other copy, if it is in B
                const int32_t ps = own ? sm : -1 - lane;
                uint32_t pm = 0;
                for_row_rotations([&](auto r) {
                    constexpr int RR = decltype(r)::value;
                    const int32_t so = row_rot<RR>(ps);
                    pm |= so == ps ? 1u << ((p - RR) & 15) : 0u;
                });
                __builtin_amdgcn_wave_barrier();
                // the lower rank first, as the sums of both orders agree
                if (pm) dsum = dc + shDc[__builtin_ctz(pm)];
            }
            if (own) shCoef[4 * (slot & 3) + (slot >> 2)] = dsum;
            // the row cache's statistics: rows of samples used before are
            // served, others filled
            if (blk == 0) {
                const bool miss =
                    lane < 16 && ((firstm >> lane) & 1u) && shSeen[lane] < 0;
                const int nm = __popcll(__ballot(miss));
                if (miss) {
                    double kq;
                    int32_t iq;
                    cand(lane, kq, iq);
                    const int32_t sq_ = SVR && iq >= n ? iq - n : iq;
                    as_global(P.seen)[sq_] = sq_;
                }
                if (nm == 0) d_served += nS;
                else d_filled += nm;
            }
            d_iter += 1;
            d_rows += nS;
            d_inner += steps;
            last_steps = steps;
            __syncthreads();
        }
        if (blk == 0 && tid == 0) {
            ws->iter = iter0 + d_iter;
            ws->res_iters += d_iter;
            ws->res_launches += 1;
            ws->rows += d_rows;
            ws->inner_total += d_inner;
            ws->cache_served += d_served;
            ws->cache_filled += d_filled;
            ws->slow_selects += d_slow;
            ws->steps = last_steps;
            ws->gap = gap_out;
            ws->m = m_out;
            ws->M = M_out;
            if (done) ws->done = done;
        }
    }

    // the state back to memory
    __syncthreads();
    for (int e = tid; e < 2 * nu; e += kSelThreads)
        if (r0 + e < n) {
            P.F[r0 + e] = Fl[e];
            P.st[r0 + e] = stl[e];
            P.alpha[r0 + e] = All[e];
            if (SVR) {
                P.st[n + r0 + e] = stl[kResRows + e];
                P.alpha[n + r0 + e] = All[kResRows + e];
            }
        }
}

size_t resident_xch_words(int R)
{
    return (size_t)2 * R * kXchBlock;
}

void launch_resident(const ResidentArgs& a, int problems, bool svr,
                     hipStream_t s)
{
    if (problems <= 0) return;
    const int64_t units = (a.n + 1) / 2;
    if (a.R < 1 || a.R > kResBlocks || a.half < 1 || a.half > 8 ||
        a.R * a.half > kResCand || (units + a.R - 1) / a.R > kResUnits)
        throw Error{SVM_E_INTERNAL, "bad resident launch"};
    const size_t lds = (size_t)(svr ? 26 : 17) * kResRows;
    const void* fn = svr ? (const void*)k_resident<true>
                         : (const void*)k_resident<false>;
    if (!raise_dynamic_lds(fn, lds))
        throw Error{SVM_E_UNSUPPORTED,
                    "resident loop needs more LDS than the device allows"};
    const uint32_t grid = (uint32_t)(problems * a.R);
    if (svr) k_resident<true><<<grid, kSelThreads, lds, s>>>(a);
    else k_resident<false><<<grid, kSelThreads, lds, s>>>(a);
}

}  // namespace msvm
