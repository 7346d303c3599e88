// Stochastic reconfiguration restricted to the highest-probability samples
// (Sec. "ANQS-tailored stochastic reconfiguration"): the SR sample set, and
// the SR-transformed gradient d = (Re S + lambda I)^{-1} F with S the quantum
// geometric tensor of Eq. qgt_definition estimated over that set with
// renormalised probabilities.
//
// With R = 2 N_SR real rows X = [sqrt(w) (O_re - Obar_re); sqrt(w) (O_im -
// Obar_im)] (N_SR x N_p each), Re S = X^T X, and since N_SR << N_p the solve
// goes through the N_SR-sized side (the identity the min-SR recipe rests
// on): (lambda I + X^T X)^{-1} F = (F - X^T (lambda I + X X^T)^{-1} X F) / lambda.
//
//   k_sr_weights  w_x = |psi_x|^2 / sum over the set, and sqrt(w_x)
//   k_sr_gram     Obar_p = sum_x w_x O_xp and the Gram matrix of [X; F] (R + 1
//                 rows) over N_p in one pass over O: each workgroup stages a
//                 slab of columns in LDS, centres it there, and its eight
//                 waves accumulate 16 x 16 tiles of the lower triangle with
//                 FP64 MFMA (v_mfma_f64_16x16x4f64); one partial Gram per
//                 workgroup, added in fixed order by k_sr_reduce
//   k_sr_chol     blocked Cholesky of X X^T + lambda I and the two triangular
//                 solves for y = (X X^T + lambda I)^{-1} X F: one workgroup,
//                 16-column panels, the trailing tiles updated with FP64 MFMA
//   k_sr_update   d_p = (F_p - sum_r X_rp y_r) / lambda
//
// The set itself: for the set sizes the solve takes, a tournament (maxima of
// interleaved chunks, the n_sr-th of them as a cut, the few values past the
// cut sorted in LDS); larger sets sort all keys.
#include "device.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eloc {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kSrWaves = 8;            // waves of a Gram workgroup
constexpr int kSrTilesPerWave = 12;    // accumulator tiles a wave holds at most
constexpr int kSrSlab = 64;            // columns of a workgroup are a multiple of this
constexpr int kSrMaxSet = 256;         // samples in the set at most (checked at the entry point)

struct SrArgs {
    int nsr;              // samples in the set
    int64_t np;           // parameters
    int R;                // rows of [X; F] = 2 nsr + 1
    int nt;               // row tiles of 16
    const double* ore;    // [nsr][np]
    const double* oim;
    const double* F;      // [np]
    const double* w;      // [nsr] weights, then [nsr] square roots
};

__global__ __launch_bounds__(256) void k_sr_weights(const double2* __restrict__ logpsi, int nsr,
                                                    double* __restrict__ w) {
    __shared__ double red[256];
    double m = -INFINITY;
    for (int x = threadIdx.x; x < nsr; x += 256) m = fmax(m, logpsi[x].x);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    m = red[0];
    __syncthreads();
    double sum = 0.0;
    for (int x = threadIdx.x; x < nsr; x += 256) sum += exp(2.0 * (logpsi[x].x - m));
    red[threadIdx.x] = sum;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    sum = red[0];
    for (int x = threadIdx.x; x < nsr; x += 256) {
        const double v = exp(2.0 * (logpsi[x].x - m)) / sum;
        w[x] = v;
        w[nsr + x] = sqrt(v);
    }
}

// v of lane l, a scalar.
__device__ __forceinline__ double bcast_d(double v, int l) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), l);
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// Tile t of the lower triangle (row tile i >= column tile j): t = i (i + 1) / 2 + j.
__device__ __forceinline__ void tile_ij(int t, int& i, int& j) {
    i = 0;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    j = t - i * (i + 1) / 2;
}

// LDS row pitch of a slab in doubles: rows start two banks apart.
constexpr int sr_pitch(int KS) { return KS + 1; }

// grid: (column ranges, tile groups); block: kSrWaves waves.  A step stages a
// slab of KS columns of [X; F] in LDS: thread (k, g) = (tid % KS, tid / KS)
// holds column k of rows g, g + G, ... in registers, the means of the columns
// are summed from those (one partial a row group, through LDS, so O is read
// once), and the next slab's values are loaded while the matrix steps work on
// this one.  FP64 matrix steps bound the set sizes in use (201 rows, 210 816
// columns: 133 us of them in 232, the rest mostly the staging between two
// barriers; a pass for the means and one with unoverlapped loads: 492).  With
// both operands of a step read from LDS that was two thirds busy too: a
// wave's tiles follow each other along the rows of the triangle and a row's
// operand stays in registers until the row changes.  NR row tiles at most, TPW
// accumulator tiles a wave: the small sets hold fewer registers and several
// workgroups share a CU.  What a row needs (its weight, its address) is in a
// table, in the lanes of a register where a row is a wave's (KS = 64) and in
// LDS where it is not: loads or branches a row leave a chain of waits longer
// than the matrix steps.  A wave short of tiles works on tile 0 and drops it.
// partial[block][tile][lane][4], the lanes' accumulators as they stand.
template <int NR, int TPW, int KS>
__global__ __launch_bounds__(64 * kSrWaves) void k_sr_gram(SrArgs A, int64_t cols_per_block,
                                                           double* __restrict__ partial, double* __restrict__ mean) {
    constexpr int kG = 64 * kSrWaves / KS;         // row groups
    constexpr int kJ = (16 * NR + kG - 1) / kG;    // rows of a thread
    constexpr int kPitch = sr_pitch(KS);
    constexpr int kStep = 32;                      // columns whose operands a wave reads at a time
    constexpr bool kLanes = KS == 64;
    static_assert(!kLanes || kJ <= 64, "a row of the wave a lane");
    constexpr int kRows = kLanes ? 1 : kG * kJ;
    extern __shared__ double slab[];   // [16 nt][kPitch]
    __shared__ double red[kSrWaves][2 * KS];
    __shared__ double wre_l[kRows], wim_l[kRows], sq_l[kRows];
    __shared__ const double* row_l[kRows];
    const int tid = static_cast<int>(threadIdx.x);
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = lane_id();
    const int ntiles = A.nt * (A.nt + 1) / 2;
    const int t0 = (static_cast<int>(blockIdx.y) * kSrWaves + wave) * TPW;
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * cols_per_block;
    const int64_t c1 = min(A.np, c0 + cols_per_block);
    const int k = tid % KS, g = KS == 64 ? wave : tid / KS;
    d4 acc[TPW];
    int ti[TPW], tj[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        acc[q] = d4{0.0, 0.0, 0.0, 0.0};
        ti[q] = 0;
        tj[q] = 0;
        if (t0 + q < ntiles) tile_ij(t0 + q, ti[q], tj[q]);
    }
    // row r: its weight in the real and in the imaginary means, its factor, its first element of the range
    auto of_row = [&](int r, double& wre, double& wim, double& sq, const double*& row) {
        const int x = r < A.nsr ? r : r - A.nsr;
        const bool of_set = r < 2 * A.nsr;
        const double w = of_set ? A.w[x] : 0.0;
        wre = r < A.nsr ? w : 0.0;
        wim = r < A.nsr ? 0.0 : w;
        sq = of_set ? A.w[A.nsr + x] : 1.0;
        row = (of_set ? (r < A.nsr ? A.ore : A.oim) + x * A.np : A.F) + c0;
    };
    double wre_v = 0.0, wim_v = 0.0, sq_v = 0.0;
    const double* row_v = nullptr;
    if constexpr (kLanes) {
        of_row(g + kG * min(lane, kJ - 1), wre_v, wim_v, sq_v, row_v);
    } else {
        for (int r = tid; r < kRows; r += 64 * kSrWaves) of_row(r, wre_l[r], wim_l[r], sq_l[r], row_l[r]);
        __syncthreads();
    }
    auto pick = [&](double lanes, const double* table, int j) __attribute__((always_inline)) {
        if constexpr (kLanes)
            return bcast_d(lanes, j);
        else
            return table[g + kG * j];
    };
    double v[kJ];
    // rows j0 .. j1 of the slab at `base`
    auto fetch = [&](int64_t base, int j0, int j1) __attribute__((always_inline)) {
        const uint32_t at = static_cast<uint32_t>(min(base + k, c1 - 1) - c0);
#pragma unroll
        for (int j = j0; j < j1 && j < kJ; ++j) {
            if constexpr (kLanes)
                v[j] = reinterpret_cast<const double*>(
                    __double_as_longlong(bcast_d(__longlong_as_double(reinterpret_cast<int64_t>(row_v)), j)))[at];
            else
                v[j] = row_l[g + kG * j][at];
        }
    };
    // the loads of a slab go among the matrix steps of the one before, some
    // after each tile but the last few: all at once they stop at what a CU
    // can have in flight, and the matrix steps behind them
    constexpr int kSteps = KS / kStep * TPW;
    constexpr int kFetch = (kJ * 5 + 4 * kSteps - 1) / (4 * kSteps);
    static_assert(kFetch * kSteps >= kJ, "every row is loaded");
    fetch(c0, 0, kJ);
    for (int64_t base = c0; base < c1; base += KS) {
        int nsr = A.nsr;
        asm volatile("" : "+s"(nsr));   // the rows' masks are made where they are used
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            sr = fma(pick(wre_v, wre_l, j), v[j], sr);
            si = fma(pick(wim_v, wim_l, j), v[j], si);
        }
#pragma unroll
        for (int m = KS; m < 64; m <<= 1) {
            sr += shfl_xor_d(sr, m);
            si += shfl_xor_d(si, m);
        }
        if (lane < KS) {
            red[wave][k] = sr;
            red[wave][KS + k] = si;
        }
        __syncthreads();   // also: every wave is past its reads of the last slab
        double mr = 0.0, mi = 0.0;
#pragma unroll
        for (int w = 0; w < kSrWaves; ++w) {
            mr += red[w][k];
            mi += red[w][KS + k];
        }
        const bool in = base + k < c1;
        if (blockIdx.y == 0 && tid < KS && in) {
            mean[base + k] = mr;
            mean[A.np + base + k] = mi;
        }
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            const int r = g + kG * j;
            const double m = r < nsr ? mr : (r < 2 * nsr ? mi : 0.0);
            const double x = pick(sq_v, sq_l, j) * (v[j] - m);
            // rows past the last tile's go with its last row, a padding one (R is odd)
            slab[min(r, 16 * A.nt - 1) * kPitch + k] = (r <= 2 * nsr && in) ? x : 0.0;
        }
        __syncthreads();
        // lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] of a 4-column
        // step: both are the slab rows' columns kk + l / 16
#pragma unroll
        for (int half = 0; half < KS; half += kStep) {
            const double* at = slab + (lane & 15) * kPitch + (lane >> 4) + half;
            double fa[kStep / 4], fb[2][kStep / 4];
            auto read = [&](double* f, int i) __attribute__((always_inline)) {
                asm volatile("" : "+s"(i));
                const double* r = at + 16 * i * kPitch;
#pragma unroll
                for (int s = 0; s < kStep / 4; ++s) f[s] = r[4 * s];
            };
            read(fa, ti[0]);
            read(fb[0], tj[0]);
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                if (q + 1 < TPW) read(fb[(q + 1) & 1], tj[q + 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < kStep / 4; ++s)
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s], fb[q & 1][s], acc[q], 0, 0, 0);
                const int u = half / kStep * TPW + q;
                fetch(base + KS, u * kFetch, (u + 1) * kFetch);   // past the range: its last column
                if (q + 1 < TPW && ti[q + 1] != ti[q]) read(fa, ti[q + 1]);   // wave-uniform
            }
        }
    }
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        if (t0 + q >= ntiles) continue;
        *reinterpret_cast<d4*>(partial + ((static_cast<int64_t>(blockIdx.x) * ntiles + t0 + q) * 64 + lane) * 4) = acc[q];
    }
}

// T[e] = the sum of the blocks' partials of element e: a workgroup takes 32
// elements, its 8 groups of 32 threads the blocks g, g + 8, ...; the groups
// are added in order.
__global__ __launch_bounds__(256) void k_sr_reduce(const double* __restrict__ partial, int nblocks, int64_t len,
                                                   double* __restrict__ T) {
    __shared__ double red[8][32];
    const int k = static_cast<int>(threadIdx.x) & 31, g = static_cast<int>(threadIdx.x) >> 5;
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 32 + k;   // len is a multiple of 256
    double s = 0.0;
#pragma unroll 8
    for (int b = g; b < nblocks; b += 8) s += partial[b * len + e];
    red[g][k] = s;
    __syncthreads();
    if (g) return;
#pragma unroll
    for (int q = 1; q < 8; ++q) s += red[q][k];
    T[e] = s;
}

// The factorisation of the augmented matrix [[A, b], [b^T, *]] (A = T[0..n)^2
// + lambda I, b = T[n][0..n)): its last row of L is z = L^{-1} b, so the
// forward substitution comes with the factorisation.  16-column panels in two
// LDS buffers; the tiles of the lower triangle go round the waves and are held
// in the accumulators' layout: register c of lane l is D[4 c + l / 16][l % 16]
// (measured layout of v_mfma_f64_16x16x4f64 on gfx950).
//
// What bounds it is the serial chain of the n pivots: a reciprocal root, and
// the broadcasts of a column to the columns after it.  So the chain runs in
// the registers of a wave, a row a lane, without a barrier in 16 pivots, and
// what the chain does to the rows of the diagonal tile is also what solves
// for a row below it and, on the columns of the identity, what inverts the
// tile: a factoring wave has the 16 diagonal rows (each wave its own copy)
// and 48 of the others.  While those waves are in panel k + 1 the rest take
// panel k off the tiles past it.  200 rows: 78 us, against 670 for a column
// and two barriers a step over a 32 x 32 grid of threads.  The inverse is kept in place of the
// diagonal tile: L^T y = z then is a product a block, from the last.
constexpr int kCholWaves = 16;
constexpr int kCholPitch = 17;
constexpr int kCholRows = 48;    // rows of a factoring wave past the diagonal ones
constexpr int kCholMaxTiles = (2 * kSrMaxSet + 1 + 15) / 16;   // row tiles

constexpr int chol_factor_waves(int nt) { return (16 * nt + kCholRows - 1) / kCholRows; }
constexpr int chol_tile_waves(int nt) { return kCholWaves - chol_factor_waves(nt); }
static_assert(chol_tile_waves(kCholMaxTiles) > 0, "waves left for the tiles of the largest set");

// sqrt(d) and 1 / sqrt(d) together, for normal d > 0: the hardware's reciprocal
// root, two steps of Goldschmidt's coupled iteration (g -> sqrt, h -> 1 / (2
// sqrt), both corrected by the one residual 1/2 - g h) and the residual of the
// root.  Half the chain of a root and a division.
__device__ __forceinline__ void root_and_inverse(double d, double& root, double& inv) {
    const double r = __builtin_amdgcn_rsq(d);
    double g = d * r, h = 0.5 * r;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const double e = fma(-h, g, 0.5);
        g = fma(g, e, g);
        h = fma(h, e, h);
    }
    root = fma(fma(-g, g, d), h, g);
    inv = h + h;
}

// TPW > 0: the tiles stay in registers, TPW a wave at most.  TPW = 0: in T.
template <int TPW>
__global__ __launch_bounds__(64 * kCholWaves) void k_sr_chol(double* __restrict__ T, int n, int nt, double lambda,
                                                             const double* __restrict__ w, double* __restrict__ y,
                                                             uint32_t* __restrict__ err) {
    extern __shared__ double pan[];   // [2][16 nt][kCholPitch]
    __shared__ double dl[16][kCholPitch];   // the inverse of the diagonal tile of the panel just factored
    __shared__ double z[16 * kCholMaxTiles];
    __shared__ double ys[16 * kCholMaxTiles];
    const int tid = static_cast<int>(threadIdx.x);
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = lane_id();
    const int lr = lane >> 4, lc = lane & 15;
    const int ntiles = nt * (nt + 1) / 2;
    const int nw = chol_tile_waves(nt);
    const int w0 = kCholWaves - nw;   // the first wave with tiles
    double* const buf0 = pan;
    double* const buf1 = pan + 16 * nt * kCholPitch;
    // panel k in b: lanes 0-15 of a wave the diagonal rows, lanes 16-31 of the
    // first wave the identity, every other lane a row below
    auto factor = [&](double* b, int k) __attribute__((always_inline)) {
        const int below = 16 * (nt - 1 - k);
        const int at = wave * kCholRows + lane - 32;   // the row below, in lanes past the fixed ones
        if (wave > 0 && wave * kCholRows - 16 >= below) return;
        const bool ident = wave == 0 && lr == 1;
        const bool is_row = lr > 0 && !ident && at < below;
        const int row = lr == 0 ? 16 * k + lc : (is_row ? 16 * (k + 1) + at : 16 * k);
        double a[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const double v = b[row * kCholPitch + c];
            a[c] = ident ? (lc == c ? 1.0 : 0.0) : v;
        }
        double dmin = 1.0;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            double d = a[c];
            if (16 * k + c >= n) d = 1.0;
            dmin = lane == c ? d : dmin;
            asm volatile("" : "+v"(dmin));
            d = bcast_d(fmax(d, 1e-300), c);
            double piv, r;
            root_and_inverse(d, piv, r);
            a[c] = lane == c ? piv : a[c] * r;
#pragma unroll
            for (int j = c + 1; j < 16; ++j) {
                a[j] = fma(-a[c], bcast_d(a[c], j), a[j]);
                // now, not when column j is used: that keeps every step's
                // broadcasts alive, past the scalar registers
                asm volatile("" : "+v"(a[j]));
            }
        }
        if (wave == 0 && lr == 0 && !(dmin > 0.0)) atomicOr(err, static_cast<uint32_t>(kErrRange));
        if (ident) {
#pragma unroll
            for (int c = 0; c < 16; ++c) dl[c][lc] = a[c];
        }
        if (is_row) {
#pragma unroll
            for (int c = 0; c < 16; ++c) b[row * kCholPitch + c] = a[c];
        }
        if (row == n && (is_row || (wave == 0 && lr == 0))) {
#pragma unroll
            for (int c = 0; c < 16; ++c) z[16 * k + c] = 16 * k + c < n ? a[c] : 0.0;
        }
    };
    // The two kinds of wave go through the same barriers: two a panel, two a
    // block of the back substitution.
    if (wave < w0) {
        for (int k = 0; k < nt; ++k) {
            double* const b = k & 1 ? buf1 : buf0;
            __syncthreads();
            factor(b, k);
            __syncthreads();
        }
        for (int k = 0; k < nt; ++k) {
            __syncthreads();
            __syncthreads();
        }
    } else {
        constexpr int kT = TPW > 0 ? TPW : 1;
        d4 acc[kT];
        int ti[kT], tj[kT];
        auto gtile = [&](int t) { return reinterpret_cast<d4*>(T + (static_cast<int64_t>(t) * 64 + lane) * 4); };
        // f(i, j, tile) over this wave's tiles
        auto each = [&](auto f) __attribute__((always_inline)) {
            if constexpr (TPW > 0) {
#pragma unroll
                for (int q = 0; q < kT; ++q) {
                    int i = ti[q], j = tj[q];
                    asm volatile("" : "+s"(i), "+s"(j));   // its addresses are made where they are used
                    if (i >= 0) f(i, j, acc[q]);
                }
            } else {
                for (int t = wave - w0; t < ntiles; t += nw) {
                    int i, j;
                    tile_ij(t, i, j);
                    f(i, j, *gtile(t));
                }
            }
        };
        if constexpr (TPW > 0) {
#pragma unroll
            for (int q = 0; q < kT; ++q) {
                ti[q] = -1;
                tj[q] = -1;
                const int t = wave - w0 + q * nw;
                if (wave >= w0 && t < ntiles) {
                    tile_ij(t, ti[q], tj[q]);
                    acc[q] = *gtile(t);
                }
            }
        }
        auto put = [&](double* b, int i, const d4& v) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < 4; ++c) b[(16 * i + 4 * c + lr) * kCholPitch + lc] = v[c];
        };
        auto update = [&](const double* b, int i, int j, d4& v) __attribute__((always_inline)) {
            const double* ra = b + (16 * i + lc) * kCholPitch + lr;
            const double* rb = b + (16 * j + lc) * kCholPitch + lr;
#pragma unroll
            for (int s = 0; s < 16; s += 4) v = __builtin_amdgcn_mfma_f64_16x16x4f64(-ra[s], rb[s], v, 0, 0, 0);
        };
        each([&](int i, int j, d4& v) __attribute__((always_inline)) {
            if (i == j) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (4 * c + lr == lc && 16 * i + lc < n) v[c] += lambda;
            }
            if (j == 0) put(buf0, i, v);
        });
        __syncthreads();
        __syncthreads();
        for (int k = 0; k < nt; ++k) {
            double* const b = k & 1 ? buf1 : buf0;
            double* const nb = k & 1 ? buf0 : buf1;
            each([&](int i, int j, d4& v) __attribute__((always_inline)) {
                if (j == k) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        v[c] = i == k ? dl[4 * c + lr][lc] : b[(16 * i + 4 * c + lr) * kCholPitch + lc];
                } else if (j == k + 1) {
                    update(b, i, j, v);
                    put(nb, i, v);
                }
            });
            if (k + 1 == nt) break;
            __syncthreads();
            each([&](int i, int j, d4& v) __attribute__((always_inline)) {
                if (j > k + 1) update(b, i, j, v);
            });
            __syncthreads();
        }
        // (tile^T x)_j for this lane's column j of the tile, rows past n left out
        auto col_dot = [&](const d4& v, const double* x, int i) __attribute__((always_inline)) {
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (16 * i + 4 * c + lr < n) s = fma(v[c], x[16 * i + 4 * c + lr], s);
            s += shfl_xor_d(s, 16);
            s += shfl_xor_d(s, 32);
            return s;
        };
        for (int k = nt - 1; k >= 0; --k) {
            each([&](int i, int j, d4& v) __attribute__((always_inline)) {
                if (i != k || j != k) return;
                const double s = col_dot(v, z, k);
                if (lr == 0) ys[16 * k + lc] = s;
            });
            __syncthreads();
            each([&](int i, int j, d4& v) __attribute__((always_inline)) {
                if (i != k || j == k) return;
                const double s = col_dot(v, ys, k);
                if (lr == 0) z[16 * j + lc] -= s;
            });
            __syncthreads();
        }
    }
    // y_r times the row's weight: what the update multiplies O - Obar by
    for (int r = tid; r < n; r += 64 * kCholWaves) y[r] = ys[r] * w[n / 2 + (r < n / 2 ? r : r - n / 2)];
}

// y: the solution times the square roots of the weights.  Memory-bound: one
// pass over O, a thread a column, 16 loads in flight (337 MB: 62 us, 5.4 TB/s;
// with the rows' kind and factors looked up for each element 118).
__global__ __launch_bounds__(256) void k_sr_update(SrArgs A, const double* __restrict__ mean,
                                                   const double* __restrict__ y, double lambda,
                                                   double* __restrict__ d) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (p >= A.np) return;
    const double mr = mean[p], mi = mean[A.np + p];
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (int x = 0; x < A.nsr; ++x) {
        sr = fma(A.ore[x * A.np + p] - mr, y[x], sr);
        si = fma(A.oim[x * A.np + p] - mi, y[A.nsr + x], si);
    }
    d[p] = (A.F[p] - (sr + si)) / lambda;
}

__global__ void k_sr_select_keys(const double2* __restrict__ logpsi, int64_t n, uint64_t* __restrict__ key,
                                 uint32_t* __restrict__ idx) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    uint64_t b = __double_as_longlong(logpsi[i].x);
    // order-preserving map of doubles to unsigned integers, then reversed so
    // that an ascending sort puts the largest Re log psi first
    b = (b >> 63) ? ~b : (b | (1ull << 63));
    key[i] = ~b;
    idx[i] = static_cast<uint32_t>(i);
}

// The tournament over (key, index), a total order.  Chunk g = the elements
// i with (i / 32) mod kTopChunks == g, so a sorted input spreads over the
// chunks.  At most nsr chunks hold a maximum at or before the nsr-th of the
// chunks' maxima, so at most nsr n / kTopChunks elements are at or before
// that cut; an input in no particular order leaves little more than nsr.
// 100 of 2^20: 23 us in four launches; the eight passes of the sort 300.
constexpr int kTopChunks = 2048;
constexpr int kTopSort = 4096;       // elements sorted in LDS at most
constexpr uint32_t kTopNone = 0xffffffffu;

__device__ __forceinline__ uint64_t top_key(double v) {
    uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    b = (b >> 63) ? ~b : (b | (1ull << 63));
    return ~b;
}
__device__ __forceinline__ bool top_before(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
    return (ka < kb) | ((ka == kb) & (ia < ib));
}

__global__ __launch_bounds__(256) void k_top_maxima(const double2* __restrict__ logpsi, int64_t n,
                                                    uint64_t* __restrict__ mk, uint32_t* __restrict__ mi) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    uint64_t bk = ~0ull;
    uint32_t bi = kTopNone;
#pragma unroll 4
    for (int64_t i = g; i < n; i += 32 * kTopChunks) {
        const uint64_t k = top_key(logpsi[i].x);
        if (top_before(k, static_cast<uint32_t>(i), bk, bi)) {
            bk = k;
            bi = static_cast<uint32_t>(i);
        }
    }
    for (int m = 16; m >= 1; m >>= 1) {
        const uint64_t ok = __shfl_xor(static_cast<unsigned long long>(bk), m);
        const uint32_t oi = __shfl_xor(bi, m);
        if (top_before(ok, oi, bk, bi)) {
            bk = ok;
            bi = oi;
        }
    }
    if ((threadIdx.x & 31) == 0) {
        mk[g / 32] = bk;
        mi[g / 32] = bi;
    }
}

// Ascending bitonic sort of m = a power of two pairs in LDS by a workgroup of 1024.
__device__ __forceinline__ void bitonic(uint64_t* k, uint32_t* v, int m) {
    for (int size = 2; size <= m; size <<= 1)
        for (int d = size >> 1; d >= 1; d >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < m / 2; t += 1024) {
                const int a = 2 * t - (t & (d - 1)), b = a + d;
                const bool up = (a & size) == 0;
                const uint64_t ka = k[a], kb = k[b];
                const uint32_t va = v[a], vb = v[b];
                if (top_before(kb, vb, ka, va) == up) {
                    k[a] = kb;
                    k[b] = ka;
                    v[a] = vb;
                    v[b] = va;
                }
            }
        }
    __syncthreads();
}

// The cut: the nsr-th of the chunks' maxima (equal ones, of empty chunks, in
// chunk order), left behind them; the count of the kept list cleared.  Found
// by rank: a wave counts what comes before one maximum (a sort in one
// workgroup is 66 barrier-bound steps: 23 us, this 4).
constexpr int kCutThreads = 64;

__global__ __launch_bounds__(256) void k_top_cut(const uint64_t* __restrict__ mk, const uint32_t* __restrict__ mi,
                                                 int nsr, uint64_t* __restrict__ cut_k, uint32_t* __restrict__ cut_i) {
    const int e = (static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x)) / kCutThreads;
    const int part = static_cast<int>(threadIdx.x) % kCutThreads;
    const uint64_t ek = mk[e];
    const uint32_t ei = mi[e];
    int rank = 0;
#pragma unroll 8
    for (int q = part; q < kTopChunks; q += kCutThreads) {
        const uint64_t k = mk[q];
        const uint32_t i = mi[q];
        rank += static_cast<int>(top_before(k, i, ek, ei)) | ((k == ek) & (i == ei) & (q < e));
    }
    for (int m = kCutThreads / 2; m >= 1; m >>= 1) rank += __shfl_xor(rank, m);
    if (part == 0 && rank == nsr - 1) {
        cut_k[0] = ek;
        cut_i[0] = ei;
        cut_i[1] = 0u;
    }
}

__global__ __launch_bounds__(256) void k_top_keep(const double2* __restrict__ logpsi, int64_t n,
                                                  const uint64_t* __restrict__ mk, uint32_t* __restrict__ mi,
                                                  uint64_t* __restrict__ kept_k, uint32_t* __restrict__ kept_i) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const uint64_t ck = mk[kTopChunks];
    const uint32_t ci = mi[kTopChunks];
    if (top_before(ck, ci, mk[g / 32], mi[g / 32])) return;
    for (int64_t i = g; i < n; i += 32 * kTopChunks) {
        const uint64_t k = top_key(logpsi[i].x);
        if (top_before(ck, ci, k, static_cast<uint32_t>(i))) continue;
        const uint32_t at = atomicAdd(mi + kTopChunks + 1, 1u);
        kept_k[at] = k;
        kept_i[at] = static_cast<uint32_t>(i);
    }
}

// The first nsr of the kept list in order.  A list past the LDS sort is first
// cut down by its digits, 8 bits of the 96 of (key, index) a pass, until the
// elements at or before the chosen prefix fit.
__global__ __launch_bounds__(1024) void k_top_order(const uint32_t* __restrict__ count,
                                                    const uint64_t* __restrict__ kept_k,
                                                    const uint32_t* __restrict__ kept_i, int nsr,
                                                    int32_t* __restrict__ out) {
    __shared__ uint64_t k[kTopSort];
    __shared__ uint32_t v[kTopSort];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t pick[3];   // digit, elements before it, elements with it
    __shared__ uint32_t put;
    const int tid = static_cast<int>(threadIdx.x);
    const uint32_t m = *count;
    uint64_t pk = 0, maskk = 0;
    uint32_t pi = 0, maski = 0;
    uint32_t upto = m, before = 0;
    for (int d = 0; upto > kTopSort && d < 12; ++d) {
        if (tid < 256) hist[tid] = 0u;
        __syncthreads();
        const int sh = d < 8 ? 56 - 8 * d : 24 - 8 * (d - 8);
        for (uint32_t e = tid; e < m; e += 1024) {
            const uint64_t ek = kept_k[e];
            const uint32_t ei = kept_i[e];
            if (((ek ^ pk) & maskk) == 0 && ((ei ^ pi) & maski) == 0)
                atomicAdd(&hist[(d < 8 ? ek >> sh : static_cast<uint64_t>(ei) >> sh) & 255], 1u);
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t run = before;
            int q = 0;
            while (q < 255 && run + hist[q] < static_cast<uint32_t>(nsr)) run += hist[q++];
            pick[0] = static_cast<uint32_t>(q);
            pick[1] = run;
            pick[2] = hist[q];
        }
        __syncthreads();
        before = pick[1];
        upto = before + pick[2];
        if (d < 8) {
            pk |= static_cast<uint64_t>(pick[0]) << sh;
            maskk |= 255ull << sh;
        } else {
            pi |= pick[0] << sh;
            maski |= 255u << sh;
        }
        __syncthreads();
    }
    int pow2 = 2;
    while (pow2 < static_cast<int>(upto)) pow2 <<= 1;
    for (int t = tid; t < pow2; t += 1024) {
        k[t] = ~0ull;
        v[t] = kTopNone;
    }
    if (tid == 0) put = 0u;
    __syncthreads();
    for (uint32_t e = tid; e < m; e += 1024) {
        const uint64_t ek = kept_k[e];
        const uint32_t ei = kept_i[e];
        if (top_before(pk, pi, ek & maskk, ei & maski)) continue;
        const uint32_t at = atomicAdd(&put, 1u);
        k[at] = ek;
        v[at] = ei;
    }
    __syncthreads();
    if (pow2 <= 256) {
        // short lists, the usual ones: by rank, four threads an element (36
        // sort steps and their barriers: 8.5 us, this 5)
        const int e = tid / 4;
        int rank = 0;
        if (e < pow2) {
            const uint64_t ek = k[e];
            const uint32_t ei = v[e];
            for (int q = tid % 4; q < pow2; q += 4) rank += top_before(k[q], v[q], ek, ei) ? 1 : 0;
        }
        rank += __shfl_xor(rank, 1);
        rank += __shfl_xor(rank, 2);
        if (tid % 4 == 0 && e < static_cast<int>(upto) && rank < nsr) out[rank] = static_cast<int32_t>(v[e]);
        return;
    }
    bitonic(k, v, pow2);
    for (int t = tid; t < nsr; t += 1024) out[t] = static_cast<int32_t>(v[t]);
}

__global__ void k_sr_take(const uint32_t* __restrict__ idx, int n, int32_t* __restrict__ out) {
    const int i = static_cast<int>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) out[i] = static_cast<int32_t>(idx[i]);
}

inline unsigned blocks256(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

}  // namespace

namespace {

int sr_tiles(int nsr) {
    const int nt = (2 * nsr + 1 + 15) / 16;
    return nt * (nt + 1) / 2;
}

// Workgroups of the Gram: one round of the chip, as many to a CU as the
// LDS slabs of this set size let in; a slab of columns at least.
int64_t gram_cols(int nsr, int64_t np) {
    const int nt = (2 * nsr + 1 + 15) / 16;
    const int64_t nb = nt <= 5 ? 768 : (nt <= 8 ? 512 : 256);
    return ((np + nb - 1) / nb + kSrSlab - 1) / kSrSlab * kSrSlab;
}

template <int NR, int TPW, int KS>
void launch_gram(const SrArgs& A, int64_t cols, double* partial, double* mean, hipStream_t st) {
    const int ntiles = A.nt * (A.nt + 1) / 2;
    const int groups = (ntiles + kSrWaves * TPW - 1) / (kSrWaves * TPW);
    const size_t lds = sizeof(double) * 16 * A.nt * sr_pitch(KS);
    hipLaunchKernelGGL((k_sr_gram<NR, TPW, KS>), dim3(static_cast<unsigned>((A.np + cols - 1) / cols), groups),
                       dim3(64 * kSrWaves), lds, st, A, cols, partial, mean);
}

template <int TPW>
void launch_chol(double* T, int n, int nt, double lambda, const double* w, double* y, uint32_t* err, hipStream_t st) {
    const size_t lds = sizeof(double) * 2 * 16 * nt * kCholPitch;
    hipLaunchKernelGGL((k_sr_chol<TPW>), dim3(1), dim3(64 * kCholWaves), lds, st, T, n, nt, lambda, w, y, err);
}

}  // namespace

int64_t sr_partial_len(int nsr, int64_t np) {
    const int64_t cols = gram_cols(nsr, np);
    return (np + cols - 1) / cols * sr_tiles(nsr) * 256;
}

int64_t sr_tile_len(int nsr) { return static_cast<int64_t>(sr_tiles(nsr)) * 256; }

bool sr_select_tournament(int64_t n, int nsr) { return nsr <= kSrMaxSet && n <= (int64_t(1) << 22); }

int64_t sr_select_scratch(int64_t n) { return std::max<int64_t>(n, kTopChunks + 2); }

// The tournament: up to the set sizes of the solve and 2^22 samples, where
// its worst case (a kept list of nsr n / 2048 elements cut down by one
// workgroup) still costs less than the eight passes of the sort.  256 of 2^22,
// sort / tournament: every value the same 456 / 153 us, a few values 721 / 108,
// descending 625 / 91, in no order 795 / 64; of 2^20 every value the same 245 /
// 131, in no order 301 / 44.
hipError_t launch_sr_select(const double2* logpsi, int64_t n, int nsr, uint64_t* key, uint32_t* val, uint64_t* key2,
                            uint32_t* val2, uint32_t* hist, int64_t* hist_off, int64_t* scan, int32_t* out,
                            hipStream_t st) {
    if (sr_select_tournament(n, nsr)) {
        const dim3 grid(32 * kTopChunks / 256), block(256);
        hipLaunchKernelGGL(k_top_maxima, grid, block, 0, st, logpsi, n, key, val);
        hipLaunchKernelGGL(k_top_cut, dim3(kTopChunks * kCutThreads / 256), dim3(256), 0, st, key, val, nsr,
                           key + kTopChunks, val + kTopChunks);
        hipLaunchKernelGGL(k_top_keep, grid, block, 0, st, logpsi, n, key, val, key2, val2);
        hipLaunchKernelGGL(k_top_order, dim3(1), dim3(1024), 0, st, val + kTopChunks + 1, key2, val2, nsr, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_sr_select_keys, dim3(blocks256(n)), dim3(256), 0, st, logpsi, n, key, val);
    int alt = 0;
    hipError_t e = launch_radix_sort_pairs(key, val, key2, val2, n, 64, hist, hist_off, scan, &alt, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sr_take, dim3(blocks256(nsr)), dim3(256), 0, st, alt ? val2 : val, nsr, out);
    return hipGetLastError();
}

hipError_t launch_sr_solve(int nsr, int64_t np, const double* ore, const double* oim, const double2* logpsi,
                           const double* F, double lambda, double* w, double* mean, double* partial, double* T,
                           double* y, double* d, uint32_t* err, hipStream_t st) {
    SrArgs A;
    A.nsr = nsr;
    A.np = np;
    A.R = 2 * nsr + 1;
    A.nt = (A.R + 15) / 16;
    A.ore = ore;
    A.oim = oim;
    A.F = F;
    A.w = w;
    hipLaunchKernelGGL(k_sr_weights, dim3(1), dim3(256), 0, st, logpsi, nsr, w);
    const int64_t cols = gram_cols(nsr, np);
    if (A.nt <= 5)
        launch_gram<5, 2, kSrSlab>(A, cols, partial, mean, st);
    else if (A.nt <= 9)
        launch_gram<9, 6, kSrSlab>(A, cols, partial, mean, st);
    else if (A.nt <= 13)
        launch_gram<13, kSrTilesPerWave, kSrSlab>(A, cols, partial, mean, st);
    else if (A.nt <= 17)
        launch_gram<17, kSrTilesPerWave, kSrSlab>(A, cols, partial, mean, st);
    else
        // 33 row tiles: 32 columns are what LDS holds
        launch_gram<kCholMaxTiles, kSrTilesPerWave, kSrSlab / 2>(A, cols, partial, mean, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t len = sr_tile_len(nsr);
    hipLaunchKernelGGL(k_sr_reduce, dim3(static_cast<unsigned>(len / 32)), dim3(256), 0, st, partial,
                       static_cast<int>((np + cols - 1) / cols), len, T);
    // tiles in registers up to the sets whose tiles they hold
    const int per_wave = (sr_tiles(nsr) + chol_tile_waves(A.nt) - 1) / chol_tile_waves(A.nt);
    if (per_wave <= 3)
        launch_chol<3>(T, 2 * nsr, A.nt, lambda, w, y, err, st);
    else if (per_wave <= 10)
        launch_chol<10>(T, 2 * nsr, A.nt, lambda, w, y, err, st);
    else
        launch_chol<0>(T, 2 * nsr, A.nt, lambda, w, y, err, st);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sr_update, dim3(blocks256(np)), dim3(256), 0, st, A, mean, y, lambda, d);
    return hipGetLastError();
}

}  // namespace eloc
