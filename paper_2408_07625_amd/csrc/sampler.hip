// Autoregressive sampling without replacement (Methods, "Autoregressive
// sampling without replacement", Algorithm ARGumbelTopK) over an ansatz of
// per-qudit perceptrons (Methods, "Ansatz architecture", "Grouping qubits
// into qudits", "Global activation", "Local pruning strategy").
//
// One level per qudit k (D_k qubits, O_k = 2^D_k outcomes), for the B kept
// prefixes, B and the selection's state on the device:
//   k_ar_net     a workgroup takes 64 prefixes; four waves evaluate the
//                qudit's perceptron for them with FP64 MFMA (16 x 16 tiles,
//                v_mfma_f64_16x16x4f64): the prefix bits as +-1 inputs (0
//                past the prefix) times W1, tanh; times W2 plus the first
//                layer's output, tanh; times W3 -> the O_k outputs z.
//   k_ar_cand    one lane per (prefix, outcome): the mean shift of z, the mask
//                of outcomes that cannot reach the electron targets, the
//                normalised log p(c | prefix), l + log p, its Gumbel
//                perturbation, the siblings' maximum Z and the conditioned
//                value Ltil; a sort key (descending Ltil, masked outcomes
//                last); the histogram of the keys' top 12 bits.
//   select       the first min(K, allowed) candidates in (key, index) order as
//                a set: the digit of the K-th (k_ar_pick), the next 12 bits
//                within it (k_ar_hist, k_ar_pick; for large K twice at need), the
//                candidates of that prefix listed (k_ar_count) and ranked in
//                one workgroup (k_ar_cut).
//   k_ar_emit    the selected candidates become the next level's prefixes
//                (key with the outcome's bits set, l, Ltil), in index order.
// Levels run one after another without a wait on the host.  At 2^16 prefixes
// of 64 outcomes a level takes 200 us (net 77, cand 86, select and emit 40); with
// the perceptrons and the candidates in one kernel (178), the selected ones
// sorted (180) and two waits it took 500.
// The last level's are sorted by key (a stable radix sort).  Sorting every
// level gives the same set in the same order as long as no two kept values of
// a level are equal: equal values come in the order of the level before, and a
// value that ties at one level ties again at the next, as the best child of a
// prefix keeps its value.  So a tie shows in the last sort, or at the cut of a
// level; then the search runs again with every level sorted (those that can be
// among its first K).  A tie at a cut, or a list past what one workgroup should
// cut down, ends the first search there: what is left of it returns at once.
#include "device.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eloc {

// State of a search on the device.  Slot `level`: the prefixes going into it,
// and its unmasked candidates.
constexpr int kArLevels = 128;
constexpr int kArBound = 4096;      // candidates that k_ar_cut ranks in LDS
constexpr uint32_t kArList = 1u << 17;   // and cuts down to that many
constexpr int kArTile = 4096;       // candidates of a counting workgroup
struct ArState {
    int64_t B[kArLevels + 1];
    unsigned long long allowed[kArLevels];
    uint32_t redo;          // this search gives way to the one with sorted levels
    uint32_t bound;         // candidates in the selected prefix
    int shift;              // the prefix is key >> shift
    uint32_t deep;          // it holds more than kArBound
    int64_t prefix, below;  // digits of the need-th candidate (one past them: all are kept), candidates below those
    uint64_t cut_key;       // the last candidate kept of that prefix
    uint32_t cut_idx;
    int64_t listed;         // candidates counted in the tiles
};

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kArH = 64;        // hidden width
constexpr int64_t kArWide = 256 * 128;   // prefixes from which the workgroups of 16 waves are most of a round

struct ArLevel {
    int N, W, D, Dk, O, level, q0;
    int n_up, n_down;           // electron targets (-1: no mask)
    int rest_up, rest_down;     // spin-up / spin-down qubits after this qudit
    uint64_t seed;
    const double* W1;           // [H][N] of this qudit
    const double* b1;           // [H]
    const double* W2;           // [H][H]
    const double* b2;
    const double* W3;           // [2^D][H] (first O rows used)
    const double* b3;
};

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Standard Gumbel variable of the node (level, prefix, outcome): the
// SplitMix64 output function chained over (seed, level, prefix words,
// outcome), u from the top 53 bits, G = -log(-log u).
__device__ __forceinline__ double gumbel(uint64_t seed, int level, const uint64_t (&prefix)[kMaxWords], int W,
                                         int outcome) {
    uint64_t h = mix64(seed + 0x9E3779B97F4A7C15ull * static_cast<uint64_t>(level + 1));
#pragma unroll
    for (int w = 0; w < kMaxWords; ++w)
        if (w < W) h = mix64(h ^ prefix[w]);
    h = mix64(h ^ static_cast<uint64_t>(outcome));
    const double u = (static_cast<double>(h >> 11) + 0.5) * 0x1.0p-53;
    return -log(-log(u));
}

// log(1 - exp(a)) for a < 0
__device__ __forceinline__ double log1mexp(double a) {
    return a > -0.69314718055994531 ? log(-expm1(a)) : log1p(-exp(a));
}

__device__ __forceinline__ int key_bit(const uint64_t* k, int q) { return static_cast<int>((k[q >> 6] >> (q & 63)) & 1ull); }

// acc[t] (the 16 x 16 output tile of columns 16 t ..) = A[rows][0..kend) *
// B[cols][0..kend)^T for t < nt, A from a callback (row, k) read once per
// k step for all tiles, B row-major [out][in] with row pitch ldb (global or
// LDS).  Lane l feeds A[l % 16][k + l / 16] and B[k + l / 16][l % 16];
// register c of lane l holds D[4 c + l / 16][l % 16] (measured layout of
// v_mfma_f64_16x16x4f64 on gfx950).
template <int NT, class AF>
__device__ __forceinline__ void tiles_mma(d4 (&acc)[NT], AF a_of, const double* __restrict__ Bw, int ldb, int ncols,
                                          int kend, int nt, int lane) {
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < kend; k += 4) {
        const int kk = k + (lane >> 4);
        const bool kin = kk < kend;
        const double a = kin ? a_of(lane & 15, kk) : 0.0;
        double b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = 16 * t + (lane & 15);
            b[t] = (t < nt && kin && col < ncols) ? Bw[col * ldb + kk] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t < nt) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[t], acc[t], 0, 0, 0);
    }
}

// Bound by the FP64 rate (2 q0 64 + 2 64 64 + 2 64 O multiply-adds and 128
// tanh a prefix) and by how many waves a CU holds to fill its gaps, which the
// LDS for a wave's hidden layer decides: the weights are staged 32 outputs at
// a time, so that one workgroup of NW = 16 waves fits where two of 4 did.
// Fewer prefixes than a round of such workgroups take NW = 4: more CUs.
constexpr int kArHalf = 32;   // outputs of a staged part of the weights

template <int NW>
__global__ __launch_bounds__(64 * NW) void k_ar_net(ArLevel A, const ArState* __restrict__ S,
                                                    const uint64_t* __restrict__ keys, double* __restrict__ zout) {
    constexpr int kRows = 16 * NW;
    extern __shared__ double lds[];
    double (*const h)[kArH + 1] = reinterpret_cast<double (*)[kArH + 1]>(lds);              // [kRows]: h1, then h2
    double (*const wb)[kArH + 1] = reinterpret_cast<double (*)[kArH + 1]>(h[kRows]);        // [kArHalf] ([out][in])
    uint64_t* const kbuf = reinterpret_cast<uint64_t*>(wb[kArHalf]);                        // [kRows][W]
    const int wave = static_cast<int>(threadIdx.x) / 64;
    const int lane = lane_id();
    const int64_t B = S->B[A.level];
    const int64_t b0 = static_cast<int64_t>(blockIdx.x) * kRows;
    if (b0 >= B || S->redo) return;
    for (int e = threadIdx.x; e < kRows * A.W; e += 64 * NW) {
        const int64_t b = min(b0 + e / A.W, B - 1);
        kbuf[e] = keys[b * A.W + e % A.W];
    }
    auto stage = [&](const double* w, int from, int upto) {
        __syncthreads();
        for (int e = threadIdx.x; e < (upto - from) * kArH; e += 64 * NW) wb[e / kArH][e % kArH] = w[from * kArH + e];
        __syncthreads();
    };
    const int r0 = 16 * wave;   // this wave's row tile
    __syncthreads();
    // layer 1: inputs +-1 for the prefix qubits (q < q0), 0 after
    {
        auto a_of = [&](int r, int q) -> double {
            return key_bit(kbuf + (r0 + r) * A.W, q) ? 1.0 : -1.0;
        };
        d4 acc[kArH / 16];
        tiles_mma(acc, a_of, A.W1, A.N, kArH, A.q0, kArH / 16, lane);
#pragma unroll
        for (int t = 0; t < kArH / 16; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int row = r0 + 4 * c + (lane >> 4), col = 16 * t + (lane & 15);
                h[row][col] = tanh(acc[t][c] + A.b1[col]);
            }
    }
    auto a_of = [&](int r, int k) -> double { return h[r0 + r][k]; };
    // layer 2 with the residual of layer 1 (the wave's own rows of h: no
    // workgroup has to wait for their change)
    {
        d4 acc[2][kArHalf / 16];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            stage(A.W2, half * kArHalf, (half + 1) * kArHalf);
            tiles_mma(acc[half], a_of, &wb[0][0], kArH + 1, kArHalf, kArH, kArHalf / 16, lane);
        }
#pragma unroll
        for (int t = 0; t < kArH / 16; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int row = r0 + 4 * c + (lane >> 4), col = 16 * t + (lane & 15);
                h[row][col] = tanh(acc[t / 2][t % 2][c] + A.b2[col] + h[row][col]);
            }
    }
    // output layer: z for the O outcomes
    for (int from = 0; from < A.O; from += kArHalf) {
        const int cols = min(kArHalf, A.O - from);
        stage(A.W3, from, from + cols);
        d4 acc[kArHalf / 16];
        const int nt = (cols + 15) / 16;
        tiles_mma(acc, a_of, &wb[0][0], kArH + 1, cols, kArH, nt, lane);
#pragma unroll
        for (int t = 0; t < kArHalf / 16; ++t) {
            if (t >= nt) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t b = b0 + r0 + 4 * c + (lane >> 4);
                const int col = 16 * t + (lane & 15);
                if (col < cols && b < B) zout[b * A.O + from + col] = acc[t][c] + A.b3[from + col];
            }
        }
    }
}

template <int NW>
void launch_net(const ArLevel& A, int64_t B, const ArState* S, const uint64_t* keys, double* z, hipStream_t st) {
    constexpr int kRows = 16 * NW;
    const size_t lds = sizeof(double) * (kRows + kArHalf) * (kArH + 1) + sizeof(uint64_t) * kRows * A.W;
    hipLaunchKernelGGL(k_ar_net<NW>, dim3(static_cast<unsigned>((B + kRows - 1) / kRows)), dim3(64 * NW), lds, st, A,
                       S, keys, z);
}

// The key's value.
__device__ __forceinline__ uint64_t key_of(double v) {
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    return ~((b >> 63) ? ~b : (b | (1ull << 63)));
}
__device__ __forceinline__ double value_of(uint64_t key) {
    const uint64_t b = ~key;
    return __longlong_as_double(static_cast<int64_t>((b >> 63) ? (b & ~(1ull << 63)) : ~b));
}

constexpr int kSelBuckets = 4096;

// cand_l: z in, l + log p out.  One lane per candidate, a prefix in O
// neighbouring lanes: bound by the eight transcendental functions a candidate,
// so it runs apart from the perceptrons, whose LDS lets in two waves a SIMD.
// hist += the top 12 bits of the unmasked keys (they are the exponent: a few
// values, counted by wave).
__global__ __launch_bounds__(256) void k_ar_cand(ArLevel A, ArState* __restrict__ S, const uint64_t* __restrict__ keys,
                                                 const double* __restrict__ lin, const double* __restrict__ Tin,
                                                 double* __restrict__ cand_l, uint64_t* __restrict__ cand_key,
                                                 uint32_t* __restrict__ hist) {
    __shared__ uint32_t cnt[kSelBuckets];
    __shared__ unsigned long long total;
    const int lane = lane_id();
    if (S->redo) return;
    if (hist)
        for (int t = threadIdx.x; t < kSelBuckets; t += 256) cnt[t] = 0u;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const int sh = A.Dk;
    const int64_t n = S->B[A.level] << sh;
    const int c = static_cast<int>(threadIdx.x) & (A.O - 1);
    unsigned long long allowed = 0;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256; i0 < n; i0 += static_cast<int64_t>(gridDim.x) * 256) {
        const int64_t i = i0 + threadIdx.x;
        const bool live = i < n;
        const int64_t b = min(i, n - 1) >> sh;
        const double z = live ? cand_l[i] : 0.0;
        double sum = z;
        for (int m = A.O / 2; m >= 1; m >>= 1) sum += shfl_xor_d(sum, m);
        const double a = 2.0 * (z - sum / A.O);
        uint64_t key[kMaxWords];
#pragma unroll
        for (int w = 0; w < kMaxWords; ++w) key[w] = w < A.W ? keys[b * A.W + w] : 0ull;
        bool ok = live;
        if (A.n_up >= 0) {
            // electrons of the prefix: even qubits spin up, odd spin down
            // (word boundaries are even, so a bit's parity is its qubit's)
            int up = 0, dn = 0;
#pragma unroll
            for (int w = 0; w < kMaxWords; ++w) {
                const int nb = min(max(A.q0 - 64 * w, 0), 64);
                const uint64_t v = key[w] & (nb >= 64 ? ~0ull : ((1ull << nb) - 1ull));
                up += __popcll(v & kEven);
                dn += __popcll(v & kOdd);
            }
            const uint64_t mine = static_cast<uint64_t>(c) << (A.q0 & 1);
            up += __popcll(mine & kEven);
            dn += __popcll(mine & kOdd);
            ok = ok && up <= A.n_up && A.n_up <= up + A.rest_up && dn <= A.n_down && A.n_down <= dn + A.rest_down;
        }
        double mx = ok ? a : -INFINITY;
        for (int m = A.O / 2; m >= 1; m >>= 1) mx = fmax(mx, shfl_xor_d(mx, m));
        double s = ok ? exp(a - mx) : 0.0;
        for (int m = A.O / 2; m >= 1; m >>= 1) s += shfl_xor_d(s, m);
        const double lc = lin[b] + (a - (mx + log(s)));
        const double Lp = lc + gumbel(A.seed, A.level, key, A.W, c);
        double Z = ok ? Lp : -INFINITY;
        for (int m = A.O / 2; m >= 1; m >>= 1) Z = fmax(Z, shfl_xor_d(Z, m));
        const double T = Tin[b];
        double Lt = T;
        if (ok && Lp < Z) {
            const double v = T - Lp + log1mexp(Lp - Z);
            Lt = T - (fmax(v, 0.0) + log1p(exp(-fabs(v))));
        }
        // masked outcomes alone have the last key (a NaN of all ones would share it)
        uint64_t k = key_of(Lt);
        if (k == ~0ull) k = ~1ull;
        if (!ok) k = ~0ull;
        if (live) {
            cand_key[i] = k;
            cand_l[i] = lc;
        }
        uint64_t left = __ballot(ok);
        allowed += static_cast<unsigned long long>(__popcll(left));
        if (hist) {
            const int d = static_cast<int>(k >> 52);
            while (left) {
                const int first = __ffsll(static_cast<unsigned long long>(left)) - 1;
                const int fd = __builtin_amdgcn_readlane(d, first);
                const uint64_t same = __ballot(ok && d == fd) & left;
                if (lane == first) atomicAdd(&cnt[fd], static_cast<uint32_t>(__popcll(same)));
                left &= ~same;
            }
        }
    }
    if (lane == 0 && allowed) atomicAdd(&total, allowed);
    __syncthreads();
    if (threadIdx.x == 0 && total) atomicAdd(&S->allowed[A.level], total);
    if (hist)
        for (int t = threadIdx.x; t < kSelBuckets; t += 256)
            if (cnt[t]) atomicAdd(hist + t, cnt[t]);
}

// The next level's prefix of candidate idx.
__device__ __forceinline__ void child_key(const uint64_t* __restrict__ keys, int64_t idx, int O, int W, int q0,
                                          uint64_t* __restrict__ out) {
    const int64_t b = idx / O;
    const uint64_t c = static_cast<uint64_t>(idx % O);
    for (int w = 0; w < W; ++w) {
        uint64_t v = keys[b * W + w];
        const int lo = q0 - 64 * w;
        if (lo >= 0 && lo < 64) v |= c << lo;
        if (lo < 0 && lo > -64) v |= c >> (-lo);
        out[w] = v;
    }
}

__global__ __launch_bounds__(1024) void k_ar_root(ArState* __restrict__ S, uint32_t* __restrict__ hist, uint64_t* keys,
                                                  int W, double* l, double* T) {
    const int t = static_cast<int>(threadIdx.x);
    for (int q = t; q < kSelBuckets; q += 1024) hist[q] = 0u;
    for (int q = t; q < kArLevels; q += 1024) S->allowed[q] = 0ull;
    if (t < W) keys[t] = 0;
    if (t == 0) {
        S->B[0] = 1;
        S->redo = 0u;
        S->bound = 0u;
        l[0] = 0.0;
        T[0] = 0.0;
    }
}

// Where the need of a level, min(K, allowed), falls among the 4096 digits of
// `total`, which is cleared for the next user: the PASS-th 12 bits of the prefix;
// the first time also B of the next level.  One workgroup, four digits a thread.
template <int PASS>
__global__ __launch_bounds__(1024) void k_ar_pick(ArState* __restrict__ S, int level, int64_t K,
                                                  uint32_t* __restrict__ total) {
    __shared__ int64_t part[16];
    const int t = static_cast<int>(threadIdx.x);
    if (PASS == 2 && !S->deep) return;
    const int64_t allowed = static_cast<int64_t>(S->allowed[level]);
    const int64_t all_need = min(K, allowed);
    const bool all = all_need == allowed;
    const int64_t above = PASS == 0 ? 0 : S->prefix, base = PASS == 0 ? 0 : S->below;
    int64_t c[4], mine = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        c[q] = total[4 * t + q];
        total[4 * t + q] = 0u;
        mine += c[q];
    }
    int64_t upto = mine;
    for (int m = 1; m < 64; m <<= 1) {
        const int64_t v = __shfl_up(static_cast<long long>(upto), m);
        if ((t & 63) >= m) upto += v;
    }
    if ((t & 63) == 63) part[t / 64] = upto;
    __syncthreads();   // also: every thread has the state of the pass before
    if (t == 0) {
        if (PASS == 0) S->B[level + 1] = all_need;
        S->bound = 0u;
        S->shift = 52 - 12 * PASS;
        if (all) {
            S->prefix = int64_t(1) << (12 * (PASS + 1));
            S->below = all_need;
            S->deep = 0u;
        }
    }
    if (all) return;
    int64_t run = upto - mine;
    for (int w = 0; w < t / 64; ++w) run += part[w];
    const int64_t need = all_need - base;
    if (run < need && need <= run + mine) {
        int q = 0;
        for (; q < 3; ++q) {
            if (run + c[q] >= need) break;
            run += c[q];
        }
        S->prefix = (above << 12) | (4 * t + q);
        S->below = base + run;
        S->deep = c[q] > kArBound ? 1u : 0u;
    }
}

// The PASS-th 12 bits of the keys with the selected bits before: per workgroup
// in LDS, then its non-zero counts added to total (the order of integer
// additions does not matter).
template <int PASS>
__global__ __launch_bounds__(1024) void k_ar_hist(const ArState* __restrict__ S, int level, int sh, int64_t K,
                                                 const uint64_t* __restrict__ key, uint32_t* __restrict__ total) {
    __shared__ uint32_t h[kSelBuckets];
    const int64_t n = S->B[level] << sh;
    if (static_cast<int64_t>(S->allowed[level]) <= K || S->redo || (PASS == 2 && !S->deep)) return;
    for (int t = threadIdx.x; t < kSelBuckets; t += 1024) h[t] = 0u;
    __syncthreads();
    const uint64_t above = static_cast<uint64_t>(S->prefix);
    const int64_t step = static_cast<int64_t>(gridDim.x) * 1024;
#pragma unroll 4
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 1024 + threadIdx.x; i < n; i += step) {
        const uint64_t k = key[i];
        if ((k >> (64 - 12 * PASS)) == above && k != ~0ull)
            atomicAdd(&h[(k >> (52 - 12 * PASS)) & (kSelBuckets - 1)], 1u);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kSelBuckets; t += 1024)
        if (h[t]) atomicAdd(total + t, h[t]);
}

// cnt[tile] = the candidates below the selected prefix.  LIST:
// those of the prefix to the list (the tiles in any order), a tile's place in it
// taken at once: with an atomic a candidate the one word is what a prefix of
// thousands waits for.  Else cnt has them too.
template <bool LIST>
__global__ __launch_bounds__(256) void k_ar_count(ArState* __restrict__ S, int level, int sh,
                                                  const uint64_t* __restrict__ key, uint32_t* __restrict__ cnt,
                                                  uint64_t* __restrict__ bkey, uint32_t* __restrict__ bidx) {
    constexpr int kPer = kArTile / 256;
    __shared__ uint32_t total, listed[4], at0;
    if (S->redo) return;
    if (threadIdx.x == 0) total = 0u;
    __syncthreads();
    const int64_t n = S->B[level] << sh;
    const uint64_t prefix = static_cast<uint64_t>(S->prefix);
    const int shift = S->shift;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kArTile;
    if (base >= n) return;
    const int wave = static_cast<int>(threadIdx.x) / 64, lane = lane_id();
    uint64_t k[kPer];
    uint32_t below = 0, mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = base + j * 256 + threadIdx.x;
        k[j] = i < n ? key[i] : ~0ull;
        below += static_cast<uint32_t>(__popcll(__ballot((k[j] >> shift) < prefix && k[j] != ~0ull)));
        mine += static_cast<uint32_t>(__popcll(__ballot((k[j] >> shift) == prefix && k[j] != ~0ull)));
    }
    if (lane == 0) {
        atomicAdd(&total, below);
        listed[wave] = mine;
    }
    __syncthreads();
    const uint32_t all = listed[0] + listed[1] + listed[2] + listed[3];
    if (threadIdx.x == 0) {
        cnt[blockIdx.x] = LIST ? total : total + all;
        if (LIST && all) at0 = atomicAdd(&S->bound, all);
    }
    if (!LIST || all == 0u) return;
    __syncthreads();
    uint32_t at = at0;
    for (int w = 0; w < wave; ++w) at += listed[w];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const bool in = (k[j] >> shift) == prefix && k[j] != ~0ull;
        const uint64_t bal = __ballot(in);
        if (in) {
            const uint32_t to = at + static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1ull)));
            bkey[to] = k[j];
            bidx[to] = static_cast<uint32_t>(base + j * 256 + threadIdx.x);
        }
        at += static_cast<uint32_t>(__popcll(bal));
    }
}

// The first need - below of the list by (key, index): the last of them is the
// cut, each counts for its tile; then cnt becomes the tiles' offsets.  One
// workgroup.  The candidates of a 24-bit prefix grow with K (a flat tail of 52
// qubits: 130 at K = 2^16, 8000 at 2^22) and with the values' distance from
// zero (most of a peaked distribution's second shell); past what is ranked in
// LDS they are cut down first, by 8 bits a pass of the key bits left and then
// the index.
__global__ __launch_bounds__(1024) void k_ar_cut(ArState* __restrict__ S, int level, int sh,
                                                 const uint64_t* __restrict__ bkey, const uint32_t* __restrict__ bidx,
                                                 uint32_t* __restrict__ cnt, int64_t* __restrict__ off) {
    __shared__ uint64_t k[kArBound];
    __shared__ uint32_t v[kArBound];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t pick[3];   // digit, listed before it, listed with it
    __shared__ uint32_t put;
    __shared__ uint64_t last, first_out;
    __shared__ int64_t part[16];
    if (S->redo) return;
    const int t = static_cast<int>(threadIdx.x);
    const int64_t need = S->B[level + 1];
    const int64_t n = S->B[level] << sh;
    const uint32_t found = S->bound;
    if (found > kArList) {
        if (t == 0) S->redo = 1u;
        return;
    }
    const int shift = S->shift, key_passes = (shift + 7) / 8;
    const uint32_t r = static_cast<uint32_t>(need - S->below);   // 1 <= r <= found where there is a list
    if (t == 0) {
        last = 0ull;
        first_out = ~0ull;
        put = 0u;
    }
    uint64_t pk = 0, maskk = 0;
    uint32_t pi = 0, maski = 0;
    uint32_t before = 0, upto = found;   // before the chosen digits, and with them
    for (int d = 0; upto - before > kArBound && d < key_passes + 4; ++d) {
        if (t < 256) hist[t] = 0u;
        __syncthreads();
        const bool of_key = d < key_passes;
        const int s = of_key ? max(shift - 8 * (d + 1), 0) : 24 - 8 * (d - key_passes);
#pragma unroll 4
        for (uint32_t e = t; e < found; e += 1024) {
            const uint64_t ek = bkey[e];
            const uint32_t ei = bidx[e];
            if (((ek ^ pk) & maskk) == 0 && ((ei ^ pi) & maski) == 0)
                atomicAdd(&hist[(of_key ? ek >> s : static_cast<uint64_t>(ei) >> s) & 255], 1u);
        }
        __syncthreads();
        if (t < 64) {
            uint32_t c[4], own = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = hist[4 * t + q];
                own += c[q];
            }
            uint32_t run = own;
            for (int m = 1; m < 64; m <<= 1) {
                const uint32_t u = __shfl_up(run, m);
                if (t >= m) run += u;
            }
            run += before - own;
            if (run < r && r <= run + own) {   // one lane
                int q = 0;
                for (; q < 3; ++q) {
                    if (run + c[q] >= r) break;
                    run += c[q];
                }
                pick[0] = static_cast<uint32_t>(4 * t + q);
                pick[1] = run;
                pick[2] = c[q];
            }
        }
        __syncthreads();
        before = pick[1];
        upto = before + pick[2];
        if (of_key) {
            pk |= static_cast<uint64_t>(pick[0]) << s;
            maskk |= 255ull << s;
        } else {
            pi |= pick[0] << s;
            maski |= 255u << s;
        }
        __syncthreads();
    }
    const int m = static_cast<int>(min(upto - before, static_cast<uint32_t>(kArBound)));
    if (maskk == 0) {
        for (int e = t; e < m; e += 1024) {
            k[e] = bkey[e];
            v[e] = bidx[e];
        }
    } else {
        __syncthreads();
        for (uint32_t e = t; e < found; e += 1024) {
            const uint64_t ek = bkey[e];
            const uint32_t ei = bidx[e];
            const uint64_t mk = ek & maskk;
            const uint32_t mi = ei & maski;
            if (mk == pk && mi == pi) {
                const uint32_t at = atomicAdd(&put, 1u);
                if (at < kArBound) {
                    k[at] = ek;
                    v[at] = ei;
                }
            } else if (mk < pk || (mk == pk && mi < pi)) {
                atomicAdd(cnt + ei / kArTile, 1u);
            }
        }
    }
    __syncthreads();
    for (int e = t; e < m; e += 1024) {
        const uint64_t ek = k[e];
        const uint32_t ei = v[e];
        uint32_t rank = before;
        for (int q = 0; q < m; ++q) rank += (k[q] < ek) | ((k[q] == ek) & (v[q] < ei));
        if (rank < r) atomicAdd(cnt + ei / kArTile, 1u);
        if (rank == r - 1) {
            S->cut_key = ek;
            S->cut_idx = ei;
            last = ek;
        }
        if (rank == r) first_out = ek;
    }
    __threadfence();
    __syncthreads();
    if (t == 0 && m && last == first_out) S->redo = 1u;
    const int64_t tiles = (n + kArTile - 1) / kArTile;
    int64_t base = 0;
    for (int64_t t0 = 0; t0 < tiles; t0 += 1024) {
        const int64_t mine = t0 + t < tiles
                                 ? static_cast<int64_t>(__hip_atomic_load(cnt + t0 + t, __ATOMIC_RELAXED,
                                                                          __HIP_MEMORY_SCOPE_AGENT))
                                 : 0;
        int64_t run = mine;
        for (int q = 1; q < 64; q <<= 1) {
            const int64_t u = __shfl_up(static_cast<long long>(run), q);
            if ((t & 63) >= q) run += u;
        }
        if ((t & 63) == 63) part[t / 64] = run;
        __syncthreads();
        int64_t first = base;
        for (int w = 0; w < 16; ++w) {
            if (w < t / 64) first += part[w];
            base += part[w];
        }
        if (t0 + t < tiles) off[t0 + t] = first + run - mine;
        __syncthreads();
    }
    if (t == 0) S->listed = base;
}

// The kept candidates, in index order, as the next level's prefixes; at the
// last level also their keys and places for the sort.  PAIRS: the candidates up
// to the prefix, as keys and indices alone.
template <bool PAIRS>
__global__ __launch_bounds__(256) void k_ar_emit(const ArState* __restrict__ S, ArLevel A, int64_t room,
                                                 const uint64_t* __restrict__ key, const double* __restrict__ cand_l,
                                                 const int64_t* __restrict__ off, const uint64_t* __restrict__ keys,
                                                 uint64_t* __restrict__ out_keys, double* __restrict__ out_l,
                                                 double* __restrict__ out_T, uint64_t* __restrict__ out_key,
                                                 uint32_t* __restrict__ out_idx) {
    constexpr int kPer = kArTile / 256;
    __shared__ uint32_t part[kPer * 4];
    if (S->redo) return;
    const int64_t n = S->B[A.level] << A.Dk;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kArTile;
    if (base >= n) return;
    const uint64_t prefix = static_cast<uint64_t>(S->prefix);
    const int shift = S->shift;
    const uint64_t ck = S->cut_key;
    const uint32_t ci = S->cut_idx;
    const int wave = static_cast<int>(threadIdx.x) / 64, lane = lane_id();
    uint64_t k[kPer];
    uint32_t keep = 0, before[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = base + j * 256 + threadIdx.x;
        k[j] = i < n ? key[i] : ~0ull;
        const bool in = k[j] != ~0ull &&
                        ((k[j] >> shift) < prefix ||
                         ((k[j] >> shift) == prefix &&
                          (PAIRS || k[j] < ck || (k[j] == ck && static_cast<uint32_t>(i) <= ci))));
        const uint64_t bal = __ballot(in);
        before[j] = static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1ull)));
        keep |= (in ? 1u : 0u) << j;
        if (lane == 0) part[4 * j + wave] = static_cast<uint32_t>(__popcll(bal));
    }
    __syncthreads();
    if (wave == 0) {
        static_assert(kPer * 4 == 64, "a part a lane");
        const uint32_t mine = part[lane];
        uint32_t upto = mine;
        for (int q = 1; q < 64; q <<= 1) {
            const uint32_t u = __shfl_up(upto, q);
            if (lane >= q) upto += u;
        }
        part[lane] = upto - mine;
    }
    __syncthreads();
    const int64_t at0 = off[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (!((keep >> j) & 1u)) continue;
        const int64_t i = base + j * 256 + threadIdx.x;
        const int64_t at = at0 + part[4 * j + wave] + before[j];
        if (at >= room) continue;
        if constexpr (PAIRS) {
            out_key[at] = k[j];
            out_idx[at] = static_cast<uint32_t>(i);
            continue;
        }
        child_key(keys, i, A.O, A.W, A.q0, out_keys + at * A.W);
        out_l[at] = cand_l[i];
        out_T[at] = value_of(k[j]);
        if (out_key) {
            out_key[at] = k[j];
            out_idx[at] = static_cast<uint32_t>(at);
        }
    }
}

// The first n sorted candidates as prefixes.
__global__ void k_ar_gather(const uint64_t* __restrict__ keys, const uint64_t* __restrict__ sorted_key,
                            const uint32_t* __restrict__ sorted_idx, int64_t n, int O, int W, int q0,
                            const double* __restrict__ cand_l, uint64_t* __restrict__ out_keys,
                            double* __restrict__ out_l, double* __restrict__ out_T) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t idx = sorted_idx[i];
    child_key(keys, idx, O, W, q0, out_keys + i * W);
    out_l[i] = cand_l[idx];
    out_T[i] = value_of(sorted_key[i]);
}

// The samples in sorted order to the caller; equal neighbours ask for the search
// with sorted levels.
__global__ void k_ar_out(ArState* __restrict__ S, const uint64_t* __restrict__ sorted_key,
                         const uint32_t* __restrict__ sorted_idx, int64_t n, int W, const uint64_t* __restrict__ keys,
                         const double* __restrict__ l, uint64_t* __restrict__ out_keys, double* __restrict__ out_l,
                         double* __restrict__ out_T) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t idx = sorted_idx[i];
    const uint64_t k = sorted_key[i];
    if (i + 1 < n && sorted_key[i + 1] == k) S->redo = 1u;
    for (int w = 0; w < W; ++w) out_keys[i * W + w] = keys[static_cast<int64_t>(idx) * W + w];
    out_l[i] = l[idx];
    if (out_T) out_T[i] = value_of(k);
}

inline unsigned blocks256(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

ArLevel level_of(const ArModelDev& M, int level, uint64_t seed) {
    ArLevel A;
    A.N = M.n_qubits;
    A.W = (M.n_qubits + 63) / 64;
    A.D = M.qudit;
    A.q0 = level * M.qudit;
    A.Dk = min(M.qudit, M.n_qubits - A.q0);
    A.O = 1 << A.Dk;
    A.level = level;
    A.n_up = M.n_up;
    A.n_down = M.n_down;
    A.rest_up = 0;
    A.rest_down = 0;
    for (int q = A.q0 + A.Dk; q < A.N; ++q) {
        if (q & 1)
            ++A.rest_down;
        else
            ++A.rest_up;
    }
    A.seed = seed;
    const int O_full = 1 << M.qudit;
    A.W1 = M.W1 + static_cast<int64_t>(level) * kArH * A.N;
    A.b1 = M.b1 + static_cast<int64_t>(level) * kArH;
    A.W2 = M.W2 + static_cast<int64_t>(level) * kArH * kArH;
    A.b2 = M.b2 + static_cast<int64_t>(level) * kArH;
    A.W3 = M.W3 + static_cast<int64_t>(level) * O_full * kArH;
    A.b3 = M.b3 + static_cast<int64_t>(level) * O_full;
    return A;
}

// The candidates of at most B prefixes (the device has the number).
void launch_candidates(const ArLevel& A, int64_t B, const ArScratch& R, int cur, uint32_t* hist, hipStream_t st) {
    if (B > kArWide)
        launch_net<16>(A, B, R.state, R.keys[cur], R.cand_l, st);
    else
        launch_net<4>(A, B, R.state, R.keys[cur], R.cand_l, st);
    const int64_t blocks = std::min<int64_t>((B * A.O + 255) / 256, 2048);
    hipLaunchKernelGGL(k_ar_cand, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, A, R.state, R.keys[cur],
                       R.l[cur], R.T[cur], R.cand_l, R.cand_key, hist);
}

}  // namespace

size_t ar_state_bytes() { return sizeof(ArState); }
int64_t ar_tiles(int64_t n) { return (n + kArTile - 1) / kArTile; }

hipError_t launch_ar_root(const ArScratch& R, int W, hipStream_t st) {
    hipLaunchKernelGGL(k_ar_root, dim3(1), dim3(1024), 0, st, R.state, R.hist, R.keys[0], W, R.l[0], R.T[0]);
    return hipGetLastError();
}

// Sets up to this size take two digits: the prefix then mostly holds some 130
// candidates, and a third digit's two launches a level, even where they return
// at once, would be 2% of it (2^16: 35 of 2190 us).
constexpr int64_t kArTwoDigits = int64_t(1) << 16;

namespace {

// The level's candidates, and the prefix of the need-th of them.  Where at most
// K can come out nothing is selected: the digit passes stay away.
void launch_select(const ArLevel& A, int64_t B, int64_t K, const ArScratch& R, int cur, hipStream_t st) {
    const int64_t n = B * A.O;
    const bool select = n > K;
    const dim3 one(1), block(1024);
    launch_candidates(A, B, R, cur, select ? R.hist : nullptr, st);
    hipLaunchKernelGGL(k_ar_pick<0>, one, block, 0, st, R.state, A.level, K, R.hist);
    if (!select) return;
    const dim3 few(static_cast<unsigned>(std::min<int64_t>((n + 8191) / 8192, 256)));   // each adds up to 4096 counts
    hipLaunchKernelGGL(k_ar_hist<1>, few, block, 0, st, R.state, A.level, A.Dk, K, R.cand_key, R.hist);
    hipLaunchKernelGGL(k_ar_pick<1>, one, block, 0, st, R.state, A.level, K, R.hist);
    if (K <= kArTwoDigits) return;
    hipLaunchKernelGGL(k_ar_hist<2>, few, block, 0, st, R.state, A.level, A.Dk, K, R.cand_key, R.hist);
    hipLaunchKernelGGL(k_ar_pick<2>, one, block, 0, st, R.state, A.level, K, R.hist);
}

}  // namespace

hipError_t launch_ar_level(const ArModelDev& M, int level, int64_t B, int64_t K, uint64_t seed, bool last,
                           const ArScratch& R, int cur, hipStream_t st) {
    const ArLevel A = level_of(M, level, seed);
    launch_select(A, B, K, R, cur, st);
    const unsigned tiles = static_cast<unsigned>(ar_tiles(B * A.O));
    hipLaunchKernelGGL(k_ar_count<true>, dim3(tiles), dim3(256), 0, st, R.state, level, A.Dk, R.cand_key, R.cnt,
                       R.bkey, R.bidx);
    hipLaunchKernelGGL(k_ar_cut, dim3(1), dim3(1024), 0, st, R.state, level, A.Dk, R.bkey, R.bidx, R.cnt, R.off);
    hipLaunchKernelGGL(k_ar_emit<false>, dim3(tiles), dim3(256), 0, st, R.state, A, K, R.cand_key, R.cand_l,
                       R.off, R.keys[cur], R.keys[cur ^ 1], R.l[cur ^ 1], R.T[cur ^ 1], last ? R.sort_key : nullptr,
                       R.sort_idx);
    return hipGetLastError();
}

hipError_t launch_ar_survivors(const ArModelDev& M, int level, int64_t B, int64_t K, uint64_t seed, const ArScratch& R,
                               int cur, hipStream_t st) {
    const ArLevel A = level_of(M, level, seed);
    launch_select(A, B, K, R, cur, st);
    const unsigned tiles = static_cast<unsigned>(ar_tiles(B * A.O));
    hipLaunchKernelGGL(k_ar_count<false>, dim3(tiles), dim3(256), 0, st, R.state, level, A.Dk, R.cand_key, R.cnt,
                       nullptr, nullptr);
    hipLaunchKernelGGL(k_ar_cut, dim3(1), dim3(1024), 0, st, R.state, level, A.Dk, nullptr, nullptr, R.cnt, R.off);
    hipLaunchKernelGGL(k_ar_emit<true>, dim3(tiles), dim3(256), 0, st, R.state, A, B * A.O, R.cand_key, nullptr,
                       R.off, nullptr, nullptr, nullptr, nullptr, R.bkey, R.bidx);
    return hipGetLastError();
}

hipError_t launch_ar_gather(const ArModelDev& M, int level, const ArScratch& R, int cur, const uint64_t* sorted_key,
                            const uint32_t* sorted_idx, int64_t n, hipStream_t st) {
    const ArLevel A = level_of(M, level, 0);
    hipLaunchKernelGGL(k_ar_gather, dim3(blocks256(n)), dim3(256), 0, st, R.keys[cur], sorted_key, sorted_idx, n, A.O,
                       A.W, A.q0, R.cand_l, R.keys[cur ^ 1], R.l[cur ^ 1], R.T[cur ^ 1]);
    return hipGetLastError();
}

hipError_t launch_ar_out(const ArScratch& R, int cur, const uint64_t* sorted_key, const uint32_t* sorted_idx,
                         int64_t n, int W, uint64_t* out_keys, double* out_l, double* out_T, hipStream_t st) {
    hipLaunchKernelGGL(k_ar_out, dim3(blocks256(n)), dim3(256), 0, st, R.state, sorted_key, sorted_idx, n, W,
                       R.keys[cur], R.l[cur], out_keys, out_l, out_T);
    return hipGetLastError();
}

hipError_t ar_read(const ArScratch& R, int level, ArResult* out, hipStream_t st) {
    ArState S;
    hipError_t e = hipMemcpyAsync(&S, R.state, sizeof(S), hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    out->B = S.B[level];
    out->listed = S.listed;
    out->redo = S.redo != 0;
    return hipSuccess;
}

}  // namespace eloc
