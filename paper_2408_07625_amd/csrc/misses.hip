// The conventional local energy's extra states (Eq. local_energy summed over
// every x', the estimator that the sample-aware form replaces): the x' =
// x ^ XY_g, x in U, that are not in U and whose matrix element is non-zero.
//
// Whether an element is non-zero (|H| > tol * sum |h_l| over the group's run;
// strings that cancel exactly, e.g. hopping strings between particle-number
// sectors, give no state) depends on few bits of the ket: the Z masks of a
// run differ by sums of a few masks, three for a double excitation, and |H|
// by the parities of the ket under those.  k_miss_rules finds the masks of a
// group and the values of H for their eight parities; a candidate then is
// three popcounts.  Groups with more masks (singles) keep the sum over the
// run.
//
// k_misses walks the same (row, XY group) candidates as LoopOverTerms: a
// wave owns kMissRows rows (keys in scalar registers), its lanes sweep 64
// groups of the row's chunk per step.  A candidate whose element is non-zero
// is looked up in U's table, and is a miss when absent.  The misses of a step
// (all rows) take one range of the output from an atomic counter and are
// written there (ballot + mbcnt), those past the capacity only counted; the
// caller reruns with a larger buffer when the count exceeds it.  The list is
// then sorted and made unique, so the order in which waves append does not
// show in the result.
//
// For one-word keys of at most 30 qubits (k_miss_bits) the states set their
// bit in a bitmap over the key space instead, U's bits are cleared after it
// (no lookups), and the set bits, read in order, are the unique states
// already sorted.  20 000 rows by 10 466 groups, a third of them non-zero:
// 3.6 ms with a lookup, the run's sum and an atomic for each, 0.5 this way.
#include "device.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eloc {

namespace {

constexpr int kMissRows = 8;

// The parities that decide whether a group's element is non-zero: bit idx of
// tab, idx = sum over k of parity(ket & mask[k]) << k.  kMissRun: evaluate
// the run.
constexpr uint32_t kMissRun = 256u;

template <int W>
struct MissRule {
    uint64_t mask[3][W];
    uint32_t tab;
    uint32_t pad;
};

struct MissArgs {
    const void* groups;      // GroupRec<W>[G]
    const uint64_t* ghash;   // lin(XY_g)
    const void* terms;       // TermRec<W>[T]
    int n_groups;
    int per_chunk;
    int chunks;
    const uint64_t* keys;
    const uint64_t* khash;
    Table ktable;
    int64_t M;
    const uint32_t* prep_err;
    double tol;
    const void* rules;       // MissRule<W>[G]
};

// |H_xx'| > tol * sum |h_l| over the group's run [b, e) (real part [b, m),
// imaginary part [m, e)), H evaluated with the ket x'.
template <int W>
__device__ __forceinline__ bool nonzero_element(const TermRec<W>* __restrict__ terms, const GroupRec<W>& gr,
                                                const uint64_t* ket, double tol) {
    double hr = 0.0, hi = 0.0, sa = 0.0;
    for (int t = gr.begin; t < gr.mid; ++t) {
        const TermRec<W> tr = terms[t];
        hr += term_f64<W>(tr, ket);
        sa += fabs(tr.h);
    }
    for (int t = gr.mid; t < gr.end; ++t) {
        const TermRec<W> tr = terms[t];
        hi += term_f64<W>(tr, ket);
        sa += fabs(tr.h);
    }
    return hypot(hr, hi) > tol * sa;
}

__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
}

template <int W>
__global__ __launch_bounds__(64) void k_miss_rules(const GroupRec<W>* __restrict__ groups,
                                                   const TermRec<W>* __restrict__ terms, int n_groups, double tol,
                                                   MissRule<W>* __restrict__ rules) {
    const int g = static_cast<int>(blockIdx.x) * 64 + static_cast<int>(threadIdx.x);
    if (g >= n_groups) return;
    const GroupRec<W> gr = groups[g];
    MissRule<W> rule{};
    int pivot[3] = {0, 0, 0};
    int rank = 0;
    // what `z` ^ the first mask of its part is a sum of; the remainder left in d
    auto reduce = [&](int t, uint64_t (&d)[W]) {
        const int first = t < gr.mid ? gr.begin : gr.mid;
        uint32_t coef = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) d[w] = terms[t].yz[w] ^ terms[first].yz[w];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k >= rank) continue;
            const uint64_t word = W == 2 && pivot[k] >= 64 ? d[W - 1] : d[0];
            if ((word >> (pivot[k] & 63)) & 1ull) {
                coef |= 1u << k;
#pragma unroll
                for (int w = 0; w < W; ++w) d[w] ^= rule.mask[k][w];
            }
        }
        return coef;
    };
    bool run = false;
    for (int t = gr.begin; t < gr.end && !run; ++t) {
        uint64_t d[W];
        reduce(t, d);
        int q = -1;
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (q < 0 && d[w]) q = 64 * w + __ffsll(static_cast<unsigned long long>(d[w])) - 1;
        if (q < 0) continue;
        if (rank == 3) {
            run = true;
            break;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == rank) {
                pivot[k] = q;
#pragma unroll
                for (int w = 0; w < W; ++w) rule.mask[k][w] = d[w];
            }
        ++rank;
    }
    if (run) {
        rule.tab = kMissRun;
    } else {
        for (uint32_t idx = 0; idx < 8u; ++idx) {
            double hr = 0.0, hi = 0.0, sa = 0.0;
            for (int t = gr.begin; t < gr.end; ++t) {
                uint64_t d[W];
                const double h = terms[t].h;
                const double v = (__popc(reduce(t, d) & idx) & 1) ? -h : h;
                (t < gr.mid ? hr : hi) += v;
                sa += fabs(h);
            }
            if (hypot(hr, hi) > tol * sa) rule.tab |= 1u << idx;
        }
    }
    rules[g] = rule;
}

template <int W>
__device__ __forceinline__ uint32_t rule_index(const MissRule<W>& rule, const uint64_t* ket) {
    uint32_t idx = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int p = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) p += __popcll(ket[w] & rule.mask[k][w]);
        idx |= (static_cast<uint32_t>(p) & 1u) << k;
    }
    return idx;
}

// Bit r: row r's element of the group is non-zero, by its run; a term is read
// once for all rows.
__device__ __forceinline__ uint32_t run_hits(const TermRec<1>* __restrict__ terms, const GroupRec<1>& gr,
                                             const uint32_t (&x)[kMissRows], uint32_t xy, double tol) {
    double hr[kMissRows] = {}, hi[kMissRows] = {}, sa = 0.0;
    for (int t = gr.begin; t < gr.mid; ++t) {
        const double h = terms[t].h;
        const uint32_t yz = static_cast<uint32_t>(terms[t].yz[0]);
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) hr[r] += (__popc(yz & (x[r] ^ xy)) & 1) ? -h : h;
        sa += fabs(h);
    }
    for (int t = gr.mid; t < gr.end; ++t) {
        const double h = terms[t].h;
        const uint32_t yz = static_cast<uint32_t>(terms[t].yz[0]);
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) hi[r] += (__popc(yz & (x[r] ^ xy)) & 1) ? -h : h;
        sa += fabs(h);
    }
    uint32_t hit = 0;
#pragma unroll
    for (int r = 0; r < kMissRows; ++r) hit |= hypot(hr[r], hi[r]) > tol * sa ? 1u << r : 0u;
    return hit;
}

// One-word keys of at most 30 qubits, all in 32 bits.  What bounds it is the
// bitmap's traffic; a bit is read before it is set, as most are set many
// times (an atomic goes past the L2s), and the reads of a step's rows are in
// flight together.
__global__ __launch_bounds__(64) void k_miss_bits(MissArgs A, uint32_t* __restrict__ bitmap) {
    const int lane = lane_id();
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kMissRows;
    const int chunk = static_cast<int>(blockIdx.y);
    if (row0 >= A.M) return;
    if (__builtin_amdgcn_readfirstlane(static_cast<int>(*A.prep_err)) != 0) return;   // U invalid: no states
    const GroupRec<1>* __restrict__ groups = static_cast<const GroupRec<1>*>(A.groups);
    const TermRec<1>* __restrict__ terms = static_cast<const TermRec<1>*>(A.terms);
    const MissRule<1>* __restrict__ rules = static_cast<const MissRule<1>*>(A.rules);
    uint32_t x[kMissRows];
#pragma unroll
    for (int r = 0; r < kMissRows; ++r) x[r] = static_cast<uint32_t>(A.keys[min(row0 + r, A.M - 1)]);
    const int g0 = chunk * A.per_chunk;
    const int g1 = min(A.n_groups, g0 + A.per_chunk);
    for (int base = g0; base < g1; base += 64) {
        const int g = min(base + lane, g1 - 1);   // lanes past the end set the last group's bits once more
        const uint32_t xy = static_cast<uint32_t>(groups[g].xy[0]);
        const MissRule<1> rule = rules[g];
        const uint32_t m0 = static_cast<uint32_t>(rule.mask[0][0]), m1 = static_cast<uint32_t>(rule.mask[1][0]),
                       m2 = static_cast<uint32_t>(rule.mask[2][0]);
        const bool run = rule.tab == kMissRun && xy != 0u;   // x itself is no miss
        uint32_t hit = 0;
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) {
            const uint32_t k = x[r] ^ xy;
            const uint32_t idx = (__popc(k & m0) & 1) | ((__popc(k & m1) & 1) << 1) | ((__popc(k & m2) & 1) << 2);
            hit |= ((rule.tab >> idx) & 1u) << r;
        }
        if (__ballot(run)) {
            if (run) hit = run_hits(terms, groups[g], x, xy, A.tol);
        }
        uint32_t word[kMissRows];
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) {
            word[r] = ~0u;
            if ((hit >> r) & 1u) word[r] = bitmap[(x[r] ^ xy) >> 5];
        }
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) {
            const uint32_t key = x[r] ^ xy, bit = 1u << (key & 31u);
            if (!(word[r] & bit)) atomicOr(bitmap + (key >> 5), bit);   // rows past the end: the last row once more
        }
    }
}

// U's own bits go.
__global__ void k_miss_clear(const uint64_t* __restrict__ keys, int64_t n, const uint32_t* __restrict__ prep_err,
                             uint32_t* __restrict__ bitmap) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n || *prep_err) return;
    const uint32_t key = static_cast<uint32_t>(keys[i]);
    atomicAnd(bitmap + (key >> 5), ~(1u << (key & 31u)));
}

template <int W, int TK>
__global__ __launch_bounds__(64) void k_misses(MissArgs A, unsigned long long* __restrict__ counter, int64_t capacity,
                                               uint64_t* __restrict__ out) {
    const int lane = lane_id();
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kMissRows;
    const int chunk = static_cast<int>(blockIdx.y);
    if (row0 >= A.M) return;
    const int nr = static_cast<int>(min(static_cast<int64_t>(kMissRows), A.M - row0));
    if (__builtin_amdgcn_readfirstlane(static_cast<int>(*A.prep_err)) != 0) return;   // U invalid: no states
    const GroupRec<W>* __restrict__ groups = static_cast<const GroupRec<W>*>(A.groups);
    const TermRec<W>* __restrict__ terms = static_cast<const TermRec<W>*>(A.terms);
    const MissRule<W>* __restrict__ rules = static_cast<const MissRule<W>*>(A.rules);
    uint64_t x[kMissRows][W];
    uint64_t hx[kMissRows];
#pragma unroll
    for (int r = 0; r < kMissRows; ++r) {
        const int64_t row = min(row0 + r, A.M - 1);
#pragma unroll
        for (int w = 0; w < W; ++w) x[r][w] = A.keys[row * W + w];
        hx[r] = A.khash[row];
    }
    const int nstash = __builtin_amdgcn_readfirstlane(static_cast<int>(A.ktable.stash->count));
    const int g0 = chunk * A.per_chunk;
    const int g1 = min(A.n_groups, g0 + A.per_chunk);
    for (int base = g0; base < g1; base += 64) {
        const int g = base + lane;
        const bool valid = g < g1;
        const GroupRec<W> gr = groups[min(g, g1 - 1)];
        const MissRule<W> rule = rules[min(g, g1 - 1)];
        const bool by_run = rule.tab == kMissRun;
        bool self = true;   // x itself is no miss
#pragma unroll
        for (int w = 0; w < W; ++w) self = self && gr.xy[w] == 0ull;
        const uint64_t gh = A.ghash[min(g, g1 - 1)];
        uint64_t m[kMissRows];
        bool miss[kMissRows];
        int total = 0;
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) {
            uint64_t xp[W];
#pragma unroll
            for (int w = 0; w < W; ++w) xp[w] = x[r][w] ^ gr.xy[w];
            miss[r] = false;
            if (valid && r < nr && !self && (by_run || ((rule.tab >> rule_index<W>(rule, xp)) & 1u) != 0u)) {
                const auto hs = salted<TK>(A.ktable, hx[r] ^ gh);
                const int j = table_settle<TK, W>(A.ktable, A.keys, load_slot<TK>(A.ktable, slot1(A.ktable, hs)),
                                                  load_slot<TK>(A.ktable, slot2(A.ktable, hs)), hs, xp, nstash);
                miss[r] = j < 0 && (!by_run || nonzero_element<W>(terms, gr, xp, A.tol));
            }
            m[r] = __ballot(miss[r]);
            total += __popcll(m[r]);
        }
        if (total == 0) continue;   // wave-uniform
        unsigned long long first = 0ull;
        if (lane == 0) first = atomicAdd(counter, static_cast<unsigned long long>(total));
        const int64_t at0 = static_cast<int64_t>(
            (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(first >> 32))))
             << 32) |
            static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(first))));
        int64_t run = 0;
#pragma unroll
        for (int r = 0; r < kMissRows; ++r) {
            if (miss[r]) {
                const int64_t at = at0 + run + lanes_below(m[r]);
                if (at < capacity) {
#pragma unroll
                    for (int w = 0; w < W; ++w) out[at * W + w] = x[r][w] ^ gr.xy[w];
                }
            }
            run += __popcll(m[r]);
        }
    }
}

// flags[i] = 1 if sorted key i differs from key i - 1 (first of its run)
template <int W>
__global__ void k_first_of_run(const uint64_t* __restrict__ sorted, int64_t n, int32_t* __restrict__ flags) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool first = i == 0;
    if (!first) {
#pragma unroll
        for (int w = 0; w < W; ++w) first = first || sorted[i * W + w] != sorted[(i - 1) * W + w];
    }
    flags[i] = first ? 1 : 0;
}

template <int W>
__global__ void k_scatter_unique(const uint64_t* __restrict__ sorted, int64_t n, const int32_t* __restrict__ flags,
                                 const int64_t* __restrict__ pos, uint64_t* __restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n || !flags[i]) return;
    const int64_t o = pos[i];
#pragma unroll
    for (int w = 0; w < W; ++w) out[o * W + w] = sorted[i * W + w];
}

inline unsigned blocks256(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

// Four words a thread: a workgroup counts a tile, so that the scan is over
// tiles (2^23 words: counts, scan and keys 140 us by words, 52 by tiles).
static_assert(kBitmapTile == 4 * 256, "a workgroup's words");
__device__ __forceinline__ uint4 tile_words(const uint32_t* __restrict__ bitmap, int64_t nwords, int64_t i) {
    if (i + 4 <= nwords) return *reinterpret_cast<const uint4*>(bitmap + i);
    uint4 b = make_uint4(0u, 0u, 0u, 0u);
    if (i < nwords) b.x = bitmap[i];
    if (i + 1 < nwords) b.y = bitmap[i + 1];
    if (i + 2 < nwords) b.z = bitmap[i + 2];
    return b;
}

__device__ __forceinline__ int popc4(const uint4& b) { return __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w); }

__global__ __launch_bounds__(256) void k_bitmap_counts(const uint32_t* __restrict__ bitmap, int64_t nwords,
                                                       int32_t* __restrict__ counts) {
    __shared__ int part[4];
    int c = popc4(tile_words(bitmap, nwords, static_cast<int64_t>(blockIdx.x) * kBitmapTile + threadIdx.x * 4));
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);
    if ((threadIdx.x & 63u) == 0) part[threadIdx.x / 64] = c;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

__global__ __launch_bounds__(256) void k_bitmap_keys(const uint32_t* __restrict__ bitmap, int64_t nwords,
                                                     const int64_t* __restrict__ pos, uint64_t* __restrict__ out) {
    __shared__ int part[4];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBitmapTile + threadIdx.x * 4;
    const uint4 b4 = tile_words(bitmap, nwords, i);
    const int mine = popc4(b4), wave = static_cast<int>(threadIdx.x) / 64;
    int upto = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(upto, d, 64);
        if (lane_id() >= d) upto += o;
    }
    if (lane_id() == 63) part[wave] = upto;
    __syncthreads();
    int64_t o = pos[blockIdx.x] + upto - mine;
    for (int w = 0; w < wave; ++w) o += part[w];
    const uint32_t words[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
    for (int u = 0; u < 4; ++u)
        for (uint32_t b = words[u]; b; b &= b - 1u)
            out[o++] = (static_cast<uint64_t>(i + u) << 5) | static_cast<uint64_t>(__builtin_ctz(b));
}

dim3 miss_grid(const MissArgs& A) {
    return dim3(static_cast<unsigned>((A.M + kMissRows - 1) / kMissRows), static_cast<unsigned>(A.chunks));
}

template <int W, int TK>
hipError_t launch_misses_t(const MissArgs& A, unsigned long long* counter, int64_t capacity, uint64_t* out,
                           hipStream_t st) {
    hipLaunchKernelGGL((k_misses<W, TK>), miss_grid(A), dim3(64), 0, st, A, counter, capacity, out);
    return hipGetLastError();
}

MissArgs miss_args(const HamDev& H, const SampleDev& S, int chunks, int per_chunk, double tol, const void* rules) {
    MissArgs A;
    A.groups = H.groups;
    A.ghash = H.group_hash;
    A.terms = H.terms;
    A.n_groups = static_cast<int>(H.n_groups);
    A.per_chunk = per_chunk;
    A.chunks = chunks;
    A.keys = S.keys;
    A.khash = S.hash;
    A.ktable = S.table;
    A.M = S.n;
    A.prep_err = S.prep_err;
    A.tol = tol;
    A.rules = rules;
    return A;
}

}  // namespace

size_t miss_rule_bytes(const HamDev& H) {
    return static_cast<size_t>(H.n_groups) * (H.W == 2 ? sizeof(MissRule<2>) : sizeof(MissRule<1>));
}

hipError_t launch_miss_rules(const HamDev& H, double tol, void* rules, hipStream_t st) {
    const int G = static_cast<int>(H.n_groups);
    if (G == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>((G + 63) / 64));
    if (H.W == 2)
        hipLaunchKernelGGL(k_miss_rules<2>, grid, dim3(64), 0, st, static_cast<const GroupRec<2>*>(H.groups),
                           static_cast<const TermRec<2>*>(H.terms), G, tol, static_cast<MissRule<2>*>(rules));
    else
        hipLaunchKernelGGL(k_miss_rules<1>, grid, dim3(64), 0, st, static_cast<const GroupRec<1>*>(H.groups),
                           static_cast<const TermRec<1>*>(H.terms), G, tol, static_cast<MissRule<1>*>(rules));
    return hipGetLastError();
}

hipError_t launch_misses(const HamDev& H, const SampleDev& S, int chunks, int per_chunk, double tol, const void* rules,
                         unsigned long long* counter, int64_t capacity, uint64_t* out, hipStream_t st) {
    const MissArgs A = miss_args(H, S, chunks, per_chunk, tol, rules);
    const int tk = table_kind(H.W, H.narrow);
    if (H.W == 2) return launch_misses_t<2, kTabVerify>(A, counter, capacity, out, st);
    if (tk == kTabNarrow) return launch_misses_t<1, kTabNarrow>(A, counter, capacity, out, st);
    return launch_misses_t<1, kTabWide>(A, counter, capacity, out, st);
}

hipError_t launch_misses_bitmap(const HamDev& H, const SampleDev& S, int chunks, int per_chunk, double tol,
                                const void* rules, uint32_t* bitmap, hipStream_t st) {
    if (H.W != 1 || H.n_qubits > kMissBitmapQubits || !bitmap) return hipErrorInvalidValue;
    const MissArgs A = miss_args(H, S, chunks, per_chunk, tol, rules);
    hipLaunchKernelGGL(k_miss_bits, miss_grid(A), dim3(64), 0, st, A, bitmap);
    hipLaunchKernelGGL(k_miss_clear, dim3(blocks256(S.n)), dim3(256), 0, st, S.keys, S.n, S.prep_err, bitmap);
    return hipGetLastError();
}

hipError_t launch_bitmap_counts(const uint32_t* bitmap, int64_t nwords, int32_t* counts, hipStream_t st) {
    hipLaunchKernelGGL(k_bitmap_counts, dim3(static_cast<unsigned>(bitmap_tiles(nwords))), dim3(256), 0, st, bitmap, nwords,
                       counts);
    return hipGetLastError();
}

hipError_t launch_bitmap_keys(const uint32_t* bitmap, int64_t nwords, const int64_t* pos, uint64_t* out,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_bitmap_keys, dim3(static_cast<unsigned>(bitmap_tiles(nwords))), dim3(256), 0, st, bitmap, nwords,
                       pos, out);
    return hipGetLastError();
}

hipError_t launch_unique_flags(int W, const uint64_t* sorted, int64_t n, int32_t* flags, hipStream_t st) {
    if (W == 2)
        hipLaunchKernelGGL(k_first_of_run<2>, dim3(blocks256(n)), dim3(256), 0, st, sorted, n, flags);
    else
        hipLaunchKernelGGL(k_first_of_run<1>, dim3(blocks256(n)), dim3(256), 0, st, sorted, n, flags);
    return hipGetLastError();
}

hipError_t launch_unique_scatter(int W, const uint64_t* sorted, int64_t n, const int32_t* flags, const int64_t* pos,
                                 uint64_t* out, hipStream_t st) {
    if (W == 2)
        hipLaunchKernelGGL(k_scatter_unique<2>, dim3(blocks256(n)), dim3(256), 0, st, sorted, n, flags, pos, out);
    else
        hipLaunchKernelGGL(k_scatter_unique<1>, dim3(blocks256(n)), dim3(256), 0, st, sorted, n, flags, pos, out);
    return hipGetLastError();
}

}  // namespace eloc
