// The conventional local energy's row sums: U's rows over a larger set X = U
// and the coupled states outside it.
//
// There most XY masks that keep a row's particle numbers lead to a state of X,
// so the work is per pair and not per candidate.  Lanes are 64 rows of U and
// the wave walks the groups, four a step: a group's mask and terms are the same
// for all lanes (scalar loads), a lane's sum stays in its registers, and only
// the table slot and the amplitude of x ^ XY are gathered.  The loop with lanes
// over groups gathers every term of every pair too, and is bound by the
// addresses of the vector memory unit (9.4e8 lines at 28 qubits, 20 000 rows,
// 3.8e6 states; here 1.4e8).  There it took 2446 us, this 994 us: 0.71 vector
// instructions per busy CU clock, 1.05e8 reads that hit L2 and 4e7 that miss.
// Of that, reading the stash only where a lookup is open was 2260 -> 990 us.
#include "full.h"

#include "device.h"

#include <algorithm>

namespace eloc {

namespace {

constexpr int kWave = 64;
constexpr int kStep = 4;                       // groups of a step
constexpr uint64_t kEvenBits = 0x5555555555555555ull;

struct FullArgs {
    const GroupRec<1>* groups;
    const uint64_t* ghash;
    const void* terms;
    int n_groups;
    const uint64_t* keys;
    const uint64_t* hash;
    Table table;
    const SampleParams* sp;
    int64_t rows;
    int64_t tiles;              // tiles of 64 rows (by partitions: at least those of all classes)
    int chunks;                 // chunks of the groups; by partitions: of a bucket
    int part_bits;              // 0: not by partitions
    int part_salt;
    const int32_t* row_perm;    // rows by class, and the classes' first positions
    const int64_t* class_off;
    const int32_t* gbucket;
};

// A run's terms are the same for all lanes: whole fours first, so that their
// records are one wide scalar load, then the rest one by one.  The order of
// the additions is the records'.
template <bool NW>
__device__ __forceinline__ double run_all(const TermRec<1>* __restrict__ terms, int b, int e, const uint64_t* ket) {
    double h = 0.0;
    int t = b;
    for (; t + 4 <= e; t += 4) {
        TermRec<1> tr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) tr[u] = terms[t + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) h += term_f64<1, NW>(tr[u], ket);
    }
    for (; t < e; ++t) h += term_f64<1, NW>(terms[t], ket);
    return h;
}
template <bool NW>
__device__ __forceinline__ F2 run_all(const TermRecF<1>* __restrict__ terms, int b, int e, const uint64_t* ket) {
    F2 h{0.f, 0.f};
    float vh, vl;
    int t = b;
    for (; t + 4 <= e; t += 4) {
        TermRecF<1> tr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) tr[u] = terms[t + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            term_f32<1, NW>(tr[u], ket, vh, vl);
            acc_add(h, vh, vl);
        }
    }
    for (; t < e; ++t) {
        term_f32<1, NW>(terms[t], ket, vh, vl);
        acc_add(h, vh, vl);
    }
    return h;
}

// One wave: 64 rows, a chunk of the groups.
template <int PREC, bool NW>
__global__ __launch_bounds__(kWave) void k_full_rows(FullArgs A, const typename Prec<PREC>::Vec* __restrict__ vec,
                                                     void* __restrict__ partial) {
    using P = Prec<PREC>;
    constexpr int TK = table_kind(1, NW);
    using HT = typename TabT<TK>::hash;
    const int lane = lane_id();
    int64_t row;
    bool on;
    int g0, g1, chunk, stride = 1;
    if (A.part_bits) {
        // workgroup w is on XCD w % 8, which takes the partitions w % 8 + 8 p
        // one after another; then (tile, chunk of the bucket).  The tile's
        // class c gives the bucket c ^ k ^ part(salt), whose candidates are
        // all in partition k
        const int nparts = 1 << A.part_bits;
        const int64_t rest = blockIdx.x / kXcds, per_pass = A.tiles * A.chunks;
        const int k = static_cast<int>(blockIdx.x % kXcds) + kXcds * static_cast<int>(rest / per_pass);
        const int sub = static_cast<int>(rest % per_pass % A.chunks);
        const int t = static_cast<int>(rest % per_pass / A.chunks);
        // lane q: class q and the tiles up to its end
        const int64_t q0 = A.class_off[min(lane, nparts)], q1 = A.class_off[min(lane + 1, nparts)];
        const int mine = static_cast<int>((q1 - q0 + kWave - 1) / kWave);
        int upto = mine;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int o = __shfl_up(upto, d, kWave);
            if (lane >= d) upto += o;
        }
        const int c = __popcll(__ballot(lane < nparts && upto <= t));
        if (k >= nparts || c >= nparts) return;   // past the classes' tiles
        const int first = __builtin_amdgcn_readlane(upto - mine, c);
        const int64_t p = A.class_off[c] + static_cast<int64_t>(t - first) * kWave + lane, end = A.class_off[c + 1];
        on = p < end;
        row = A.row_perm[min(p, end - 1)];
        const int r = rev_bits(c ^ k ^ A.part_salt, A.part_bits);
        const int bs = A.gbucket[r << (kMaxPartBits - A.part_bits)];
        const int be = A.gbucket[(r + 1) << (kMaxPartBits - A.part_bits)];
        const int per = (be - bs + A.chunks - 1) / A.chunks;
        g0 = __builtin_amdgcn_readfirstlane(min(be, bs + sub * per));
        g1 = __builtin_amdgcn_readfirstlane(min(be, bs + sub * per + per));
        chunk = k * A.chunks + sub;
    } else {
        chunk = static_cast<int>(blockIdx.x / A.tiles);
        const int64_t p = (blockIdx.x % A.tiles) * kWave + lane;
        on = p < A.rows;
        row = min(p, A.rows - 1);
        // every chunks-th group: the long runs come one after another
        g0 = chunk;
        g1 = A.n_groups;
        stride = A.chunks;
    }
    const Table& T = A.table;
    const SlotReader<TK> slots(T);
    const int nstash = __builtin_amdgcn_readfirstlane(static_cast<int>(T.stash->count));
    const bool any = __builtin_amdgcn_readfirstlane(A.sp->sig_all) != 0;
    const uint32_t sig_pa = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(A.sp->sig_pa)),
                   sig_n = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(A.sp->sig_n)),
                   rad_max = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(A.sp->rad_max));
    const uint64_t ref = A.sp->rad_ref[0];
    const auto* __restrict__ terms = static_cast<const typename P::template Term<1>*>(A.terms);
    const uint64_t x = A.keys[row];
    const uint64_t hx = A.hash[row] ^ T.salt;
    typename P::Acc acc{};
    for (int g = g0; g < g1; g += kStep * stride) {
        GroupRec<1> gr[kStep];
        uint64_t xp[kStep];
        HT hs[kStep];
        typename TabT<TK>::slot v1[kStep], v2[kStep];
        int j[kStep];
        typename P::Vec v[kStep];
        bool ok[kStep];
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            const int gg = min(g + u * stride, g1 - 1);
            gr[u] = A.groups[gg];
            hs[u] = static_cast<HT>(hx ^ A.ghash[gg]);
        }
        // X's signature, where it has a single one, else its radius
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            xp[u] = x ^ gr[u].xy[0];
            bool pass;
            if (any) {
                const uint32_t d = NW ? __popc(static_cast<uint32_t>(xp[u]) ^ static_cast<uint32_t>(ref))
                                      : popc64(xp[u] ^ ref);
                pass = d <= rad_max;
            } else {
                uint32_t pa, pn;
                if constexpr (NW) {
                    pa = __popc(static_cast<uint32_t>(xp[u]) & static_cast<uint32_t>(kEvenBits));
                    pn = __popc(static_cast<uint32_t>(xp[u]));
                } else {
                    pa = popc64(xp[u] & kEvenBits);
                    pn = popc64(xp[u]);
                }
                pass = pa == sig_pa && pn == sig_n;
            }
            ok[u] = on && g + u * stride < g1 && pass;
            v1[u] = slots.load(slot1(T, hs[u]), ok[u]);
        }
#pragma unroll
        for (int u = 0; u < kStep; ++u) v2[u] = slots.load(slot2(T, hs[u]), need_slot2<TK>(T, v1[u], hs[u]));
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            j[u] = wave_settle<TK>(T, v1[u], v2[u], hs[u], nstash);
            v[u] = typename P::Vec{};
            if (j[u] >= 0) v[u] = vec[j[u]];
        }
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            if (__ballot(j[u] >= 0) == 0) continue;
            const auto hr = run_all<NW>(terms, gr[u].begin, gr[u].mid, &xp[u]);
            const auto hi = run_all<NW>(terms, gr[u].mid, gr[u].end, &xp[u]);
            if (j[u] >= 0) P::madd(acc, hr, hi, v[u]);
        }
    }
    if (on) store_acc(partial, static_cast<int64_t>(chunk) * A.rows + row, acc);
}

// X by partition class.  28 qubits, 20 000 rows, 3.8e6 states: a call 2940 us
// without, 2745 with it (L2 misses of the sums 6.8e7 -> 4.1e7; the order itself
// about 0.2 ms).
__global__ __launch_bounds__(256) void k_full_order(int64_t n, const int32_t* __restrict__ perm,
                                                    const uint64_t* __restrict__ keys,
                                                    const uint64_t* __restrict__ hash, uint64_t* __restrict__ keys_to,
                                                    uint64_t* __restrict__ hash_to) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t p = perm[i];
    keys_to[i] = keys[p];
    hash_to[i] = hash[p];
}

__global__ __launch_bounds__(256) void k_full_vec(int64_t n, const int32_t* __restrict__ perm,
                                                  const double2* __restrict__ from, double2* __restrict__ to) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) to[i] = from[perm[i]];
}

}  // namespace

hipError_t launch_full_order(int64_t n, const int32_t* perm, const uint64_t* keys, const uint64_t* hash,
                             uint64_t* keys_to, uint64_t* hash_to, hipStream_t st) {
    hipLaunchKernelGGL(k_full_order, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, n, perm, keys, hash,
                       keys_to, hash_to);
    return hipGetLastError();
}

hipError_t launch_full_vec(int64_t n, const int32_t* perm, const double2* from, double2* to, hipStream_t st) {
    hipLaunchKernelGGL(k_full_vec, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, n, perm, from, to);
    return hipGetLastError();
}

// By partitions only with enough rows for whole tiles in every class (two, of
// 64).  About 16 384 waves, at least eight chunks, so that no lane's sum is one
// long chain, and at most 128, whose sum is one thread's.  In order the long
// runs of the single excitations are one chunk's: 30 qubits, 2000 rows, a call
// 2000 us; dealt out 1490, the loop over groups 1530.
Plan full_plan(const HamDev& H, int64_t rows, int part_bits) {
    Plan P;
    const int64_t nparts = int64_t(1) << part_bits;
    P.rows_per_block = kWave;
    const int64_t tiles = (rows + kWave - 1) / kWave;
    P.part = part_bits > 0 && rows >= 128 * nparts;
    if (P.part) {
        P.part_sub = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(4, 16384 / (tiles * nparts))));
        P.chunks = static_cast<int>(nparts) * P.part_sub;
        return P;
    }
    const int64_t steps = (H.n_groups + kStep - 1) / kStep;
    const int64_t chunks = std::min({steps, int64_t(128), std::max<int64_t>(8, (16384 + tiles - 1) / tiles)});
    P.chunks = static_cast<int>(chunks);
    return P;
}

hipError_t launch_full_rows(int precision, const HamDev& H, const SampleDev& S, const Plan& P, const double2* vec,
                            const float4* vecf, void* partial, hipStream_t st) {
    FullArgs A{};
    A.groups = static_cast<const GroupRec<1>*>(P.part ? H.part.groups : H.groups);
    A.ghash = P.part ? H.part.ghash : H.group_hash;
    A.terms = precision == 0 ? H.terms : H.terms_f;
    A.n_groups = static_cast<int>(H.n_groups);
    A.keys = S.keys;
    A.hash = S.hash;
    A.table = S.table;
    A.sp = S.params;
    A.rows = S.rows > 0 ? S.rows : S.n;
    A.tiles = (A.rows + kWave - 1) / kWave;
    A.chunks = P.part ? P.part_sub : P.chunks;
    int64_t blocks = A.tiles * P.chunks;
    if (P.part) {
        const int64_t nparts = int64_t(1) << S.part.bits;
        A.part_bits = S.part.bits;
        A.part_salt = hash_part(S.table.salt, H.part.shift, A.part_bits);
        A.row_perm = S.part.row_perm;
        A.class_off = S.part.class_off;
        A.gbucket = H.part.bucket_dev;
        A.tiles += nparts;
        blocks = A.tiles * A.chunks * nparts;
    }
    const dim3 grid(static_cast<unsigned>(blocks)), block(kWave);
    if (precision == 0) {
        if (H.narrow)
            hipLaunchKernelGGL((k_full_rows<0, true>), grid, block, 0, st, A, vec, partial);
        else
            hipLaunchKernelGGL((k_full_rows<0, false>), grid, block, 0, st, A, vec, partial);
    } else if (H.narrow) {
        hipLaunchKernelGGL((k_full_rows<1, true>), grid, block, 0, st, A, vecf, partial);
    } else {
        hipLaunchKernelGGL((k_full_rows<1, false>), grid, block, 0, st, A, vecf, partial);
    }
    return hipGetLastError();
}

}  // namespace eloc
