// Pair kernels by spin strings, for Hamiltonians whose XY masks factor into
// few spin-up and spin-down parts (electronic structure: a mask flips none,
// two or four orbitals of a spin).
//
// With (a, b) the spin-up and spin-down parts of x ^ x':
//   (0, b) and (a, 0): x' has one of x's two strings.  The samples are sorted
//     by spin-up string and again by spin-down string, and a wave scans
//     for up to 16 rows of one string its own bucket (the range of that string):
//     a column passes by popcount, and a table lookup of its part decides.
//   (a, b): the spin-up string of x' is that of x ^ a, whose bucket one
//     lookup finds.  Light buckets (few samples) are scanned like the own one.
//     A column of a heavy spin-up bucket is found from its spin-down bucket
//     instead, if that is light, and else in a table over (heavy spin-up
//     string, heavy spin-down string), where a row has few candidates.  Every
//     pair is met exactly once.
//
// Scanning costs a XOR, a popcount, a compare and a carry add per row and 64
// columns, in 32 bits for one-word keys, and nearly every column that passes
// is a pair; LoopOverTerms spends 14 instructions per row and 64 XY masks.
#include "device.h"

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eloc {

namespace {

constexpr int kWave = 64;
constexpr int kAccCols = 16;    // accumulator columns per row
constexpr int kSmall = 8;       // buckets up to this size are gathered before they are scanned
constexpr int kQueue = 2 * kWave;

struct JoinArgs {
    const void* terms;
    JoinHamDev H;
    JoinDev U;
    int chunks;      // 0: spin-down order; 1: heavy-heavy table; the rest: alist
    int per_chunk;   // masks of alist per chunk
    int64_t tiles;
    uint32_t own_up, own_down;   // longest own bucket scanned, by order (sums)
};

__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
}
__device__ __forceinline__ uint32_t pop(uint32_t v) { return static_cast<uint32_t>(__popc(v)); }
__device__ __forceinline__ uint32_t pop(uint64_t v) { return static_cast<uint32_t>(__popcll(v)); }
__device__ __forceinline__ uint32_t rdlane(uint32_t v, int l) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ uint64_t rdlane(uint64_t v, int l) {
    return (static_cast<uint64_t>(rdlane(static_cast<uint32_t>(v >> 32), l)) << 32) |
           rdlane(static_cast<uint32_t>(v), l);
}

// Element at a 32-bit byte offset (base in scalar registers).
template <class T>
__device__ __forceinline__ T ld(const void* base, uint32_t off) {
    return *reinterpret_cast<const T*>(static_cast<const char*>(base) + off);
}
// 2 v + the lane's bit of m.
__device__ __forceinline__ uint32_t shift_in(uint32_t v, uint64_t m) {
    uint32_t o;
    uint64_t carry;
    asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(o), "=&s"(carry) : "v"(v), "s"(m));
    return o;
}

// p += v in LDS.
__device__ __forceinline__ void lds_add(double* p, double v) {
    typedef __attribute__((address_space(3))) double* lds_ptr;
    (void)__builtin_amdgcn_ds_atomic_fadd_f64((lds_ptr)p, v);
}

// Bucket of string k (start, len; len 0 where no sample has it).  The table
// is at most half full, so every probe sequence ends at an empty slot.
template <class ST>
__device__ __forceinline__ uint2 find_bucket(const JoinBucket* __restrict__ slots, int bits, ST k) {
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t s = join_hash(k, bits);
    for (uint32_t t = 0; t <= mask; ++t, s = (s + 1) & mask) {
        const uint4 v = reinterpret_cast<const uint4*>(slots)[s];
        if (v.w == 0u) break;
        if ((static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32)) == static_cast<uint64_t>(k))
            return make_uint2(v.z, v.w);
    }
    return make_uint2(0u, 0u);
}

template <int W>
__device__ __forceinline__ uint32_t find_part(const JoinSlot<W>* __restrict__ slots, int bits, JoinStr<W> k) {
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t s = join_hash(k, bits);
    for (uint32_t t = 0; t <= mask; ++t, s = (s + 1) & mask) {
        const JoinSlot<W> v = slots[s];
        if (static_cast<uint32_t>(v.id) == kJoinNone) break;
        if (v.key == k) return static_cast<uint32_t>(v.id);
    }
    return kJoinNone;
}

// kModeSumPairs: the sums, and the number of pairs (1.2% of 52 qubits, 2^20
// samples, so only where a caller wants it)
enum { kModeSum = 0, kModeCount = 1, kModeFill = 2, kModeSumPairs = 3 };

struct JoinOut {
    void* partial;             // kModeSum
    unsigned long long* pairs; // kModeSumPairs: += the pairs, over kJoinPairSlots words
    int32_t* counts;           // kModeCount
    const int64_t* offsets;    // kModeFill
    uint64_t* pkey;
    uint32_t* pval;
    int jbits;
};

template <int W, int PREC, bool ADJ, bool NW, int MODE, int kRows>
__global__ __launch_bounds__(kWave) void k_join(JoinArgs A, JoinOut O) {
    using ST = JoinStr<W>;
    using P = Prec<PREC>;
    using Acc = typename P::Acc;
    using Vec = typename P::Vec;
    using Term = typename P::template Term<W>;
    // a heavy spin-down string next to a row: its table column | row << 24, the string
    struct Near {
        uint32_t at;
        ST s;
    };
    constexpr bool kSums = MODE == kModeSum || MODE == kModeSumPairs;
    constexpr int kList = kWave * kSmall;                                   // gathered columns
    constexpr int kNear = kList * 4 / static_cast<int>(sizeof(Near));
    // queued columns: position | row << 24, place base, the two strings
    __shared__ uint2 q[kQueue];
    __shared__ ST qs[kQueue][2];
    __shared__ uint2 lq[kSums ? kQueue : 1];   // pairs of linear places: position | row << 24, place
    __shared__ uint64_t buf[kList / 2];             // list, or near
    __shared__ ST rowstr[kRows][2];   // the rows' scanned string, their order's string
    __shared__ double2 acc_raw[kSums ? kRows * kAccCols : 1];
    static_assert(sizeof(Acc) == sizeof(double2), "accumulators are 16 bytes");
    uint32_t* list = reinterpret_cast<uint32_t*>(buf);   // position | mask lane << 24
    Near* near = reinterpret_cast<Near*>(buf);
    Acc* acc = reinterpret_cast<Acc*>(acc_raw);
    const int lane = lane_id();
    const int chunk = static_cast<int>(blockIdx.x / static_cast<uint64_t>(A.tiles));
    const int64_t tile = static_cast<int64_t>(blockIdx.x) - chunk * A.tiles;
    const int64_t M = A.U.M;
    const int64_t row0 = tile * kRows;
    const int n = static_cast<int>(min(static_cast<int64_t>(kRows), M - row0));
    const bool down = chunk == 0, core = chunk == 1;
    const int64_t at = down ? M : 0;                // the order's first position
    const int32_t* __restrict__ perm = A.U.perm + at;
    const ST* __restrict__ scan = static_cast<const ST*>(A.U.scan) + at;
    const double2* __restrict__ vec = A.U.vec + at;
    const JoinBucket* __restrict__ slots = A.U.slots + (down ? (int64_t(1) << A.U.bits) : 0);
    const Term* __restrict__ terms = static_cast<const Term*>(A.terms);
    const bool bad = __builtin_amdgcn_readfirstlane(static_cast<int>(*A.U.prep_err)) != 0;
    const uint32_t heavy_min = rdlane(A.U.heavy->min, 0);
    const uint32_t core_row = rdlane(A.U.heavy->n[1], 0);
    const int heavy_bits0 = static_cast<int>(rdlane(A.U.heavy->bits[0], 0)),
              heavy_bits1 = static_cast<int>(rdlane(A.U.heavy->bits[1], 0));
    const int64_t rpos = row0 + min(lane, n - 1);
    const int32_t row = perm[rpos];
    int cnt[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) cnt[r] = 0;
    int64_t fill_at = 0;
    if constexpr (MODE == kModeFill) fill_at = O.offsets[static_cast<int64_t>(row) * A.chunks + chunk];
    const bool huge = !kSums && rdlane(A.U.heavy->huge, 0) != 0u;   // not listed here
    if (bad || huge || (core && heavy_min == kJoinNone)) {   // invalid samples: no pairs
        if constexpr (MODE == kModeCount)
            if (lane < n) O.counts[static_cast<int64_t>(row) * A.chunks + chunk] = huge && !bad ? -1 : 0;
        if constexpr (kSums)
            if (lane < n) store_acc(O.partial, static_cast<int64_t>(chunk) * M + row, Acc{});
        return;
    }
    const ST gl = (static_cast<const ST*>(A.U.group) + at)[rpos];
    const ST sl = scan[rpos];
    if (lane < kRows) {
        rowstr[lane][0] = sl;
        rowstr[lane][1] = gl;
    }
    if constexpr (kSums)
        for (int i = lane; i < kRows * kAccCols; i += kWave) acc[i] = Acc{};
    ST srow[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        srow[r] = rdlane(sl, r);
        // kept in vector registers: the scalar ones are all taken, and a
        // spilled one would cost a lane read per row and step
        asm("" : "+v"(srow[r]));
    }
    wave_sync();

    // v into row r's column lane % kAccCols.  The lanes that share a column
    // add one after another (FP64: LDS adds, which a wave issues in order)
    auto add = [&](int r, const Acc& v, bool on) __attribute__((always_inline)) {
        Acc* a = acc + r * kAccCols + (lane & (kAccCols - 1));
#pragma unroll
        for (int ph = 0; ph < kWave; ph += kAccCols) {
            if (on && (lane & ~(kAccCols - 1)) == ph) {
                if constexpr (PREC == 0) {
                    lds_add(&a->re, v.re);
                    lds_add(&a->im, v.im);
                } else {
                    Acc t = *a;
                    acc_plus(t, v);
                    *a = t;
                }
            }
            wave_sync();
        }
    };
    // acc += h v for a real matrix element
    auto product = [&](Acc& sum, double h, const Vec& v) __attribute__((always_inline)) {
        if constexpr (PREC == 0) {
            sum.re = h * v.x;
            sum.im = h * v.y;
        } else {
            const float hh = static_cast<float>(h);
            P::madd(sum, F2{hh, static_cast<float>(h - static_cast<double>(hh))}, F2{0.f, 0.f}, v);
        }
    };
    int qn = 0;   // queued columns (wave-uniform)
    int ln = 0;   // queued pairs of linear places
    int found = 0;   // pairs (kModeSumPairs)
    // the last m of them: a table entry per nibble of the ket's strings
    auto drain_linear = [&](int m) __attribute__((always_inline)) {
        wave_sync();
        const bool on = lane < m;
        const uint2 e = lq[ln - m + (on ? lane : 0)];
        ln -= m;
        const int r = static_cast<int>(e.x >> 24);
        const uint32_t p = e.x & 0xFFFFFFu;
        const Vec v = ld<Vec>(vec, p * 16u);
        const ST s = rowstr[r][0], t = rowstr[r][1];
        const JoinPlace<W> pl = ld<JoinPlace<W>>(A.H.place, e.y * static_cast<uint32_t>(sizeof(JoinPlace<W>)));
        const ST cs = ld<ST>(scan, p * static_cast<uint32_t>(sizeof(ST)));
        const ST ct = ld<ST>(static_cast<const ST*>(A.U.group) + at, p * static_cast<uint32_t>(sizeof(ST)));
        const ST ks = ADJ ? s : cs, kt = ADJ ? t : ct;
        const uint32_t mp = pop(static_cast<ST>(ks & (s ^ cs))) + pop(static_cast<ST>(kt & (t ^ ct)));
        const ST ka = down ? ks : kt, kb = down ? kt : ks;
        const uint32_t zp = pop(static_cast<ST>(ka & pl.za)) + pop(static_cast<ST>(kb & pl.zb));
        const uint32_t half = static_cast<uint32_t>(A.H.nibbles) * 128u;
        uint32_t cell = (pl.lo * 2u + (mp & 1u)) * half * 2u;
        double h = 0.0;
        for (int b = 0; b < A.H.nibbles; ++b, cell += 128u) {
            h += ld<double>(A.H.linear, cell + (static_cast<uint32_t>(ka >> (4 * b)) & 15u) * 8u);
            h += ld<double>(A.H.linear, cell + half + (static_cast<uint32_t>(kb >> (4 * b)) & 15u) * 8u);
        }
        h = (zp & 1u) ? -h : h;
        Acc sum{};
        if (on) product(sum, h, v);
        add(r, sum, on);
    };
    // Queued columns are drained in two halves, so that a batch's loads are
    // in flight while the next one is found: `issue` takes the last m columns
    // off the queue and requests what their places hold, `consume` does with
    // them what the mode asks for.
    struct Batch {
        uint32_t at;       // position | row << 24
        uint32_t place;    // kJoinNone: not a pair
        ST ka, kb;         // the ket's strings
        bool by_idx;       // T from `sign`
        JoinPlace<W> pl;
        Vec v;
        uint64_t t;
    } pend;
    bool pending = false;
    auto issue = [&](int m) __attribute__((always_inline)) {
        wave_sync();
        const bool on = lane < m;
        const int qi = qn - m + (on ? lane : 0);
        const uint2 e = q[qi];
        const ST cs = qs[qi][0], ct = qs[qi][1];
        qn -= m;
        const int r = static_cast<int>(e.x >> 24);
        const bool own = (e.y & kJoinFull) != 0u;   // a one-spin mask
        const ST rs = rowstr[r][0], rt = rowstr[r][1];
        const ST d = cs ^ rs;
        // the place: by position, or by lookup
        uint32_t id = kJoinNone, stride = 1u;
        if (A.H.direct) {
            const uint32_t c = pop(d);
            if (on && !own && c == 2u) id = join_pair_id(d);
            if (__ballot(on && own)) {
                if (on && own && !(c & 1u)) id = join_even_id(d, static_cast<uint32_t>(A.H.string_bits));
            }
            if (down && !own) stride = A.H.stride;
        } else if (on) {
            const JoinSlot<W>* tab = static_cast<const JoinSlot<W>*>(A.H.b_cross);
            int bits = A.H.b_cross_bits;
            if (own) {
                tab = static_cast<const JoinSlot<W>*>(down ? A.H.a_own : A.H.b_own);
                bits = down ? A.H.a_own_bits : A.H.b_own_bits;
            }
            id = find_part<W>(tab, bits, d);
        }
        const uint32_t place = id == kJoinNone ? 0u : (e.y & ~kJoinFull) + id * stride;
        pend.at = e.x;
        pend.place = id == kJoinNone ? kJoinNone : place;
        pend.pl = ld<JoinPlace<W>>(A.H.place, place * static_cast<uint32_t>(sizeof(JoinPlace<W>)));
        if constexpr (kSums) {
            pend.v = ld<Vec>(vec, (e.x & 0xFFFFFFu) * 16u);
            const ST ks = ADJ ? rs : cs, kt = ADJ ? rt : ct;
            pend.ka = down ? ks : kt;
            pend.kb = down ? kt : ks;
            // T: with the place where both parities are odd, else by idx
            const uint32_t ps = pop(static_cast<ST>(ks & d)) & 1u, pt = pop(static_cast<ST>(kt & (ct ^ rt))) & 1u;
            uint32_t idx = down ? ps | (pt << 1) : pt | (ps << 1);
            pend.by_idx = own || idx != kJoinMain;
            if (__ballot(pend.by_idx)) {
                ST p1, p3;
                join_parity_masks(d, p1, p3);
                const uint32_t i2 = (pop(static_cast<ST>(ks & p1)) & 1u) | (ps << 1) |
                                    ((pop(static_cast<ST>(ks & p3)) & 1u) << 2);
                idx = own ? i2 : idx;
                if (pend.by_idx) pend.t = ld<uint64_t>(A.H.sign, (idx * A.H.places + place) * 8u);
            }
        }
        pending = true;
    };
    auto consume = [&]() __attribute__((always_inline)) {
        pending = false;
        const int r = static_cast<int>(pend.at >> 24);
        const uint32_t p = pend.at & 0xFFFFFFu;
        const uint32_t place = pend.place;
        const bool tag = (pend.pl.hi & kJoinTag) == kJoinTag;
        const uint32_t kind = place == kJoinNone ? static_cast<uint32_t>(kJoinEmpty)
                              : tag              ? pend.pl.hi & 7u
                                                 : static_cast<uint32_t>(kJoinSign);
        if constexpr (MODE == kModeCount) {
            const bool hit = kind != kJoinEmpty;
#pragma unroll
            for (int k = 0; k < kRows; ++k) cnt[k] += __popcll(__ballot(hit && r == k));
        } else if constexpr (MODE == kModeFill) {
            const bool hit = kind != kJoinEmpty;
            for (int k = 0; k < n; ++k) {
                const uint64_t mk = __ballot(hit && r == k);
                const int64_t base = static_cast<int64_t>(rdlane(static_cast<uint64_t>(fill_at), k));
                if (hit && r == k) {
                    const int64_t o = base + lanes_below(mk);
                    O.pkey[o] = (static_cast<uint64_t>(static_cast<uint32_t>(perm[row0 + k])) << O.jbits) |
                                static_cast<uint64_t>(static_cast<uint32_t>(perm[p]));
                    O.pval[o] = static_cast<uint32_t>(A.H.gids[place]);
                }
                if (lane == k) fill_at += __popcll(mk);
            }
        } else {
            const Vec v = pend.v;
            const uint32_t zp = pop(static_cast<ST>(pend.ka & pend.pl.za)) + pop(static_cast<ST>(pend.kb & pend.pl.zb));
            const uint64_t hb =
                pend.by_idx ? pend.t : (static_cast<uint64_t>(pend.pl.hi) << 32) | pend.pl.lo;
            double h;
            __builtin_memcpy(&h, &hb, sizeof(h));
            h = (zp & 1u) ? -h : h;
            const bool sign = kind == kJoinSign;
            if constexpr (MODE == kModeSumPairs) found += __popcll(__ballot(kind != kJoinEmpty));
            Acc sum{};
            if (sign) product(sum, h, v);
            add(r, sum, sign);
            // linear places wait for a whole wave of them
            const bool lin = kind == kJoinLinear;
            const uint64_t mlin = __ballot(lin);
            if (mlin) {
                if (lin) lq[ln + lanes_below(mlin)] = make_uint2(pend.at, place);
                ln += __popcll(mlin);
                if (ln >= kWave) drain_linear(kWave);
            }
            // other runs one at a time, the terms over the lanes
            uint64_t ml = __ballot(kind == kJoinRunKind);
            while (ml) {
                const int l = __ffsll(static_cast<unsigned long long>(ml)) - 1;
                ml &= ml - 1;
                const int rr = static_cast<int>(rdlane(static_cast<uint32_t>(r), l));
                const JoinRun jr = A.H.runs[rdlane(place, l)];
                const int tb = static_cast<int>(jr.begin), tm = tb + static_cast<int>(jr.lens & 0xFFFFu),
                          te = tm + static_cast<int>(jr.lens >> 16);
                const int64_t x = ADJ ? __shfl(row, rr, kWave) : perm[rdlane(p, l)];
                uint64_t k1[W];
#pragma unroll
                for (int w = 0; w < W; ++w) k1[w] = A.U.keys[x * W + w];
                typename P::H hr, hi;
                melem<W, NW>(terms, tb, tm, te, lane, kWave, k1, hr, hi);
                Acc one{};
                P::madd(one, hr, hi, lane_shfl(v, l));
                add(rr, one, true);
            }
        }
    };
    // a batch through both halves, one behind the other
    auto drain = [&](int m) __attribute__((always_inline)) {
        if (pending) consume();
        issue(m);
    };
    // column p (strings s, t) with row r, where `hit`: into the queue
    auto push = [&](uint64_t mk, bool hit, uint32_t p, uint32_t r, uint32_t base, ST s, ST t)
                    __attribute__((always_inline)) {
        if (hit) {
            const int i = qn + lanes_below(mk);
            q[i] = make_uint2(p | (r << 24), base);
            qs[i][0] = s;
            qs[i][1] = t;
        }
        qn += __popcll(mk);
    };

    // the masks of this work item: own bucket first in the spin-down order
    const int ka = down ? -1 : core ? 0 : (chunk - 2) * A.per_chunk;
    const int kb = down ? (heavy_min == kJoinNone ? 0 : A.H.n_b) : core ? A.H.n_a : min(A.H.n_a, (chunk - 1) * A.per_chunk);
    const uint32_t own_pen = down ? 0u - A.H.a_pmin : 0u;
    uint32_t rem = (1u << n) - 1u;
    while (rem) {   // the tile's distinct strings, in order
        const ST g = rdlane(gl, __ffs(rem) - 1);
        const uint32_t piece = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(gl == g)) & rem;
        rem &= ~piece;
        const uint32_t rlast = 31u - static_cast<uint32_t>(__builtin_clz(piece));   // rows of a string are neighbours
        int next_row = __ffs(piece) - 1, next_part = 0;   // core: first (row, part) not yet looked up
        do {
            int nn = 0;   // strings in `near`
            if (core) {
                while (next_row <= static_cast<int>(rlast) && nn <= kNear - kWave) {
                    const int j = next_part + lane;
                    const bool on = j < A.H.n_b;
                    const ST s = static_cast<const ST*>(A.H.blist)[on ? j : 0] ^ rdlane(sl, next_row);
                    const uint32_t id = find_part<W>(static_cast<const JoinSlot<W>*>(A.U.heavy_slots) + kJoinHeavySlots,
                                                     heavy_bits1, s);
                    const bool hit = on && id != kJoinNone;
                    const uint64_t mk = __ballot(hit);
                    if (hit) near[nn + lanes_below(mk)] = Near{id | (static_cast<uint32_t>(next_row) << 24), s};
                    nn += __popcll(mk);
                    next_part += kWave;
                    if (next_part >= A.H.n_b) {
                        next_part = 0;
                        ++next_row;
                    }
                }
                wave_sync();
                if (nn == 0) continue;
            }
            for (int k0 = ka; k0 < kb; k0 += kWave) {
                // lane: one mask and its bucket
                const int k = min(k0 + lane, kb - 1);
                JoinMask mask{A.H.a_base | kJoinFull, A.H.a_span};
                ST t = g;
                if (down && k >= 0) {
                    mask = A.H.bmask[k];
                    t ^= static_cast<const ST*>(A.H.blist)[k];
                } else if (!down) {
                    mask = A.H.amask[k];
                    t ^= static_cast<const ST*>(A.H.alist)[k];
                }
                const bool own = (mask.base & kJoinFull) != 0u;
                const bool own0 = rdlane(mask.base, 0) & kJoinFull;   // only lane 0 can have the own bucket
                const bool on = k0 + lane < kb && !(down && own && !A.H.has_a_own);
                uint2 b = make_uint2(0u, 0u);
                uint32_t total = 0;
                if (core) {
                    const uint32_t id = on && !own ? find_part<W>(static_cast<const JoinSlot<W>*>(A.U.heavy_slots),
                                                                  heavy_bits0, t)
                                                   : kJoinNone;
                    if (id != kJoinNone) b = make_uint2(id * core_row, 1u);
                } else {
                    // heavy buckets are left to the spin-down order and the
                    // table, own ones past the limit to k_join_own
                    if (on) b = find_bucket<ST>(slots, A.U.bits, t);
                    if (own ? kSums && b.y > (down ? A.own_down : A.own_up) : b.y >= heavy_min) b.y = 0u;
                }
                if (!core) {
                    // the small buckets' columns are gathered side by side
                    const uint32_t mine = !own && b.y <= kSmall ? b.y : 0u;
                    uint32_t before = mine;
#pragma unroll
                    for (int d = 1; d < kWave; d <<= 1) {
                        const uint32_t o = __shfl_up(before, d, kWave);
                        if (lane >= d) before += o;
                    }
                    total = rdlane(before, kWave - 1);
                    before -= mine;
                    for (uint32_t c = 0; __ballot(c < mine); ++c)
                        if (c < mine) list[before + c] = (b.x + c) | (static_cast<uint32_t>(lane) << 24);
                    wave_sync();
                }
                // the other buckets one by one, then the gathered columns: one
                // column per lane against the rows of the piece; for the table,
                // one near string per lane.  A step's columns are requested a
                // step ahead, across buckets
                uint64_t big = __ballot(b.y > (own || core ? 0u : static_cast<uint32_t>(kSmall)));
                bool gathered = total > 0, more = false, range = false;
                uint32_t st = 0, len = 0, c = 0;   // the next step's source and offset
                int l0 = 0;
                uint32_t pn = 0;                   // what it reads: position and mask lane,
                ST fn = 0, sn = 0;                 // the column's string; table: its cell, the near string
                auto pick = [&]() __attribute__((always_inline)) {
                    range = big != 0;
                    more = range || gathered;
                    c = 0;
                    if (range) {
                        l0 = __ffsll(static_cast<unsigned long long>(big)) - 1;
                        big &= big - 1;
                        st = rdlane(b.x, l0);
                        len = core ? static_cast<uint32_t>(nn) : rdlane(b.y, l0);
                    } else {
                        gathered = false;
                        len = total;
                    }
                };
                auto fetch = [&]() __attribute__((always_inline)) {
                    const uint32_t o = min(c + lane, len - 1);
                    if (core) {
                        const Near e = near[o];
                        pn = e.at;
                        sn = e.s;
                        fn = ld<uint32_t>(A.U.core, (st + (e.at & 0xFFFFFFu)) * 4u);
                    } else {
                        // a light bucket of a spin-down string holds columns with
                        // light spin-up strings, which are met from those
                        const bool crossed = down && !(range && own0 && l0 == 0);
                        pn = range ? st + o : list[o];
                        fn = ld<ST>(crossed ? A.U.cross : static_cast<const void*>(scan),
                                    (pn & 0xFFFFFFu) * static_cast<uint32_t>(sizeof(ST)));
                    }
                };
                pick();
                if (more) fetch();
                while (more) {
                    // this step, before the next one's columns are requested
                    const bool whole = range;
                    const int l = l0;
                    const bool valid = c + lane < len;
                    uint32_t p = pn & 0xFFFFFFu;
                    const uint32_t tag = pn >> 24, cell = static_cast<uint32_t>(fn);
                    const ST s = core ? sn : fn;
                    c += kWave;
                    if (c >= len) pick();
                    if (more) fetch();
                    uint32_t span = rdlane(mask.span, l), base = rdlane(mask.base, l);
                    ST col = rdlane(t, l);
                    uint32_t rows = 0;   // bit i: the column passes against row rlast - i
                    if (core) {
                        if (valid && cell) rows = 1u << (rlast - tag);
                        p = cell - 1u;
                    } else {
                        if (!whole) {
                            span = __shfl(mask.span, static_cast<int>(tag), kWave);
                            base = __shfl(mask.base, static_cast<int>(tag), kWave);
                            col = lane_shfl(t, static_cast<int>(tag));
                        }
                        // 2^16 on idle lanes, else less the smallest popcount:
                        // one for two-spin masks
                        const uint32_t pen = !valid ? 0x10000u : (base & kJoinFull) ? own_pen : ~0u;
                        if (piece == (1u << kRows) - 1u) {
#pragma unroll
                            for (int r = 0; r < kRows; ++r)
                                rows = shift_in(rows, __builtin_amdgcn_ballot_w64(
                                                          pop(static_cast<ST>(s ^ srow[r])) + pen <= span));
                        } else {
                            for (uint32_t rr = piece; rr; rr &= rr - 1u)
                                rows = shift_in(rows, __builtin_amdgcn_ballot_w64(
                                                          pop(static_cast<ST>(s ^ rdlane(sl, __ffs(rr) - 1))) + pen <= span));
                        }
                    }
                    for (uint64_t mk = __ballot(rows != 0u); mk; mk = __ballot(rows != 0u)) {
                        push(mk, rows != 0u, p, rlast - static_cast<uint32_t>(__ffs(rows) - 1), base, s, col);
                        rows &= rows - 1u;
                        if (qn >= kWave) drain(kWave);
                    }
                }
                wave_sync();
            }
        } while (core && next_row <= static_cast<int>(rlast));
    }
    if (qn > 0) drain(qn);
    if (pending) consume();
    if constexpr (kSums)
        if (ln > 0) drain_linear(ln);
    wave_sync();
    if constexpr (MODE == kModeCount) {
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            if (lane == r && r < n) O.counts[static_cast<int64_t>(row) * A.chunks + chunk] = cnt[r];
    }
    if constexpr (kSums) {
        // kPer lanes a row: some columns each, then pairwise
        constexpr int kPer = kWave / kRows;
        const int mine = lane / kPer, sub = lane % kPer;
        Acc t{};
        for (int c = 0; c < kAccCols; c += kPer) acc_plus(t, acc[mine * kAccCols + c + sub]);
#pragma unroll
        for (int m = kPer / 2; m >= 1; m >>= 1) {
            const Acc o = lane_shfl(t, lane ^ m);
            Acc first = (lane & m) ? o : t;
            acc_plus(first, (lane & m) ? t : o);
            t = first;
        }
        const int32_t id = __shfl(row, mine, kWave);
        if (sub == 0 && mine < n) store_acc(O.partial, static_cast<int64_t>(chunk) * M + id, t);
        if (MODE == kModeSumPairs && lane == 0 && found)
            atomicAdd(O.pairs + (blockIdx.x % kJoinPairSlots) * kJoinPairStride, static_cast<unsigned long long>(found));
    }
}

// ---------------------------------------------------------------------------
// Matrix elements of given pairs
// ---------------------------------------------------------------------------
// One pair per lane: its place by position, then a record and a T or the
// nibble tables; the diagonal's term run by the whole wave.  CSR: pairs as
// emitted; else given indices, checked.
template <int W, bool CSR>
__global__ __launch_bounds__(256) void k_join_elements(JoinHamDev H, const TermRec<W>* __restrict__ terms,
                                                       const uint64_t* __restrict__ keys, int64_t M, int64_t n,
                                                       const int32_t* __restrict__ pi, const int32_t* __restrict__ pj,
                                                       const uint64_t* __restrict__ pkey, int jbits,
                                                       double2* __restrict__ out, int32_t* __restrict__ cnt,
                                                       int32_t* __restrict__ grp, uint32_t* __restrict__ err) {
    using ST = JoinStr<W>;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const bool on = t < n;
    int64_t i = 0, j = 0;
    if (on && CSR) {
        i = static_cast<int64_t>(pkey[t] >> jbits);
        j = static_cast<int64_t>(pkey[t] & ((1ull << jbits) - 1ull));
    } else if (on) {
        i = pi[t];
        j = pj[t];
    }
    const bool ok = CSR || (i >= 0 && j >= 0 && i < M && j < M);
    if (!ok) {
        atomicOr(err, static_cast<uint32_t>(kErrIndex));
        i = j = 0;
    }
    uint64_t ket[W];
#pragma unroll
    for (int w = 0; w < W; ++w) ket[w] = keys[j * W + w];
    ST ia, ib, ka, kb;
    spin_strings<W>(keys + i * W, ia, ib);
    spin_strings<W>(ket, ka, kb);
    const ST a = ia ^ ka, b = ib ^ kb;
    const uint32_t ca = pop(a), cb = pop(b), sb = static_cast<uint32_t>(H.string_bits);
    uint32_t place = kJoinNone;
    const bool one = a == 0 || b == 0;
    // keys with bits past the qubits (reported by eloc_check) may get here, and
    // a part with such a bit has no place: its number would lie past the tables
    const bool known = ((a | b) & ~join_string_mask<ST>(sb)) == 0;
    if (known && one && ca + cb <= 4u && !((ca + cb) & 1u))
        place = (a == 0 ? 0u : H.a_base) + join_even_id(static_cast<ST>(a | b), sb);
    if (known && ca == 2u && cb == 2u) place = H.cross + join_pair_id(a) * H.stride + join_pair_id(b);
    if (!on || !ok) place = kJoinNone;
    JoinPlace<W> pl{0, 0, 0, kJoinTag};
    if (place != kJoinNone) pl = static_cast<const JoinPlace<W>*>(H.place)[place];
    const uint32_t kind = (pl.hi & kJoinTag) == kJoinTag ? pl.hi & 7u : static_cast<uint32_t>(kJoinSign);
    const uint32_t pa = pop(static_cast<ST>(ka & a)) & 1u, pb = pop(static_cast<ST>(kb & b)) & 1u;
    const bool flip = (pop(static_cast<ST>(ka & pl.za)) + pop(static_cast<ST>(kb & pl.zb))) & 1u;
    double h = 0.0, hi = 0.0;
    if (kind == kJoinSign) {
        uint32_t idx = pa | (pb << 1);
        if (one) {
            ST p1, p3;
            join_parity_masks(static_cast<ST>(a | b), p1, p3);
            const ST k = a == 0 ? kb : ka;
            idx = (pop(static_cast<ST>(k & p1)) & 1u) | ((pa ^ pb) << 1) | ((pop(static_cast<ST>(k & p3)) & 1u) << 2);
        }
        h = H.sign[static_cast<int64_t>(idx) * H.places + place];
    } else if (kind == kJoinLinear) {
        const double* F = H.linear + (static_cast<int64_t>(pl.lo) * 2 + ((pa ^ pb) & 1u)) * 2 * H.nibbles * 16;
        for (int q = 0; q < H.nibbles; ++q) {
            h += F[q * 16 + (static_cast<uint32_t>(ka >> (4 * q)) & 15u)];
            h += F[(H.nibbles + q) * 16 + (static_cast<uint32_t>(kb >> (4 * q)) & 15u)];
        }
    }
    if (flip) h = -h;
    JoinRun run{0u, 0u};
    if (kind == kJoinRunKind) run = H.runs[place];
    const int rb = static_cast<int>(run.begin), rm = rb + static_cast<int>(run.lens & 0xFFFFu),
              re = rm + static_cast<int>(run.lens >> 16);
    double hr, hm;
    wave_melem<W, false>(terms, rb, rm, re, ket, hr, hm);
    if (kind == kJoinRunKind) {
        h = hr;
        hi = hm;
    }
    if (!on) return;
    out[t] = make_double2(h, hi);
    if constexpr (CSR) cnt[t] = static_cast<int32_t>(j);   // the column
    if (!CSR && cnt) {
        const bool hit = kind != kJoinEmpty;
        const JoinRun r = hit ? H.runs[place] : JoinRun{0u, 0u};
        cnt[t] = static_cast<int32_t>((r.lens & 0xFFFFu) + (r.lens >> 16));
        grp[t] = hit ? H.gids[place] : -1;
    }
}

// ---------------------------------------------------------------------------
// Index of U
// ---------------------------------------------------------------------------
constexpr int kBlock = 256;
constexpr uint32_t kHeavyLeast = 16;   // no string of fewer samples is heavy

// Sort keys of both orders, and the tables cleared.
template <int W>
__global__ __launch_bounds__(kBlock) void k_join_keys(JoinBuild B, int sbits) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t step = static_cast<int64_t>(gridDim.x) * kBlock;
    uint4* slots = reinterpret_cast<uint4*>(B.slots);
    for (int64_t s = t; s < (int64_t(2) << B.bits); s += step) slots[s] = make_uint4(0u, 0u, 0u, 0u);
    uint4* core = reinterpret_cast<uint4*>(B.core);
    if (B.split)
        for (int64_t s = t; s < kJoinCore / 4; s += step) core[s] = make_uint4(0u, 0u, 0u, 0u);
    if (B.filter)
        for (int64_t s = t; s < B.filter_words; s += step) B.filter[s] = 0u;
    JoinSlot<W>* hs = static_cast<JoinSlot<W>*>(B.heavy_slots);
    if (B.split)
        for (int64_t s = t; s < 2 * static_cast<int64_t>(kJoinHeavySlots); s += step) hs[s] = JoinSlot<W>{0, kJoinNone};
    for (int64_t s = t; s < static_cast<int64_t>(sizeof(JoinHeavy) / 4); s += step)
        reinterpret_cast<uint32_t*>(B.heavy)[s] = s == 0 ? kJoinNone : 0u;
    if (t >= B.M) return;
    JoinStr<W> a, b;
    spin_strings<W>(B.keys + t * W, a, b);
    // bits past the string (invalid keys, reported elsewhere) stay out of the order bit
    const uint64_t m = (1ull << sbits) - 1ull;
    B.key[t] = a & m;
    B.key[B.M + t] = (b & m) | (1ull << sbits);
    B.val[t] = static_cast<uint32_t>(t);
    B.val[B.M + t] = static_cast<uint32_t>(t);
}

// Positions of both orders: strings, keys, and for the first position of
// every run of equal strings the bucket, inserted by linear probing (the
// table is at most half full).
template <int W>
__global__ __launch_bounds__(kBlock) void k_join_index(JoinBuild B, int sbits, const uint64_t* __restrict__ key,
                                                       const uint32_t* __restrict__ val) {
    using ST = JoinStr<W>;
    const int64_t M = B.M;
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= 2 * M) return;
    const bool down = p >= M;
    const int64_t o0 = down ? M : 0;
    const uint64_t k = key[p];
    const uint32_t i = val[p];
    const uint64_t* x = B.keys + static_cast<int64_t>(i) * W;
    ST a, b;
    spin_strings<W>(x, a, b);
    B.perm[p] = static_cast<int32_t>(i);
    const ST g = static_cast<ST>(k & ((1ull << sbits) - 1ull));
    static_cast<ST*>(B.group)[p] = g;
    static_cast<ST*>(B.scan)[p] = down ? a : b;
    if (p > o0 && key[p - 1] == k) return;
    // end of the run: doubling steps, then bisection
    int64_t lo = p, step = 1;   // key[lo] == k
    while (lo + step < o0 + M && key[lo + step] == k) {
        lo += step;
        step <<= 1;
    }
    int64_t hi = min(lo + step, o0 + M);   // hi == end or key[hi] != k
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (key[mid] == k)
            lo = mid;
        else
            hi = mid;
    }
    const uint32_t len = static_cast<uint32_t>(hi - p);
    if (len > (down ? B.own_limit[1] : B.own_limit[0])) B.heavy->huge = 1u;
    if (B.split && len >= kHeavyLeast) atomicAdd(&B.heavy->hist[down ? 1 : 0][31 - __clz(static_cast<int>(len))], 1u);
    const uint64_t word = static_cast<uint64_t>(p - o0) | (static_cast<uint64_t>(len) << 32);
    JoinBucket* tab = B.slots + (down ? (int64_t(1) << B.bits) : 0);
    const uint32_t mask = (1u << B.bits) - 1u;
    uint32_t s = join_hash(g, B.bits);
    for (uint32_t t = 0; t <= mask; ++t, s = (s + 1) & mask) {
        auto* w = reinterpret_cast<unsigned long long*>(&tab[s].start);
        if (atomicCAS(w, 0ull, static_cast<unsigned long long>(word)) == 0ull) {
            tab[s].key = g;
            return;
        }
    }
}

// The smallest power of two from which on the heavy-heavy table and the
// tables of the heavy strings have room.
__global__ void k_join_heavy_min(JoinHeavy* __restrict__ h) {
    uint64_t n[2] = {0, 0};
    uint32_t least = kJoinNone;
    for (int c = 25; (1 << c) >= static_cast<int>(kHeavyLeast); --c) {
        n[0] += h->hist[0][c];
        n[1] += h->hist[1][c];
        if (n[0] * n[1] > kJoinCore || 4 * n[0] > kJoinHeavySlots || 4 * n[1] > kJoinHeavySlots) break;
        if (n[0] * n[1] == 0) continue;
        least = 1u << c;
        for (int o = 0; o < 2; ++o) {
            h->n[o] = static_cast<uint32_t>(n[o]);
            uint32_t bits = 2;
            while ((1u << bits) < 4u * h->n[o]) ++bits;
            h->bits[o] = bits;
        }
    }
    h->min = least;
}

// The heavy strings numbered, in their tables (at most a quarter full).
template <int W>
__global__ __launch_bounds__(kBlock) void k_join_heavy_ids(JoinBuild B) {
    using ST = JoinStr<W>;
    using AT = std::conditional_t<W == 1, uint32_t, unsigned long long>;
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= 2 * B.M) return;
    const int o = p >= B.M ? 1 : 0;
    const int64_t o0 = o ? B.M : 0;
    const ST* group = static_cast<const ST*>(B.group);
    const ST g = group[p];
    if (p > o0 && group[p - 1] == g) return;
    const uint2 b = find_bucket<ST>(B.slots + (o ? (int64_t(1) << B.bits) : 0), B.bits, g);
    if (b.y < B.heavy->min) return;
    const uint32_t id = atomicAdd(&B.heavy->taken[o], 1u);
    JoinSlot<W>* tab = static_cast<JoinSlot<W>*>(B.heavy_slots) + (o ? kJoinHeavySlots : 0);
    const uint32_t mask = (1u << B.heavy->bits[o]) - 1u;
    uint32_t s = join_hash(g, static_cast<int>(B.heavy->bits[o]));
    for (uint32_t t = 0; t <= mask; ++t, s = (s + 1) & mask)
        if (atomicCAS(reinterpret_cast<AT*>(&tab[s].id), static_cast<AT>(kJoinNone), static_cast<AT>(id)) ==
            static_cast<AT>(kJoinNone)) {
            tab[s].key = g;
            return;
        }
}

// The samples with two heavy strings into the table; in the spin-down order
// the scan strings for two-spin masks, all ones above the string where the
// spin-up string is light.
template <int W>
__global__ __launch_bounds__(kBlock) void k_join_core(JoinBuild B, int sbits) {
    using ST = JoinStr<W>;
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= 2 * B.M) return;
    const uint32_t least = B.heavy->min;
    const ST* group = static_cast<const ST*>(B.group);
    const ST* scan = static_cast<const ST*>(B.scan);
    const JoinBucket* up = B.slots;
    if (p >= B.M) {
        const ST a = scan[p];
        const bool light = find_bucket<ST>(up, B.bits, a).y < least;
        static_cast<ST*>(B.cross)[p - B.M] = light ? static_cast<ST>(a | (~ST(0) << sbits)) : a;
        return;
    }
    if (least == kJoinNone) return;
    const JoinSlot<W>* tab = static_cast<const JoinSlot<W>*>(B.heavy_slots);
    const uint32_t a = find_part<W>(tab, static_cast<int>(B.heavy->bits[0]), group[p]);
    if (a == kJoinNone) return;
    const uint32_t b = find_part<W>(tab + kJoinHeavySlots, static_cast<int>(B.heavy->bits[1]), scan[p]);
    if (b != kJoinNone) B.core[a * B.heavy->n[1] + b] = static_cast<uint32_t>(p) + 1u;
}

// The pairs inside own buckets past the limit, for the row sums: a row looks its
// masks of that order up in U's table, as the loop over masks does but over a
// ninth of them.  A wave takes 64 positions and of their rows those that have
// such a bucket, four at a time (a step's 64 masks are read once for them); with
// none in U every wave ends at once.  A candidate passes U's signature and a
// Bloom filter that stays in the L2s, and those that pass are queued and looked
// up 64 at a time.  What bounds it are the L2s' requests and misses, of the
// slots and amplitudes (2^20 samples: 1.3e10 and 3.2e9 in 70 ms; looked up
// unfiltered and evaluated from their terms where they were found 150).
// Energies, all electrons of one spin, by scans / here / by the loop: 52 qubits,
// 2^18 samples 17.0 / 12.2 / 15.0 ms, 2^20 225 / 81 / 70; 56 qubits, 2^20 and
// 2^21 here 73 and 218, by the loop 83 and 192.
constexpr int kOwnRows = 4;

template <int W, int PREC, bool ADJ, bool NW>
__global__ __launch_bounds__(kBlock) void k_join_own(JoinArgs A, JoinOwn T, const typename Prec<PREC>::Vec* __restrict__ vec,
                                                     void* __restrict__ partial, unsigned long long* __restrict__ pairs) {
    using P = Prec<PREC>;
    using ST = JoinStr<W>;
    using Acc = typename P::Acc;
    constexpr int TK = table_kind(W, NW);
    using HT = typename TabT<TK>::hash;
    struct Cand {   // of a row: the mask's number and part, the candidate's salted hash
        uint32_t at;
        ST part;
        HT hs;
    };
    __shared__ Cand queue[kBlock / kWave][kOwnRows][kQueue];
    if (*A.U.prep_err != 0u || A.U.heavy->huge == 0u) return;
    const int lane = lane_id();
    Cand (*const q)[kQueue] = queue[threadIdx.x / kWave];
    const int64_t M = A.U.M, tiles = (M + kWave - 1) / kWave;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kBlock / kWave);
    const TermRec<W>* __restrict__ terms = static_cast<const TermRec<W>*>(T.terms);
    const uint32_t* __restrict__ filter = A.U.filter;
    const uint32_t fmask = A.U.filter_mask;
    const int nstash = __builtin_amdgcn_readfirstlane(static_cast<int>(T.table.stash->count));
    const bool sig = T.params && __builtin_amdgcn_readfirstlane(T.params->sig_all) == 0;
    unsigned long long found = 0;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) +
                     __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
         t < 2 * tiles; t += waves) {
        // the rows of an order's buckets in the other order, that of the strings
        // that differ
        const int o = t >= tiles ? 1 : 0;
        const int64_t p0 = (t - (o ? tiles : 0)) * kWave;
        const bool in = p0 + lane < M;
        const int64_t p = (o ? 0 : M) + min(p0 + lane, M - 1);
        const ST g = static_cast<const ST*>(A.U.scan)[p];
        const uint2 b = find_bucket<ST>(A.U.slots + (o ? (int64_t(1) << A.U.bits) : 0), A.U.bits, g);
        const int32_t sample = A.U.perm[p];
        const JoinOwnDev own = o ? A.H.own[1] : A.H.own[0];
        const JoinOwnMask<W>* __restrict__ masks = static_cast<const JoinOwnMask<W>*>(own.masks);
        const GroupRec<W>* __restrict__ groups = static_cast<const GroupRec<W>*>(own.groups);
        const JoinPlace<W>* __restrict__ places = static_cast<const JoinPlace<W>*>(own.place);
        const int n = own.n;
        const ST scanned = static_cast<const ST*>(A.U.group)[p];
        uint64_t rows = __ballot(in && b.y > (o ? A.own_down : A.own_up));
        while (rows) {
            int64_t x[kOwnRows];
            uint64_t hx[kOwnRows];
            ST str[kOwnRows], grp[kOwnRows];   // the row's scanned string, its order's
            uint32_t ones[kOwnRows];
            Acc acc[kOwnRows];
            int qn[kOwnRows], nr = 0;
#pragma unroll
            for (int r = 0; r < kOwnRows; ++r) {   // past the last: the tile's first, without candidates
                const int l = rows ? __ffsll(static_cast<unsigned long long>(rows)) - 1 : 0;
                nr += rows ? 1 : 0;
                rows &= rows - 1;
                x[r] = __shfl(sample, l, kWave);
                str[r] = rdlane(scanned, l);
                grp[r] = rdlane(g, l);
                ones[r] = pop(str[r]);
                hx[r] = T.khash[x[r]];
                acc[r] = Acc{};
                qn[r] = 0;
            }
            // the last m of row r's candidates
            auto drain = [&](int r, int m) __attribute__((always_inline)) {
                wave_sync();
                const bool on = lane < m;
                const Cand e = q[r][qn[r] - m + (on ? lane : 0)];
                qn[r] -= m;
                const int c = static_cast<int>(e.at);
                const HT hs = e.hs;
                typename TabT<TK>::slot v1 = 0, v2 = 0;
                if (on) v1 = load_slot<TK>(T.table, slot1(T.table, hs));
                const JoinPlace<W> pl = places[c];
                const ST ks = ADJ ? str[r] : static_cast<ST>(str[r] ^ e.part);
                ST p1, p3;
                join_parity_masks(e.part, p1, p3);
                const uint32_t idx = (pop(static_cast<ST>(ks & p1)) & 1u) | ((pop(static_cast<ST>(ks & e.part)) & 1u) << 1) |
                                     ((pop(static_cast<ST>(ks & p3)) & 1u) << 2);
                double hr = own.sign[static_cast<int64_t>(idx) * n + c], hi = 0.0;
                if (need_slot2<TK>(T.table, v1, hs)) v2 = load_slot<TK>(T.table, slot2(T.table, hs));
                const uint32_t zp = pop(static_cast<ST>(ks & (o ? pl.za : pl.zb))) + pop(static_cast<ST>(grp[r] & (o ? pl.zb : pl.za)));
                hr = (zp & 1u) ? -hr : hr;
                const bool by_run = (pl.hi & kJoinTag) == kJoinTag && (pl.hi & 7u) != static_cast<uint32_t>(kJoinSign);
                uint64_t row[W], xp[W];
                GroupRec<W> gr{};
                if (TK == kTabVerify || __ballot(by_run)) {
                    gr = groups[c];
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        row[w] = A.U.keys[x[r] * W + w];
                        xp[w] = row[w] ^ gr.xy[w];
                    }
                }
                int j;
                if constexpr (TK == kTabVerify)
                    j = table_settle<TK, W>(T.table, A.U.keys, v1, v2, hs, xp, nstash, on);
                else
                    j = wave_settle<TK>(T.table, v1, v2, hs, nstash);
                const bool hit = on && j >= 0;
                found += static_cast<unsigned long long>(__popcll(__ballot(hit)));
                const typename P::Vec v = vec[hit ? j : 0];
                if (__ballot(hit && by_run)) {   // runs not told by signs: single excitations, the diagonal
                    const bool run = hit && by_run;
                    double rr, ri;
                    wave_melem<W, NW>(terms, run ? gr.begin : 0, run ? gr.mid : 0, run ? gr.end : 0, ADJ ? row : xp, rr, ri);
                    if (by_run) {
                        hr = rr;
                        hi = ri;
                    }
                }
                if (hit) {
                    if constexpr (PREC == 0) {
                        mac(acc[r], hr, hi, v);
                    } else {
                        const float4 h = split_c(hr, hi);
                        mac(acc[r], F2{h.x, h.y}, F2{h.z, h.w}, v);
                    }
                }
                wave_sync();
            };
            for (int j0 = 0; j0 < n; j0 += kWave) {
                const JoinOwnMask<W> mask = masks[min(j0 + lane, n - 1)];
                bool ok[kOwnRows];
                uint32_t word[kOwnRows], bits[kOwnRows];
#pragma unroll
                for (int r = 0; r < kOwnRows; ++r) {
                    ok[r] = j0 + lane < n && r < nr && (!sig || pop(static_cast<ST>(str[r] ^ mask.part)) == ones[r]);
                    const uint32_t hf = static_cast<uint32_t>((hx[r] ^ mask.hash) >> 32);
                    bits[r] = bloom_bits(hf);
                    word[r] = 0u;
                    if (ok[r]) word[r] = filter[bloom_word(hf, fmask)];
                }
#pragma unroll
                for (int r = 0; r < kOwnRows; ++r) {
                    const bool pass = ok[r] && (word[r] & bits[r]) == bits[r];
                    const uint64_t mk = __ballot(pass);
                    if (pass)
                        q[r][qn[r] + lanes_below(mk)] = Cand{static_cast<uint32_t>(j0 + lane), mask.part,
                                                             static_cast<HT>(hx[r] ^ mask.hash ^ T.table.salt)};
                    qn[r] += __popcll(mk);
                    if (qn[r] >= kWave) drain(r, kWave);
                }
            }
#pragma unroll
            for (int r = 0; r < kOwnRows; ++r) {
                if (r >= nr) continue;
                if (qn[r] > 0) drain(r, qn[r]);
                wave_sum(acc[r]);
                // the row's sum of the chunk that has its own bucket
                if (lane == 0) {
                    const int64_t to = (o ? 0 : 2) * M + x[r];
                    Acc sum;
                    __builtin_memcpy(&sum, static_cast<const double2*>(partial) + to, sizeof(sum));
                    acc_plus(sum, acc[r]);
                    store_acc(partial, to, sum);
                }
            }
        }
    }
    if (pairs && lane == 0 && found)
        atomicAdd(pairs + (blockIdx.x % kJoinPairSlots) * kJoinPairStride, found);
}

// The amplitudes in both orders; with huge buckets in U also its filter.
__global__ __launch_bounds__(kBlock) void k_join_vec(JoinDev U, const uint64_t* __restrict__ khash,
                                                     const double2* __restrict__ in) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= 2 * U.M) return;
    const int32_t i = U.perm[p];
    U.vec[p] = in[i];
    if (U.filter && p < U.M && U.heavy->huge) {
        const uint32_t hf = static_cast<uint32_t>(khash[i] >> 32);
        atomicOr(U.filter + bloom_word(hf, U.filter_mask), bloom_bits(hf));
    }
}

inline unsigned div_up(int64_t n, int64_t d) { return static_cast<unsigned>((n + d - 1) / d); }

JoinArgs make_args(const void* terms, const JoinHamDev& JH, const JoinDev& J, const Plan& P) {
    JoinArgs A;
    A.terms = terms;
    A.H = JH;
    A.U = J;
    A.chunks = P.chunks;
    A.per_chunk = P.per_chunk;
    A.tiles = (J.M + P.rows_per_block - 1) / P.rows_per_block;
    A.own_up = A.own_down = kJoinNone;
    return A;
}

template <int W, bool NW>
void launch_own(bool adjoint, int precision, const JoinArgs& A, const JoinOwn& T, const double2* vec, const float4* vecf,
                void* partial, unsigned long long* pairs, hipStream_t st) {
    // one round of the chip at most, four waves a SIMD
    const int64_t tiles = 2 * ((A.U.M + kWave - 1) / kWave);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>((tiles + 3) / 4, 1024))), block(kBlock);
    if (precision == 0 && adjoint)
        hipLaunchKernelGGL((k_join_own<W, 0, true, NW>), grid, block, 0, st, A, T, vec, partial, pairs);
    else if (precision == 0)
        hipLaunchKernelGGL((k_join_own<W, 0, false, NW>), grid, block, 0, st, A, T, vec, partial, pairs);
    else if (adjoint)
        hipLaunchKernelGGL((k_join_own<W, 1, true, NW>), grid, block, 0, st, A, T, vecf, partial, pairs);
    else
        hipLaunchKernelGGL((k_join_own<W, 1, false, NW>), grid, block, 0, st, A, T, vecf, partial, pairs);
}

template <int W, int PREC, bool ADJ, bool NW, int MODE>
hipError_t launch_rows(int rows, const JoinArgs& A, const JoinOut& O, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(A.tiles * A.chunks));
    if (rows == 16)
        hipLaunchKernelGGL((k_join<W, PREC, ADJ, NW, MODE, 16>), grid, dim3(kWave), 0, st, A, O);
    else
        hipLaunchKernelGGL((k_join<W, PREC, ADJ, NW, MODE, 8>), grid, dim3(kWave), 0, st, A, O);
    return hipGetLastError();
}

template <int W, bool ADJ, bool NW>
hipError_t launch_sum(int precision, int rows, const JoinArgs& A, const JoinOut& O, hipStream_t st) {
    if constexpr (!ADJ)
        if (O.pairs)
            return precision == 0 ? launch_rows<W, 0, ADJ, NW, kModeSumPairs>(rows, A, O, st)
                                  : launch_rows<W, 1, ADJ, NW, kModeSumPairs>(rows, A, O, st);
    return precision == 0 ? launch_rows<W, 0, ADJ, NW, kModeSum>(rows, A, O, st)
                          : launch_rows<W, 1, ADJ, NW, kModeSum>(rows, A, O, st);
}

template <int MODE>
hipError_t launch_list(const HamDev& H, int rows, const JoinArgs& A, const JoinOut& O, hipStream_t st) {
    return H.W == 2 ? launch_rows<2, 0, false, false, MODE>(rows, A, O, st)
                    : launch_rows<1, 0, false, false, MODE>(rows, A, O, st);
}

}  // namespace

template <int W>
static hipError_t join_index(const JoinBuild& B, hipStream_t st) {
    const int sbits = join_string_bits(B.n_qubits);
    const dim3 rows(div_up(B.M, kBlock)), both(div_up(2 * B.M, kBlock)), block(kBlock);
    hipLaunchKernelGGL(k_join_keys<W>, rows, block, 0, st, B, sbits);
    int alt = 0;
    const hipError_t e = launch_radix_sort_pairs(B.key, B.val, B.key2, B.val2, 2 * B.M, sbits + 1, B.hist, B.hist_off,
                                                 B.hist_scan, &alt, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_join_index<W>, both, block, 0, st, B, sbits, alt ? B.key2 : B.key, alt ? B.val2 : B.val);
    if (B.split) {
        hipLaunchKernelGGL(k_join_heavy_min, dim3(1), dim3(1), 0, st, B.heavy);
        hipLaunchKernelGGL(k_join_heavy_ids<W>, both, block, 0, st, B);
        hipLaunchKernelGGL(k_join_core<W>, both, block, 0, st, B, sbits);
    }
    return hipGetLastError();
}

hipError_t launch_join_index(int W, const JoinBuild& B, hipStream_t st) {
    return W == 1 ? join_index<1>(B, st) : join_index<2>(B, st);
}

static hipError_t join_sums(bool adjoint, int precision, const HamDev& H, const JoinArgs& A, const JoinOut& O, int rows,
                            hipStream_t st) {
    if (H.W == 2)
        return adjoint ? launch_sum<2, true, false>(precision, rows, A, O, st)
                       : launch_sum<2, false, false>(precision, rows, A, O, st);
    if (H.n_qubits <= 32)
        return adjoint ? launch_sum<1, true, true>(precision, rows, A, O, st)
                       : launch_sum<1, false, true>(precision, rows, A, O, st);
    return adjoint ? launch_sum<1, true, false>(precision, rows, A, O, st)
                   : launch_sum<1, false, false>(precision, rows, A, O, st);
}

hipError_t launch_join_pairs(bool adjoint, int precision, const HamDev& H, const JoinHamDev& JH, const JoinDev& J,
                             const Plan& P, const JoinOwn& own, const double2* vec, const float4* vecf, void* partial,
                             hipStream_t st, unsigned long long* pairs) {
    if (adjoint && pairs) return hipErrorInvalidValue;   // the forward sums count
    JoinArgs A = make_args(precision == 0 ? H.terms : H.terms_f, JH, J, P);
    const bool huge = J.filter != nullptr;
    if (huge) {
        A.own_up = join_own_limit(JH.own[0].n);
        A.own_down = join_own_limit(JH.own[1].n);
    }
    JoinOut O{};
    O.partial = partial;
    O.pairs = pairs;
    static_assert(sizeof(double2) == sizeof(float4), "one copy serves both precisions");
    hipLaunchKernelGGL(k_join_vec, dim3(div_up(2 * J.M, kBlock)), dim3(kBlock), 0, st, J, own.khash,
                       precision == 0 ? vec : reinterpret_cast<const double2*>(vecf));
    const hipError_t e = join_sums(adjoint, precision, H, A, O, P.rows_per_block, st);
    if (e != hipSuccess || !huge) return e;
    if (H.W == 2)
        launch_own<2, false>(adjoint, precision, A, own, vec, vecf, partial, pairs, st);
    else if (own.narrow)
        launch_own<1, true>(adjoint, precision, A, own, vec, vecf, partial, pairs, st);
    else
        launch_own<1, false>(adjoint, precision, A, own, vec, vecf, partial, pairs, st);
    return hipGetLastError();
}

hipError_t launch_join_count(const HamDev& H, const JoinHamDev& JH, const JoinDev& J, const Plan& P, int32_t* counts,
                             hipStream_t st) {
    JoinOut O{};
    O.counts = counts;
    return launch_list<kModeCount>(H, P.rows_per_block, make_args(H.terms, JH, J, P), O, st);
}

hipError_t launch_join_elements(const HamDev& H, const JoinHamDev& JH, const SampleDev& S, int64_t n,
                                const int32_t* i_idx, const int32_t* j_idx, double2* h_out, int32_t* cnt, int32_t* grp,
                                uint32_t* err, hipStream_t st) {
    const dim3 grid(div_up(n, 256)), block(256);
    if (H.W == 2)
        hipLaunchKernelGGL((k_join_elements<2, false>), grid, block, 0, st, JH, static_cast<const TermRec<2>*>(H.terms),
                           S.keys, S.n, n, i_idx, j_idx, nullptr, 0, h_out, cnt, grp, err);
    else
        hipLaunchKernelGGL((k_join_elements<1, false>), grid, block, 0, st, JH, static_cast<const TermRec<1>*>(H.terms),
                           S.keys, S.n, n, i_idx, j_idx, nullptr, 0, h_out, cnt, grp, err);
    return hipGetLastError();
}

hipError_t launch_join_to_csr(const HamDev& H, const JoinHamDev& JH, const SampleDev& S, int64_t n,
                              const uint64_t* pkey, int jbits, int32_t* col, double2* h, hipStream_t st) {
    const dim3 grid(div_up(n, 256)), block(256);
    if (H.W == 2)
        hipLaunchKernelGGL((k_join_elements<2, true>), grid, block, 0, st, JH, static_cast<const TermRec<2>*>(H.terms),
                           S.keys, S.n, n, nullptr, nullptr, pkey, jbits, h, col, nullptr, nullptr);
    else
        hipLaunchKernelGGL((k_join_elements<1, true>), grid, block, 0, st, JH, static_cast<const TermRec<1>*>(H.terms),
                           S.keys, S.n, n, nullptr, nullptr, pkey, jbits, h, col, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_join_fill(const HamDev& H, const JoinHamDev& JH, const JoinDev& J, const Plan& P, int jbits,
                            const int64_t* offsets, uint64_t* pkey, uint32_t* pval, hipStream_t st) {
    JoinOut O{};
    O.offsets = offsets;
    O.pkey = pkey;
    O.pval = pval;
    O.jbits = jbits;
    return launch_list<kModeFill>(H, P.rows_per_block, make_args(H.terms, JH, J, P), O, st);
}

}  // namespace eloc
