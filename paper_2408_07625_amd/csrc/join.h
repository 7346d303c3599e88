// Host side of the spin-string join (join.hip): the Hamiltonian's XY masks by
// their spin-up and spin-down parts.
#pragma once

#include "ham.h"
#include "host.h"
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

namespace eloc {

// A function on a thread of its own, joined at the end of the scope at the
// latest; run in place where no thread can be had.
class BesideThread {
public:
    template <class F>
    explicit BesideThread(F f) {
        try {
            t_ = std::thread(f);
        } catch (const std::system_error&) {
            f();
        }
    }
    ~BesideThread() { wait(); }
    void wait() {
        if (t_.joinable()) t_.join();
    }

private:
    std::thread t_;
};

template <int W>
struct HostJoin {
    using ST = JoinStr<W>;
    bool ok = false;
    std::vector<ST> alist, blist;
    std::vector<JoinMask> amask, bmask;
    bool direct = false;
    uint32_t stride = 0;
    std::vector<JoinSlot<W>> b_cross, b_own, a_own;   // spin part -> id
    // by place
    std::vector<JoinPlace<W>> place;
    std::vector<double> sign;         // [kJoinIdx][places]
    std::vector<double> linear;       // [tables][2][2 nibbles][16]
    std::vector<JoinRun> runs;
    std::vector<int32_t> gids;
    struct Own {
        std::vector<JoinOwnMask<W>> masks;
        std::vector<GroupRec<W>> groups;
        std::vector<JoinPlace<W>> place;
        std::vector<double> sign;
    } own[2];                         // the masks (0, b); (a, 0) with a != 0
    int nibbles = 0;
    uint32_t cross = 0;               // first place of the two-spin masks
    uint32_t a_base = 0;              // places of the masks (a, 0)
    uint32_t a_pmin = 0, a_span = 0;  // their smallest popcount, largest less smallest
    uint32_t cross_span = 0;          // largest popcount of a part of a two-spin mask
};

// Slots of a table of n spin parts (load at most 1/4).
inline uint64_t join_capacity(size_t n) { return pow2_at_least(4 * std::max<uint64_t>(n, 2)); }

template <int W>
inline void join_insert(std::vector<JoinSlot<W>>& t, JoinStr<W> key, uint32_t id) {
    const int bits = bits_for(t.size() - 1);
    size_t s = join_hash(key, bits);
    while (t[s].id != kJoinNone) s = (s + 1) & (t.size() - 1);
    t[s].key = key;
    t[s].id = id;
}

// T[idx] of a group whose terms share z; false where the dependence on ket & m
// does not go through idx.  mixed: y is y0 (ya0, yb0) with the spin-up part,
// the spin-down part, both or neither flipped, idx holds the parities of the
// parts, and the sign of y0 is left to the caller (where a Jordan-Wigner string
// of one spin passes over a flipped orbital of the other, y0 is not empty); else
// y is an even subset of at most four bits, and idx holds the parities of
// join_parity_masks and of all.
template <int W>
inline bool join_signs(const HostHam<W>& hh, const GroupRec<W>& gr, JoinStr<W> a, JoinStr<W> b, bool mixed,
                       JoinStr<W> ya0, JoinStr<W> yb0, double (&T)[kJoinIdx]) {
    using ST = JoinStr<W>;
    const ST w = a | b;
    if (!mixed && join_count(w) > 4) return false;
    ST ket[kJoinIdx];   // ket bits of every idx: l1 clear, the rest follows
    if (!mixed) {
        ST bit[4], v = w;
        for (int i = 0; i < 4; ++i) {
            bit[i] = v & (~v + 1);
            v &= v - 1;
        }
        for (uint32_t i = 0; i < kJoinIdx; ++i) {
            ST k = 0;
            if (i & 1u) k |= bit[0];
            if (i & 4u) k |= bit[2];
            if ((join_count(k) & 1u) != ((i >> 1) & 1u)) k |= bit[3];
            ket[i] = k;
        }
    }
    double c[4] = {0.0, 0.0, 0.0, 0.0};   // mixed: by (y has the spin-up part, the spin-down part)
    for (double& t : T) t = 0.0;
    for (int t = gr.begin; t < gr.end; ++t) {
        const TermRec<W>& tr = hh.terms[static_cast<size_t>(t)];
        uint64_t y[W];
        for (int q = 0; q < W; ++q) y[q] = tr.yz[q] & gr.xy[q];
        ST ya, yb;
        spin_strings<W>(y, ya, yb);
        if (mixed) {
            ya ^= ya0;
            yb ^= yb0;
            if ((ya != 0 && ya != a) || (yb != 0 && yb != b)) return false;
            c[(ya != 0 ? 1 : 0) + (yb != 0 ? 2 : 0)] += tr.h;
        } else {
            const ST yy = ya | yb;
            if (join_count(yy) & 1u) return false;
            for (size_t i = 0; i < kJoinIdx; ++i) T[i] += (join_count(static_cast<ST>(ket[i] & yy)) & 1u) ? -tr.h : tr.h;
        }
    }
    for (size_t i = 0; i < kJoinIdx; ++i) {
        if (mixed) {
            const double pa = (i & 1u) ? -1.0 : 1.0, pb = (i & 2u) ? -1.0 : 1.0;
            T[i] = (c[0] + pa * c[1]) + pb * (c[2] + pa * c[3]);
        }
        if (!std::isfinite(T[i])) return false;
    }
    return true;
}

template <int W>
inline JoinPlace<W> join_tag(JoinKind kind, uint32_t number = 0) {
    return JoinPlace<W>{0, 0, number, kJoinTag | static_cast<uint32_t>(kind)};
}
inline JoinKind join_kind_of(uint32_t hi) {
    return (hi & kJoinTag) == kJoinTag ? static_cast<JoinKind>(hi & 7u) : kJoinSign;
}

// One place's evaluation where its terms share the bits outside the mask; false
// where they do not.  Writes that place alone.
template <int W>
bool join_place_one(const HostHam<W>& hh, const GroupRec<W>& gr, size_t place, bool mixed, HostJoin<W>& out) {
    using ST = JoinStr<W>;
    const size_t P = out.place.size();
    JoinPlace<W>& pl = out.place[place];
    pl = join_tag<W>(kJoinRunKind);
    if (gr.end != gr.mid) return true;
    ST a, b;
    spin_strings<W>(gr.xy, a, b);
    uint64_t z[W];
    bool one = true;
    for (int w = 0; w < W; ++w) {
        z[w] = hh.terms[static_cast<size_t>(gr.begin)].yz[w] & ~gr.xy[w];
        for (int t = gr.begin + 1; t < gr.end; ++t)
            one = one && ((hh.terms[static_cast<size_t>(t)].yz[w] & ~gr.xy[w]) == z[w]);
    }
    if (!one) return false;
    double T[kJoinIdx];
    uint64_t y0[W];
    for (int w = 0; w < W; ++w) y0[w] = hh.terms[static_cast<size_t>(gr.begin)].yz[w] & gr.xy[w];
    ST ya0 = 0, yb0 = 0;
    if (mixed) {   // with each part's fewer bits
        spin_strings<W>(y0, ya0, yb0);
        if (2 * join_count(ya0) > join_count(a)) ya0 ^= a;
        if (2 * join_count(yb0) > join_count(b)) yb0 ^= b;
    }
    if (!join_signs<W>(hh, gr, a, b, mixed, ya0, yb0, T)) return true;
    pl = join_tag<W>(kJoinSign);
    spin_strings<W>(z, pl.za, pl.zb);
    pl.za ^= ya0;
    pl.zb ^= yb0;
    for (size_t i = 0; i < kJoinIdx; ++i) out.sign[i * P + place] = T[i];
    if (mixed) {
        uint64_t bits;
        std::memcpy(&bits, &T[kJoinMain], sizeof(bits));
        pl.lo = static_cast<uint32_t>(bits);
        pl.hi = static_cast<uint32_t>(bits >> 32);
    }
    return true;
}

// The others: a majority z and one further bit, by the linear table `number`
// (zeros so far; left so where the place keeps its run).
template <int W>
void join_place_linear(const HostHam<W>& hh, const GroupRec<W>& gr, size_t place, size_t number, HostJoin<W>& out) {
    JoinPlace<W>& pl = out.place[place];
    uint64_t z[W];
    const int n = gr.end - gr.begin;
    bool any = false;
    for (int w = 0; w < W; ++w) any = any || gr.xy[w] != 0;
    if (n < 8 || !any || number >= (size_t(1) << 16)) return;
    {   // a bit of the majority z is the majority of the bits
        int c[64 * W] = {};
        for (int t = gr.begin; t < gr.end; ++t)
            for (int w = 0; w < W; ++w)
                for (uint64_t v = hh.terms[static_cast<size_t>(t)].yz[w] & ~gr.xy[w]; v; v &= v - 1)
                    ++c[64 * w + __builtin_ctzll(v)];
        for (int w = 0; w < W; ++w) {
            z[w] = 0;
            for (int q = 0; q < 64; ++q)
                if (2 * c[64 * w + q] > n) z[w] |= 1ull << q;
        }
    }
    const size_t half = static_cast<size_t>(out.nibbles) * 16, per = 2 * half;
    double* const tab = out.linear.data() + number * 2 * per;
    for (int t = gr.begin; t < gr.end; ++t) {
        const TermRec<W>& tr = hh.terms[static_cast<size_t>(t)];
        int bit = -1, extra = 0;
        bool none = true, all = true;
        for (int w = 0; w < W; ++w) {
            const uint64_t e = (tr.yz[w] & ~gr.xy[w]) ^ z[w], y = tr.yz[w] & gr.xy[w];
            extra += __builtin_popcountll(e);
            if (e) bit = 64 * w + __builtin_ctzll(e);
            none = none && y == 0;
            all = all && y == gr.xy[w];
        }
        if (extra > 1 || !(none || all)) {
            std::fill(tab, tab + 2 * per, 0.0);
            return;
        }
        const int q = bit < 0 ? 0 : bit / 2;   // bit of the string
        for (int par = 0; par < 2; ++par) {
            const double h = (all && par) ? -tr.h : tr.h;
            double* F = tab + static_cast<size_t>(par) * per + (bit >= 0 && (bit & 1) ? half : 0) +
                        static_cast<size_t>(q / 4) * 16;
            for (int v = 0; v < 16; ++v) F[v] += (bit >= 0 && ((v >> (q % 4)) & 1)) ? -h : h;
        }
    }
    pl = join_tag<W>(kJoinLinear, static_cast<uint32_t>(number));
    spin_strings<W>(z, pl.za, pl.zb);
}

// ok stays false where the masks do not factor well: more places than four
// times the groups, or over an eighth of the groups summed term by term.
template <int W>
void build_host_join(const HostHam<W>& hh, int n_qubits, HostJoin<W>& out) {
    using ST = JoinStr<W>;
    const int64_t G = hh.G;
    if (hh.maxpart >= kNarrowMaxPart) return;   // a run's part lengths travel in 16 bits
    // distinct parts: of the two-spin masks, and of the one-spin masks
    const auto number = [](XYMap& map, std::vector<ST>& vals, ST v) {
        const uint64_t k = v;
        const int64_t i = map.find_or_insert(&k, static_cast<int64_t>(vals.size()));
        if (i == static_cast<int64_t>(vals.size())) vals.push_back(v);
        return i;
    };
    std::vector<ST> as(static_cast<size_t>(G)), bs(static_cast<size_t>(G));
    XYMap amap(1), bmap(1), aomap(1), bomap(1);
    std::vector<ST> avals, bvals, aown, bown;
    std::vector<int32_t> bid(static_cast<size_t>(G));
    bool zero = false, pairs = true;   // pairs: every mask has ids by position
    // what `number` gave the parts of two bits, by position
    const size_t by_two = static_cast<size_t>(32 * W) * (32 * W - 1) / 2;
    std::vector<int64_t> atwo(by_two, -1), btwo(by_two, -1);
    const auto number_part = [&](XYMap& map, std::vector<ST>& vals, std::vector<int64_t>& two, ST v, uint32_t count) {
        if (count != 2u) return number(map, vals, v);
        int64_t& id = two[join_pair_id(v)];
        if (id < 0) id = number(map, vals, v);
        return id;
    };
    for (int64_t g = 0; g < G; ++g) {
        ST a, b;
        spin_strings<W>(&hh.gkeys[static_cast<size_t>(g * W)], a, b);
        as[static_cast<size_t>(g)] = a;
        bs[static_cast<size_t>(g)] = b;
        int64_t id;
        const uint32_t pa = join_count(a), pb = join_count(b);
        if (a == 0 || b == 0) {
            zero = zero || a == 0;
            id = a == 0 ? number(bomap, bown, b) : number(aomap, aown, a);
            pairs = pairs && (pa + pb) % 2 == 0 && pa + pb <= 4;
        } else {
            (void)number_part(amap, avals, atwo, a, pa);
            id = number_part(bmap, bvals, btwo, b, pb);
            pairs = pairs && pa == 2 && pb == 2;
            out.cross_span = std::max(out.cross_span, std::max(pa, pb));
        }
        bid[static_cast<size_t>(g)] = static_cast<int32_t>(id);
    }
    out.alist.assign(avals.begin(), avals.end());
    std::sort(out.alist.begin(), out.alist.end());
    out.blist.assign(bvals.begin(), bvals.end());
    std::sort(out.blist.begin(), out.blist.end());
    if (zero) out.alist.insert(out.alist.begin(), ST(0));
    const int64_t na = static_cast<int64_t>(out.alist.size());
    const int sb = join_string_bits(n_qubits);
    const int64_t n_pairs = static_cast<int64_t>(sb) * (sb - 1) / 2, n_even = join_even_count(sb);
    // ids by position unless that leaves too many places empty
    const auto size = [&](bool direct) {
        if (direct) return 2 * n_even + n_pairs * n_pairs;
        return static_cast<int64_t>(bown.size() + aown.size()) + static_cast<int64_t>(avals.size() * bvals.size());
    };
    out.direct = pairs && size(true) <= 4 * G + 4096;
    const int64_t places = size(out.direct);
    if (na < 1 || places > 4 * G + 4096 || places >= (int64_t(1) << 25)) return;
    out.stride = static_cast<uint32_t>(out.direct ? n_pairs : static_cast<int64_t>(bvals.size()));
    const uint32_t cross = out.cross = static_cast<uint32_t>(out.direct ? n_even : static_cast<int64_t>(bown.size()));
    out.a_base = static_cast<uint32_t>(places - (out.direct ? n_even : static_cast<int64_t>(aown.size())));
    const auto a_index = [&](ST a) {   // of a two-spin mask's spin-up part
        return static_cast<uint32_t>(std::lower_bound(out.alist.begin(), out.alist.end(), a) - out.alist.begin());
    };
    const auto a_base_of = [&](ST a) {
        const uint32_t i = out.direct ? join_pair_id(a) : a_index(a) - (zero ? 1u : 0u);
        return cross + i * out.stride;
    };
    out.amask.resize(static_cast<size_t>(na));
    for (int64_t k = 0; k < na; ++k) {
        const ST a = out.alist[static_cast<size_t>(k)];
        out.amask[static_cast<size_t>(k)] = JoinMask{a == 0 ? kJoinFull : a_base_of(a), 0u};
    }
    out.bmask.resize(out.blist.size());
    for (size_t k = 0; k < out.blist.size(); ++k)
        out.bmask[k] = JoinMask{out.direct ? cross + join_pair_id(out.blist[k]) : 0u, out.cross_span - 1u};
    out.nibbles = (sb + 3) / 4;
    out.runs.assign(static_cast<size_t>(places), JoinRun{0, 0});
    out.gids.assign(static_cast<size_t>(places), -1);
    out.place.assign(static_cast<size_t>(places), join_tag<W>(kJoinEmpty));
    out.sign.assign(static_cast<size_t>(places) * kJoinIdx, 0.0);
    std::vector<uint32_t> at(static_cast<size_t>(G));
    uint32_t pmin = ~0u, pmax = 0;
    for (int64_t g = 0; g < G; ++g) {
        const ST a = as[static_cast<size_t>(g)], b = bs[static_cast<size_t>(g)];
        size_t place = static_cast<size_t>(bid[static_cast<size_t>(g)]);
        if (a == 0) {
            JoinMask& m = out.amask[0];
            m.span = std::max(m.span, join_count(b));
            if (out.direct) place = join_even_id(b, static_cast<uint32_t>(sb));
        } else if (b == 0) {
            if (out.direct) place = join_even_id(a, static_cast<uint32_t>(sb));
            place += out.a_base;
            pmin = std::min(pmin, join_count(a));
            pmax = std::max(pmax, join_count(a));
        } else {
            JoinMask& m = out.amask[out.direct ? 0 : a_index(a)];
            if (!out.direct) m.span = std::max<uint32_t>(m.span, join_count(b) - 1u);
            place = a_base_of(a) + (out.direct ? join_pair_id(b) : place);
        }
        const GroupRec<W>& gr = hh.groups[static_cast<size_t>(g)];
        out.runs[place] = JoinRun{static_cast<uint32_t>(gr.begin),
                                  static_cast<uint32_t>(gr.mid - gr.begin) |
                                      (static_cast<uint32_t>(gr.end - gr.mid) << 16)};
        out.gids[place] = static_cast<int32_t>(g);
        at[static_cast<size_t>(g)] = static_cast<uint32_t>(place);
    }
    // the evaluations, a part of the groups a thread (each writes its own
    // places and tables)
    const auto in_parts = [](int64_t n, int64_t least, const auto& part) {
        const int64_t per = std::max<int64_t>(least, (n + 3) / 4);
        std::vector<std::unique_ptr<BesideThread>> others;
        for (int64_t i0 = per; i0 < n; i0 += per)
            others.push_back(std::make_unique<BesideThread>([&part, i0, i1 = std::min(n, i0 + per)] { part(i0, i1); }));
        part(0, std::min(n, per));
    };
    std::vector<uint8_t> more(static_cast<size_t>(G), 0);
    in_parts(G, 4096, [&](int64_t g0, int64_t g1) {
        for (int64_t g = g0; g < g1; ++g) {
            const size_t i = static_cast<size_t>(g);
            more[i] = join_place_one<W>(hh, hh.groups[i], at[i], as[i] != 0 && bs[i] != 0, out) ? 0 : 1;
        }
    });
    std::vector<int64_t> rest;
    for (int64_t g = 0; g < G; ++g)
        if (more[static_cast<size_t>(g)]) rest.push_back(g);
    out.linear.assign(std::min<size_t>(rest.size(), size_t(1) << 16) * 4 * static_cast<size_t>(out.nibbles) * 16, 0.0);
    in_parts(static_cast<int64_t>(rest.size()), 64, [&](int64_t k0, int64_t k1) {
        for (int64_t k = k0; k < k1; ++k) {
            const size_t i = static_cast<size_t>(rest[static_cast<size_t>(k)]);
            join_place_linear<W>(hh, hh.groups[i], at[i], static_cast<size_t>(k), out);
        }
    });
    int64_t by_run = 0;
    for (int64_t g = 0; g < G; ++g)
        by_run += join_kind_of(out.place[at[static_cast<size_t>(g)]].hi) == kJoinRunKind;
    if (8 * by_run > G) return;
    for (int o = 0; o < 2; ++o) {
        std::vector<size_t> list;
        for (size_t i = 0; i < static_cast<size_t>(G); ++i)
            if (o == 0 ? as[i] == 0 : as[i] != 0 && bs[i] == 0) list.push_back(i);
        std::stable_sort(list.begin(), list.end(), [&](size_t x, size_t y) {
            return hh.groups[x].end - hh.groups[x].begin > hh.groups[y].end - hh.groups[y].begin;
        });
        typename HostJoin<W>::Own& own = out.own[o];
        own.sign.resize(kJoinIdx * list.size());
        for (size_t k = 0; k < list.size(); ++k) {
            const size_t i = list[k];
            own.masks.push_back(JoinOwnMask<W>{o == 0 ? bs[i] : as[i], hh.ghash[i]});
            own.groups.push_back(hh.groups[i]);
            own.place.push_back(out.place[at[i]]);
            for (size_t q = 0; q < kJoinIdx; ++q)
                own.sign[q * list.size() + k] = out.sign[q * static_cast<size_t>(places) + at[i]];
        }
    }
    if (out.direct)
        for (int64_t k = zero ? 1 : 0; k < na; ++k) out.amask[static_cast<size_t>(k)].span = 1u;
    if (!aown.empty()) {
        out.a_pmin = pmin;
        out.a_span = pmax - pmin;
    }
    const auto table = [](std::vector<JoinSlot<W>>& t, const std::vector<ST>& vals) {
        t.assign(join_capacity(vals.size()), JoinSlot<W>{0, kJoinNone});
        for (size_t i = 0; i < vals.size(); ++i) join_insert<W>(t, vals[i], static_cast<uint32_t>(i));
    };
    table(out.b_cross, bvals);
    table(out.b_own, bown);
    table(out.a_own, aown);
    out.ok = true;
}

// The masks by spin part, where the strings are short enough and there is the
// memory for them; else hj.ok stays false.
template <int W>
inline void build_host_join_if(const HostHam<W>& hh, int n_qubits, HostJoin<W>& hj) {
    if (n_qubits > kJoinMaxQubits) return;
    try {
        build_host_join<W>(hh, n_qubits, hj);
    } catch (const std::bad_alloc&) {
        hj = HostJoin<W>{};
    }
}

// Whether the join is taken for M samples where the loop would meet `loop`
// candidates.  The loops take about 6.5e8 candidates a millisecond (|U| |XY|
// for LoopOverTerms, |U|^2 for LoopOverBatch; LoopOverTrie costs about eight of
// them per |U| |XY|), the join about 0.2 ms for U's two orders and 6 ns a sample
// at 28 qubits, 17 at 52, 26 at 74, 60 at 100, where the masks are many more.
// Samples that share a spin string make it longer (join_own_limit).  Measured,
// loop / join: LoopOverTerms, 28 qubits, 65 536 samples
// (6.9e8) 1.09 / 0.53 ms; 52 qubits, 2^20 (1.4e11) 97 / 18 ms; LoopOverBatch,
// 40 qubits, 9999 samples (1.0e8) 0.16 / 0.24 ms.
// `beside`: in a batch the join's many small launches run beside the others'
// items, which is worth about half of the fixed part: 26 qubits, 29 882 samples
// (2.3e8) in a batch of 16, 1.29 ms for the batch with its loop, 1.06 with the join.
inline bool join_pays(int64_t M, int64_t loop, bool beside = false) {
    return loop >= (int64_t(1) << (beside ? 26 : 27)) + (M << 12);
}

// Launch geometry for M rows.  Chunk 0: the spin-down order; chunk 1: the
// heavy-heavy table; then alist in chunks of at least 16 masks.  16 rows a wave
// share a scanned column and a bucket lookup, but a heavy string's wave then
// runs long: 52 qubits, 2^20 samples, 18.8 ms with 16 rows, 19.3 with 8; 28
// qubits, 65 536, 0.63 with 8, 0.66 with 16.
inline Plan join_plan(int n_a, int64_t M) {
    Plan P;
    P.rows_per_block = M >= (int64_t(1) << 17) ? 16 : 8;
    const int64_t target = 32768;   // waves
    const int64_t tiles = (M + P.rows_per_block - 1) / P.rows_per_block;
    const int64_t chunks = std::max<int64_t>(1, std::min<int64_t>((n_a + 15) / 16, (target + tiles - 1) / tiles - 2));
    P.per_chunk = static_cast<int>((n_a + chunks - 1) / chunks);
    if (P.per_chunk > 64) P.per_chunk = (P.per_chunk + 63) / 64 * 64;
    P.chunks = 2 + (n_a + P.per_chunk - 1) / P.per_chunk;
    return P;
}

// The masks on the device.
struct JoinMasks {
    JoinHamDev dev;
    bool split = false;   // the pairs allow the heavy / light split
    DevBuf all;           // its arrays in one allocation and one copy

    template <int W>
    hipError_t upload(const HostJoin<W>& hj, int n_qubits) {
        dev = JoinHamDev{};
        split = false;
        if (!hj.ok) return hipSuccess;
        std::vector<unsigned char> host;
        const auto put = [&](const auto& v) {
            const size_t at = (host.size() + 255) / 256 * 256, bytes = v.size() * sizeof(v[0]);
            host.resize(at + bytes);
            if (bytes) std::memcpy(host.data() + at, v.data(), bytes);
            return at;
        };
        const auto size = [](const auto& v) { return v.size() * sizeof(v[0]) + 256; };
        hipError_t e = hipSuccess;
        size_t at[20];
        try {
            size_t own_bytes = 0;
            for (const auto& own : hj.own)
                own_bytes += size(own.masks) + size(own.groups) + size(own.place) + size(own.sign);
            host.reserve(size(hj.alist) + size(hj.amask) + size(hj.blist) + size(hj.bmask) + size(hj.b_cross) +
                         size(hj.b_own) + size(hj.a_own) + size(hj.place) + size(hj.sign) + size(hj.linear) +
                         size(hj.runs) + size(hj.gids) + own_bytes);
            at[0] = put(hj.alist);
            at[1] = put(hj.amask);
            at[2] = put(hj.blist);
            at[3] = put(hj.bmask);
            at[4] = put(hj.b_cross);
            at[5] = put(hj.b_own);
            at[6] = put(hj.a_own);
            at[7] = put(hj.place);
            at[8] = put(hj.sign);
            at[9] = put(hj.linear);
            at[10] = put(hj.runs);
            at[11] = put(hj.gids);
            for (int o = 0; o < 2; ++o) {
                at[12 + 4 * o] = put(hj.own[o].masks);
                at[13 + 4 * o] = put(hj.own[o].groups);
                at[14 + 4 * o] = put(hj.own[o].place);
                at[15 + 4 * o] = put(hj.own[o].sign);
            }
            e = all.ensure(host.size());
        } catch (const std::bad_alloc&) {
            return hipSuccess;   // the loops serve
        }
        if (e == hipErrorOutOfMemory) {   // the loops serve
            (void)hipGetLastError();
            return hipSuccess;
        }
        if (e == hipSuccess) e = hipMemcpy(all.p, host.data(), host.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return e;
        const auto part = [&](int k) -> void* { return all.as<unsigned char>() + at[k]; };
        JoinHamDev H;
        H.ok = true;
        H.n_a = static_cast<int>(hj.alist.size());
        H.alist = part(0);
        H.amask = static_cast<const JoinMask*>(part(1));
        H.n_b = static_cast<int>(hj.blist.size());
        H.blist = part(2);
        H.bmask = static_cast<const JoinMask*>(part(3));
        H.direct = hj.direct;
        H.stride = hj.stride;
        H.b_cross = part(4);
        H.b_own = part(5);
        H.a_own = part(6);
        H.b_cross_bits = bits_for(hj.b_cross.size() - 1);
        H.b_own_bits = bits_for(hj.b_own.size() - 1);
        H.a_own_bits = bits_for(hj.a_own.size() - 1);
        H.place = part(7);
        H.string_bits = join_string_bits(n_qubits);
        H.sign = static_cast<const double*>(part(8));
        H.linear = static_cast<const double*>(part(9));
        H.runs = static_cast<const JoinRun*>(part(10));
        H.gids = static_cast<const int32_t*>(part(11));
        H.places = static_cast<uint32_t>(hj.place.size());
        H.cross = hj.cross;
        H.nibbles = hj.nibbles;
        H.a_base = hj.a_base;
        H.a_pmin = hj.a_pmin;
        H.a_span = hj.a_span;
        H.has_a_own = hj.a_base < hj.place.size();
        for (int o = 0; o < 2; ++o) {
            H.own[o].n = static_cast<int>(hj.own[o].masks.size());
            H.own[o].masks = part(12 + 4 * o);
            H.own[o].groups = part(13 + 4 * o);
            H.own[o].place = part(14 + 4 * o);
            H.own[o].sign = static_cast<const double*>(part(15 + 4 * o));
        }
        split = join_splits(n_qubits, H, hj.cross_span);
        dev = H;
        return hipSuccess;
    }
    void release() { all.release(); }
};

// U in two sorted orders: the buffers (with their own sort scratch) and the
// index built in them.
struct JoinIndex {
    JoinDev dev;
    DevBuf key, val, key2, val2, hist, hist_off, hist_scan;
    DevBuf perm, group, scan, cross, vec, slots, heavy, heavy_slots, core, filter;
    int64_t filter_words = 0;

    // Room for n samples; nothing is allocated when the index is built.
    hipError_t room(int W, int64_t n, const JoinMasks& masks) {
        const size_t st = W == 1 ? sizeof(uint32_t) : sizeof(uint64_t);
        const int64_t tiles = radix_tiles(2 * n);
        hipError_t e = hipSuccess;
        const auto need = [&](DevBuf& b, size_t bytes) {
            if (e == hipSuccess) e = b.ensure(bytes);
        };
        need(key, sizeof(uint64_t) * 2 * n);
        need(key2, sizeof(uint64_t) * 2 * n);
        need(val, sizeof(uint32_t) * 2 * n);
        need(val2, sizeof(uint32_t) * 2 * n);
        need(hist, sizeof(uint32_t) * 256 * tiles);
        need(hist_off, sizeof(int64_t) * (256 * tiles + 1));
        need(hist_scan, sizeof(int64_t) * scan_scratch_len(256 * tiles));
        need(perm, sizeof(int32_t) * 2 * n);
        need(group, st * 2 * n);
        need(scan, st * 2 * n);
        need(vec, sizeof(double2) * 2 * n);
        need(slots, sizeof(JoinBucket) * (size_t(2) << join_bucket_bits(n)));
        need(cross, st * n);
        need(heavy, sizeof(JoinHeavy));
        need(heavy_slots, 2 * st * 2 * kJoinHeavySlots);
        need(core, sizeof(uint32_t) * kJoinCore);
        filter_words = join_filter_words(masks.dev, n);
        if (filter_words) need(filter, sizeof(uint32_t) * filter_words);
        return e;
    }
    // The index of keys[n][W]; enqueued.
    hipError_t build(int W, const uint64_t* keys, int64_t n, int n_qubits, const JoinMasks& masks,
                     const uint32_t* prep_err, hipStream_t st) {
        JoinBuild B;
        B.keys = keys;
        B.M = n;
        B.n_qubits = n_qubits;
        B.split = masks.split;
        for (int o = 0; o < 2; ++o) B.own_limit[o] = join_own_limit(masks.dev.own[o].n);
        B.filter = filter_words ? filter.as<uint32_t>() : nullptr;
        B.filter_words = filter_words;
        B.key = key.as<uint64_t>();
        B.key2 = key2.as<uint64_t>();
        B.val = val.as<uint32_t>();
        B.val2 = val2.as<uint32_t>();
        B.hist = hist.as<uint32_t>();
        B.hist_off = hist_off.as<int64_t>();
        B.hist_scan = hist_scan.as<int64_t>();
        B.perm = perm.as<int32_t>();
        B.group = group.p;
        B.scan = scan.p;
        B.cross = cross.p;
        B.slots = slots.as<JoinBucket>();
        B.bits = join_bucket_bits(n);
        B.heavy = heavy.as<JoinHeavy>();
        B.heavy_slots = heavy_slots.p;
        B.core = core.as<uint32_t>();
        const hipError_t e = launch_join_index(W, B, st);
        if (e != hipSuccess) return e;
        JoinDev J;
        J.M = n;
        J.perm = B.perm;
        J.group = B.group;
        J.scan = B.scan;
        J.cross = B.cross;
        J.vec = vec.as<double2>();
        J.keys = B.keys;
        J.slots = B.slots;
        J.bits = B.bits;
        J.heavy = B.heavy;
        J.heavy_slots = B.heavy_slots;
        J.core = B.core;
        J.filter = B.filter;
        J.filter_mask = static_cast<uint32_t>(filter_words - 1);
        J.prep_err = prep_err;
        dev = J;
        return hipSuccess;
    }
    void release() {
        for (DevBuf* b : {&key, &val, &key2, &val2, &hist, &hist_off, &hist_scan, &perm, &group, &scan, &cross, &vec, &slots,
                          &heavy, &heavy_slots, &core, &filter})
            b->release();
    }
};

}  // namespace eloc
