// Enumeration of the sector's members in a range of candidates, with jumps
// over the candidates that a rejection rules out together (Section 5.2 tests
// every candidate).
//
// A candidate s is a member iff no group image is smaller and every element
// fixing s has character 1.  Let an image v = g(s) be smaller than s, and d
// the highest bit where they differ.  The comparison reads only the bits of
// s at d and above and the bits that g moves to d and above.  With m the
// lowest of all these positions, every candidate that agrees with s on the
// bits m and above has the same smaller image, so the walk goes on at the
// first candidate whose bits m and above are larger.  Near the bottom of the
// order, where most members are, m is small; above, one test rules out
// millions of candidates (the prefix pruning of necklace generation, here
// for any group).  Bound by the VALU, and by lanes waiting for the busiest of
// their wavefront.  Counting 3.4e10 candidates of the 40-spin chain: 351 ms
// testing each, 20 ms with the jumps; the 6x6 sector's build 82 ms then, 11 now.
#pragma once

#include "orbit.hpp"

namespace ls {

template <typename W>
__device__ __forceinline__ uint32_t top_bit(W v) {
    if constexpr (sizeof(W) == 4) return 31u - static_cast<uint32_t>(__builtin_clz(static_cast<uint32_t>(v)));
    else return 63u - static_cast<uint32_t>(__builtin_clzll(static_cast<uint64_t>(v)));
}

template <typename W>
__device__ __forceinline__ uint32_t pop_count(W v) {
    if constexpr (sizeof(W) == 4) return static_cast<uint32_t>(__builtin_popcount(static_cast<uint32_t>(v)));
    else return static_cast<uint32_t>(__builtin_popcountll(static_cast<uint64_t>(v)));
}

template <typename W>
__device__ __forceinline__ W next_combination(W x) {
    const W c = x & (~x + 1);
    const W r = x + c;
    const int z = sizeof(W) == 4 ? __builtin_ctz(static_cast<uint32_t>(x))
                                 : __builtin_ctzll(static_cast<uint64_t>(x));
    return (((r ^ x) >> 2) >> z) | r;
}

// The candidates of one lane: from the first one up to, not including, the
// 64-bit value `end`; `last` is the greatest candidate of the whole sector.
template <typename W>
struct CandRange {
    uint64_t end;
    W last;
    bool gosper;     // fixed weight: the candidates are the weight-w words

    // Moves s past every candidate that agrees with it on the bits m and
    // above; false when the range ends there.  s grows with every call.
    __device__ __forceinline__ bool skip(W &s, uint32_t m) const {
        const W low = (static_cast<W>(1) << m) - 1;
        W top;       // the greatest candidate with these high bits
        if (gosper) {
            const uint32_t c = pop_count<W>(s & low);
            top = (s & ~low) | (low & ~((static_cast<W>(1) << (m - c)) - 1));
        } else {
            top = s | low;
        }
        if (top >= last) return false;
        s = gosper ? next_combination<W>(top) : static_cast<W>(top + 1);
        return static_cast<uint64_t>(s) < end;
    }
};

// Any group: one iteration tests one image (with its spin-flipped partner) of
// the lane's current candidate, and a lane goes on as soon as its candidate is
// decided, so a wavefront runs at the pace of its slowest lane's total and not
// of the slowest candidate at every step.  Images in the order coset, y-shift,
// x-shift; P.skip gives m by (image, d).  hit(s, stabilizer size) is called
// for every member, in increasing order.
template <typename W, typename Hit>
__device__ __forceinline__ void walk_images(const PlanDev &P, W s, const CandRange<W> &R, Hit &&hit) {
    const W full = static_cast<W>(P.full);
    const bool pf = P.pair_flip != 0;
    const uint32_t nz = pf ? 2u : 1u;
    const uint32_t n = P.n_sites, lx = P.lx, ly = P.ly, nc = P.n_cosets;
    uint32_t a = 0, b = 0, p = 0, img = 0, stab = 0;
    W ub = s, v = s;   // cosets[0] is the identity
    for (;;) {
        const W vf = static_cast<W>(v ^ full);
        const W lo = pf ? min(v, vf) : v;
        const bool less = lo < s;
        const W diff = lo ^ s;
        bool out = less;
        if (lo == s) {
            const uint32_t code = img * nz + (v == s ? 0u : 1u);
            ++stab;
            out = !chi_is_one(P, code);
        }
        const uint32_t here = img;
        bool end = false;
        ++img;
        if (++a < lx) {
            v = xrot<W>(v, P);
        } else {
            a = 0;
            if (++b < ly) {
                ub = yrot<W>(ub, P);
                v = ub;
            } else {
                b = 0;
                if (++p < nc) {
                    ub = apply_coset<W>(P.cosets[p], s, P);
                    v = ub;
                } else {
                    end = true;
                }
            }
        }
        if (out || end) {
            if (!out) hit(s, stab);
            const uint32_t m = less ? P.skip[here * n + top_bit<W>(diff)] : 0u;
            if (!R.skip(s, m)) break;
            a = b = p = img = stab = 0;
            ub = v = s;
        }
    }
}

// Rings (all rotations, with or without the reversal; ring_walk): the smallest
// rotation puts one of the longest zero runs on top, with spin inversion one
// of the longest zero or one runs.  With L leading zeros, a run of L + 1
// zeros (or ones) anywhere rejects s; among the words that pass, only the
// rotations that lift another run of exactly L are compared, forward and
// reversed.  An iteration takes the windows of a new candidate and then one
// run.  m: a run starting at bit i is read from bit i up; the rotation by k
// reads bit j - k for bit j, so d - k when d >= k (else it wraps and reads
// bit 0); the reversed rotation by k reads bits n-1-j+k, so k when d >= k.
template <typename W, typename Hit>
__device__ __forceinline__ void walk_ring(const PlanDev &P, W s, const CandRange<W> &R, Hit &&hit) {
    const uint32_t n = P.n_sites;
    const W full = static_cast<W>(P.full);
    const bool pf = P.pair_flip != 0, mirror = P.n_cosets == 2;
    const uint32_t nz = pf ? 2u : 1u;
    // rotation of the low n bits left by k < n
    auto rotl = [&](W w, uint32_t k) -> W {
        return static_cast<W>(((w << k) | ((w >> 1) >> (n - 1 - k))) & full);
    };
    auto reversed = [&](W w) -> W { return bit_reverse<W>(w, n); };
    W zs = 0, os = 0;        // runs of the current candidate still to compare
    uint32_t L = 0, stab = 0;
    bool fresh = true;
    for (;;) {
        uint32_t m = 0;
        bool out = false, done = false;
        if (fresh) {
            stab = 0;
            os = 0;
            if (s == 0 || s == full) {
                // every rotation and reversal is s; of all ones, the flip is smaller
                zs = 0;
                const uint32_t rot = n * (mirror ? 2u : 1u);
                if (s == full && pf) {
                    out = true;
                } else {
                    for (uint32_t c = 0; c < rot; ++c)
                        if (!chi_is_one(P, c * nz)) out = true;
                    stab = rot;
                }
                done = true;
            } else {
                L = n - 1 - top_bit<W>(s);
                W z = ~s & full, o = pf ? s : static_cast<W>(0);
                uint32_t len = 1;
                while (len < L) {
                    const uint32_t st = min(len, L - len);
                    z &= z >> st;
                    o &= o >> st;
                    len += st;
                }
                // windows of L + 1 (L = 0: single zeros and ones)
                const W zv = L == 0 ? z : static_cast<W>(z & (z >> 1));
                const W ov = L == 0 ? o : static_cast<W>(o & (o >> 1));
                const W bad = zv | ov;
                if (bad) {
                    out = true;
                    m = top_bit<W>(bad);
                } else if ((s & 1) == 0) {
                    out = true;      // the top run goes on at bit 0
                } else {
                    zs = z;
                    os = o;
                }
            }
        }
        if (!out && !done) {
            // the highest run left: its rotation, and the reversed one
            const bool one = os > zs;
            W &set = one ? os : zs;
            const uint32_t i = top_bit<W>(set);
            set ^= static_cast<W>(1) << i;
            const W w = one ? static_cast<W>(s ^ full) : s;
            const uint32_t k = n - i - L;          // <= n - 1 (L >= 1); 0 for the top run itself
            const W v = rotl(w, k);
            const W u = mirror ? rotl(reversed(w), i) : full;
            const uint32_t f = one ? 1u : 0u;
            if (v < s) {
                const uint32_t d = top_bit<W>(static_cast<W>(v ^ s));
                out = true;
                m = d >= k ? d - k : 0u;
            }
            if (u < s) {
                const uint32_t d = top_bit<W>(static_cast<W>(u ^ s));
                out = true;
                m = max(m, d >= i ? i : 0u);
            }
            if (v == s) {
                ++stab;
                if (!chi_is_one(P, k * nz + f)) out = true;
            }
            if (mirror && u == s) {
                ++stab;
                if (!chi_is_one(P, (n + i) * nz + f)) out = true;
            }
            done = (zs | os) == 0;
        }
        fresh = out || done;
        if (fresh) {
            if (!out) hit(s, stab);
            if (!R.skip(s, m)) break;
        }
    }
}

// Tori with a pair table (lx = 3..6, ly >= 2): the top two rows of the smallest
// image are the smallest pair of rows over every base image, y-shift, flip
// and row operation, and the pair table gives the smallest value of a pair.
// An iteration takes one base image of the lane's candidate: ly table reads
// decide all its images (a smaller pair rejects, with the m of the two rows
// it is made of; the largest m of the base's smaller pairs is taken), and only
// the images that equal s in the top two rows are formed and compared.
template <typename W, typename Hit>
__device__ __forceinline__ void walk_torus(const PlanDev &P, W s, const CandRange<W> &R, Hit &&hit) {
    const W full = static_cast<W>(P.full);
    const uint32_t n = P.n_sites, L = P.lx, ly = P.ly, nt = P.n_trans;
    const uint32_t nz = P.pair_flip ? 2u : 1u;
    const uint32_t low = n - 2 * L;                    // bits below the top two rows
    uint32_t p = 0, stab = 0;
    for (;;) {
        const W u = p == 0 ? s : apply_coset<W>(P.bases[p], s, P);
        const uint32_t own = static_cast<uint32_t>(s >> low);
        const uint32_t coset = P.op_code[p * 4] & 0xFFu;
        uint32_t m = 0;
        bool out = false;
        uint64_t tie = 0, tief = 0;                    // y-shifts: plain, flipped
        W v = u;
        for (uint32_t b = 0; b < ly; ++b) {
            const uint32_t e = P.pair_lut[static_cast<uint32_t>(v >> low)];
            const uint32_t k0 = e & 0xFFFFu, k1 = nz == 2 ? e >> 16 : ~0u;
            if (min(k0, k1) < own) {
                out = true;
                m = max(m, static_cast<uint32_t>(P.skip[(coset * nt + L * b) * n + low]));
            }
            tie |= (k0 == own ? 1ull : 0ull) << b;
            tief |= (k1 == own ? 1ull : 0ull) << b;
            v = yrot<W>(v, P);
        }
        if (out) tie = tief = 0;
        while (tie | tief) {
            const uint32_t f = tie ? 0u : 1u;
            uint64_t &set = tie ? tie : tief;
            const uint32_t b = static_cast<uint32_t>(__builtin_ctzll(set));
            set &= set - 1;
            W c = u;
            if (b) c = ((c << (L * b)) | (c >> (n - L * b))) & full;
            if (f) c ^= full;
            uint32_t am = P.pair_arg[static_cast<uint32_t>(c >> low)];
            W cr = 0;                                  // the rows' bits reversed
            for (uint32_t x = 0; x < L; ++x) cr |= ((c >> x) & static_cast<W>(P.col0)) << (L - 1 - x);
            while (am) {
                const uint32_t j = static_cast<uint32_t>(__builtin_ctz(am));
                am &= am - 1;
                const uint32_t o = j >> 3, a = j & 7u;
                W z = (o == 1 || o == 2) ? cr : c;
                if (o >= 2) {
                    // reversed, and the pair (now at the bottom) rotated to the top
                    z = bit_reverse<W>(z, n);
                    if (ly > 2) z = ((z << low) | (z >> (n - low))) & full;
                }
                if ((P.op_flips >> o) & 1u) z ^= full;
                const W ma = static_cast<W>(P.col_ge[a]);
                z = ((z << a) & ma) | ((z >> (L - a)) & ~ma & full);
                if (z > s) continue;
                const uint32_t oc = P.op_code[p * 4 + o];
                uint32_t x = ((oc >> 8) & 0xFFu) + a, y = ((oc >> 16) & 0xFFu) + (o >= 2 ? 2 * ly - 2 - b : b);
                if (x >= L) x -= L;
                while (y >= ly) y -= ly;
                const uint32_t img = (oc & 0xFFu) * nt + x + L * y;
                if (z < s) {
                    out = true;
                    m = max(m, static_cast<uint32_t>(P.skip[img * n + top_bit<W>(static_cast<W>(z ^ s))]));
                } else {
                    ++stab;
                    if (!chi_is_one(P, img * nz + (f ^ (oc >> 24)))) out = true;
                }
            }
        }
        if (out || ++p >= P.n_base) {
            if (!out) hit(s, stab);
            if (!R.skip(s, m)) break;
            p = stab = 0;
        }
    }
}

// Rings that walk_ring takes: translations of a ring, alone or with the plain
// reversal (the group's split then holds no other coset).
inline bool ring_walk(const GroupPlan &p) {
    return p.ly == 1 && p.lx == p.n_sites && p.n_sites > 1 &&
           (p.cosets.size() == 1 ||
            (p.cosets.size() == 2 && p.cosets[1].kind == kCosetReverse && p.cosets[1].flip == 0));
}

// The walk of a group's enumeration.
enum WalkKind : int { kWalkImages = 0, kWalkRing = 1, kWalkTorus = 2 };
inline int walk_kind(const GroupPlan &p) {
    return ring_walk(p) ? kWalkRing : p.row_tables ? kWalkTorus : kWalkImages;
}

}  // namespace ls
