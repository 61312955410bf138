// Device helpers: group action, orbit search and stateToIndex.
//
// Every lane owns one basis state.  The general walk visits the whole group in
// registers: for each coset representative p (identity, full bit reversal or a
// Benes network of delta swaps), the translated images tau_t(p(s)) are produced
// by shifts (x-rotation of every row, rotation of the word by one row), and
// with spin inversion in the group each image v is paired with v ^ full.  The
// representative is the minimum image (the orbit minimum).  Rings and tori find
// it from a few images (ring_fold, torus_orbit_min).
#pragma once

#include <type_traits>

#include "ls_internal.hpp"

namespace ls {

// Memory that no kernel writes while it is read this way: at an index that is
// the same in all lanes, the reads are scalar loads.
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ ConstPtr<T> as_const(const T *p) {
    return (ConstPtr<T>)p;
}

// Structure kinds the kernels are specialised for.
enum OrbitKind : int {
    kOrbitGeneric = 0,   // runtime lx, ly (ring, torus, or no translations)
    kOrbitRing32 = 1,    // N <= 32 ring: all rotations from one funnel shift each
    kOrbitTorus = 2,     // lx = 3..6, ly >= 2 torus: pruned by the pair table (torus_orbit_min)
    kOrbitRing64 = 3,    // 32 < N < 64 ring whose words' longest runs show in 64 bits when doubled
    kOrbitRing64T = 4,   // other 32 < N < 64 rings: the words are turned (ring_fold)
};

// A value that is the same in every active lane, moved to a scalar register.
// Loop counters of the group walk are uniform, but the walk runs inside
// each lane's own element loop, where the compiler cannot prove it; scalar
// counters keep coset masks in scalar loads and index arithmetic off the
// vector ALU.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

template <typename W>
__device__ __forceinline__ W benes_apply(W x, const uint64_t *m) {
    if constexpr (sizeof(W) == 4) {
        constexpr int dl[9] = {16, 8, 4, 2, 1, 2, 4, 8, 16};
#pragma unroll
        for (int s = 0; s < 9; ++s) {
            const W t = ((x >> dl[s]) ^ x) & static_cast<W>(m[s]);
            x ^= t ^ (t << dl[s]);
        }
    } else {
        constexpr int dl[11] = {32, 16, 8, 4, 2, 1, 2, 4, 8, 16, 32};
#pragma unroll
        for (int s = 0; s < 11; ++s) {
            const W t = ((x >> dl[s]) ^ x) & static_cast<W>(m[s]);
            x ^= t ^ (t << dl[s]);
        }
    }
    return x;
}

template <typename W>
__device__ __forceinline__ W bit_reverse(W x, uint32_t n) {
    if constexpr (sizeof(W) == 4)
        return static_cast<W>(__builtin_bitreverse32(static_cast<uint32_t>(x)) >> (32u - n));
    else
        return static_cast<W>(__builtin_bitreverse64(static_cast<uint64_t>(x)) >> (64u - n));
}

template <typename W>
__device__ __forceinline__ W apply_coset(const CosetRep &c, W s, const PlanDev &P) {
    W u;
    if (c.kind == kCosetIdentity)
        u = s;
    else if (c.kind == kCosetReverse)
        u = bit_reverse<W>(s, P.n_sites);
    else
        u = benes_apply<W>(s, c.masks);
    if (c.flip) u ^= static_cast<W>(P.full);
    return u;
}

// (x, y) -> (x + 1, y) for every row of an lx-wide layout
template <typename W>
__device__ __forceinline__ W xrot(W v, const PlanDev &P) {
    const W c0 = static_cast<W>(P.col0), full = static_cast<W>(P.full);
    return ((v << 1) & ~c0 & full) | ((v >> (P.lx - 1)) & c0);
}

// (x, y) -> (x, y + 1): rotate the N-bit word by one row
template <typename W>
__device__ __forceinline__ W yrot(W v, const PlanDev &P) {
    return ((v << P.lx) | (v >> (P.n_sites - P.lx))) & static_cast<W>(P.full);
}

__device__ __forceinline__ bool chi_is_one(const PlanDev &P, uint32_t code) {
    return (P.chi_one[code >> 5] >> (code & 31)) & 1u;
}

// Visit every group image of s: f(v, code).  Returning false from f stops.
template <typename W, int KIND, typename F>
__device__ __forceinline__ void for_each_image(const PlanDev &P, W s, F &&f) {
    const uint32_t nz = P.pair_flip ? 2u : 1u;
    const W full = static_cast<W>(P.full);
    for (uint32_t p0 = 0; p0 < P.n_cosets; ++p0) {
        const uint32_t p = uni(p0);
        const CosetRep c = P.cosets[p];
        W u = apply_coset<W>(c, s, P);
        if constexpr (KIND == kOrbitRing32) {
            // u doubled into 64 bits: rotating right by t is one funnel shift
            const uint32_t n = P.n_sites;
            const uint64_t uu = static_cast<uint64_t>(u) | (static_cast<uint64_t>(u) << n);
            const uint32_t lo = static_cast<uint32_t>(uu), hi = static_cast<uint32_t>(uu >> 32);
            for (uint32_t t0 = 0; t0 < n; ++t0) {
                const uint32_t t = uni(t0);
                const W v = static_cast<W>(__builtin_amdgcn_alignbit(hi, lo, t)) & full;
                // right rotation by t is the translation a = (n - t) mod n
                const uint32_t a = t == 0 ? 0u : n - t;
                const uint32_t base = uni((p * n + a) * nz);
                if (!f(v, base)) return;
                if (P.pair_flip && !f(static_cast<W>(v ^ full), base + 1)) return;
            }
        } else {
            for (uint32_t b = 0; b < P.ly; ++b) {
                W v = u;
                for (uint32_t a = 0; a < P.lx; ++a) {
                    const uint32_t base = uni((p * P.n_trans + a + P.lx * b) * nz);
                    if (!f(v, base)) return;
                    if (P.pair_flip && !f(static_cast<W>(v ^ full), base + 1)) return;
                    if (a + 1 < P.lx) v = xrot<W>(v, P);
                }
                if (b + 1 < P.ly) u = yrot<W>(u, P);
            }
        }
    }
}

// What a search found beside the smallest image: with TRACK the code of an
// element reaching it, with COUNT how many images equal it (the stabilizer
// size of the orbit's states) and whether two elements that reach it have
// characters that differ (the projector annihilates the orbit).
struct OrbitInfo {
    uint32_t code = 0, count = 0;
    bool mixed = false;
};

// Notes the image v of the element with code `code` (given as a function): the
// smallest so far, and with COUNT how many are equal to it, the smallest of
// their codes, and whether their characters differ (of trivial characters
// only how many).
template <bool TRACK, bool COUNT, typename W, typename Code>
__device__ __forceinline__ void fold_image(const PlanDev &P, W v, Code &&code, W &best, OrbitInfo &info) {
    const bool chars = TRACK && !(COUNT && P.chi_trivial);
    if constexpr (COUNT) {
        if (v == best && info.count) {
            ++info.count;
            if (chars) {
                const uint32_t c = code();
                const double2 c0 = P.chi[info.code], c1 = P.chi[c];
                info.mixed = info.mixed || fabs(c0.x - c1.x) + fabs(c0.y - c1.y) > 1e-6;
                info.code = min(info.code, c);
            }
        }
    }
    if (v < best || (COUNT && info.count == 0)) {
        best = v;
        if (chars) info.code = code();
        if constexpr (COUNT) {
            info.count = 1;
            info.mixed = false;
        }
    }
}

// Folds the rotations of the ring word w (n <= 32, or 32 < n < 64 in 64 bits)
// that can be the orbit's smallest into `best`; with `mirror` also those of
// the reversed word, with spin inversion also of the flipped ones.  The
// smallest image has the longest zero run on top.  With spin inversion the
// runs of equal spins are the zero runs of the boundaries w ^ (w >> 1), so
// one search finds the zero and the one runs: doubled windows, then binary
// lifting of the length.  For a run starting at bit i, the rotation y of the
// (flipped) word that brings it to the bottom gives both images: y >> length
// has the run on top, and so has y reversed.  Code of rotating left by k:
// code0 + k * |Z| + flip, mirrored mcode0 + i * |Z| + flip.
// Windows that wrap are plain shifts of the doubled word, which holds them as
// far as 64 bits go.  Where the sector has longer runs (ring_turns), the word is
// turned instead so that no run wraps (TURN).
// About 45 instructions and 15 to 25 a run, where 32 sites took 4 for each of
// 128 images (32-site ring product 1.34 ms) and more sites 118 for each of the
// zero and the one runs (38-spin chain 75 ms, VALU busy all the time).
// Constant words: every rotation is the word (false with COUNT: the caller
// counts every image).
template <typename W, bool TRACK, bool COUNT, bool TURN>
__device__ __forceinline__ bool ring_fold(const PlanDev &P, W w, bool mirror, uint32_t code0, uint32_t mcode0, W &best,
                                          OrbitInfo &info) {
    constexpr bool SMALL = sizeof(W) == 4;
    const uint32_t n = P.n_sites, pf = P.pair_flip ? 1u : 0u, nz = 1u + pf;
    const W full = static_cast<W>(P.full);
    uint32_t turn = 0;       // bit i of the turned word is bit i + turn (mod n) of the word
    if constexpr (TURN) {
        // (the last bit of a constant word that is looked at stays its own)
        const W edges = static_cast<W>((w ^ (w >> 1)) | static_cast<W>(1) << (n - 2));
        turn = static_cast<uint32_t>(__builtin_ctzll(static_cast<uint64_t>(edges))) + 1;
        w = ((w >> turn) | (w << (n - turn))) & full;
    }
    uint64_t ext = static_cast<uint64_t>(w);
    if constexpr (!TURN) ext |= static_cast<uint64_t>(w) << (SMALL ? n : n & 63u);
    const uint32_t seen = (SMALL ? 2 * n : TURN ? n : 64u) - pf;      // bits of z that tell
    const uint64_t z = ~(pf ? ext ^ (ext >> 1) : ext) & (~0ull >> (64 - seen));
    const uint64_t z2 = z & (z >> 1), z4 = z2 & (z2 >> 2), z8 = z4 & (z4 >> 4);
    uint64_t cur = z;
    uint32_t len = 1;
    auto lift = [&](uint64_t zl, uint32_t l) {
        const uint64_t t = cur & (zl >> len);
        if (t != 0) {
            cur = t;
            len += l;
        }
    };
    if constexpr (TURN) {
        const uint64_t z16 = z8 & (z8 >> 8);
        lift(z16 & (z16 >> 16), 32);
        lift(z16, 16);
    }
    lift(z8, 8);
    lift(z4, 4);
    lift(z2, 2);
    lift(z, 1);
    if (z == 0) {                                          // no two equal neighbours
        cur = P.full;
        len = 0;
    } else if (!TURN && len == 16) {
        while (len < n && (cur & (z >> len)) != 0) {
            cur &= z >> len;
            ++len;
        }
    }
    if (w == 0 || w == full) {
        if constexpr (!COUNT) {
            fold_image<TRACK, COUNT>(P, w, [&] { return code0; }, best, info);
            if (pf) fold_image<TRACK, COUNT>(P, static_cast<W>(w ^ full), [&] { return code0 + 1; }, best, info);
        }
        return !COUNT;
    }
    const uint32_t run = len + pf;
    W starts = static_cast<W>(cur) & full;
    while (starts) {
        const uint32_t i = SMALL ? static_cast<uint32_t>(__builtin_ctz(static_cast<uint32_t>(starts)))
                                 : static_cast<uint32_t>(__builtin_ctzll(static_cast<uint64_t>(starts)));
        starts &= starts - 1;
        const uint32_t f = pf ? static_cast<uint32_t>(w >> i) & 1u : 0u;
        W y;
        if constexpr (SMALL) {
            y = static_cast<W>((f ? ~ext : ext) >> i) & full;
        } else {
            const W wf = f ? w ^ full : w;
            y = ((wf >> i) | (wf << (n - i))) & full;
        }
        const uint32_t at = !TURN || i + turn < n ? i + turn : i + turn - n;      // the run's start in the word
        fold_image<TRACK, COUNT>(P, static_cast<W>(y >> run), [&] {
            const uint32_t k = 2 * n - at - run;
            return code0 + (k >= n ? k - n : k) * nz + f;
        }, best, info);
        if (mirror) {
            fold_image<TRACK, COUNT>(P, bit_reverse<W>(y, n), [&] { return mcode0 + at * nz + f; }, best, info);
        }
    }
    return true;
}

// The orbit minimum of a ring word by ring_fold over the cosets (the plain
// reversal folded into the identity's); false: a constant word with COUNT.
template <typename W, bool TRACK, bool COUNT, bool TURN>
__device__ __forceinline__ bool ring_orbit_min(const PlanDev &P, W s, W &best, OrbitInfo &info) {
    const uint32_t nz = P.pair_flip ? 2u : 1u, per = P.n_sites * nz;
    if (P.n_cosets == 2 && P.cosets[1].kind == kCosetReverse && P.cosets[1].flip == 0)
        return ring_fold<W, TRACK, COUNT, TURN>(P, s, true, 0, per, best, info);
    for (uint32_t p0 = 0; p0 < P.n_cosets; ++p0) {
        const uint32_t p = uni(p0);
        const W u = p == 0 ? s : apply_coset<W>(P.cosets[p], s, P);
        if (!ring_fold<W, TRACK, COUNT, TURN>(P, u, false, p * per, 0, best, info)) return false;
    }
    return true;
}

// Orbit minimum; with TRACK also the code of an element reaching it.
template <typename W, int KIND, bool TRACK>
__device__ __forceinline__ W orbit_min(const PlanDev &P, W s, uint32_t &code) {
    if constexpr (KIND == kOrbitRing32 || KIND == kOrbitRing64 || KIND == kOrbitRing64T) {
        OrbitInfo info;
        W least = static_cast<W>(~static_cast<W>(0));
        (void)ring_orbit_min<W, TRACK, false, KIND == kOrbitRing64T>(P, s, least, info);
        code = info.code;
        return least;
    } else {
        code = 0;
        if (P.n_elements == 1) return s;
        W best = s;
        uint32_t arg = 0;
        for_each_image<W, KIND>(P, s, [&](W v, uint32_t c) {
            if constexpr (TRACK) {
                if (v < best) { best = v; arg = c; }
            } else {
                best = v < best ? v : best;
            }
            return true;
        });
        code = arg;
        return best;
    }
}

// Byte offset of the 4-byte table entry of the top two rows of tau_{0,b}(u),
// rows ly-1-b and ly-2-b (mod ly) of an L-wide word.
template <typename W>
__device__ __forceinline__ uint32_t pair_offset(W u, uint32_t b, uint32_t L, uint32_t ly) {
    // bits [sh, sh + 32) of u shifted up by 2
    auto x4 = [&](uint32_t sh) -> uint32_t {
        return sh >= 2 ? static_cast<uint32_t>(u >> (sh - 2)) : static_cast<uint32_t>(u) << (2 - sh);
    };
    const uint32_t rm = (1u << L) - 1u, m2 = (1u << (2 * L)) - 1u, ty = ly - 1 - b;
    if (ty >= 1) return x4(L * (ty - 1)) & (m2 << 2);
    return ((static_cast<uint32_t>(u) & rm) << (L + 2)) | (x4(L * (ly - 1)) & (rm << 2));
}

// Pruned orbit minimum on an lx-by-ly torus (lx = 3..6, ly >= 2).
//
// The group is row operations (x-shifts, the reversal of the rows' bits, the
// reversal of the rows' order) after y-shifts of a few base images (the
// identity; on square tori a transposition as well).  The base images of a
// neighbour are p(r) ^ pi_p(f), from the row's images p(r) (pr[]) and the flip
// images pi_p(f) (cf[p * cstride]).  Pass 1 reads the pair table for every
// base image p and y-shift b: the entry of two neighbouring rows holds, for
// the pair and for its spin-flipped partner, the smallest value they take as
// top rows over all row operations (the key).  The minimum image has the
// smallest key, so only the (p, b, f) that reach it are looked at further:
// 1.09 of 24 on average in a 6x6 sector, at most 2.3 over a wavefront.  Their
// table `arg` names the operations and x-shifts that reach the key (1.5 images
// in all), and only the rows below the top two are formed and compared, 24
// bits for 6x6.  With a table of x-shifts only the 6x6 search made 48 reads,
// one per coset and y-shift, against 12: the 6x6 product took 30.6 ms, now
// 25.7 (69% of the cycles issue a VALU instruction; 168 GB of L2 misses at 6.5
// TB/s).
// LX, LY, NZ are the layout and |Z| when known at compile time (0: read from
// the plan); the compile-time shapes have two base images and no operation
// that comes with a flip of its own.
//   lut   pair table in LDS: key(q) | key(q ^ all-ones) << 16;
//   arg   bit m * 8 + a for every operation m and x-shift a reaching key(q);
//   lcol  col_ge masks.
constexpr uint32_t kTorusMaxBases = kTorusCosetSlots;

template <typename W, bool TRACK, bool COUNT, uint32_t LX, uint32_t LY, uint32_t NZ, typename FlipPtr>
__device__ __forceinline__ W torus_orbit_min(const PlanDev &P, const W *pr, FlipPtr cf, uint32_t cstride,
                                             const uint32_t *lut, const uint32_t *arg, const uint64_t *lcol,
                                             OrbitInfo &info) {
    // the rows below the top two, in 32 bits where they fit
    constexpr bool SMALL = sizeof(W) == 4 || (LX != 0 && LX * (LY - 2) < 32);
    using T = typename std::conditional<SMALL, uint32_t, uint64_t>::type;
    const uint32_t L = LX ? LX : P.lx, Ly = LY ? LY : P.ly;
    const uint32_t nz = NZ ? NZ : (P.pair_flip ? 2u : 1u);
    const uint32_t nb = LX ? 2u : P.n_base;
    const uint32_t n = LX ? LX * LY : P.n_sites, tb = L * (Ly - 2);
    const W full = static_cast<W>(P.full);
    const T tmask = static_cast<T>((static_cast<uint64_t>(1) << tb) - 1);
    const T col0 = static_cast<T>(P.col0) & tmask;
    using u16x2 = unsigned short __attribute__((ext_vector_type(2)));
    auto entry = [&](W u, uint32_t b) -> uint32_t {
        return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const unsigned char *>(lut) +
                                                   pair_offset<W>(u, b, L, Ly));
    };
    T tail = static_cast<T>(~static_cast<T>(0));
    uint32_t won = 0;    // base << 16 | y-shift << 8 | flip << 7 | operation << 3 | x-shift
    auto code_of = [&](uint32_t w) -> uint32_t {
        const uint32_t i = w >> 16, b = (w >> 8) & 0xFFu, f = (w >> 7) & 1u, m = (w >> 3) & 3u, a = w & 7u;
        const uint32_t c = P.op_code[i * 4 + m];
        uint32_t x = ((c >> 8) & 0xFFu) + a, y = ((c >> 16) & 0xFFu) + (m >= 2 ? 2 * Ly - 2 - b : b);
        if (x >= L) x -= L;
        while (y >= Ly) y -= Ly;
        return ((c & 0xFFu) * P.n_trans + x + L * y) * nz + (f ^ (c >> 24));
    };
    // the images of base image u, y-shift b and flip f that reach the key
    auto visit = [&](W u, uint32_t i, uint32_t b, uint32_t f) {
        W v = u;
        if (LX || b) v = ((v << (L * b)) | (v >> (n - L * b))) & full;
        if (f) v ^= full;
        uint32_t am = arg[static_cast<uint32_t>(v >> tb)];
        const T t = static_cast<T>(v) & tmask;
        T tr = 0;        // the rows' bits reversed (bases that are all the cosets: no operation reverses)
        if (LX || nb != P.n_cosets) {
#pragma unroll
            for (uint32_t x = 0; x < 6; ++x)
                if (x < L) tr |= ((t >> x) & col0) << (L - 1 - x);
        }
        while (am) {
            const uint32_t j = static_cast<uint32_t>(__builtin_ctz(am));
            am &= am - 1;
            const uint32_t m = j >> 3, a = j & 7u;
            // operation 3 reverses all bits, 2 is 3 after 1
            T z = (m == 1 || m == 2) ? tr : t;
            if (m >= 2) {
                if constexpr (SMALL) z = tb ? __builtin_bitreverse32(z) >> ((32 - tb) & 31) : 0;
                else z = tb ? __builtin_bitreverse64(z) >> ((64 - tb) & 63) : 0;
            }
            if (LX == 0 && ((P.op_flips >> m) & 1u)) z ^= tmask;
            const T ma = static_cast<T>(lcol[a]);
            z = ((z << a) & ma & tmask) | ((z >> (L - a)) & ~ma);
            const uint32_t w = i << 16 | b << 8 | f << 7 | j;
            if constexpr (COUNT) {
                fold_image<true, true>(P, z, [&] { return code_of(w); }, tail, info);
            } else if (z < tail) {
                tail = z;
                if constexpr (TRACK) won = w;
            }
        }
    };
    uint32_t best;
    if constexpr (LX != 0) {
        W u[2];
        uint32_t e[2 * LY];
#pragma unroll
        for (uint32_t i = 0; i < 2; ++i) {
            u[i] = pr[i] ^ static_cast<W>(cf[i * cstride]);
#pragma unroll
            for (uint32_t b = 0; b < LY; ++b) e[i * LY + b] = entry(u[i], b);
        }
        u16x2 mn = __builtin_bit_cast(u16x2, e[0]);
#pragma unroll
        for (uint32_t k = 1; k < 2 * LY; ++k) mn = __builtin_elementwise_min(mn, __builtin_bit_cast(u16x2, e[k]));
        best = NZ == 2 ? min(static_cast<uint32_t>(mn.x), static_cast<uint32_t>(mn.y)) : static_cast<uint32_t>(mn.x);
        // bit k: entry k misses the key, bit 16 + k: its flipped partner does
        const uint32_t pat = best << 16 | best;
        const u16x2 one = {1, 1};
        uint32_t miss = 0;
#pragma unroll
        for (uint32_t k = 0; k < 2 * LY; ++k)
            miss |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, e[k] ^ pat), one))
                    << k;
        constexpr uint32_t all = (1u << (2 * LY)) - 1u;
        uint32_t hits = ~miss & (NZ == 2 ? all << 16 | all : all);
        while (hits) {
            const uint32_t k = static_cast<uint32_t>(__builtin_ctz(hits));
            hits &= hits - 1;
            const uint32_t f = k >> 4, p = k & 15u, i = p >= LY ? 1u : 0u;
            visit(i ? u[1] : u[0], i, p - (i ? LY : 0u), f);
        }
    } else {
        u16x2 mn = {0xFFFFu, 0xFFFFu};
#pragma unroll
        for (uint32_t i = 0; i < kTorusMaxBases; ++i) {
            if (i >= nb) continue;
            const W u = pr[i] ^ static_cast<W>(cf[i * cstride]);
            for (uint32_t b = 0; b < Ly; ++b)
                mn = __builtin_elementwise_min(mn, __builtin_bit_cast(u16x2, entry(u, uni(b))));
        }
        best = nz == 2 ? min(static_cast<uint32_t>(mn.x), static_cast<uint32_t>(mn.y)) : static_cast<uint32_t>(mn.x);
        // bit i * Ly + b: plain, flipped; without flips the second word has the
        // odd base images (bases * Ly * |Z| is at most 128)
        uint64_t hp = 0, hf = 0;
#pragma unroll
        for (uint32_t i = 0; i < kTorusMaxBases; ++i) {
            if (i >= nb) continue;
            const W u = pr[i] ^ static_cast<W>(cf[i * cstride]);
            uint64_t m0 = 0, m1 = 0;
            for (uint32_t b0 = 0; b0 < Ly; ++b0) {
                const uint32_t b = uni(b0), e = entry(u, b);
                m0 |= ((e & 0xFFFFu) == best ? 1ull : 0ull) << b;
                m1 |= (nz == 2 && (e >> 16) == best ? 1ull : 0ull) << b;
            }
            if (nz == 2) {
                hp |= m0 << (i * Ly);
                hf |= m1 << (i * Ly);
            } else if (i & 1u) {
                hf |= m0 << ((i >> 1) * Ly);
            } else {
                hp |= m0 << ((i >> 1) * Ly);
            }
        }
        while (hp | hf) {
            const uint32_t second = hp ? 0u : 1u;
            uint64_t &h = hp ? hp : hf;
            uint32_t i = 0, b = static_cast<uint32_t>(__builtin_ctzll(h));
            h &= h - 1;
            while (b >= Ly) {
                b -= Ly;
                ++i;
            }
            if (nz == 1) i = 2 * i + second;
            const uint32_t f = nz == 2 ? second : 0u;
            W u = pr[0];
#pragma unroll
            for (uint32_t q = 1; q < kTorusMaxBases; ++q) u = (q < nb && i == q) ? pr[q] : u;
            visit(u ^ static_cast<W>(cf[i * cstride]), i, b, f);
        }
    }
    if constexpr (TRACK && !COUNT) info.code = code_of(won);
    return static_cast<W>(static_cast<W>(best) << tb) | static_cast<W>(tail);
}

// Binomial coefficient table [65][65] in device memory.
__device__ __forceinline__ uint64_t binom(const uint64_t *t, uint32_t n, uint32_t k) {
    return t[n * 65u + k];
}

// Position of the weight-w word s among the weight-w words in increasing
// order, kRankBits bits at a time: tab[((b << kRankBits) + v) * (w + 1) + k] is
// what the bits of chunk b with value v add when k bits are set below it.  The
// reads do not depend on each other (a loop over the set bits waits for one
// read a bit: 16-site ring product without symmetry 25.7 us, with this and the
// row groups in steps 16.3 us), and a chunk's values lie in a few KB of L1
// (whole bytes, 67 KB for 20 sites, were slower than the loop there).
__device__ __forceinline__ uint64_t colex_rank(uint64_t s, uint32_t n_sites, uint32_t w, const uint64_t *tab) {
    uint64_t r = 0;
    uint32_t k = 0;
    for (uint32_t b = 0; kRankBits * b < n_sites; ++b) {
        const uint32_t v = static_cast<uint32_t>(s >> (kRankBits * b)) & ((1u << kRankBits) - 1);
        r += tab[((b << kRankBits) + v) * (w + 1) + k];
        k += static_cast<uint32_t>(__builtin_popcount(v));
    }
    return r;
}

// Home line of a group of key blocks in a hash index of 2^(64 - shift) lines:
// Fibonacci hashing (the top bits of group * 2^64/phi).
__host__ __device__ __forceinline__ uint64_t line_of(uint64_t group, uint32_t shift) {
    return (group * 0x9E3779B97F4A7C15ULL) >> shift;
}
__device__ __forceinline__ uint64_t group_of(const SearchDev &S, uint64_t key) {
    return key >> (S.low_bits() + S.group_bits());
}
__device__ __forceinline__ uint64_t home_line(const SearchDev &S, uint64_t key) {
    return line_of(group_of(S, key), S.hash_shift);
}

// Number of the key's block among all entries of the table, in line `line`.
__device__ __forceinline__ uint64_t block_at(const SearchDev &S, uint64_t line, uint64_t key) {
    return line << S.group_bits() | ((key >> S.low_bits()) & ((1u << S.group_bits()) - 1));
}

// One probe of the hash index: the entry of the key's block in line `line`.
__device__ __forceinline__ uint4 load_block(const SearchDev &S, uint64_t line, uint64_t key) {
    return *reinterpret_cast<const uint4 *>(S.table + block_at(S, line, key));
}

// Number of a key among the keys its block can hold.
__device__ __forceinline__ uint32_t low_rank(const SearchDev &S, uint64_t key) {
    return S.low_rank[static_cast<uint32_t>(key) & ((1u << S.low_bits()) - 1)];
}

// Position and stabilizer size of a key from the probe e of its home line
// (further lines are read where another group holds it), q = low_rank(key);
// -1: not a representative.  The table always has free lines, so every probe
// sequence ends.
__device__ __forceinline__ int64_t resolve_block(const SearchDev &S, uint64_t key, uint64_t line, uint4 e, uint32_t q,
                                                 uint32_t &stab) {
    const uint64_t g = group_of(S, key);
    const uint32_t g_lo = static_cast<uint32_t>(g), g_hi = static_cast<uint32_t>(g >> 32);
    while (e.w != g_lo || (e.y >> S.tag_shift()) != g_hi) {
        if ((e.w & e.z) == 0xFFFFFFFFu) return -1;      // a free line (no position is ~0)
        line = (line + 1) & S.hash_mask;
        e = load_block(S, line, key);
    }
    // the members up to and with the key, the key on top
    const uint64_t members = static_cast<uint64_t>(e.x) | static_cast<uint64_t>(e.y & ((1u << (kBlockKeys - 32)) - 1)) << 32;
    const uint64_t upto = members << (63u - q);
    if (static_cast<int64_t>(upto) >= 0) return -1;
    const uint32_t idx = e.z + static_cast<uint32_t>(__builtin_popcountll(upto)) - 1u;
    stab = __builtin_amdgcn_ubfe(e.y, kBlockStab - 32, S.stab_bits());   // (no bits: 0)
    int64_t found = static_cast<int64_t>(idx);
    if (stab == 0) {
        if ((e.y >> (kBlockDropped - 32)) & 1u)
            for (uint64_t k = 1; k <= S.dropped[0]; ++k) found |= S.dropped[k] == key ? -1ll : 0ll;
        stab = S.stab[idx];
    }
    return found;
}

__device__ __forceinline__ int64_t lookup_hash(const SearchDev &S, uint64_t key, uint32_t &stab) {
    const uint64_t line = home_line(S, key);
    const uint4 e = load_block(S, line, key);
    return resolve_block(S, key, line, e, low_rank(S, key), stab);
}

// Binary search for key among reps[lo, end) (one bucket of the sorted array).
__device__ __forceinline__ int64_t search_bucket(const uint64_t *reps, uint32_t lo, uint32_t end, uint64_t key) {
    uint32_t hi = end;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (reps[mid] < key) lo = mid + 1; else hi = mid;
    }
    return (lo < end && reps[lo] == key) ? static_cast<int64_t>(lo) : -1;
}

// stateToIndex: hash index, or bucket of the key's high bits then binary
// search, or (PLAIN: groups of one element) the colex rank or the state itself.
template <bool PLAIN = true>
__device__ __forceinline__ int64_t lookup_index(const SearchDev &S, uint64_t key) {
    if (S.mode == kLookupHash) {
        // a block's numbering holds for keys of the sector's weight only
        if (key < S.kmin || key > S.kmax || (S.weight >= 0 && __builtin_popcountll(key) != S.weight)) return -1;
        uint32_t st;
        return lookup_hash(S, key, st);
    }
    if constexpr (PLAIN) {
        if (S.mode == kLookupIdentity)
            return (S.n_sites == 64 || (key >> S.n_sites) == 0) ? static_cast<int64_t>(key) : -1;
        if (S.mode == kLookupRank) {
            if ((S.n_sites < 64 && (key >> S.n_sites) != 0) || __builtin_popcountll(key) != S.weight) return -1;
            return static_cast<int64_t>(colex_rank(key, S.n_sites, static_cast<uint32_t>(S.weight), S.rank));
        }
    }
    if (key < S.kmin || key > S.kmax) return -1;
    const uint64_t b = (key - S.kmin) >> S.shift;
    return search_bucket(S.reps, S.buckets[b], S.buckets[b + 1], key);
}

// The bucket search with the bucket table staged in LDS (lb, S.n_bkt
// entries): the bucket's bounds are LDS reads, only the search inside the
// bucket reads reps.
__device__ __forceinline__ int64_t lookup_staged(const SearchDev &S, const uint32_t *lb, uint64_t key) {
    if (key < S.kmin || key > S.kmax) return -1;
    const uint32_t b = static_cast<uint32_t>((key - S.kmin) >> S.shift);
    return search_bucket(S.reps, lb[b], lb[b + 1], key);
}

// Index and stabilizer size of a key of the sector's weight (terms conserve
// it; the hash index holds both in one entry).
template <bool PLAIN = true>
__device__ __forceinline__ int64_t lookup_index_stab(const SearchDev &S, uint64_t key, const uint16_t *stab_arr,
                                                     uint32_t &stab) {
    if (S.mode == kLookupHash) {
        if (key > S.kmax) return -1;
        return lookup_hash(S, key, stab);
    }
    const int64_t j = lookup_index<PLAIN>(S, key);
    if (j >= 0) stab = stab_arr[j];
    return j;
}

}  // namespace ls
