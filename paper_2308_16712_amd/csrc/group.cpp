// Host-side group compiler: validation of a symmetry sector, Benes routing
// of bit permutations, and the coset split used by the device orbit search.
//
// The paper builds symmetry groups in its Haskell front end and leaves the
// representative test to the literature (Section 4 "Multiple languages",
// Section 5.2).  Here a group arrives as explicit permutations with
// characters; it is checked to be a group with a one-dimensional
// representation and compiled for the GPU.
//
// Benes networks: a permutation of n = 2^k wires is realised by 2k-1 stages
// of conditional exchanges (Benes 1964); on a machine word every stage is a
// "delta swap" (exchange bit j with bit j+d wherever mask bit j is set),
// stage distances n/2, ..., 2, 1, 2, ..., n/2.  The masks are found with the
// classic looping algorithm: the two wires of every input pair must enter
// different half-size subnetworks, and so must the two sources of every
// output pair; following these constraints around each cycle 2-colours the
// wires, then each half is routed recursively.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <unordered_map>

#include "ls_internal.hpp"

namespace ls {

namespace {

struct Elem {
    std::vector<uint16_t> perm;
    uint8_t flip;
};

std::string key_of(const uint16_t *perm, uint32_t n, uint8_t flip) {
    std::string k(reinterpret_cast<const char *>(perm), n * sizeof(uint16_t));
    k.push_back(static_cast<char>(flip));
    return k;
}

// Recursive looping-algorithm router on block [off, off+m) at a given level.
void route_block(const std::vector<int> &pi, int off, int m, int level, int n_levels,
                 uint64_t *masks) {
    if (m == 2) {
        if (pi[0] == 1) masks[level] |= 1ULL << off;
        return;
    }
    const int h = m / 2;
    std::vector<int> inv(m), side(m, -1);
    for (int i = 0; i < m; ++i) inv[pi[i]] = i;
    for (int j = 0; j < h; ++j) {
        if (side[j] >= 0) continue;
        int i = j;
        int s = 0;
        while (side[i] < 0) {
            side[i] = s;
            // the other source of i's output pair goes to the other half
            int o2 = pi[i] ^ h;
            int i2 = inv[o2];
            if (side[i2] >= 0) break;
            side[i2] = 1 - s;
            // the input partner of i2 goes to the half opposite to i2
            i = i2 ^ h;
            s = s;  // i2's partner gets 1 - (1 - s) = s
        }
    }
    std::vector<int> sub0(h), sub1(h);
    const int first = level, last = 2 * (n_levels - 1) - level;
    for (int i = 0; i < m; ++i) {
        const int pos_in = i & (h - 1);
        const int pos_out = pi[i] & (h - 1);
        if (side[i] == 0) {
            sub0[pos_in] = pos_out;
            if (i >= h) masks[first] |= 1ULL << (off + pos_in);   // bottom input moved up
            if (pi[i] >= h) masks[last] |= 1ULL << (off + pos_out);
        } else {
            sub1[pos_in] = pos_out;
            if (i < h) masks[first] |= 1ULL << (off + pos_in);     // top input moved down
        }
    }
    route_block(sub0, off, h, level + 1, n_levels, masks);
    route_block(sub1, off + h, h, level + 1, n_levels, masks);
}

}  // namespace

int benes_route(const std::vector<int> &dest, int n, uint64_t *masks) {
    int k = 0;
    while ((1 << k) < n) ++k;
    const int n_stages = 2 * k - 1;
    for (int s = 0; s < kMaxStages; ++s) masks[s] = 0;
    route_block(dest, 0, n, 0, k, masks);
    return n_stages;
}

uint64_t benes_apply_host(uint64_t x, const uint64_t *masks, int n_stages, int n) {
    const int k = (n_stages + 1) / 2;
    for (int s = 0; s < n_stages; ++s) {
        const int lvl = s < k ? s : 2 * (k - 1) - s;
        const int d = n >> (lvl + 1);
        const uint64_t t = ((x >> d) ^ x) & masks[s];
        x ^= t ^ (t << d);
    }
    if (n < 64) x &= (1ULL << n) - 1ULL;
    return x;
}

GroupPlan compile_group(const ls_sector_desc &d) {
    const uint32_t n = d.n_sites;
    LS_REQUIRE(n >= 1 && n <= 64, "n_sites must be in 1..64");
    LS_REQUIRE(d.hamming_weight >= -1 && d.hamming_weight <= static_cast<int32_t>(n),
               "hamming_weight must be -1 or in 0..n_sites");
    LS_REQUIRE(d.hamming_weight >= 0 || n <= 36, "without U(1) the library enumerates 2^N states; N must be <= 36");
    LS_REQUIRE(d.n_elements >= 1 && d.n_elements <= 4096, "n_elements must be in 1..4096");
    LS_REQUIRE(d.perm && d.flip && d.chi, "perm, flip and chi must not be NULL");
    const uint32_t ng = d.n_elements;

    std::unordered_map<std::string, int> index;
    index.reserve(ng * 2);
    for (uint32_t g = 0; g < ng; ++g) {
        const uint16_t *p = d.perm + static_cast<size_t>(g) * n;
        std::vector<char> seen(n, 0);
        for (uint32_t i = 0; i < n; ++i) {
            LS_REQUIRE(p[i] < n, "perm entry out of range");
            LS_REQUIRE(!seen[p[i]], "perm is not a bijection");
            seen[p[i]] = 1;
        }
        LS_REQUIRE(d.flip[g] <= 1, "flip must be 0 or 1");
        if (d.flip[g]) LS_REQUIRE(d.hamming_weight < 0 || 2 * d.hamming_weight == static_cast<int32_t>(n),
                                  "spin inversion needs hamming_weight = n_sites / 2");
        const double re = d.chi[2 * g], im = d.chi[2 * g + 1];
        LS_REQUIRE(std::isfinite(re) && std::isfinite(im) && std::fabs(std::hypot(re, im) - 1.0) < 1e-9,
                   "characters must have modulus 1");
        auto ins = index.emplace(key_of(p, n, d.flip[g]), static_cast<int>(g));
        LS_REQUIRE(ins.second, "duplicate group element");
    }
    // identity present with character 1
    std::vector<uint16_t> ident(n);
    for (uint32_t i = 0; i < n; ++i) ident[i] = static_cast<uint16_t>(i);
    auto it_id = index.find(key_of(ident.data(), n, 0));
    LS_REQUIRE(it_id != index.end(), "the group must contain the identity");
    {
        const int g = it_id->second;
        LS_REQUIRE(std::fabs(d.chi[2 * g] - 1.0) < 1e-9 && std::fabs(d.chi[2 * g + 1]) < 1e-9,
                   "the identity must have character 1");
    }
    // closure and homomorphism: chi(g h) = chi(g) chi(h) for all pairs.  The
    // product of a pair is found through generators: right multiplication by
    // a generator takes |G| compositions and lookups, a product by h = h' s is
    // the product by h' times s, so only |G| x (generators) permutations are
    // composed instead of |G|^2 (6x6 torus, 576 elements: 15 ms of a build).
    // A list that is not closed is composed pair by pair for its error.
    std::vector<uint16_t> comp(n);
    auto product = [&](uint32_t g, uint32_t h) -> int {
        const uint16_t *pg = d.perm + static_cast<size_t>(g) * n, *ph = d.perm + static_cast<size_t>(h) * n;
        for (uint32_t i = 0; i < n; ++i) comp[i] = pg[ph[i]];
        auto it = index.find(key_of(comp.data(), n, d.flip[g] ^ d.flip[h]));
        return it == index.end() ? -1 : it->second;
    };
    auto check_pair = [&](uint32_t g, uint32_t h, int gh) {
        LS_REQUIRE(gh >= 0, "the elements are not closed under composition");
        const double are = d.chi[2 * g], aim = d.chi[2 * g + 1];
        const double bre = d.chi[2 * h], bim = d.chi[2 * h + 1];
        const double pre = are * bre - aim * bim, pim = are * bim + aim * bre;
        LS_REQUIRE(std::fabs(pre - d.chi[2 * gh]) < 1e-9 && std::fabs(pim - d.chi[2 * gh + 1]) < 1e-9,
                   "chi is not a one-dimensional representation (chi(gh) != chi(g) chi(h))");
    };
    {
        // right[k][g] = g * generator k; reached: h = from[h] * generator via[h]
        std::vector<std::vector<int>> right;
        std::vector<int> from(ng, -1), via(ng, -1), order;
        std::vector<char> reached(ng, 0);
        order.push_back(it_id->second);
        reached[it_id->second] = 1;
        bool closed = true;
        for (uint32_t g = 0; g < ng && closed; ++g) {
            if (reached[g]) continue;
            std::vector<int> r(ng);
            for (uint32_t a = 0; a < ng && closed; ++a) {
                r[a] = product(a, g);
                closed = r[a] >= 0;
            }
            if (!closed) break;
            right.push_back(std::move(r));
            // all words in the generators so far
            for (size_t at = 0; at < order.size(); ++at)
                for (size_t k = 0; k < right.size(); ++k) {
                    const int h = right[k][order[at]];
                    if (!reached[h]) {
                        reached[h] = 1;
                        from[h] = order[at];
                        via[h] = static_cast<int>(k);
                        order.push_back(h);
                    }
                }
        }
        if (!closed) {
            for (uint32_t g = 0; g < ng; ++g)
                for (uint32_t h = 0; h < ng; ++h) check_pair(g, h, product(g, h));
        }
        // by[h][g] = g * h along the words (a word's beginning comes first)
        std::vector<std::vector<int>> by(ng);
        for (int h : order) {
            by[h].resize(ng);
            for (uint32_t g = 0; g < ng; ++g)
                by[h][g] = from[h] < 0 ? static_cast<int>(g) : right[via[h]][by[from[h]][g]];
        }
        for (uint32_t h = 0; h < ng; ++h)
            for (uint32_t g = 0; g < ng; ++g) check_pair(g, h, by[h][g]);
    }

    GroupPlan P;
    P.n_sites = n;
    P.n_elements = ng;
    P.full = n == 64 ? ~0ULL : ((1ULL << n) - 1ULL);
    P.n_stages = n <= 32 ? 9 : 11;
    const int wires = n <= 32 ? 32 : 64;

    auto find_elem = [&](const std::vector<uint16_t> &perm, uint8_t flip) -> int {
        auto it = index.find(key_of(perm.data(), n, flip));
        return it == index.end() ? -1 : it->second;
    };

    // spin inversion pairing
    P.pair_flip = find_elem(ident, 1) >= 0 ? 1 : 0;

    // translation layout: lx * ly = n, every (x,y) -> (x+a, y+b) present
    auto trans_perm = [&](uint32_t lx, uint32_t ly, uint32_t a, uint32_t b) {
        std::vector<uint16_t> p(n);
        if (lx * ly != n) {   // no translation layout: T = {identity}
            for (uint32_t i = 0; i < n; ++i) p[i] = static_cast<uint16_t>(i);
            return p;
        }
        for (uint32_t y = 0; y < ly; ++y)
            for (uint32_t x = 0; x < lx; ++x)
                p[x + lx * y] = static_cast<uint16_t>(((x + a) % lx) + lx * ((y + b) % ly));
        return p;
    };
    std::vector<uint32_t> shapes;
    shapes.push_back(n);
    for (uint32_t lx = n - 1; lx >= 2; --lx)
        if (n % lx == 0) shapes.push_back(lx);
    P.lx = 1;
    P.ly = 1;
    if (ng > 1) {
        for (uint32_t lx : shapes) {
            const uint32_t ly = n / lx;
            if (lx == 1) continue;
            bool ok = true;
            for (uint32_t b = 0; b < ly && ok; ++b)
                for (uint32_t a = 0; a < lx && ok; ++a)
                    ok = find_elem(trans_perm(lx, ly, a, b), 0) >= 0;
            if (ok) { P.lx = lx; P.ly = ly; break; }
        }
    }
    for (uint32_t y = 0; y < P.ly; ++y) P.col0 |= 1ULL << (P.lx * y);
    const uint32_t nt = P.lx * P.ly;
    const uint32_t nz = P.pair_flip ? 2 : 1;

    // the elements of (Z x T) o g
    auto coset_of = [&](int g) {
        std::vector<int> out;
        const uint16_t *pg = d.perm + static_cast<size_t>(g) * n;
        for (uint32_t t = 0; t < nt; ++t) {
            auto tp = trans_perm(P.lx, P.ly, t % P.lx, t / P.lx);
            std::vector<uint16_t> c(n);
            for (uint32_t i = 0; i < n; ++i) c[i] = tp[pg[i]];
            for (uint32_t z = 0; z < nz; ++z) {
                int e = find_elem(c, static_cast<uint8_t>(d.flip[g] ^ z));
                if (e < 0) throw Error{LS_EINTERNAL, "coset element missing from a closed group"};
                out.push_back(e);
            }
        }
        return out;
    };
    std::vector<uint16_t> reverse(n);
    for (uint32_t i = 0; i < n; ++i) reverse[i] = static_cast<uint16_t>(n - 1 - i);
    const int rev_elem = find_elem(reverse, 0);

    std::vector<char> covered(ng, 0);
    std::vector<int> reps;
    auto take = [&](int g) {
        auto c = coset_of(g);
        int best = -1, rank = 4;
        for (int e : c) {
            int r;
            if (e == it_id->second) r = 0;
            else if (e == rev_elem) r = 1;
            else if (d.flip[e] == 0) r = 2;
            else r = 3;
            if (r < rank || (r == rank && e < best)) { rank = r; best = e; }
        }
        for (int e : c) {
            if (covered[e]) throw Error{LS_EINTERNAL, "cosets overlap"};
            covered[e] = 1;
        }
        reps.push_back(best);
    };
    take(it_id->second);
    for (uint32_t g = 0; g < ng; ++g)
        if (!covered[g]) take(static_cast<int>(g));

    // Benes networks for the coset representatives
    for (int e : reps) {
        CosetRep cr{};
        cr.flip = d.flip[e];
        const uint16_t *pe = d.perm + static_cast<size_t>(e) * n;
        bool is_id = true, is_rev = true;
        for (uint32_t i = 0; i < n; ++i) {
            is_id = is_id && pe[i] == i;
            is_rev = is_rev && pe[i] == n - 1 - i;
        }
        if (is_id) {
            cr.kind = kCosetIdentity;
        } else if (is_rev) {
            cr.kind = kCosetReverse;
        } else {
            cr.kind = kCosetBenes;
            std::vector<int> dest(wires);
            for (int i = 0; i < wires; ++i) dest[i] = i < static_cast<int>(n) ? pe[i] : i;
            const int st = benes_route(dest, wires, cr.masks);
            if (st != static_cast<int>(P.n_stages)) throw Error{LS_EINTERNAL, "Benes stage count"};
            for (int i = 0; i < wires; ++i) {
                const uint64_t got = benes_apply_host(1ULL << i, cr.masks, st, wires);
                if (got != (1ULL << dest[i])) throw Error{LS_EINTERNAL, "Benes routing self-check failed"};
            }
        }
        P.cosets.push_back(cr);
    }

    // character table by code ((p * nt) + t) * nz + f, element F^f o tau_t o p
    const uint32_t ncode = static_cast<uint32_t>(P.cosets.size()) * nt * nz;
    if (ncode != ng) throw Error{LS_EINTERNAL, "coset split does not cover the group"};
    P.chi.assign(2 * ng, 0.0);
    P.chi_one.assign((ng + 31) / 32, 0u);
    P.code_to_index.assign(ng, -1);
    P.skip.assign(static_cast<size_t>(P.cosets.size()) * nt * n, 0);
    std::vector<char> hit(ng, 0);
    bool trivial = true, real = true;
    for (uint32_t p = 0; p < P.cosets.size(); ++p) {
        const uint16_t *pp = d.perm + static_cast<size_t>(reps[p]) * n;
        for (uint32_t t = 0; t < nt; ++t) {
            auto tp = trans_perm(P.lx, P.ly, t % P.lx, t / P.lx);
            std::vector<uint16_t> c(n);
            for (uint32_t i = 0; i < n; ++i) c[i] = tp[pp[i]];
            std::vector<uint16_t> from(n);
            for (uint32_t i = 0; i < n; ++i) from[c[i]] = static_cast<uint16_t>(i);
            uint32_t lowest = n;
            for (uint32_t d = n; d-- > 0;) {
                lowest = std::min<uint32_t>(lowest, from[d]);
                P.skip[(static_cast<size_t>(p) * nt + t) * n + d] = static_cast<uint8_t>(std::min(lowest, d));
            }
            for (uint32_t f = 0; f < nz; ++f) {
                const uint32_t code = (p * nt + t) * nz + f;
                const int e = find_elem(c, static_cast<uint8_t>(d.flip[reps[p]] ^ f));
                if (e < 0 || hit[e]) throw Error{LS_EINTERNAL, "code table is not a bijection"};
                hit[e] = 1;
                P.code_to_index[code] = e;
                double re = d.chi[2 * e], im = d.chi[2 * e + 1];
                const bool one = std::fabs(re - 1.0) < 1e-9 && std::fabs(im) < 1e-9;
                if (!one) trivial = false;
                if (std::fabs(im) >= 1e-9) real = false;
                P.chi[2 * code] = re;
                P.chi[2 * code + 1] = im;
                if (one) P.chi_one[code / 32] |= 1u << (code % 32);
            }
        }
    }
    P.chi_mode = trivial ? kChiTrivial : (real ? kChiReal : kChiComplex);

    // Tables of the torus search: the row operations present, the base
    // images that the other cosets are row operations of, and for each pair
    // of rows the smallest value over operations and x-shifts.
    if (P.lx >= 3 && P.lx <= 6 && P.ly >= 2 && P.cosets.size() <= 8 && P.cosets.size() * P.ly * nz <= 128) {
        const uint32_t L = P.lx, rm = (1u << L) - 1u;
        std::vector<uint32_t> code_of(ng);
        for (uint32_t c = 0; c < ng; ++c) code_of[P.code_to_index[c]] = c;
        // code of row operation m (its flip g) after the element e; -1: not in the group
        auto op_after = [&](uint32_t m, uint8_t g, int e) -> int {
            const uint16_t *pe = d.perm + static_cast<size_t>(e) * n;
            std::vector<uint16_t> c(n);
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t x = pe[i] % L, y = pe[i] / L;
                c[i] = static_cast<uint16_t>(((m & 1) ? L - 1 - x : x) + L * ((m & 2) ? P.ly - 1 - y : y));
            }
            const int h = find_elem(c, static_cast<uint8_t>(g ^ d.flip[e]));
            return h < 0 ? -1 : static_cast<int>(code_of[h]);
        };
        const uint32_t per_coset = nt * nz;
        uint32_t ops[4] = {}, n_ops = 0;
        std::vector<char> seen(P.cosets.size(), 0);
        for (uint32_t m = 0; m < 4; ++m)
            for (uint8_t g = 0; g < 2; ++g) {
                const int c = op_after(m, g, it_id->second);
                if (c < 0 || seen[c / per_coset]) continue;   // absent, or a translation of another
                seen[c / per_coset] = 1;
                ops[n_ops++] = m;
                if (g) P.op_flips |= 1u << m;
            }
        std::vector<char> taken(P.cosets.size(), 0);
        bool split = true;
        for (uint32_t p = 0; p < P.cosets.size(); ++p) {
            if (taken[p]) continue;
            P.base_coset.push_back(p);
            P.op_code.resize(P.base_coset.size() * 4, 0);
            for (uint32_t k = 0; k < n_ops; ++k) {
                const int c = op_after(ops[k], (P.op_flips >> ops[k]) & 1u, reps[p]);
                if (c < 0 || taken[c / per_coset]) {
                    split = false;
                    break;
                }
                taken[c / per_coset] = 1;
                const uint32_t t = (static_cast<uint32_t>(c) / nz) % nt, f = static_cast<uint32_t>(c) % nz;
                P.op_code[(P.base_coset.size() - 1) * 4 + ops[k]] =
                    static_cast<uint32_t>(c) / per_coset | (t % L) << 8 | (t / L) << 16 | f << 24;
            }
        }
        if (!split) throw Error{LS_EINTERNAL, "row operations do not split the cosets"};
        // The searches compare few images as fast one by one, and two rows of
        // few sites tie often: 3x12 without point group, 36 images: product
        // 24.9 ms by the tables, 12.6 by all images; 5x8, 40 images: 1.14 and
        // 0.91; 4x16, 64 images: 0.65 and 0.65; 3x9 full, 108 images: 0.62 and
        // 0.77.  (2x14, full point group and inversion: 2.00 and 0.80 ms, and
        // the enumeration by images is as fast: no tables two sites wide.)
        P.row_tables = true;
        P.torus = P.lx == 6 || P.cosets.size() * nt >= 64;
        auto rot = [&](uint32_t v, uint32_t a) { return a == 0 ? v : (((v << a) | (v >> (L - a))) & rm); };
        auto rev = [&](uint32_t v) {
            uint32_t r = 0;
            for (uint32_t x = 0; x < L; ++x) r |= ((v >> x) & 1u) << (L - 1 - x);
            return r;
        };
        const uint32_t nq = 1u << (2 * L);
        std::vector<uint32_t> key(nq);
        P.pair_arg.assign(nq, 0);
        for (uint32_t q = 0; q < nq; ++q) {
            uint32_t best = ~0u;
            for (uint32_t k = 0; k < n_ops; ++k) {
                const uint32_t m = ops[k], w = ((P.op_flips >> m) & 1u) ? q ^ (nq - 1) : q;
                uint32_t top = w >> L, second = w & rm;
                if (m & 1) { top = rev(top); second = rev(second); }
                if (m & 2) std::swap(top, second);
                for (uint32_t a = 0; a < L; ++a) {
                    const uint32_t v = (rot(top, a) << L) | rot(second, a);
                    if (v < best) { best = v; P.pair_arg[q] = 0; }
                    if (v == best) P.pair_arg[q] |= 1u << (m * 8 + a);
                }
            }
            key[q] = best;
        }
        // each entry also carries the key of the spin-flipped pair
        P.pair_lut.resize(nq);
        for (uint32_t q = 0; q < nq; ++q) P.pair_lut[q] = key[q] | (key[q ^ (nq - 1)] << 16);
        for (uint32_t a = 0; a < L; ++a) {
            const uint64_t rowpat = static_cast<uint64_t>(rm & ~((1u << a) - 1u));
            uint64_t m = 0;
            for (uint32_t y = 0; y < P.ly; ++y) m |= rowpat << (L * y);
            P.col_ge[a] = m;
        }
    }
    if (P.chi_mode != kChiComplex) {
        // characters within 1e-9 of +-1 are used as exactly +-1
        for (uint32_t c = 0; c < ng; ++c) {
            P.chi[2 * c] = P.chi[2 * c] > 0 ? 1.0 : -1.0;
            P.chi[2 * c + 1] = 0.0;
        }
    }
    return P;
}

}  // namespace ls
