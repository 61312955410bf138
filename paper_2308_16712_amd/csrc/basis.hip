// Basis construction (Section 5.2), state_info and stateToIndex kernels.
//
// Enumeration: the candidates are all weight-w bitstrings in increasing
// order (colex rank 0 .. C(N,w)-1), or 0 .. 2^N-1 without U(1).  The paper
// splits this range into chunks, filters each chunk and then places the
// survivors with a histogram -> cumulative sum -> offsets scheme (Section
// 5.1 "Block to hashed", Section 5.2).  On one GPU the same scheme becomes
// an order-preserving stream compaction:
//   pass 1  every lane walks a run of consecutive candidates (enumerate.hpp:
//           jumps over those one test rules out together) and counts its
//           members; a workgroup reduction gives per-chunk counts;
//   scan    an exclusive scan of the chunk counts gives chunk offsets;
//   pass 2  a workgroup scan of the lanes' counts gives each lane's offset;
//           the lane walks its run again and writes its members and their
//           stabilizer sizes, or steps through the candidates that pass 1
//           marked (marked_build), and the stabilizers follow in a pass of
//           their own.  No atomics; the output is sorted by construction.
// The "condition" kept by the filter: s is the minimum of its orbit, and P
// does not annihilate it (every stabilizer element has character 1).

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <string>

#include "enumerate.hpp"

namespace ls {

namespace {

constexpr int kBlock = 256;
constexpr uint64_t kMarkCandidates = 1ull << 33;       // most candidates of one (1 GiB of marks)

__device__ uint64_t unrank_colex(uint64_t rank, uint32_t n, int32_t w, const uint64_t *tab) {
    uint64_t s = 0;
    uint32_t k = static_cast<uint32_t>(w);
    for (int p = static_cast<int>(n) - 1; p >= 0 && k > 0; --p) {
        const uint64_t c = binom(tab, static_cast<uint32_t>(p), k);
        if (c <= rank) {
            s |= 1ULL << p;
            rank -= c;
            --k;
        }
    }
    return s;
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (t < s) sh[t] += sh[t + s];
        __syncthreads();
    }
    const uint32_t r = sh[0];
    __syncthreads();
    return r;
}

// exclusive scan over the block
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const uint32_t add = t >= off ? sh[t - off] : 0u;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    const uint32_t incl = sh[t];
    __syncthreads();
    return incl - v;
}

struct EnumArgs {
    PlanDev plan;
    const uint64_t *binom;
    uint64_t begin, total;    // candidate ranks [begin, total)
    uint32_t per_lane;        // consecutive candidates of a lane
    uint32_t n_sites;
    int32_t weight;
    uint32_t *lane_counts;    // [lanes]
    uint64_t *marks;          // [lanes], marked builds: the members among up to 64 candidates
    uint32_t *counts;         // [blocks]
    const uint64_t *offsets;  // [blocks], pass 2
    uint64_t *reps;           // pass 2
    uint16_t *stab;           // pass 2
};

template <typename W>
__device__ __forceinline__ W candidate(const EnumArgs &a, uint64_t rank) {
    return a.weight >= 0 ? static_cast<W>(unrank_colex(rank, a.n_sites, a.weight, a.binom)) : static_cast<W>(rank);
}

// Walks the lane's candidates; hit(s, stab) for every member in order.  A
// lane's range ends where its neighbour's starts: one unranking a lane.
template <typename W, int WALK, typename Hit>
__device__ __forceinline__ void walk_lane(const EnumArgs &a, uint64_t *sh, Hit &&hit) {
    const uint64_t lane0 = static_cast<uint64_t>(blockIdx.x) * kBlock;
    const uint64_t start = a.begin + (lane0 + threadIdx.x) * a.per_lane;
    const bool live = start < a.total;
    const W s = live ? candidate<W>(a, start) : static_cast<W>(0);
    sh[threadIdx.x] = live ? static_cast<uint64_t>(s) : ~0ULL;
    if (threadIdx.x == 0) {
        const uint64_t stop = a.begin + (lane0 + kBlock) * a.per_lane;
        sh[kBlock] = stop < a.total ? static_cast<uint64_t>(candidate<W>(a, stop)) : ~0ULL;
    }
    __syncthreads();
    uint64_t end = sh[threadIdx.x + 1];
    __syncthreads();
    if (!live) return;
    CandRange<W> R;
    R.gosper = a.weight >= 0;
    const W full = static_cast<W>(a.plan.full);
    // the sector's greatest candidate: all its up spins on top
    R.last = full;
    if (R.gosper && a.weight < static_cast<int32_t>(a.n_sites)) R.last = static_cast<W>(full & ~(full >> a.weight));
    // a range that ends before the sector does, without a neighbour lane
    if (end == ~0ULL && start + a.per_lane >= a.total) {
        const W stop = candidate<W>(a, a.total - 1);
        if (stop < R.last) end = static_cast<uint64_t>(stop) + 1;
    }
    R.end = end;
    if constexpr (WALK == kWalkRing) walk_ring<W>(a.plan, s, R, hit);
    else if constexpr (WALK == kWalkTorus) walk_torus<W>(a.plan, s, R, hit);
    else walk_images<W>(a.plan, s, R, hit);
}

// Pass 1 of the build.
template <typename W, int WALK>
__global__ void __launch_bounds__(kBlock) k_enum_mark(EnumArgs a) {
    __shared__ uint64_t ends[kBlock + 1];
    __shared__ uint32_t sh[kBlock];
    uint32_t c = 0;
    walk_lane<W, WALK>(a, ends, [&](W, uint32_t) { ++c; });
    const uint64_t lane = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    a.lane_counts[lane] = c;
    const uint32_t t = block_sum(c, sh);
    if (threadIdx.x == 0) a.counts[blockIdx.x] = t;
}

// Pass 1 of a marked build (up to 64 candidates a lane): one bit a candidate, so
// that pass 2 need not walk again.
template <typename W, int WALK>
__global__ void __launch_bounds__(kBlock) k_enum_mark_bits(EnumArgs a) {
    __shared__ uint64_t ends[kBlock + 1];
    __shared__ uint32_t sh[kBlock];
    const uint64_t lane = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x, start = lane * a.per_lane;
    uint64_t mask = 0;
    walk_lane<W, WALK>(a, ends, [&](W s, uint32_t) {
        uint64_t rank = static_cast<uint64_t>(s);
        if (a.weight >= 0) {
            rank = 0;
            uint32_t k = 0;
            for (uint64_t left = static_cast<uint64_t>(s); left != 0; left &= left - 1)
                rank += binom(a.binom, static_cast<uint32_t>(__builtin_ctzll(left)), ++k);
        }
        mask |= 1ull << (rank - start);
    });
    if (start < a.total) a.marks[lane] = mask;
    const uint32_t c = block_sum(static_cast<uint32_t>(__builtin_popcountll(mask)), sh);
    if (threadIdx.x == 0) a.counts[blockIdx.x] = c;
}

// Pass 2 of a marked build: a lane steps through its candidates up to the last
// member.
template <typename W>
__global__ void __launch_bounds__(kBlock) k_enum_write_bits(EnumArgs a) {
    __shared__ uint32_t sh[kBlock];
    const uint64_t lane = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x, start = lane * a.per_lane;
    uint64_t mask = start < a.total ? a.marks[lane] : 0ull;
    const uint32_t local = block_exclusive_scan(static_cast<uint32_t>(__builtin_popcountll(mask)), sh);
    if (mask == 0) return;
    uint64_t pos = a.offsets[blockIdx.x] + local;
    for (W s = candidate<W>(a, start);;) {
        if (mask & 1) a.reps[pos++] = static_cast<uint64_t>(s);
        mask >>= 1;
        if (mask == 0) break;
        s = a.weight >= 0 ? next_combination<W>(s) : static_cast<W>(s + 1);
    }
}

// Stabilizer sizes of a marked build's members.
template <typename W>
__global__ void __launch_bounds__(kBlock) k_stab(PlanDev P, const uint64_t *reps, uint64_t d, uint16_t *stab) {
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= d) return;
    const W r = static_cast<W>(reps[i]);
    uint32_t c = 0;
    for_each_image<W, kOrbitGeneric>(P, r, [&](W v, uint32_t) {
        c += v == r ? 1u : 0u;
        return true;
    });
    stab[i] = static_cast<uint16_t>(c);
}

// Count only: block totals are added into *acc (integer atomic adds: the
// total does not depend on their order), so launches on one stream over
// consecutive ranges accumulate.
template <typename W, int WALK>
__global__ void __launch_bounds__(kBlock) k_enum_count(EnumArgs a, unsigned long long *acc) {
    __shared__ uint64_t ends[kBlock + 1];
    __shared__ uint32_t sh[kBlock];
    uint32_t c = 0;
    walk_lane<W, WALK>(a, ends, [&](W, uint32_t) { ++c; });
    const uint32_t t = block_sum(c, sh);
    if (threadIdx.x == 0 && t != 0) atomicAdd(acc, static_cast<unsigned long long>(t));
}

// Pass 2 of the build.
template <typename W, int WALK>
__global__ void __launch_bounds__(kBlock) k_enum_write(EnumArgs a) {
    __shared__ uint64_t ends[kBlock + 1];
    __shared__ uint32_t sh[kBlock];
    if (a.counts[blockIdx.x] == 0) return;
    const uint64_t lane = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const uint32_t local = block_exclusive_scan(a.lane_counts[lane], sh);
    uint64_t pos = a.offsets[blockIdx.x] + local;
    walk_lane<W, WALK>(a, ends, [&](W s, uint32_t st) {
        a.reps[pos] = static_cast<uint64_t>(s);
        a.stab[pos] = static_cast<uint16_t>(st);
        ++pos;
    });
}

// Single-workgroup exclusive scan of n counts (n up to a few million).
__global__ void __launch_bounds__(1024) k_scan_counts(const uint32_t *counts, uint64_t n, uint64_t *offsets,
                                                      uint64_t *total) {
    __shared__ uint64_t sh[1024];
    const int t = threadIdx.x;
    const uint64_t per = (n + 1023) / 1024;
    const uint64_t b = min<uint64_t>(n, per * t), e = min<uint64_t>(n, b + per);
    uint64_t s = 0;
    for (uint64_t i = b; i < e; ++i) s += counts[i];
    sh[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t add = t >= off ? sh[t - off] : 0ull;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    uint64_t run = sh[t] - s;
    for (uint64_t i = b; i < e; ++i) {
        offsets[i] = run;
        run += counts[i];
    }
    if (t == 1023) *total = sh[1023];
}

// buckets[k] = first index whose key reaches bucket k (k = 0 .. nb; entry
// nb is d): one binary search per bucket, so empty stretches of the key
// range cost no more than full ones.
__global__ void __launch_bounds__(kBlock) k_buckets(const uint64_t *reps, uint64_t d, uint64_t kmin, uint32_t shift,
                                                    uint64_t nb, uint32_t *buckets) {
    const uint64_t k = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (k > nb) return;
    uint64_t lo = 0, hi = d;
    if (k < nb) {
        while (lo < hi) {
            const uint64_t mid = (lo + hi) >> 1;
            if (((reps[mid] - kmin) >> shift) < k) lo = mid + 1; else hi = mid;
        }
    } else {
        lo = d;
    }
    buckets[k] = static_cast<uint32_t>(lo);
}

__global__ void k_clear_u64(unsigned long long *p) { *p = 0ull; }

// Groups of the hash index among the sorted representatives (integer atomic
// adds: the total does not depend on their order).
__global__ void __launch_bounds__(kBlock) k_count_groups(const uint64_t *reps, uint64_t d, uint32_t shift,
                                                         unsigned long long *total) {
    __shared__ uint32_t sh[kBlock];
    uint32_t heads = 0;
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * kBlock;
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x; i < d; i += stride)
        heads += (i == 0 || (reps[i] >> shift) != (reps[i - 1] >> shift)) ? 1u : 0u;
    const uint32_t c = block_sum(heads, sh);
    if (threadIdx.x == 0 && c != 0) atomicAdd(total, static_cast<unsigned long long>(c));
}

// Whether an entry belongs to group g.
__device__ __forceinline__ bool holds_group(const SearchDev &S, const IndexBlock &B, uint64_t g) {
    return B.tag == static_cast<uint32_t>(g) && (B.bits >> (S.tag_shift() + 32)) == (g >> 32);
}

// Hash index, first pass: the first representative of every group claims the
// first free line of the group's probe sequence with a compare-and-swap
// (groups are distinct and the table has more lines than groups, so every
// sequence ends) and marks its blocks as the group's, empty.
__global__ void __launch_bounds__(kBlock) k_index_claim(SearchDev S, IndexBlock *table) {
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= S.dim) return;
    const uint64_t key = S.reps[i], g = group_of(S, key);
    if (i > 0 && group_of(S, S.reps[i - 1]) == g) return;
    const uint32_t tag = static_cast<uint32_t>(g);
    uint64_t line = home_line(S, key);
    for (;;) {
        // tag and position of the line's first block: ~0 while it is free
        unsigned long long *w = reinterpret_cast<unsigned long long *>(&table[line << S.group_bits()].base);
        const unsigned long long mine = static_cast<unsigned long long>(tag) << 32;
        if (atomicCAS(w, ~0ull, mine) == ~0ull) break;
        line = (line + 1) & S.hash_mask;
    }
    for (uint32_t b = 0; b < (1u << S.group_bits()); ++b) {
        IndexBlock &B = table[line << S.group_bits() | b];
        B.bits = (g >> 32) << (S.tag_shift() + 32);
        if (b) {
            B.base = 0;
            B.tag = tag;
        }
    }
}

// Second pass: the first representative of every block fills it.
__global__ void __launch_bounds__(kBlock) k_index_fill(SearchDev S, IndexBlock *table) {
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= S.dim) return;
    const uint64_t first = S.reps[i], blk = first >> S.low_bits(), g = group_of(S, first);
    if (i > 0 && (S.reps[i - 1] >> S.low_bits()) == blk) return;
    uint64_t key = first, bits = 0, stab = S.stab[i];
    bool one = true;
    for (uint64_t j = i;;) {
        bits |= 1ull << low_rank(S, key);
        one = one && S.stab[j] == stab;
        if (++j >= S.dim) break;
        key = S.reps[j];
        if ((key >> S.low_bits()) != blk) break;
    }
    if (one) bits |= (stab & ((1ull << S.stab_bits()) - 1)) << kBlockStab;
    uint64_t line = home_line(S, first);
    for (;;) {
        IndexBlock &B = table[block_at(S, line, first)];
        if (holds_group(S, B, g)) {
            B.bits |= bits;
            B.base = static_cast<uint32_t>(i);
            return;
        }
        line = (line + 1) & S.hash_mask;
    }
}

// Test hook: `key` joins the dropped keys and its block gets the mark that
// makes lookups compare with them.  One thread; the walk is bounded by the
// table size.
__global__ void k_drop_key(SearchDev S, IndexBlock *table, uint64_t *dropped, uint64_t key) {
    uint64_t line = home_line(S, key);
    for (uint64_t n = 0; n <= S.hash_mask; ++n) {
        IndexBlock &B = table[block_at(S, line, key)];
        if (holds_group(S, B, group_of(S, key))) {
            dropped[++dropped[0]] = key;
            B.bits &= ~(((1ull << S.stab_bits()) - 1) << kBlockStab);
            B.bits |= 1ull << kBlockDropped;
            return;
        }
        line = (line + 1) & S.hash_mask;
    }
}

// Flip images of a state taken by itself: none.
struct NoFlips {
    __device__ __forceinline__ uint64_t operator[](uint32_t) const { return 0; }
};

// Representative, character and norm of each state, from the products'
// searches or a walk of all images (launch_state_info).  As many elements take s
// to its representative as fix s, so a search's number of images that equal the
// minimum is the stabilizer size, and the projector annihilates the orbit when
// two of them have different characters (`mixed`).  Walking all images took 864 us for 4.2e6 states of a 6x6 sector
// (576 elements).  Tori: the tables lie in LDS and the workgroups stay for many
// states.
template <int KIND>
constexpr int state_block() {
    return KIND == kOrbitTorus ? 1024 : kBlock;
}
template <typename W, int KIND, uint32_t LX, uint32_t LY, uint32_t NZ>
__global__ void __launch_bounds__(state_block<KIND>())
    k_state_info(PlanDev P, int32_t weight, uint64_t n, const uint64_t *states, uint64_t *reps, double *chi,
                 double *norm) {
    constexpr int BLOCK = state_block<KIND>();
    __shared__ uint32_t lut[KIND == kOrbitTorus ? 4096 : 1], arg[KIND == kOrbitTorus ? 4096 : 1];
    __shared__ uint64_t col[8];
    if constexpr (KIND == kOrbitTorus) {
        for (uint32_t q = threadIdx.x; q < 1u << (2 * P.lx); q += BLOCK) {
            lut[q] = P.pair_lut[q];
            arg[q] = P.pair_arg[q];
        }
        if (threadIdx.x < 8) col[threadIdx.x] = P.col_ge[threadIdx.x];
        __syncthreads();
    }
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * BLOCK) {
        const uint64_t s64 = states[i];
        const bool inside = P.n_sites == 64 || (s64 >> P.n_sites) == 0;
        double2 c = make_double2(0.0, 0.0);
        double nrm = 0.0;
        uint64_t rep = s64;
        if (inside) {
            const W s = static_cast<W>(s64);
            OrbitInfo info;
            W best = static_cast<W>(~static_cast<W>(0));
            bool found = false;
            if constexpr (KIND == kOrbitTorus) {
                W pr[kTorusMaxBases] = {};
                pr[0] = s;
#pragma unroll
                for (uint32_t p = 1; p < (LX ? 2u : kTorusMaxBases); ++p)
                    if (LX || p < P.n_base) pr[p] = apply_coset<W>(P.bases[p], s, P);
                best = torus_orbit_min<W, true, true, LX, LY, NZ>(P, pr, NoFlips{}, 0, lut, arg, col, info);
                found = true;
            } else if constexpr (KIND == kOrbitRing32 || KIND == kOrbitRing64T) {
                found = ring_orbit_min<W, true, true, KIND == kOrbitRing64T>(P, s, best, info);
            }
            if (!found) {
                // every image, the stabilizer from those that are s itself
                constexpr int WALK = KIND == kOrbitRing32 ? kOrbitRing32 : kOrbitGeneric;
                info = OrbitInfo{};
                best = s;
                for_each_image<W, WALK>(P, s, [&](W v, uint32_t code) {
                    if (v < best) {
                        best = v;
                        info.code = code;
                    }
                    if (v == s) {
                        ++info.count;
                        info.mixed = info.mixed || !chi_is_one(P, code);
                    }
                    return true;
                });
            }
            rep = static_cast<uint64_t>(best);
            if (!info.mixed && (weight < 0 || __builtin_popcountll(s64) == weight)) {
                c = P.chi[info.code];
                nrm = __dsqrt_rn(__ddiv_rn(static_cast<double>(info.count), static_cast<double>(P.n_elements)));
            }
        }
        reps[i] = rep;
        chi[2 * i] = c.x;
        chi[2 * i + 1] = c.y;
        norm[i] = nrm;
    }
}

__global__ void __launch_bounds__(kBlock) k_index_lookup(SearchDev S, uint64_t n, const uint64_t *keys, int64_t *out) {
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    out[i] = lookup_index(S, keys[i]);
}

uint64_t grid_for(uint64_t n) { return (n + kBlock - 1) / kBlock; }

// Device scratch of a build, allocated and released in order on the build's
// stream: unlike hipFree, hipFreeAsync does not wait for the whole device,
// so a build beside running products (the serving loop) is not held up by
// them.
struct StreamBuf {
    void *p = nullptr;
    hipStream_t st;
    StreamBuf(size_t bytes, hipStream_t s) : st(s) { LS_HIP_CHECK(hipMallocAsync(&p, bytes, s)); }
    ~StreamBuf() {
        if (p) (void)hipFreeAsync(p, st);
    }
    StreamBuf(const StreamBuf &) = delete;
    StreamBuf &operator=(const StreamBuf &) = delete;
    template <class T>
    T *as() const {
        return static_cast<T *>(p);
    }
};

// Candidates of a lane.  The members crowd at the low ranks, so few candidates
// a lane balance the walk; but a lane pays about a thousand instructions to
// unrank its first one.  Rings: 3.4e10 candidates of the 40-spin chain take
// 22.4 ms at 512 a lane, 24.8 at 256, 28.8 at 128, 50.6 at 32.  Members of the
// other groups cost more each: a 6x6 build takes 45.6 ms at 512, 36.5 at 128,
// 38.0 at 64, 43.4 at 32.
uint32_t cand_per_lane(uint64_t candidates, int walk) {
    const uint64_t most = walk == kWalkRing ? 512 : 128;
    return static_cast<uint32_t>(std::min<uint64_t>(most, std::max<uint64_t>(4, candidates >> 20)));
}

// Whether the build marks the members, for pass 2 to step through the
// candidates, or walks twice.  Members cost a walk every image, so a second
// walk costs most where they are many: 30-site ring in scrambled order, 60
// images, 1.6e8 candidates: 6.4 ms walked twice, 2.9 marked; 4x9, 144 images: 5.1
// and 2.9; 6x6, 12 up, 288 images, 1.3e9 candidates: 6.2 and 4.8; 6x6, 18 up, 9e9:
// 11.2 and 15.2.  Rings walk their members by a few runs (32 sites: 3 ms).
bool marked_build(int walk, uint64_t total) { return walk != kWalkRing && total <= kMarkCandidates; }

// Sorted representatives and their stabilizer sizes.
template <typename W, int WALK>
void enumerate_impl(ls_basis *b, hipStream_t st, uint64_t total) {
    const bool marked = marked_build(WALK, total);
    EnumArgs a{};
    a.plan = b->plan_dev;
    a.binom = b->d_binom;
    a.begin = 0;
    a.total = total;
    a.per_lane = marked ? std::min(64u, cand_per_lane(total, WALK)) : cand_per_lane(total, WALK);
    a.n_sites = b->plan.n_sites;
    a.weight = b->weight;
    const uint64_t lanes = (total + a.per_lane - 1) / a.per_lane;
    const uint64_t blocks = grid_for(lanes);
    // a count or 64 marks of every lane
    StreamBuf lanes_b(std::max<uint64_t>(blocks, 1) * kBlock * (marked ? sizeof(uint64_t) : sizeof(uint32_t)), st);
    StreamBuf counts_b(std::max<uint64_t>(blocks, 1) * sizeof(uint32_t), st);
    StreamBuf offsets_b(std::max<uint64_t>(blocks, 1) * sizeof(uint64_t), st);
    StreamBuf total_b(sizeof(uint64_t), st);
    a.lane_counts = lanes_b.as<uint32_t>();
    a.marks = lanes_b.as<uint64_t>();
    a.counts = counts_b.as<uint32_t>();
    a.offsets = offsets_b.as<uint64_t>();
    uint64_t dim = 0;
    if (blocks > 0) {
        if constexpr (WALK != kWalkRing) {
            if (marked) hipLaunchKernelGGL((k_enum_mark_bits<W, WALK>), dim3(blocks), dim3(kBlock), 0, st, a);
        }
        if (!marked) hipLaunchKernelGGL((k_enum_mark<W, WALK>), dim3(blocks), dim3(kBlock), 0, st, a);
        LS_HIP_CHECK(hipGetLastError());
        hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, st, a.counts, blocks, offsets_b.as<uint64_t>(),
                           total_b.as<uint64_t>());
        LS_HIP_CHECK(hipGetLastError());
        LS_HIP_CHECK(hipMemcpyAsync(&dim, total_b.p, sizeof(uint64_t), hipMemcpyDeviceToHost, st));
        LS_HIP_CHECK(hipStreamSynchronize(st));
    }
    if (dim >= 0xFFFFFFFFull) throw Error{LS_EINVAL, "basis dimension must be below 2^32 - 1"};
    b->d_reps = dev_alloc_n<uint64_t>(std::max<uint64_t>(dim, 1), st);
    b->d_stab = dev_alloc_n<uint16_t>(std::max<uint64_t>(dim, 1), st);
    a.reps = b->d_reps;
    a.stab = b->d_stab;
    if (dim > 0 && marked) {
        hipLaunchKernelGGL((k_enum_write_bits<W>), dim3(blocks), dim3(kBlock), 0, st, a);
        hipLaunchKernelGGL((k_stab<W>), dim3(grid_for(dim)), dim3(kBlock), 0, st, b->plan_dev, b->d_reps, dim, b->d_stab);
        LS_HIP_CHECK(hipGetLastError());
    } else if (dim > 0) {
        hipLaunchKernelGGL((k_enum_write<W, WALK>), dim3(blocks), dim3(kBlock), 0, st, a);
        LS_HIP_CHECK(hipGetLastError());
    }
    b->dim = dim;
}

template <int WALK>
void enumerate_words(ls_basis *b, hipStream_t st, uint64_t total) {
    if (b->plan.n_sites <= 32) enumerate_impl<uint32_t, WALK>(b, st, total);
    else enumerate_impl<uint64_t, WALK>(b, st, total);
}

uint64_t host_binom(uint32_t n, uint32_t k) {
    if (k > n) return 0;
    uint64_t r = 1;
    for (uint32_t i = 1; i <= k; ++i) r = r * (n - k + i) / i;   // exact: r*(n-k+i) divisible by i
    return r;
}

}  // namespace

// Lines of the hash index, a power of two, and the bits of a block's number
// in its line, within the bytes of a table of one 16-byte slot a key (load 1/8
// within 8 GiB, 1/4 within 64 GiB, 1/2 or 3/4 within 128 GiB; the admission of
// the serving loop reserves them): 128-byte lines at load 1/4 where they fit,
// which they do in dense sectors with room to spare (about 20 keys a line), else
// one block a line, as many lines as fit.  0: over 128 GiB.
uint64_t index_lines(uint64_t dim, uint64_t groups, uint32_t *group_bits) {
    struct Tier {
        uint64_t num, den, limit;   // slots >= dim * num / den while slots * 16 <= limit
    };
    const Tier tiers[] = {{8, 1, 8ULL << 30}, {4, 1, 64ULL << 30}, {2, 1, 128ULL << 30}, {4, 3, 128ULL << 30}};
    uint64_t slots = 0;
    for (const Tier &t : tiers) {
        uint64_t cap = 1024;
        while (cap * t.den < t.num * dim) cap <<= 1;
        if (cap * 16 <= t.limit) {
            slots = cap;
            break;
        }
    }
    uint64_t lines = 8;
    while (lines < 4 * groups) lines <<= 1;
    *group_bits = kGroupBits;
    if (lines << kGroupBits <= slots) return lines;
    *group_bits = 0;
    return slots;
}

// Whether the ring search of a sector's words turns them: a doubled word of
// 64 bits shows runs up to 64 - N zeros, and with spin inversion (runs of equal
// spins, taken by their boundaries) as many spins.  A word with `weight` up
// spins has at most N - weight zeros in a row.  Turning costs 5% where it is
// not needed (34 sites, 17 up: 7.41 ms turned, 7.04 doubled).  Doubling every
// word first and searching again where a run is longer makes a wavefront take
// both searches (44 sites, 7 up: 308 us, turned 257; 60 sites, 6 up: 448 and
// 312).
bool ring_turns(const GroupPlan &gp, int32_t weight) {
    return weight < 0 || gp.n_sites - static_cast<uint32_t>(weight) + gp.n_sites > 64;
}

namespace {

// Host images of the device tables of a compiled group, shared by
// upload_plan (device allocations) and the allocation-free count (static
// scratch): binomial table [65][65], coset representatives, characters by
// code, chi == 1 bitset.
struct PlanTables {
    std::vector<uint64_t> binom;
};

PlanTables plan_tables() {
    PlanTables t;
    t.binom.assign(65 * 65, 0);
    for (uint32_t i = 0; i <= 64; ++i)
        for (uint32_t k = 0; k <= i; ++k)
            t.binom[i * 65 + k] = k == 0 || k == i ? 1 : t.binom[(i - 1) * 65 + k - 1] + t.binom[(i - 1) * 65 + k];
    return t;
}

// PlanDev fields that do not point into device memory.
void fill_plan_dev(const GroupPlan &gp, PlanDev &pd) {
    pd.n_sites = gp.n_sites;
    pd.lx = gp.lx;
    pd.ly = gp.ly;
    pd.n_trans = gp.lx * gp.ly;
    pd.n_cosets = static_cast<uint32_t>(gp.cosets.size());
    pd.pair_flip = gp.pair_flip;
    pd.n_stages = gp.n_stages;
    pd.n_elements = gp.n_elements;
    pd.full = gp.full;
    pd.col0 = gp.col0;
    pd.pair_lut = pd.pair_arg = pd.op_code = nullptr;
    pd.bases = nullptr;
    pd.n_base = static_cast<uint32_t>(gp.base_coset.size());
    pd.op_flips = gp.op_flips;
    pd.chi_trivial = gp.chi_mode == kChiTrivial ? 1 : 0;
    pd.skip = nullptr;
    for (int a = 0; a < 8; ++a) pd.col_ge[a] = gp.col_ge[a];
    pd.n_stab_cls = 0;
    pd.stab_cls = nullptr;
    pd.stab_ratio = nullptr;
}

// Tables of the torus search, in one block: base images, pair table, argument
// table, codes of the operations.
std::vector<unsigned char> torus_tables(const GroupPlan &gp) {
    std::vector<unsigned char> t;
    auto add = [&](const void *p, size_t bytes) {
        const unsigned char *c = static_cast<const unsigned char *>(p);
        t.insert(t.end(), c, c + bytes);
    };
    for (uint32_t p : gp.base_coset) add(&gp.cosets[p], sizeof(CosetRep));
    add(gp.pair_lut.data(), gp.pair_lut.size() * sizeof(uint32_t));
    add(gp.pair_arg.data(), gp.pair_arg.size() * sizeof(uint32_t));
    add(gp.op_code.data(), gp.op_code.size() * sizeof(uint32_t));
    return t;
}

void set_torus_tables(const GroupPlan &gp, const unsigned char *d, PlanDev &pd) {
    pd.bases = reinterpret_cast<const CosetRep *>(d);
    pd.pair_lut = reinterpret_cast<const uint32_t *>(d + gp.base_coset.size() * sizeof(CosetRep));
    pd.pair_arg = pd.pair_lut + gp.pair_lut.size();
    pd.op_code = pd.pair_arg + gp.pair_arg.size();
}

// Stabilizer-ratio table of a group: the class of every divisor of |G|
// (0xFF for the other sizes) followed, at offset kStabMapBytes, by the
// correctly rounded sqrt(d_b / d_a) over pairs of divisors (IEEE division
// and square root, the bits the kernels' own division and square root give).
// Empty when |G| or its number of divisors is above the table's limits.
std::vector<unsigned char> stab_table(uint32_t ng, uint32_t &n_cls) {
    n_cls = 0;
    if (ng > kStabMapMax) return {};
    std::vector<uint32_t> div;
    for (uint32_t d = 1; d <= ng; ++d)
        if (ng % d == 0) div.push_back(d);
    if (div.size() > kStabClsMax) return {};
    const uint32_t nd = static_cast<uint32_t>(div.size());
    std::vector<unsigned char> t(kStabMapBytes + static_cast<size_t>(nd) * nd * sizeof(double), 0xFF);
    for (uint32_t c = 0; c < nd; ++c) t[div[c]] = static_cast<unsigned char>(c);
    double *r = reinterpret_cast<double *>(t.data() + kStabMapBytes);
    for (uint32_t a = 0; a < nd; ++a)
        for (uint32_t c = 0; c < nd; ++c)
            r[a * nd + c] = std::sqrt(static_cast<double>(div[c]) / static_cast<double>(div[a]));
    n_cls = nd;
    return t;
}

}  // namespace

void upload_plan(ls_basis *b, hipStream_t st) {
    const GroupPlan &gp = b->plan;
    const PlanTables t = plan_tables();
    b->d_binom = dev_alloc_n<uint64_t>(t.binom.size(), st);
    LS_HIP_CHECK(hipMemcpyAsync(b->d_binom, t.binom.data(), t.binom.size() * sizeof(uint64_t), hipMemcpyHostToDevice, st));
    const size_t ncos = gp.cosets.size();
    b->d_cosets = dev_alloc_n<CosetRep>(ncos, st);
    LS_HIP_CHECK(hipMemcpyAsync(b->d_cosets, gp.cosets.data(), ncos * sizeof(CosetRep), hipMemcpyHostToDevice, st));
    b->d_chi = dev_alloc_n<double2>(gp.n_elements, st);
    LS_HIP_CHECK(hipMemcpyAsync(b->d_chi, gp.chi.data(), gp.n_elements * sizeof(double2), hipMemcpyHostToDevice, st));
    // (rings take m from the rotation, one element never rejects)
    if (gp.n_elements > 1 && walk_kind(gp) != kWalkRing) {
        b->d_skip = dev_alloc_n<uint8_t>(gp.skip.size(), st);
        LS_HIP_CHECK(hipMemcpyAsync(b->d_skip, gp.skip.data(), gp.skip.size(), hipMemcpyHostToDevice, st));
    }
    b->d_chi_one = dev_alloc_n<uint32_t>(gp.chi_one.size(), st);
    LS_HIP_CHECK(hipMemcpyAsync(b->d_chi_one, gp.chi_one.data(), gp.chi_one.size() * sizeof(uint32_t),
                                hipMemcpyHostToDevice, st));
    PlanDev &pd = b->plan_dev;
    fill_plan_dev(gp, pd);
    pd.cosets = b->d_cosets;
    pd.chi = b->d_chi;
    pd.chi_one = b->d_chi_one;
    pd.skip = b->d_skip;
    if (gp.row_tables) {
        const std::vector<unsigned char> t = torus_tables(gp);
        b->d_torus = dev_alloc_n<unsigned char>(t.size(), st);
        LS_HIP_CHECK(hipMemcpyAsync(b->d_torus, t.data(), t.size(), hipMemcpyHostToDevice, st));
        LS_HIP_CHECK(hipStreamSynchronize(st));
        set_torus_tables(gp, b->d_torus, pd);
    }
    uint32_t n_cls = 0;
    const std::vector<unsigned char> stab = stab_table(gp.n_elements, n_cls);
    if (n_cls) {
        unsigned char *d = dev_alloc_n<unsigned char>(stab.size(), st);
        b->d_stab_tab = d;
        LS_HIP_CHECK(hipMemcpyAsync(d, stab.data(), stab.size(), hipMemcpyHostToDevice, st));
        pd.n_stab_cls = n_cls;
        pd.stab_cls = d;
        pd.stab_ratio = reinterpret_cast<const double *>(d + kStabMapBytes);
    }
    // the host tables are released on return: the copies complete first
    LS_HIP_CHECK(hipStreamSynchronize(st));
}

uint64_t candidate_count(const ls_basis *b) {
    const uint32_t n = b->plan.n_sites;
    if (b->weight >= 0) return host_binom(n, static_cast<uint32_t>(b->weight));
    return n == 64 ? ~0ULL : (1ULL << n);
}

namespace {

// Members among the candidates of rank [begin, end) (end within range),
// accumulated into *acc (device, 8 bytes; cleared here by a fill kernel);
// the plan's tables must be on the device.
template <typename W>
uint64_t count_impl(const GroupPlan &gp, const PlanDev &pd, const uint64_t *binom, int32_t weight, uint64_t begin,
                    uint64_t end, unsigned long long *acc, hipStream_t st) {
    // a launch covers up to 2^20 workgroups (at most 1.4e11 candidates)
    constexpr uint64_t kSpanBlocks = 1ull << 20;
    unsigned long long total = 0;
    hipLaunchKernelGGL(k_clear_u64, dim3(1), dim3(1), 0, st, acc);
    LS_HIP_CHECK(hipGetLastError());
    EnumArgs a{};
    a.plan = pd;
    a.binom = binom;
    a.per_lane = cand_per_lane(end - begin, walk_kind(gp));
    a.n_sites = gp.n_sites;
    a.weight = weight;
    const uint64_t span = kSpanBlocks * kBlock * a.per_lane;
    for (uint64_t lo = begin; lo < end;) {
        const uint64_t hi = end - lo > span ? lo + span : end;
        a.begin = lo;
        a.total = hi;
        const uint64_t lanes = (hi - lo + a.per_lane - 1) / a.per_lane;
        const uint32_t blocks = static_cast<uint32_t>(grid_for(lanes));
        switch (walk_kind(gp)) {
            case kWalkRing:
                hipLaunchKernelGGL((k_enum_count<W, kWalkRing>), dim3(blocks), dim3(kBlock), 0, st, a, acc);
                break;
            case kWalkTorus:
                hipLaunchKernelGGL((k_enum_count<W, kWalkTorus>), dim3(blocks), dim3(kBlock), 0, st, a, acc);
                break;
            default: hipLaunchKernelGGL((k_enum_count<W, kWalkImages>), dim3(blocks), dim3(kBlock), 0, st, a, acc);
        }
        LS_HIP_CHECK(hipGetLastError());
        lo = hi;
    }
    LS_HIP_CHECK(hipMemcpyAsync(&total, acc, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    LS_HIP_CHECK(hipStreamSynchronize(st));
    return static_cast<uint64_t>(total);
}

uint64_t candidates_of(const GroupPlan &gp, int32_t weight) {
    const uint32_t n = gp.n_sites;
    if (weight >= 0) return host_binom(n, static_cast<uint32_t>(weight));
    return n == 64 ? ~0ULL : (1ULL << n);
}

}  // namespace

uint64_t count_members(ls_basis *b, uint64_t begin, uint64_t end, hipStream_t st) {
    const uint64_t total = candidate_count(b);
    end = std::min(end, total);
    if (begin >= end) return 0;
    StreamBuf acc_b(sizeof(unsigned long long), st);
    unsigned long long *acc = acc_b.as<unsigned long long>();
    const GroupPlan &gp = b->plan;
    return gp.n_sites <= 32 ? count_impl<uint32_t>(gp, b->plan_dev, b->d_binom, b->weight, begin, end, acc, st)
                            : count_impl<uint64_t>(gp, b->plan_dev, b->d_binom, b->weight, begin, end, acc, st);
}

// ---- the allocation-free count --------------------------------------------
//
// The same count for callers that cannot allocate device memory: the
// compiled group's tables and the accumulator live in `scratch`, a
// file-scope device array (kCountScratchBytes, and the walk's tables after
// them) that each GPU holds for the life of the process.  Host code never passes the array's name to a
// kernel or a copy (on the host it is only a stand-in symbol): the device
// address of each GPU's copy is taken once with hipGetSymbolAddress, with
// that GPU current, and used everywhere.  Calls are serialised by a
// process-wide lock, since every call on a GPU shares its array; calls from
// several processes on one GPU use separate arrays.

constexpr size_t kCountScratchBytes = 256 * 1024;
// the skip table of the walk lies after them: at most 4096 images of 64 bits
constexpr size_t kSkipBytes = 4096 * 64;
// and the torus tables: at most 8 base images, twice 4^6 entries, 32 codes
constexpr size_t kTorusBytes = 8 * sizeof(CosetRep) + 2 * 4096 * sizeof(uint32_t) + 32 * sizeof(uint32_t);
static __device__ __align__(256) unsigned char scratch[kCountScratchBytes + kSkipBytes + kTorusBytes];

namespace {

std::mutex g_scratch_mu;
void *g_scratch_ptr[256] = {};   // per device ordinal

void *scratch_address(int dev) {
    if (dev < 0 || dev >= 256) throw Error{LS_EDEVICE, "device ordinal out of range"};
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr)
            throw Error{LS_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

uint64_t count_members_noalloc(const GroupPlan &gp, int32_t weight, uint64_t begin, uint64_t end, hipStream_t st,
                               uint64_t *n_candidates) {
    const uint64_t total = candidates_of(gp, weight);
    if (n_candidates) *n_candidates = total;
    end = std::min(end, total);
    // layout: accumulator | binomials | cosets | characters | chi == 1 bits
    const PlanTables t = plan_tables();
    const size_t o_binom = 256;
    const size_t o_cos = align_up(o_binom + t.binom.size() * sizeof(uint64_t), 256);
    const size_t o_chi = align_up(o_cos + gp.cosets.size() * sizeof(CosetRep), 256);
    const size_t o_one = align_up(o_chi + gp.chi.size() / 2 * sizeof(double2), 256);
    const size_t need = align_up(o_one + gp.chi_one.size() * sizeof(uint32_t), 256);
    if (need > kCountScratchBytes)
        throw Error{LS_EINVAL, "the compiled group needs " + std::to_string(need) + " bytes of device tables, above the " +
                                   std::to_string(kCountScratchBytes) +
                                   "-byte scratch of the allocation-free count (use ls_sector_count)"};
    const std::vector<unsigned char> rows = gp.row_tables ? torus_tables(gp) : std::vector<unsigned char>();
    if (gp.skip.size() > kSkipBytes || rows.size() > kTorusBytes)
        throw Error{LS_EINTERNAL, "the walk's tables pass their scratch"};
    if (begin >= end) return 0;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    int dev = 0;
    LS_HIP_CHECK(hipGetDevice(&dev));
    unsigned char *base = static_cast<unsigned char *>(scratch_address(dev));
    auto put = [&](size_t off, const void *src, size_t bytes) {
        if (bytes) LS_HIP_CHECK(hipMemcpyAsync(base + off, src, bytes, hipMemcpyHostToDevice, st));
    };
    put(o_binom, t.binom.data(), t.binom.size() * sizeof(uint64_t));
    put(o_cos, gp.cosets.data(), gp.cosets.size() * sizeof(CosetRep));
    put(o_chi, gp.chi.data(), gp.chi.size() * sizeof(double));
    put(o_one, gp.chi_one.data(), gp.chi_one.size() * sizeof(uint32_t));
    put(kCountScratchBytes, gp.skip.data(), gp.skip.size());
    PlanDev pd{};
    fill_plan_dev(gp, pd);
    pd.cosets = reinterpret_cast<const CosetRep *>(base + o_cos);
    pd.chi = reinterpret_cast<const double2 *>(base + o_chi);
    pd.chi_one = reinterpret_cast<const uint32_t *>(base + o_one);
    pd.skip = base + kCountScratchBytes;
    if (!rows.empty()) {
        put(kCountScratchBytes + kSkipBytes, rows.data(), rows.size());
        set_torus_tables(gp, base + kCountScratchBytes + kSkipBytes, pd);
    }
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(base);
    const uint64_t *binom = reinterpret_cast<const uint64_t *>(base + o_binom);
    return gp.n_sites <= 32 ? count_impl<uint32_t>(gp, pd, binom, weight, begin, end, acc, st)
                            : count_impl<uint64_t>(gp, pd, binom, weight, begin, end, acc, st);
}

void build_basis(ls_basis *b, hipStream_t st) {
    const GroupPlan &gp = b->plan;
    const uint32_t n = gp.n_sites;
    upload_plan(b, st);

    const uint64_t total = candidate_count(b);
    switch (walk_kind(gp)) {
        case kWalkRing: enumerate_words<kWalkRing>(b, st, total); break;
        case kWalkTorus: enumerate_words<kWalkTorus>(b, st, total); break;
        default: enumerate_words<kWalkImages>(b, st, total);
    }

    // search layout
    SearchDev &S = b->search_dev;
    S.n_sites = n;
    S.weight = b->weight;
    S.dim = b->dim;
    S.reps = b->d_reps;
    std::vector<uint64_t> rank;   // host table of the rank layout, until the last synchronisation
    if (gp.n_elements == 1 && b->weight < 0) {
        S.mode = kLookupIdentity;
    } else if (gp.n_elements == 1) {
        S.mode = kLookupRank;
        const uint32_t w = static_cast<uint32_t>(b->weight);
        const std::vector<uint64_t> pascal = plan_tables().binom;
        const uint32_t chunks = (n + kRankBits - 1) / kRankBits;
        rank.assign((static_cast<size_t>(chunks) << kRankBits) * (w + 1), 0);
        for (uint32_t c = 0; c < chunks; ++c)
            for (uint32_t v = 0; v < (1u << kRankBits); ++v)
                for (uint32_t k = 0; k <= w; ++k) {
                    uint64_t r = 0;
                    uint32_t set = k;
                    for (uint32_t i = 0; i < kRankBits; ++i)
                        if (((v >> i) & 1u) && kRankBits * c + i < n && set < w) r += pascal[(kRankBits * c + i) * 65 + ++set];
                    rank[((static_cast<size_t>(c) << kRankBits) + v) * (w + 1) + k] = r;
                }
        b->d_rank = dev_alloc_n<uint64_t>(rank.size(), st);
        S.rank = b->d_rank;
        LS_HIP_CHECK(hipMemcpyAsync(b->d_rank, rank.data(), rank.size() * sizeof(uint64_t), hipMemcpyHostToDevice, st));
    } else {
        uint64_t kmin = 0, kmax = 0;
        if (b->dim > 0) {
            LS_HIP_CHECK(hipMemcpyAsync(&kmin, b->d_reps, sizeof(uint64_t), hipMemcpyDeviceToHost, st));
            LS_HIP_CHECK(hipMemcpyAsync(&kmax, b->d_reps + (b->dim - 1), sizeof(uint64_t), hipMemcpyDeviceToHost, st));
            LS_HIP_CHECK(hipStreamSynchronize(st));
        }
        S.kmin = kmin;
        S.kmax = kmax;
        // Hash index (index_lines); when it would pass 128 GiB, or when asked
        // for, the bucket search.
        const char *env = std::getenv("LS_ED_SEARCH");
        const bool want_buckets = env != nullptr && std::string(env) == "buckets";
        const uint32_t low_bits = b->weight >= 0 ? 7 : 5;
        uint32_t group_bits = 0;
        uint64_t lines = 0;
        if (!want_buckets) {
            StreamBuf groups_b(sizeof(uint64_t), st);
            unsigned long long *d_groups = groups_b.as<unsigned long long>(), groups = 0;
            hipLaunchKernelGGL(k_clear_u64, dim3(1), dim3(1), 0, st, d_groups);
            if (b->dim > 0)
                // (a workgroup a 256 rows: 0.74 ms of atomic adds for 6x6)
                hipLaunchKernelGGL(k_count_groups, dim3(std::min<uint64_t>(2048, grid_for(b->dim))), dim3(kBlock), 0,
                                   st, b->d_reps, b->dim, low_bits + kGroupBits, d_groups);
            LS_HIP_CHECK(hipGetLastError());
            LS_HIP_CHECK(hipMemcpyAsync(&groups, d_groups, sizeof(groups), hipMemcpyDeviceToHost, st));
            LS_HIP_CHECK(hipStreamSynchronize(st));
            lines = index_lines(b->dim, groups, &group_bits);
        }
        if (lines != 0) {
            S.mode = kLookupHash;
            S.hash_mask = lines - 1;
            S.hash_shift = 64;
            for (uint64_t c = lines; c > 1; c >>= 1) --S.hash_shift;
            // wide groups leave the entries no room for stabilizer sizes
            const bool wide = (kmax >> (low_bits + group_bits)) > kMaxGroup;
            S.index_format = low_bits | group_bits << 8 | ((wide ? kBlockTagWide : kBlockTag) - 32) << 16 |
                             (wide ? 0 : kBlockStabBits) << 24;
            // a key's number in its block: its low bits, or their rank among
            // those of their popcount
            uint8_t rank[128] = {}, next[8] = {};
            for (uint32_t v = 0; v < (1u << S.low_bits()); ++v)
                rank[v] = b->weight >= 0 ? next[__builtin_popcount(v)]++ : static_cast<uint8_t>(v);
            b->d_low_rank = dev_alloc_n<uint8_t>(sizeof(rank), st);
            LS_HIP_CHECK(hipMemcpyAsync(b->d_low_rank, rank, sizeof(rank), hipMemcpyHostToDevice, st));
            b->d_dropped = dev_alloc_n<uint64_t>(1 + kMaxDropped, st);
            hipLaunchKernelGGL(k_clear_u64, dim3(1), dim3(1), 0, st,
                               reinterpret_cast<unsigned long long *>(b->d_dropped));
            b->d_table = dev_alloc_n<IndexBlock>(lines << S.group_bits(), st);
            LS_HIP_CHECK(hipMemsetAsync(b->d_table, 0xFF, (lines << S.group_bits()) * sizeof(IndexBlock), st));
            S.table = b->d_table;
            S.low_rank = b->d_low_rank;
            S.stab = b->d_stab;
            S.dropped = b->d_dropped;
            if (b->dim > 0) {
                hipLaunchKernelGGL(k_index_claim, dim3(grid_for(b->dim)), dim3(kBlock), 0, st, S, b->d_table);
                hipLaunchKernelGGL(k_index_fill, dim3(grid_for(b->dim)), dim3(kBlock), 0, st, S, b->d_table);
            }
            LS_HIP_CHECK(hipGetLastError());
            LS_HIP_CHECK(hipStreamSynchronize(st));
            return;
        }
        S.mode = kLookupSearch;
        // about 4 keys per bucket, 2^8 .. 2^22 buckets
        uint32_t bits = 8;
        while (bits < 22 && (1ULL << bits) * 4 < b->dim) ++bits;
        const uint64_t range = kmax - kmin;
        uint32_t len = 0;
        while (len < 64 && (range >> len) != 0) ++len;
        S.bits = bits;
        S.shift = len > bits ? len - bits : 0;
        const uint64_t nb = (range >> S.shift) + 1;   // buckets 0 .. nb-1
        b->d_buckets = dev_alloc_n<uint32_t>(nb + 1, st);
        hipLaunchKernelGGL(k_buckets, dim3(grid_for(nb + 1)), dim3(kBlock), 0, st, b->d_reps, b->dim, kmin, S.shift,
                           nb, b->d_buckets);
        LS_HIP_CHECK(hipGetLastError());
        S.buckets = b->d_buckets;
    }
    LS_HIP_CHECK(hipStreamSynchronize(st));
}

void drop_key(ls_basis *b, uint64_t index, hipStream_t st) {
    const SearchDev &S = b->search_dev;
    LS_REQUIRE(S.mode == kLookupHash, "only a hash search layout can drop a key");
    LS_REQUIRE(b->n_dropped < kMaxDropped, "no more keys can be dropped");
    uint64_t key = 0;
    LS_HIP_CHECK(hipMemcpyAsync(&key, b->d_reps + index, sizeof(uint64_t), hipMemcpyDeviceToHost, st));
    LS_HIP_CHECK(hipStreamSynchronize(st));
    hipLaunchKernelGGL(k_drop_key, dim3(1), dim3(1), 0, st, S, b->d_table, b->d_dropped, key);
    ++b->n_dropped;
    LS_HIP_CHECK(hipGetLastError());
    LS_HIP_CHECK(hipStreamSynchronize(st));
}

namespace {

template <typename W, int KIND, uint32_t LX = 0, uint32_t LY = 0, uint32_t NZ = 0>
void run_state_info(const ls_basis *b, uint64_t n, const uint64_t *states, uint64_t *reps, double *chi, double *norm,
                    hipStream_t st) {
    constexpr uint64_t block = state_block<KIND>();
    // tori: two workgroups a CU, each staging the tables once
    const uint64_t most = KIND == kOrbitTorus ? 512 : ~0ull;
    const uint64_t grid = std::min<uint64_t>(most, (n + block - 1) / block);
    hipLaunchKernelGGL((k_state_info<W, KIND, LX, LY, NZ>), dim3(static_cast<uint32_t>(grid)), dim3(block), 0, st,
                       b->plan_dev, b->weight, n, states, reps, chi, norm);
}

}  // namespace

void launch_state_info(const ls_basis *b, uint64_t n, const uint64_t *states, uint64_t *reps, double *chi,
                       double *norm, hipStream_t st) {
    if (n == 0) return;
    const GroupPlan &gp = b->plan;
    const bool ring = gp.ly == 1 && gp.lx == gp.n_sites && gp.n_sites < 64;
    // The torus search looks at every image that ties with the smallest in two
    // rows, which with few spins a row are many; a walk of all images is as fast
    // for few of them and in small sectors, whose states have many symmetries
    // (1e6 states, search and walk: 6x6, 18 up, 288 images: 50 and 268 us; 6x5,
    // 11 up, 120 images: 70 and 81; 4x7, 14 up, 112: 111 and 102; 6x8, 7 up: 156
    // and 129; 6x10, 5 up: 238 and 159; 4x4: 234 and 179).
    const uint32_t images = gp.n_elements / (gp.pair_flip ? 2 : 1), w = static_cast<uint32_t>(b->weight);
    const bool search = gp.torus && gp.n_sites > 16 && images >= 120 &&
                        (b->weight < 0 || 5 * std::min(w, gp.n_sites - w) >= 6 * gp.ly);
    if (gp.n_sites <= 32) {
        if (ring) run_state_info<uint32_t, kOrbitRing32>(b, n, states, reps, chi, norm, st);
        else if (search) run_state_info<uint32_t, kOrbitTorus>(b, n, states, reps, chi, norm, st);
        else run_state_info<uint32_t, kOrbitGeneric>(b, n, states, reps, chi, norm, st);
    } else if (ring) {
        run_state_info<uint64_t, kOrbitRing64T>(b, n, states, reps, chi, norm, st);
    } else if (search && square_torus(gp) && gp.lx == 6) {
        run_state_info<uint64_t, kOrbitTorus, 6, 6, 2>(b, n, states, reps, chi, norm, st);
    } else if (search) {
        run_state_info<uint64_t, kOrbitTorus>(b, n, states, reps, chi, norm, st);
    } else {
        run_state_info<uint64_t, kOrbitGeneric>(b, n, states, reps, chi, norm, st);
    }
    LS_HIP_CHECK(hipGetLastError());
}

void launch_index_lookup(const ls_basis *b, uint64_t n, const uint64_t *keys, int64_t *index, hipStream_t st) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_index_lookup, dim3(grid_for(n)), dim3(kBlock), 0, st, b->search_dev, n, keys, index);
    LS_HIP_CHECK(hipGetLastError());
}

}  // namespace ls
