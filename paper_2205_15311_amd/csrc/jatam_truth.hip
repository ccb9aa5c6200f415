// jatam_truth.hip - the true class of a genotype: every growth order followed.
//
// The k runs of §3.2 sample growth orders, so a genotype whose every sampled
// run ends in one shape can still have an order that meets an ambiguous site
// or ends in another shape; the paper measures how this misclassification
// falls as k grows (§4.1).  The true class needs every order:
//   DET  every order ends in one shape without an event (size, D4 hash),
//   ND   some order meets an event (a bondable ring site, an ambiguous
//        site) or ends in a second shape (occupancy, without rotation).
//
// Three stages.
//   first       run 0 of every genotype (any order will do; solo_kernel's first
//               runs).  An event in it is reachable: ND.  A run that never
//               chose between two sites is the only order: DET.  A guarded
//               shape (no conflicting neighbour can be placed before the cell
//               it conflicts with, so every order places the same tiles) is
//               DET.  Anything else is queued.
//   narrow<W>   queued genotypes, sixteen lanes each: breadth first over the
//               event-free states (sets of placed (cell, tile) pairs), level by
//               level (a state of level L has L + 1 tiles, so states of one
//               level are only ever reached from the level before), a state in
//               each lane's own LDS grid, with its frontier.  An event ends the
//               search (ND), an empty frontier is a terminal shape, compared
//               with the first one found.  Successors are deduplicated in an
//               open-addressing table in LDS whose 64-bit slots hold a 32-bit
//               state hash and the successor itself (parent, cell, tile), so
//               equal hashes are settled by comparing the two states exactly and
//               no lane ever waits for another.  More than `cap` states:
//               undecided.  A level of more than sixteen states: to the next
//               stage.
//   wide<W>     the same search, one wave per genotype, with the levels in
//               device memory; a state's frontier is rebuilt from its tiles.
#include <new>

#include "jatam_assembly.hpp"
#include "jatam_internal.hpp"
#include "jatam_waves.hpp"

namespace jatam {

namespace {

// Words of one stored state: occupancy bitmap, 4-bit tiles of the occupied
// cells (zero elsewhere), and the state's hash.
template <int W>
struct StateLayout {
    using Geo = Geometry<W>;
    static constexpr int kOcc = 0;
    static constexpr int kPend = Geo::kWords;
    static constexpr int kHash = Geo::kWords + Geo::kPendWords;
    static constexpr int kWords = kHash + 1;
};

// Hash of one placed (cell, tile) pair; a state's hash is the XOR over its
// pairs, so a successor's hash is its parent's XOR one term.
__device__ __forceinline__ uint32_t pair_mix(uint32_t cell, uint32_t tile)
{
    uint32_t h = (cell * 16u + tile) * 0x9E3779B1u + 0x7F4A7C15u;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// Packed successor: parent index (bits 14..31), cell (4..13), tile (0..3).

__device__ __forceinline__ uint32_t succ_pack(uint32_t parent, uint32_t cell, uint32_t tile)
{
    return (parent << 14) | (cell << 4) | tile;   // parent < kMaxTruthLevel = 2^18
}

template <int W>
__device__ __forceinline__ uint32_t state_word(const uint32_t* parent, int w, uint32_t cell,
                                               uint32_t tile)
{
    using L = StateLayout<W>;
    uint32_t v = parent[w];
    if (w == L::kOcc + (int)(cell >> 5))
        v |= 1u << (cell & 31u);
    if (w == L::kPend + (int)(cell >> 3))
        v |= tile << ((cell & 7u) * 4u);
    return v;
}

// Whether parent_a + (cell_a, tile_a) and parent_b + (cell_b, tile_b) are the
// same set of pairs.
template <int W>
__device__ bool same_state(const uint32_t* level, uint32_t a, uint32_t b)
{
    using L = StateLayout<W>;
    const uint32_t pa = a >> 14, pb = b >> 14;
    if (pa == pb)
        return a == b;
    const uint32_t* sa = level + (size_t)pa * L::kWords;
    const uint32_t* sb = level + (size_t)pb * L::kWords;
    const uint32_t ca = (a >> 4) & 1023u, cb = (b >> 4) & 1023u;
    for (int w = 0; w < L::kHash; ++w)
        if (state_word<W>(sa, w, ca, a & 15u) != state_word<W>(sb, w, cb, b & 15u))
            return false;
    return true;
}

// Genotype i of the call.
__device__ __forceinline__ uint64_t truth_genome(const TruthArgs& a, uint64_t i)
{
    return a.genomes != nullptr ? a.genomes[i] : a.first + i;
}

}  // namespace

// ---------------------------------------------------------------------------
// Narrow searches: sixteen lanes per queued genotype, everything in LDS.
//
// Bound by the chain of LDS reads and writes per level (copying a state's grid,
// placing a tile, checking its neighbours), whatever the width.  A search has
// seven states on average over S_{2,8}, at most 19, and never more than sixteen a
// level, so a wave takes four at once.  The 35,553 searches of a quarter of
// S_{2,8}: 72 us; one wave a search with its levels in device memory (the wide
// search, 256 waves) 5.4 ms.
// ---------------------------------------------------------------------------
constexpr int kNarrow = 16;          // states per level, and lanes per genotype
constexpr int kNarrowSlots = 2 * kNarrow;

// Whether two successors of states in the wave's grids are the same set of pairs.
// The PEND nibble of the successor's new cell, on the frontier of its parent, is
// the tile placed there, so its parent's nibbles are the successor's too.
template <int W>
__device__ __forceinline__ bool same_successor(const uint32_t* states, uint32_t a, uint32_t b)
{
    using Geo = Geometry<W>;
    if ((a >> 14) == (b >> 14))
        return a == b;
    const uint32_t* const sa = states + (a >> 14);
    const uint32_t* const sb = states + (b >> 14);
    const uint32_t ca = (a >> 4) & 1023u, cb = (b >> 4) & 1023u;
    for (uint32_t w = 0; w < (uint32_t)Geo::kWords; ++w) {
        const uint32_t oa = sa[(Geo::kOcc + w) * 64] | ((ca >> 5) == w ? 1u << (ca & 31u) : 0u);
        const uint32_t ob = sb[(Geo::kOcc + w) * 64] | ((cb >> 5) == w ? 1u << (cb & 31u) : 0u);
        if (oa != ob)
            return false;
        if (oa == 0)
            continue;
        uint32_t differ = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            uint32_t cells = (oa >> (8 * k)) & 0xFFu;   // one bit a nibble
            cells = (cells | (cells << 12)) & 0x000F000Fu;
            cells = (cells | (cells << 6)) & 0x03030303u;
            cells = (cells | (cells << 3)) & 0x11111111u;
            const uint32_t at = (Geo::kPend + 4 * w + k) * 64;
            differ |= (sa[at] ^ sb[at]) & (cells * 15u);
        }
        if (differ != 0)
            return false;
    }
    return true;
}

template <int W, class M>
__global__ __launch_bounds__(64) void truth_narrow_kernel(TruthArgs a)
{
    using Geo = Geometry<W>;
    constexpr int kGroups = 64 / kNarrow;
    constexpr int kCopy = 8;   // words copied at a time: all read, then all written
    static_assert(Geo::kLaneWords % kCopy == 0, "whole copies");
    __shared__ uint32_t smem[Geo::kLaneWords * 64];
    __shared__ unsigned long long tables[kGroups][kNarrowSlots];
    __shared__ uint32_t lists[kGroups][kNarrow];     // the next level's states
    __shared__ uint32_t refs[kGroups][Geo::kWords];  // the first terminal shapes
    __shared__ uint32_t nexts[kGroups];
    const uint32_t lane = (uint32_t)lane_id(), sub = lane % kNarrow, grp = lane / kNarrow;
    const uint32_t lead = grp * kNarrow;
    const uint64_t mates = ((1ull << kNarrow) - 1) << lead;   // the group's lanes
    unsigned long long* const table = tables[grp];
    LaneGrid<W, 64> g{smem + lane};
    g.clear_all();
    RunState st{};
    const int G = a.grid;
    const uint32_t nq = a.counters[0];
    uint64_t k = (uint64_t)blockIdx.x * kGroups + grp;
    // uniform over the group
    bool busy = false, have_ref = false;
    uint32_t i = 0, width = 0;
    int64_t total = 0;
    int ref_size = 0;
    M m{};
    // the lane's state: its hash, and the event met in reaching it
    uint32_t hash = 0;
    int ev = kEvNone;
    for (;;) {
        // -- groups without a genotype take their next one --------------------
        while (!busy && k < nq) {
            i = a.queue[k];
            k += (uint64_t)gridDim.x * kGroups;
            const uint64_t genome = truth_genome(a, i);
            m = build_bonds<M>(genome, a.t, a.bits, a.c);
            busy = true;
            if constexpr (M::kManyIds) {
                // the first stage may not know where the sixteenth oriented tile
                // lies and proves nothing then: its proof is made up for here
                if (a.t == 4) {
                    bool guarded = false;
                    if (sub == 0) {
                        const uint64_t rid = genome | ((uint64_t)(uint32_t)a.t << 56);
                        run_assembly(m, g, st, G,
                                     RunKey{a.key0, a.key1, (uint32_t)rid,
                                            (uint32_t)(rid >> 32), 0});
                        uint64_t key = 0;
                        int x0 = 0, y0 = 0;
                        const bool fits = shape_key8(g, st, G, st.size(), key, x0, y0);
                        guarded = shape_is_guarded(m, g, TileIds{true, 0ull}, G, fits, key, x0, y0);
                        if (guarded)
                            a.out[i] = jatam_result_t{JATAM_DET, st.size(), shape_hash(g, G), 0};
                    }
                    busy = (__ballot(guarded) & mates) == 0;
                }
            }
            if (busy) {
                // level 0: the seed alone (tile id 0: tile 0 unrotated)
                if (sub == 0) {
                    ev = run_start(m, g, st, G);
                    hash = pair_mix((uint32_t)((G / 2 - 1) * W + (G / 2 - 1)), 0u);
                }
                width = 1;
                total = 1;
                have_ref = false;
            }
        }
        if (__ballot(busy) == 0)
            break;
        // -- the level's events and terminal shapes, and its successors --------
        const bool mine = busy && sub < width;
        const bool event = (__ballot(mine && ev != kEvNone) & mates) != 0;
        const bool terminal = mine && !event && st.nf == 0;
        for (uint32_t j = sub; j < (uint32_t)kNarrowSlots; j += kNarrow)
            table[j] = 0ull;
        if (sub == 0)
            nexts[grp] = 0;
        wave_lds_sync();
        bool wide = false;
        if (mine && !event && !terminal) {
            for (uint32_t fs = st.touched<W>(); fs != 0; fs &= fs - 1) {
                const int w = __builtin_ctz(fs);
                for (uint32_t cells = g.fr(w); cells != 0; cells &= cells - 1) {
                    const uint32_t q = (uint32_t)((w << 5) | __builtin_ctz(cells));
                    const uint32_t tile = g.tile_id((int)q);
                    const uint32_t succ = succ_pack(sub, q, tile);
                    const uint32_t h = hash ^ pair_mix(q, tile);
                    const unsigned long long key = ((unsigned long long)(h | 1u) << 32) | succ;
                    uint32_t slot = h % kNarrowSlots;
                    uint32_t probe = 0;
                    for (; probe < (uint32_t)kNarrowSlots; ++probe) {
                        const unsigned long long old = atomicCAS(&table[slot], 0ull, key);
                        if (old == 0ull) {
                            const uint32_t pos = atomicAdd(&nexts[grp], 1u);
                            if (pos < (uint32_t)kNarrow && pos < a.max_level)
                                lists[grp][pos] = succ;
                            else
                                wide = true;
                            break;
                        }
                        if ((old >> 32) == (key >> 32) &&
                            same_successor<W>(smem + lead, (uint32_t)old, succ))
                            break;   // already inserted by another path
                        slot = (slot + 1u) % kNarrowSlots;
                    }
                    wide = wide || probe == (uint32_t)kNarrowSlots;   // table full
                }
            }
        }
        wave_lds_sync();
        const uint32_t found = nexts[grp];
        const bool too_wide = (__ballot(wide) & mates) != 0;
        const uint64_t tm = __ballot(terminal) & mates;
        const uint32_t first = tm != 0 ? (uint32_t)__builtin_ctzll(tm) : lane;
        const int first_size = __shfl(st.size(), (int)first);
        if (tm != 0 && !have_ref) {
            if (lane == first)
                for (int w = 0; w < Geo::kWords; ++w)
                    refs[grp][w] = g.occ(w);
            have_ref = true;
            ref_size = first_size;
        }
        wave_lds_sync();
        bool other = false;
        if (terminal)
            for (int w = 0; w < Geo::kWords; ++w)
                other = other || g.occ(w) != refs[grp][w];
        const bool second = (__ballot(other) & mates) != 0;
        // -- the end of the search ---------------------------------------------
        bool stop = true, report = true;
        int verdict = -2;   // undecided
        if (event)
            verdict = JATAM_ND_SITE;
        else if (too_wide)
            report = false;
        else if (second)
            verdict = JATAM_ND_SITE;
        else if (total + (int64_t)found > a.cap)
            verdict = -2;
        else if (found == 0)
            verdict = have_ref ? JATAM_DET : -2;
        else
            stop = false;
        if (busy && stop && sub == 0) {
            if (report) {
                jatam_result_t rec{verdict, 0, 0u,
                                   (int32_t)(total < 0x7FFFFFFF ? total : 0x7FFFFFFF)};
                if (verdict == JATAM_DET) {
                    // without successors every state of the level is terminal
                    rec.size = ref_size;
                    rec.hash = shape_hash(g, G);
                }
                a.out[i] = rec;
            } else {
                a.wide[atomicAdd(a.counters + 1, 1u)] = i;
            }
        }
        busy = busy && !stop;
        // -- the next level's states, each in the grid of its lane ----------------
        const bool child = busy && sub < found;
        const uint32_t succ = child ? lists[grp][sub] : sub << 14;
        const uint32_t from = lead + (succ >> 14);
        const uint32_t* const src = smem + from;
        wave_lds_sync();
#pragma unroll 1
        for (int w = 0; w < Geo::kLaneWords; w += kCopy) {
            uint32_t v[kCopy];
#pragma unroll
            for (int j = 0; j < kCopy; ++j)
                v[j] = src[(w + j) * 64];
            wave_lds_sync();
            if (child)
#pragma unroll
                for (int j = 0; j < kCopy; ++j)
                    g.word(w + j) = v[j];
            wave_lds_sync();
        }
        const uint32_t nf = (uint32_t)__shfl((int)st.nf, (int)from);
        const uint32_t osum = (uint32_t)__shfl((int)st.osum, (int)from);
        const int steps = __shfl(st.steps, (int)from);
        const uint32_t parent_hash = (uint32_t)__shfl((int)hash, (int)from);
        if (child) {
            const uint32_t q = (succ >> 4) & 1023u, tile = succ & 15u;
            st.nf = nf - 1u;
            st.osum = osum | (1u << (q >> 5));
            st.steps = steps + 1;
            hash = parent_hash ^ pair_mix(q, tile);
            g.occ((int)(q >> 5)) |= 1u << (q & 31u);
            g.fr((int)(q >> 5)) &= ~(1u << (q & 31u));
            ev = update_site(m, g, st, G, (int)q, m.oriented(tile));
        }
        if (busy) {
            width = found;
            total += found;
        }
    }
}

// ---------------------------------------------------------------------------
// Wide searches: one wave per genotype, the levels in device memory.
// ---------------------------------------------------------------------------
template <int W, class M>
__global__ __launch_bounds__(64) void truth_wide_kernel(TruthArgs a)
{
    using Geo = Geometry<W>;
    using L = StateLayout<W>;
    __shared__ uint32_t smem[Geo::kLaneWords * 64];
    __shared__ uint32_t s_next, s_terms, s_flags;   // flags: 1 event/second shape, 2 overflow
    __shared__ uint32_t s_ref[Geo::kWords];         // the first terminal shape
    const int lane = (int)threadIdx.x;
    LaneGrid<W, 64> g{smem + lane};
    const uint32_t maxw = a.max_level;
    uint32_t* const level0 = a.arena + (size_t)blockIdx.x * 2 * maxw * L::kWords;
    uint32_t* const level1 = level0 + (size_t)maxw * L::kWords;
    uint32_t* const list = a.lists + (size_t)blockIdx.x * maxw;
    uint32_t* const terms = a.terms + (size_t)blockIdx.x * maxw;
    unsigned long long* const table = a.tables + ((size_t)blockIdx.x << a.table_log2);
    const uint32_t tmask = (1u << a.table_log2) - 1u;

    for (;;) {
        uint32_t k = 0;
        if (lane == 0)
            k = atomicAdd(a.counters + 2, 1u);
        k = (uint32_t)__shfl((int)k, 0);
        if (k >= a.counters[1])
            break;
        const uint32_t i = a.wide[k];
        const uint64_t genome = truth_genome(a, i);
        const M m = build_bonds<M>(genome, a.t, a.bits, a.c);
        const int G = a.grid;
        const int seed = (G / 2 - 1) * W + (G / 2 - 1);
        // level 0: the seed alone (tile id 0: tile 0 unrotated)
        for (int w = lane; w < L::kWords; w += 64) {
            uint32_t v = 0;
            if (w == L::kOcc + (seed >> 5))
                v = 1u << (seed & 31);
            if (w == L::kHash)
                v = pair_mix((uint32_t)seed, 0u);
            level0[w] = v;
        }
        uint32_t* cur = level0;
        uint32_t* nxt = level1;
        uint32_t width = 1;
        int64_t total = 1;
        bool have_ref = false;
        int ref_size = 0;
        int verdict = -2;   // undecided until the search ends
        if (lane == 0)
            s_flags = 0;
        __syncthreads();
        for (;;) {
            if (lane == 0) {
                s_next = 0;
                s_terms = 0;
            }
            __syncthreads();
            // -- analyse the level's states, insert their successors --------
            for (uint32_t s = (uint32_t)lane; s < width; s += 64) {
                const uint32_t* src = cur + (size_t)s * L::kWords;
                RunState st{};
                for (int w = 0; w < Geo::kWords; ++w) {
                    const uint32_t o = src[L::kOcc + w];
                    g.occ(w) = o;
                    g.fr(w) = 0;
                    st.osum |= (o != 0 ? 1u : 0u) << w;
                }
                for (int w = 0; w < Geo::kPendWords; ++w)
                    g.word(Geo::kPend + w) = src[L::kPend + w];
                int ev = kEvNone;
                for (uint32_t os = st.osum; os != 0; os &= os - 1) {
                    const int w = __builtin_ctz(os);
                    for (uint32_t cells = g.occ(w); cells != 0; cells &= cells - 1) {
                        const int p = (w << 5) | __builtin_ctz(cells);
                        const uint32_t id =
                            (g.pend_word(p) >> ((uint32_t)(p & 7) * 4u)) & 15u;
                        const int e = update_site(m, g, st, G, p, m.oriented(id));
                        ev = e != kEvNone ? e : ev;
                    }
                }
                if (ev != kEvNone) {
                    atomicOr(&s_flags, 1u);
                } else if (st.nf == 0) {
                    const uint32_t pos = atomicAdd(&s_terms, 1u);
                    terms[pos] = s;
                } else {
                    const uint32_t h0 = src[L::kHash];
                    for (uint32_t fs = st.touched<W>(); fs != 0; fs &= fs - 1) {
                        const int w = __builtin_ctz(fs);
                        for (uint32_t cells = g.fr(w); cells != 0; cells &= cells - 1) {
                            const uint32_t q = (uint32_t)((w << 5) | __builtin_ctz(cells));
                            const uint32_t tile = (g.pend_word((int)q) >> ((q & 7u) * 4u)) & 15u;
                            const uint32_t succ = succ_pack(s, q, tile);
                            const uint32_t h = h0 ^ pair_mix(q, tile);
                            const unsigned long long key =
                                ((unsigned long long)(h | 1u) << 32) | succ;
                            uint32_t slot = h & tmask;
                            for (uint32_t probe = 0;; ++probe) {
                                if (probe > tmask) {   // table full
                                    atomicOr(&s_flags, 2u);
                                    break;
                                }
                                const unsigned long long old = atomicCAS(&table[slot], 0ull, key);
                                if (old == 0ull) {
                                    const uint32_t pos = atomicAdd(&s_next, 1u);
                                    if (pos < maxw)
                                        list[pos] = slot;
                                    else
                                        atomicOr(&s_flags, 2u);
                                    break;
                                }
                                if ((old >> 32) == (key >> 32) &&
                                    same_state<W>(cur, (uint32_t)old, succ))
                                    break;   // already inserted by another path
                                slot = (slot + 1u) & tmask;
                            }
                        }
                    }
                }
            }
            __syncthreads();
            const uint32_t flags = s_flags;
            const uint32_t nnext = s_next < maxw ? s_next : maxw;
            const uint32_t nterms = s_terms;
            // -- terminal shapes: the first one is the reference ------------
            if (flags == 0 && nterms > 0) {
                if (!have_ref) {
                    const uint32_t* r = cur + (size_t)terms[0] * L::kWords;
                    for (int w = lane; w < Geo::kWords; w += 64)
                        s_ref[w] = r[L::kOcc + w];
                    __syncthreads();
                    have_ref = true;
                    ref_size = 0;
                    for (int w = 0; w < Geo::kWords; ++w)
                        ref_size += __popc(s_ref[w]);
                }
                for (uint32_t j = (uint32_t)lane; j < nterms; j += 64) {
                    const uint32_t* r = cur + (size_t)terms[j] * L::kWords;
                    bool same = true;
                    for (int w = 0; w < Geo::kWords; ++w)
                        same = same && r[L::kOcc + w] == s_ref[w];
                    if (!same)
                        atomicOr(&s_flags, 1u);
                }
                __syncthreads();
            }
            const uint32_t flags2 = s_flags;
            bool stop = false;
            if (flags2 & 1u) {
                verdict = JATAM_ND_SITE;
                stop = true;
            } else if ((flags2 & 2u) || total + (int64_t)nnext > a.cap) {
                verdict = -2;
                stop = true;
            } else if (nnext == 0) {
                verdict = have_ref ? JATAM_DET : -2;
                stop = true;
            }
            if (stop) {
                // leave the table empty for the next genotype
                if (flags2 & 2u) {
                    for (uint32_t j = (uint32_t)lane; j <= tmask; j += 64)
                        table[j] = 0ull;
                } else {
                    for (uint32_t j = (uint32_t)lane; j < nnext; j += 64)
                        table[list[j]] = 0ull;
                }
                __syncthreads();
                break;
            }
            // -- the next level's states, written out; table emptied ----------
            for (uint32_t j = (uint32_t)lane; j < nnext; j += 64) {
                const uint32_t slot = list[j];
                const uint32_t succ = (uint32_t)table[slot];
                table[slot] = 0ull;
                const uint32_t* src = cur + (size_t)(succ >> 14) * L::kWords;
                const uint32_t cell = (succ >> 4) & 1023u, tile = succ & 15u;
                uint32_t* dst = nxt + (size_t)j * L::kWords;
                for (int w = 0; w < L::kHash; ++w)
                    dst[w] = state_word<W>(src, w, cell, tile);
                dst[L::kHash] = src[L::kHash] ^ pair_mix(cell, tile);
            }
            __syncthreads();
            uint32_t* tmp = cur;
            cur = nxt;
            nxt = tmp;
            width = nnext;
            total += nnext;
        }
        if (lane == 0) {
            jatam_result_t rec{verdict, 0, 0u, (int32_t)(total < 0x7FFFFFFF ? total : 0x7FFFFFFF)};
            if (verdict == JATAM_DET)
                rec.size = ref_size;
            a.out[i] = rec;
        }
        if (verdict == JATAM_DET) {
            // the D4 hash of the reference shape, on lane 0's LDS grid
            if (lane == 0) {
                for (int w = 0; w < Geo::kWords; ++w)
                    g.occ(w) = s_ref[w];
                a.out[i].hash = shape_hash(g, G);
            }
        }
        __syncthreads();
    }
}

// Words of the counters and, after them, one class's claim counters.
constexpr int kTruthCounters = 64;
constexpr int kTruthReset = kTruthCounters + kClaimCounters * kClaimStride;

__global__ void truth_reset_kernel(uint32_t* counters)
{
    for (int k = (int)threadIdx.x; k < kTruthReset; k += (int)blockDim.x)
        counters[k] = 0;
}

template <int W, class M>
static void launch_truth_t(const TruthArgs& a, int narrow, int wide, hipStream_t s)
{
    // (a queue that holds every genotype gives each group of lanes one)
    const uint64_t most = ((uint64_t)a.n * kNarrow + 63) / 64;
    const uint32_t blocks = most < (uint64_t)narrow ? (uint32_t)most : (uint32_t)narrow;
    hipLaunchKernelGGL((truth_narrow_kernel<W, M>), dim3(blocks), dim3(64), 0, s, a);
    hipLaunchKernelGGL((truth_wide_kernel<W, M>), dim3(wide), dim3(64), 0, s, a);
}

template <class M>
static void truth_waves_t(TruthWaves& w, int geno, int cus)
{
    w.narrow[0][geno] = cus * resident_per_cu(truth_narrow_kernel<16, M>);
    w.narrow[1][geno] = cus * resident_per_cu(truth_narrow_kernel<32, M>);
}

static bool truth_waves(TruthWaves& w)
{
    int dev = -1, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
        return false;
    solo_occupancy(w.first);
    for (auto& klass : w.first)
        for (int& n : klass)
            n *= cus;
    truth_waves_t<Bonds2>(w, kGenoTwo, cus);
    truth_waves_t<Bonds4>(w, kGenoFour, cus);
    truth_waves_t<BondsC16>(w, kGenoC16, cus);
    return true;
}

int launch_truth(const TruthArgs& a, const Params& p, const TruthWaves& waves, hipStream_t s)
{
    if (a.max_level > kMaxTruthLevel || a.max_level == 0)
        return JATAM_E_INVALID_ARG;
    const int geno = geno_kind(a.t, a.c), klass = a.grid <= 16 ? 0 : 1;
    hipLaunchKernelGGL(truth_reset_kernel, dim3(1), dim3(256), 0, s, a.counters);
    // the first stage's chunks are claimed as in the classification's first runs
    // (a quarter of S_{2,8} 0.37 ms, all of them dealt out 0.50)
    DeviceWorkspace ws{};
    uint32_t* const claims = a.counters + kTruthCounters;
    ws.run_claim = claims - klass * kClaimCounters * kClaimStride;
    const jatam_tuning_t tuning = default_tuning(klass);
    constexpr int64_t kPiece = (int64_t)1 << 31;
    for (int64_t at = 0; at < a.n; at += kPiece) {
        BatchArgs b =
            batch_args_for(p, a.n - at < kPiece ? a.n - at : kPiece, a.out + at, nullptr, ws);
        b.dyn16 = tuning.claim_share;
        b.claim_chunks = tuning.claim_chunks;
        if (at > 0)
            launch_clear(claims, nullptr, s);
        b.genomes = a.genomes != nullptr ? a.genomes + at : nullptr;
        b.first = a.first + (uint64_t)at;
        launch_first_open(b, waves.first[klass][geno], geno,
                          OpenList{a.queue, a.counters, (uint32_t)at}, s);
    }
    const int narrow = waves.narrow[klass][geno];
    if (klass == 0) {
        if (geno == kGenoTwo)
            launch_truth_t<16, Bonds2>(a, narrow, waves.wide, s);
        else if (geno == kGenoFour)
            launch_truth_t<16, Bonds4>(a, narrow, waves.wide, s);
        else
            launch_truth_t<16, BondsC16>(a, narrow, waves.wide, s);
    } else {
        if (geno == kGenoTwo)
            launch_truth_t<32, Bonds2>(a, narrow, waves.wide, s);
        else if (geno == kGenoFour)
            launch_truth_t<32, Bonds4>(a, narrow, waves.wide, s);
        else
            launch_truth_t<32, BondsC16>(a, narrow, waves.wide, s);
    }
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam

// ---------------------------------------------------------------------------
// C ABI.
// ---------------------------------------------------------------------------
struct jatam_truth {
    int64_t max_n;
    uint32_t max_level;
    jatam::TruthWaves waves;
    void* region;
    jatam::TruthArgs a;   // workspace pointers
};

namespace {

int truth_launch(jatam_truth_t* w, const uint64_t* genotypes, uint64_t first, int64_t n, int t,
                 int c, int grid_limit, int64_t cap, jatam_result_t* out, void* stream)
{
    if (w == nullptr || n < 0 || n > w->max_n || cap < 1 || (n > 0 && out == nullptr))
        return JATAM_E_INVALID_ARG;
    jatam::Params p;
    const int rc = jatam::make_params(t, c, grid_limit, 1, 1, &p);
    if (rc != JATAM_OK)
        return rc;
    if (n == 0)
        return JATAM_OK;
    jatam::TruthArgs a = w->a;
    a.genomes = genotypes;
    a.first = first;
    a.n = n;
    a.t = p.t;
    a.c = p.c;
    a.bits = p.bits;
    a.genome_bits = p.genome_bits;
    a.grid = p.grid;
    a.key0 = p.key0;
    a.key1 = p.key1;
    a.cap = cap;
    a.out = out;
    return jatam::launch_truth(a, p, w->waves, (hipStream_t)stream);
}

}  // namespace

extern "C" {

int jatam_truth_create(int64_t max_n, int32_t max_level, int32_t waves, jatam_truth_t** out)
{
    if (out == nullptr)
        return JATAM_E_INVALID_ARG;
    *out = nullptr;
    if (max_n < 1 || max_n > (int64_t(1) << 32) || max_level < 1 ||
        (uint32_t)max_level > jatam::kMaxTruthLevel || waves < 1 || waves > 4096)
        return JATAM_E_INVALID_ARG;
    jatam_truth_t* w = new (std::nothrow) jatam_truth_t();
    if (w == nullptr)
        return JATAM_E_HIP;
    w->max_n = max_n;
    w->max_level = (uint32_t)max_level;
    w->waves.wide = waves;
    if (!jatam::truth_waves(w->waves)) {
        delete w;
        return JATAM_E_HIP;
    }
    int tl = 1;
    while ((int64_t(1) << tl) < 2 * (int64_t)max_level)
        ++tl;
    // both grid classes fit the 32 x 32 state size
    const size_t sw = (size_t)jatam::truth_state_words(32);
    const size_t counters = ((size_t)jatam::kTruthReset * 4 + 255) / 256 * 256;
    const size_t queue = ((size_t)max_n * 4 + 255) / 256 * 256;
    const size_t arena = (size_t)waves * 2 * max_level * sw * 4;
    const size_t lists = ((size_t)waves * max_level * 4 + 255) / 256 * 256;
    const size_t tables = (size_t)waves * (size_t(1) << tl) * 8;
    const size_t total = counters + 2 * queue + 2 * lists + arena + tables;
    uint8_t* base = nullptr;
    if (hipMalloc((void**)&base, total) != hipSuccess) {
        delete w;
        return JATAM_E_HIP;
    }
    // the tables start empty and every call leaves them empty
    if (hipMemset(base, 0, total) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        (void)hipFree(base);
        delete w;
        return JATAM_E_HIP;
    }
    w->region = base;
    jatam::TruthArgs& a = w->a;
    a = jatam::TruthArgs{};
    size_t off = 0;
    a.counters = (uint32_t*)(base + off);
    off += counters;
    a.tables = (unsigned long long*)(base + off);
    off += tables;
    a.queue = (uint32_t*)(base + off);
    off += queue;
    a.wide = (uint32_t*)(base + off);
    off += queue;
    a.lists = (uint32_t*)(base + off);
    off += lists;
    a.terms = (uint32_t*)(base + off);
    off += lists;
    a.arena = (uint32_t*)(base + off);
    a.max_level = (uint32_t)max_level;
    a.table_log2 = tl;
    *out = w;
    return JATAM_OK;
}

int jatam_truth_destroy(jatam_truth_t* w)
{
    if (w == nullptr)
        return JATAM_OK;
    const hipError_t e = hipFree(w->region);
    delete w;
    return e == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

int jatam_true_class(jatam_truth_t* w, const uint64_t* genotypes, int64_t n, int t, int c,
                     int grid_limit, int64_t cap, jatam_result_t* out, void* stream)
{
    if (n > 0 && genotypes == nullptr)
        return JATAM_E_INVALID_ARG;
    return truth_launch(w, genotypes, 0, n, t, c, grid_limit, cap, out, stream);
}

int jatam_true_class_range(jatam_truth_t* w, uint64_t first, int64_t n, int t, int c,
                           int grid_limit, int64_t cap, jatam_result_t* out, void* stream)
{
    if (n > 0) {
        jatam::Params p;
        const int rc = jatam::make_params(t, c, grid_limit, 1, 1, &p);
        if (rc != JATAM_OK)
            return rc;
        const uint64_t last = first + (uint64_t)(n - 1);
        if (last < first || (p.genome_bits < 64 && (last >> p.genome_bits) != 0))
            return JATAM_E_INVALID_ARG;
    }
    return truth_launch(w, nullptr, first, n, t, c, grid_limit, cap, out, stream);
}

}  // extern "C"
