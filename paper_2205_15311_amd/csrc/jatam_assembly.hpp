// jatam_assembly.hpp - one lane's assembly run on gfx950, shared by the one-launch,
// the pipeline's and the variants' kernels.
//
// A lane's grid lives in LDS as
//   OCC   occupancy bitmap, W*W bits
//   FR    frontier bitmap (sites with exactly one admissible tile), W*W bits
//   PEND  the pending tile of every frontier site, 4 bits per cell
// in a lane-interleaved layout (word k of the lane with thread index j at
// smem[k*B + j]), so a wave's 64 lanes always touch 64 consecutive dwords and
// never conflict in a bank, whatever cells they address.
//
// Grid layout.  The bounded (G-1)-square is stored at cells (x, y) in
// [0, G-2]^2 of a W x W torus (W = 16 or 32 >= G), cell index y*W + x.  Its
// ring - the sites just outside the box - is every cell with x >= G-1 or
// y >= G-1: stepping E or S off the box lands on x or y = G-1, and stepping W
// or N off it wraps (mod W*W) onto x or y = W-1.  Cell order y*W + x is the
// row-major frontier order.  Only the words a run touched are cleared for the
// next run (the paper finds 83% of its time in re-initialising grids and
// proposes exactly this, §5.2).
#pragma once

#include "jatam_device.hpp"
#include "jatam_shapes.hpp"

namespace jatam {

template <int W>
struct Geometry {
    static_assert(W == 16 || W == 32, "W must be 16 or 32");
    static constexpr int kLogW = W == 16 ? 4 : 5;
    static constexpr int kCells = W * W;
    static constexpr int kWords = kCells / 32;       // bitmap words
    static constexpr int kPendWords = kCells / 8;    // 4-bit cells
    static constexpr int kOcc = 0;
    static constexpr int kFr = kWords;
    static constexpr int kPend = 2 * kWords;
    static constexpr int kLaneWords = 2 * kWords + kPendWords;
};

// LDS atomic OR without return: sets bits with no read on the critical path.
__device__ __forceinline__ void set_bits(uint32_t& w, uint32_t bits)
{
    __hip_atomic_fetch_or(&w, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Per-lane view of the workgroup's LDS.
template <int W, int B>
struct LaneGrid {
    using Geo = Geometry<W>;
    static constexpr int kW = W;
    static constexpr bool kLean = false;
    static constexpr int kPend = Geo::kPend;
    uint32_t* base;   // &smem[threadIdx.x]

    __device__ __forceinline__ uint32_t& word(int k) { return base[k * B]; }
    __device__ __forceinline__ uint32_t& occ(int w) { return word(Geo::kOcc + w); }
    __device__ __forceinline__ uint32_t& fr(int w) { return word(Geo::kFr + w); }

    __device__ __forceinline__ bool occupied(int p) { return (occ(p >> 5) >> (p & 31)) & 1u; }
    // every word of the lane's grid, PEND included (kernel start)
    __device__ __forceinline__ void clear_all()
    {
        for (int k = 0; k < Geo::kLaneWords; ++k)
            word(k) = 0;
    }
    __device__ __forceinline__ uint32_t& pend_word(int p) { return word(Geo::kPend + (p >> 3)); }
    // the tile's id at an occupied cell
    __device__ __forceinline__ uint32_t tile_id(int p)
    {
        return (pend_word(p) >> ((uint32_t)(p & 7) * 4u)) & 15u;
    }
    __device__ __forceinline__ uint32_t row(int y)
    {
        if constexpr (W == 32) {
            return occ(y);
        } else {
            return (occ(y >> 1) >> ((y & 1) * 16)) & 0xFFFFu;
        }
    }
};

// The grid of the first-run kernel, one wave a workgroup: FR and PEND only,
// 40 words a lane instead of 48 (16 x 16) or 160 instead of 192 (32 x 32),
// which lets 14 waves instead of 10, or 4 instead of 3, share a CU's LDS.  A
// nibble holds tag = id + 1 (mod 16), and a cell off the frontier is occupied
// exactly when its nibble is not zero: so a step reads, tests and writes three
// words less too.  Id 15 has tag 0, which is fine on the frontier (FR tells);
// a cell placed with it takes the tag 1 instead, that of id 0, and the run's tiles
// count as lost: its shape waits for a proof of its own, in which shape_ids tells
// the two apart from their neighbours.
// The occupied cells near the seed are kept as a bitmap in a register
// (RunState::near) for the shape at the run's end.
//
// Row W-1 is never part of the box: the words that only it uses (`spare`,
// spare_words() of them) are free for the wave's own data.  A step may read
// them and write them back unchanged, and nothing clears them.
template <int W>
struct LeanGrid {
    using Geo = Geometry<W>;
    static constexpr int kW = W;
    static constexpr bool kLean = true;
    static constexpr int kFr = 0;
    static constexpr int kPend = Geo::kWords;
    static constexpr int kLaneWords = Geo::kWords + Geo::kPendWords;
    // all lanes' PEND words of row W-1, and (W = 32) its FR word
    static constexpr int kSpare = (kLaneWords - W / 8) * 64;
    static constexpr int kSpareFr = W == 32 ? (W - 1) * 64 : -1;
    uint32_t* base;   // &smem[lane]

    __device__ __forceinline__ uint32_t& word(int k) { return base[k * 64]; }
    __device__ __forceinline__ uint32_t& fr(int w) { return word(kFr + w); }
    __device__ __forceinline__ uint32_t& pend_word(int p) { return word(kPend + (p >> 3)); }
    __device__ __forceinline__ void clear_all()
    {
        for (int k = 0; k < kLaneWords; ++k)
            word(k) = 0;
    }
    // Once no frontier is left: whether a cell is occupied, and the tile's id there.
    __device__ __forceinline__ uint32_t nibble(int p)
    {
        return (pend_word(p) >> ((uint32_t)(p & 7) * 4u)) & 15u;
    }
    __device__ __forceinline__ bool occupied(int p) { return nibble(p) != 0; }
    __device__ __forceinline__ uint32_t tile_id(int p) { return (nibble(p) - 1u) & 15u; }
    // Row y's occupied cells, once no frontier is left.
    __device__ __forceinline__ uint32_t row(int y)
    {
        uint32_t r = 0;
#pragma unroll
        for (int h = 0; h < W / 16; ++h) {
            const int at = kPend + y * (W / 8) + 2 * h;
            uint64_t v = ((uint64_t)word(at + 1) << 32) | word(at);
            v |= v >> 2;
            v = (v | (v >> 1)) & 0x1111111111111111ull;
            v = (v | (v >> 3)) & 0x0303030303030303ull;
            v = (v | (v >> 6)) & 0x000F000F000F000Full;
            v = (v | (v >> 12)) & 0x000000FF000000FFull;
            r |= (uint32_t)((v | (v >> 24)) & 0xFFFFu) << (16 * h);
        }
        return r;
    }
};

enum { kEvNone = 0, kEvUnbound = 1, kEvAmbig = 2, kEvCorrupt = 3 };

// For one-wave workgroups: LDS writes made by the wave before this point are
// seen by its LDS reads after it.  A wave's LDS operations are performed in
// order, so only the compiler must not move accesses across the point: no
// s_barrier, and no wait for the wave's outstanding global stores, which the
// workgroup-scope fence of __syncthreads adds.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Assembly state of one run, in registers.
struct RunState {
    uint32_t nf;       // frontier size
    uint32_t osum;     // bit w set: occupancy word w may be nonzero
    int steps;         // placements so far: the structure has steps + 1 tiles
    bool choice;
    // 32 x 32 layout: frontier sites per group of four rows, byte k for rows
    // 4k .. 4k+3 (at most 4 * 31 sites), the frontier select's first level
    uint64_t groups;
    // LeanGrid: the occupied cells of the 8 x 8 window whose cell (3, 3) is the
    // seed, and whether a placed tile's id was lost
    uint64_t near;
    uint32_t lost;

    __device__ __forceinline__ int size() const { return steps + 1; }
    // Words that may hold a touched cell: frontier sites lie next to occupied
    // cells, so in the occupied words or the ones before and after them.
    template <int W>
    __device__ __forceinline__ uint32_t touched() const
    {
        const uint32_t t = osum | (osum << 1) | (osum >> 1);
        return W == 16 ? t & 0xFFu : t;
    }
};

// 32 x 32 layout: one more frontier site at cell q, or one less.  Nothing in
// the 16 x 16 layout.
template <int W>
__device__ __forceinline__ void frontier_group_add(RunState& st, int q, bool add)
{
    if constexpr (W == 32) {
        const uint64_t one = 1ull << (8 * (q >> 7));
        st.groups += add ? one : 0ull - one;
    }
}

// The tile `tuple` lies at p: check its empty neighbours (§3.2).
// A bondable site on the ring means the structure leaves the box; a site
// that two distinct tiles can fill is ambiguous; otherwise a free site with
// one admissible tile joins the frontier with that tile pending.
//
// Invariant: the PEND nibble of a free cell is zero unless the cell is on
// the frontier, so a new pending tile is written with one LDS atomic OR.  An
// occupied cell keeps the tile placed there in its nibble.
//
// `added`, if given, receives bit d for every direction d whose site joined
// the frontier (the movelist traversal pushes those sites).
//
// This is the general form, one direction at a time; run_step below does the
// same for the four directions of a fresh placement at once.
template <int W, int B, class Src>
__device__ __forceinline__ int update_site(const Src& m, LaneGrid<W, B>& g, RunState& st,
                                           int G, int p, uint32_t tuple,
                                           uint32_t* added = nullptr)
{
    constexpr int kMask = W * W - 1;
    int q[4];
    uint32_t ow[4], fw[4], pw[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int delta = d == 0 ? -W : d == 1 ? 1 : d == 2 ? W : -1;
        q[d] = (p + delta) & kMask;
        ow[d] = g.occ(q[d] >> 5);
        fw[d] = g.fr(q[d] >> 5);
        pw[d] = g.pend_word(q[d]);
    }
    const uint32_t codes = m.codes(tuple);
    // p lies in the box ([0, G-2]^2), so a neighbour is on the ring exactly
    // when p is on the box's edge in that direction (N and W wrap round the
    // torus onto row or column W-1)
    const int px = p & (W - 1), py = p >> Geometry<W>::kLogW;
    bool unbound = false, ambiguous = false;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const SiteOpts opt = split_code(codes >> (8 * d));
        const bool ring = d == 0 ? py == 0 : d == 1 ? px == G - 2 : d == 2 ? py == G - 2 : px == 0;
        const uint32_t bit = (uint32_t)q[d] & 31u;
        const bool free = ((ow[d] >> bit) & 1u) == 0;
        const bool live = opt.has && !ring && free;
        const bool in_f = ((fw[d] >> bit) & 1u) != 0;
        const uint32_t sh = ((uint32_t)q[d] & 7u) * 4u;
        const uint32_t pending = (pw[d] >> sh) & 15u;
        unbound = unbound | (opt.has & ring);
        ambiguous = ambiguous | (live & (opt.multi | (in_f & (pending != opt.id))));
        if (live && !opt.multi && !in_f) {
            set_bits(g.fr(q[d] >> 5), 1u << bit);
            set_bits(g.pend_word(q[d]), opt.id << sh);
            st.nf += 1;
            frontier_group_add<W>(st, q[d], true);
            if (added != nullptr)
                *added |= 1u << d;
        }
    }
    return unbound ? kEvUnbound : ambiguous ? kEvAmbig : kEvNone;
}

// Clears what the previous run touched and places the seed (tile 0,
// unrotated) at the centre; returns the seed's cell.
template <class Grid>
__device__ __forceinline__ int run_clear(Grid& g, RunState& st, int G)
{
    constexpr int W = Grid::kW;
    // occupied cells keep their tiles in PEND, and a run that ended on an
    // event leaves frontier cells (with their PEND nibbles) behind: clear all
    // (but row W-1, which no run touches)
    uint32_t touched = st.touched<W>();
    if constexpr (W == 32)
        touched &= 0x7FFFFFFFu;
    for (uint32_t s = touched; s; s &= s - 1) {
        const int w = __builtin_ctz(s);
        if constexpr (!Grid::kLean)
            g.occ(w) = 0;
        g.fr(w) = 0;
        const int second = W == 16 && w == 7 ? 0 : 2;
        g.word(Grid::kPend + 4 * w) = 0;
        g.word(Grid::kPend + 4 * w + 1) = 0;
        g.word(Grid::kPend + 4 * w + second) = 0;
        g.word(Grid::kPend + 4 * w + second + 1) = 0;
    }
    st.nf = 0;
    st.groups = 0;
    st.steps = 0;
    st.choice = false;
    const int seed_pos = (G / 2 - 1) * W + (G / 2 - 1);
    if constexpr (Grid::kLean) {
        g.pend_word(seed_pos) = 1u << ((seed_pos & 7) * 4);   // id 0
        st.near = 1ull << 27;
        st.lost = 0;
    } else {
        g.occ(seed_pos >> 5) = 1u << (seed_pos & 31);
    }
    st.osum = 1u << (seed_pos >> 5);
    return seed_pos;
}

// Starts a run whose seed has the four site codes `codes` (Bonds::codes of
// the seed's tuple): clears what the previous run touched, places the seed
// (tile 0, unrotated) at the centre and puts its sites on the frontier.  In
// the cleared grid they are free and off the frontier, and with G >= 8 the
// ring is at least three cells away.
template <class Grid>
__device__ __forceinline__ int run_start_known(Grid& g, RunState& st, int G, uint32_t codes)
{
    constexpr int W = Grid::kW;
    const int p = run_clear(g, st, G);
    if ((codes & kSiteMulti) != 0)
        return kEvAmbig;
    st.nf = (uint32_t)__popc(codes & kSiteAny);
    // a site without an option is written too, as zero bits
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int q = p + (d == 0 ? -W : d == 1 ? 1 : d == 2 ? W : -1);
        const uint32_t code = codes >> (8 * d), any = (code >> 7) & 1u;
        const uint32_t nibble = Grid::kLean ? (code + any) & 15u : code & 15u;
        set_bits(g.fr(q >> 5), any << (q & 31));
        set_bits(g.pend_word(q), nibble << ((q & 7) * 4));
        if constexpr (W == 32)
            st.groups += (uint64_t)any << (8 * (q >> 7));
    }
    return kEvNone;
}

// Starts a run of genotype m.
template <class Grid, class Src>
__device__ __forceinline__ int run_start(const Src& m, Grid& g, RunState& st, int G)
{
    return run_start_known(g, st, G, m.codes(m.seed()));
}

// A run is over once an event happened or the frontier is empty.  Every step
// fills a new cell of the box, so (G-1)^2 steps also end it (never reached).
__device__ __forceinline__ bool run_over(int ev, const RunState& st, int G)
{
    return ev != kEvNone || st.nf == 0 || st.steps >= (G - 1) * (G - 1);
}

// What draws a run's random words: its Philox key and stream.
struct RunKey {
    uint32_t key0, key1, rid_lo, rid_hi;
    int run;
};

// Index of the first of four inclusive prefix counts p0 <= p1 <= p2 (<= p3)
// above j (j < p3): which of four words holds site j.  *below receives the
// count before that word.
__device__ __forceinline__ uint32_t pick4(uint32_t j, uint32_t p0, uint32_t p1, uint32_t p2,
                                          uint32_t& below)
{
    const bool up = j >= p1;
    const uint32_t q = up ? p2 : p0;
    const bool odd = j >= q;
    below = odd ? q : up ? p1 : 0u;
    return (up ? 2u : 0u) + (odd ? 1u : 0u);
}

// The check of a fresh placement's four neighbours (§3.2), all at once: byte d
// of every word belongs to direction d.
//   codes   Bonds::codes of the placed tile
//   inside  bit 7 set where the neighbour lies in the box (not on its ring)
//   occ, fr bit 7 set where it is occupied, on the frontier
//   pend    its PEND nibble
//   tags    the nibbles that the placed tile's sites would have
// fresh receives bit 7 where a site joins the frontier.  Returns the events as
// bits: bit 7 of a byte where the structure leaves the box, bit 6 where a site
// is ambiguous (event_of gives the event; the rules as in update_site).
__device__ __forceinline__ uint32_t check_sites(uint32_t codes, uint32_t inside, uint32_t occ,
                                                uint32_t fr, uint32_t pend, uint32_t tags,
                                                uint32_t& fresh)
{
    const uint32_t has = codes & kSiteAny;
    const uint32_t live = has & inside & ~occ;
    // nibbles that differ: their XOR is 1..15, so adding 0x7F sets bit 7
    const uint32_t differ = ((pend ^ tags) & 0x0F0F0F0Fu) + 0x7F7F7F7Fu;
    const uint32_t ambiguous = live & ((codes << 1) | (fr & differ));
    fresh = live & ~fr;
    return (has & ~inside) | (ambiguous >> 1);
}

// The event of a step's bits: bit 0 set, the grid is corrupt; else check_sites'.
__device__ __forceinline__ int event_of(uint32_t bits)
{
    return bits == 0 ? kEvNone : (bits & 1u) ? kEvCorrupt
           : (bits & kSiteAny) != 0 ? kEvUnbound : kEvAmbig;
}

// Bit 7 of byte d set where cell (x, y)'s neighbour in direction d lies in the
// box [0, G-2]^2.
__device__ __forceinline__ uint32_t inside_box(uint32_t x, uint32_t y, int G)
{
    // the distances to the four edges, at most 30: zero ones stay below 0x80
    const uint32_t far = (uint32_t)(G - 2) * 0x00010100u;
    const uint32_t room = (y | (x << 24)) + (far - ((x << 8) | (y << 16)));
    return room + 0x7F7F7F7Fu;
}

// One step: take the frontier site of rank floor(u*|F|/2^32) in row-major
// order (u = Philox word `steps` of this run's stream; with one site any word
// gives rank 0), place its pending tile and check the new neighbours.
//
// A wave is bound here by the instructions it issues and, with few waves or
// few lanes left, by the length of their chain: two rounds of LDS reads (the
// frontier words, then the placed cell's and its neighbours' words) and one
// straight line of integer work without branches, the neighbours' words read
// as the rows around the cell, the four sites checked together and the
// touched words written back whole.  About 150 instructions, where one site at
// a time with branches around each insertion took about 270 (16 x 16) to 350
// (32 x 32).  Measured with the bond lookup of Bonds: all of S_{2,8} in one
// call 1.31 -> 1.07 ms, a generation of 65,536 three-tile genotypes at G = 32
// (its longest run, one placement after the other) 0.93 -> 0.63 ms.
//
// Returns the step's event bits (event_of).
template <class Grid, class Src>
__device__ __forceinline__ uint32_t run_step(const Src& m, Grid& g, RunState& st, int G,
                                             uint32_t u)
{
    constexpr int W = Grid::kW;
    constexpr bool kLean = Grid::kLean;
    const uint32_t nf = st.nf;
    const uint32_t j = __umulhi(u, nf);
    st.choice = st.choice | (nf >= 2);
    // the j-th frontier site in row-major order: its word w (fw), then the
    // bit.  The bitmap's count always equals nf; were it not so, the run
    // would end as corrupt (and every address below stays in the lane's grid)
    uint32_t w, fw, below, total;
    if constexpr (W == 16) {
        // the eight frontier words and their prefix counts, halved thrice
        const uint32_t f0 = g.fr(0), f1 = g.fr(1), f2 = g.fr(2), f3 = g.fr(3);
        const uint32_t f4 = g.fr(4), f5 = g.fr(5), f6 = g.fr(6), f7 = g.fr(7);
        const uint32_t p0 = __popc(f0), p1 = p0 + __popc(f1), p2 = p1 + __popc(f2);
        const uint32_t p3 = p2 + __popc(f3), p4 = p3 + __popc(f4), p5 = p4 + __popc(f5);
        const uint32_t p6 = p5 + __popc(f6);
        total = p6 + __popc(f7);
        const bool up = j >= p3;
        const uint32_t a0 = up ? f4 : f0, a1 = up ? f5 : f1, a2 = up ? f6 : f2, a3 = up ? f7 : f3;
        const uint32_t q1 = up ? p5 : p1;
        uint32_t in_half;
        const uint32_t k = pick4(j, up ? p4 : p0, q1, up ? p6 : p2, in_half);
        below = k != 0 ? in_half : up ? p3 : 0u;
        const uint32_t b0 = (k & 2u) ? a2 : a0, b1 = (k & 2u) ? a3 : a1;
        fw = (k & 1u) ? b1 : b0;
        w = (up ? 4u : 0u) + k;
    } else {
        // two levels: the counts of the eight groups of four rows (one byte
        // each, in registers) pick the group, its four words the row
        const uint32_t ga = (uint32_t)st.groups, gb = (uint32_t)(st.groups >> 32);
        const uint32_t p0 = ga & 0xFFu;
        const uint32_t p1 = __builtin_amdgcn_udot4(ga, 0x00000101u, 0u, false);
        const uint32_t p2 = __builtin_amdgcn_udot4(ga, 0x00010101u, 0u, false);
        const uint32_t p3 = __builtin_amdgcn_udot4(ga, 0x01010101u, 0u, false);
        const uint32_t p4 = __builtin_amdgcn_udot4(gb, 0x00000001u, p3, false);
        const uint32_t p5 = __builtin_amdgcn_udot4(gb, 0x00000101u, p3, false);
        const uint32_t p6 = __builtin_amdgcn_udot4(gb, 0x00010101u, p3, false);
        total = __builtin_amdgcn_udot4(gb, 0x01010101u, p3, false);
        const bool up = j >= p3;
        uint32_t in_half;
        const uint32_t k = pick4(j, up ? p4 : p0, up ? p5 : p1, up ? p6 : p2, in_half);
        const uint32_t before = k != 0 ? in_half : up ? p3 : 0u;
        const uint32_t w0 = 4u * ((up ? 4u : 0u) + k);
        const uint32_t f0 = g.fr(w0), f1 = g.fr(w0 + 1), f2 = g.fr(w0 + 2), f3 = g.fr(w0 + 3);
        const uint32_t c0 = __popc(f0), c1 = c0 + __popc(f1), c2 = c1 + __popc(f2);
        uint32_t in_group;
        const uint32_t r = pick4(j - before, c0, c1, c2, in_group);
        below = before + in_group;
        const uint32_t b0 = (r & 2u) ? f2 : f0, b1 = (r & 2u) ? f3 : f1;
        fw = (r & 1u) ? b1 : b0;
        w = w0 + r;
    }
    // the site's bit: its rank in the word is nearly always 0..2, so clearing
    // the lowest bit that often beats a fixed binary search; the first three
    // without a branch
    uint32_t rest = fw;
    int rank = (int)(j - below);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        rest &= (rest - 1u) | (uint32_t)((rank - 1) >> 31);
        rank = max(rank - 1, 0);
    }
    for (; rank > 0; --rank)
        rest &= rest - 1u;
    const uint32_t bit = (uint32_t)__builtin_ctz(rest | 0x80000000u);
    uint32_t ev, x, y, fresh;
    if constexpr (W == 16) {
        // a word holds two rows.  The cell's own word and the next (odd row)
        // or previous one (even row) as 64 bits hold the rows above and below
        // too: shifted so that N is bit 0, W is bit 15, the cell 16, E 17 and
        // S 32 (off the torus' rim they show ring cells, which are masked)
        const uint32_t odd = bit >> 4, wa = (w + 2u * odd - 1u) & 7u, shift = bit ^ 16u;
        x = bit & 15u;
        y = 2u * w + odd;
        const uint32_t fa = g.fr(wa);
        // the row's 16 PEND nibbles, and the words above and below the cell
        const uint32_t prow = Grid::kPend + 2u * y, half = x >> 3;
        const uint32_t n_at = Grid::kPend + 2u * ((y - 1u) & 15u) + half;
        const uint32_t s_at = Grid::kPend + 2u * ((y + 1u) & 15u) + half;
        uint64_t row = ((uint64_t)g.word(prow + 1) << 32) | g.word(prow);
        const uint32_t pn = g.word(n_at), ps = g.word(s_at), sh = 4u * (x & 7u);
        uint64_t fr2 = odd ? ((uint64_t)fa << 32) | fw : ((uint64_t)fw << 32) | fa;
        auto around = [](uint64_t u) -> uint32_t {
            const uint32_t a = (uint32_t)u, b = (uint32_t)(u >> 32);
            return ((a << 7) & 0x80u) | ((a >> 2) & 0x8000u) | ((b << 23) & 0x800000u) |
                   ((a << 16) & 0x80000000u);
        };
        const uint32_t fr = around(fr2 >> shift);
        // nibbles: 0 the W neighbour, 1 the cell, 2 the E neighbour
        const uint32_t near = (uint32_t)((row << 4) >> (4u * x)), own = (near >> 4) & 15u;
        const uint32_t pend = ((pn >> sh) & 15u) | (near & 0xF00u) | (((ps >> sh) & 15u) << 16) |
                              ((near & 15u) << 24);
        uint32_t codes, tags, occ, mark = 0;
        if constexpr (kLean) {
            codes = m.codes(m.oriented(own - 1u));
            tags = codes + 0x01010101u;
            occ = (pend + 0x7F7F7F7Fu) & ~fr;
            if constexpr (Src::kManyIds) {   // id 15: see LeanGrid
                mark = (own - 1u) >> 31;
                st.lost |= mark;
            }
        } else {
            const uint32_t o = g.occ(w), oa = g.occ(wa);
            codes = m.codes(m.oriented(own));
            tags = codes;
            occ = around((odd ? ((uint64_t)oa << 32) | o : ((uint64_t)o << 32) | oa) >> shift);
            g.occ(w) = o | (1u << bit);
        }
        ev = check_sites(codes, inside_box(x, y, G), occ, fr, pend, tags, fresh);
        // the cell leaves the frontier, fresh sites (none of them on it) join
        const uint32_t flip = ((fresh >> 7) & 1u) | ((fresh >> 16) & 0x8000u) | 0x10000u |
                              ((fresh << 2) & 0x20000u);
        fr2 ^= (((uint64_t)((fresh >> 23) & 1u) << 32) | flip) << shift;
        g.fr(w) = odd ? (uint32_t)fr2 : (uint32_t)(fr2 >> 32);
        g.fr(wa) = odd ? (uint32_t)(fr2 >> 32) : (uint32_t)fr2;
        const uint32_t ones = fresh >> 7, ids = tags & ((ones << 4) - ones);
        row |= ((uint64_t)((ids >> 24) | (mark << 4) | (ids & 0xF00u)) << (4u * x)) >> 4;
        g.word(prow) = (uint32_t)row;
        g.word(prow + 1) = (uint32_t)(row >> 32);
        g.word(n_at) = pn | ((ids & 15u) << sh);
        g.word(s_at) = ps | (((ids >> 16) & 15u) << sh);
    } else {
        // a word holds one row
        x = bit;
        y = w;
        const uint32_t yn = (y - 1u) & 31u, ys = (y + 1u) & 31u;
        const uint32_t fn = g.fr(yn), fs = g.fr(ys);
        // eight PEND nibbles a word: the cell's word and the next one in its
        // row (right half) or the one before (left half) hold E and W
        const uint32_t at = x >> 3, k = x & 7u, sh = 4u * k;
        const bool right = k >= 4u;
        const uint32_t prow = Grid::kPend + 4u * y, pa = prow + ((right ? at + 1u : at - 1u) & 3u);
        const uint32_t n_at = Grid::kPend + 4u * yn + at, s_at = Grid::kPend + 4u * ys + at;
        const uint32_t po = g.word(prow + at), pj = g.word(pa), pn = g.word(n_at);
        const uint32_t ps = g.word(s_at);
        uint64_t row = right ? ((uint64_t)pj << 32) | po : ((uint64_t)po << 32) | pj;
        const uint32_t rsh = right ? sh - 4u : sh + 28u;
        // nibbles: 0 the W neighbour, 1 the cell, 2 the E neighbour
        const uint32_t near = (uint32_t)(row >> rsh), own = (near >> 4) & 15u;
        const uint32_t pend = ((pn >> sh) & 15u) | (near & 0xF00u) | (((ps >> sh) & 15u) << 16) |
                              ((near & 15u) << 24);
        // rows rotated so that W is bit 0, the cell 1, E 2
        auto around = [x](uint32_t n, uint32_t o, uint32_t s) -> uint32_t {
            const uint32_t a = __builtin_amdgcn_alignbit(o, o, x - 1u);
            return (((n >> x) & 1u) << 7) | ((a << 13) & 0x8000u) | (((s >> x) & 1u) << 23) |
                   (a << 31);
        };
        const uint32_t fr = around(fn, fw, fs);
        uint32_t codes, tags, occ, mark = 0;
        if constexpr (kLean) {
            codes = m.codes(m.oriented(own - 1u));
            tags = codes + 0x01010101u;
            occ = (pend + 0x7F7F7F7Fu) & ~fr;
            if constexpr (Src::kManyIds) {   // id 15: see LeanGrid
                mark = (own - 1u) >> 31;
                st.lost |= mark;
            }
        } else {
            const uint32_t on = g.occ(yn), o = g.occ(y), os = g.occ(ys);
            codes = m.codes(m.oriented(own));
            tags = codes;
            occ = around(on, o, os);
            g.occ(y) = o | (1u << x);
        }
        ev = check_sites(codes, inside_box(x, y, G), occ, fr, pend, tags, fresh);
        const uint32_t flip = (fresh >> 31) | 2u | ((fresh >> 13) & 4u);
        const uint32_t up = (fresh >> 7) & 1u, down = (fresh >> 23) & 1u;
        g.fr(y) = fw ^ __builtin_amdgcn_alignbit(flip, flip, 1u - x);
        g.fr(yn) = fn | (up << x);
        g.fr(ys) = fs | (down << x);
        const uint32_t ones = fresh >> 7, ids = tags & ((ones << 4) - ones);
        row |= (uint64_t)((ids >> 24) | (mark << 4) | (ids & 0xF00u)) << rsh;
        g.word(prow + at) = right ? (uint32_t)row : (uint32_t)(row >> 32);
        g.word(pa) = right ? (uint32_t)(row >> 32) : (uint32_t)row;
        g.word(n_at) = pn | ((ids & 15u) << sh);
        g.word(s_at) = ps | (((ids >> 16) & 15u) << sh);
        st.groups += (uint64_t)(uint32_t)__popc(fresh & 0x80008000u) << (8u * (y >> 2));
        st.groups -= 1ull << (8u * (y >> 2));
        st.groups += (uint64_t)up << (8u * (yn >> 2));
        st.groups += (uint64_t)down << (8u * (ys >> 2));
    }
    if constexpr (kLean) {
        // the cell in the window at the seed (cells before it wrap to large
        // numbers)
        const uint32_t dx = x - (uint32_t)(G / 2 - 4), dy = y - (uint32_t)(G / 2 - 4);
        st.near |= (uint64_t)((dx | dy) < 8u ? 1u : 0u) << ((8u * dy + dx) & 63u);
    }
    st.nf = nf + (uint32_t)__popc(fresh) - 1u;
    st.osum |= 1u << w;
    st.steps += 1;
    return ev | min(total ^ nf, 1u);
}

// Up to four steps of a run that is not over and whose steps so far are a
// multiple of four, so that one Philox block holds their words.  A wave whose
// lanes all start their runs between such groups computes the generator once
// a group with every running lane taking part, and tests for finished lanes
// once a group.
template <class Grid, class Src>
__device__ __forceinline__ int run_four(const Src& m, Grid& g, RunState& st, int G,
                                        const RunKey& k)
{
    const Words4 u = philox4x32_10((uint32_t)st.steps >> 2, (uint32_t)k.run, k.rid_lo, k.rid_hi,
                                   k.key0, k.key1);
    uint32_t ev = run_step(m, g, st, G, u.w[0]);
    if (ev == 0 && st.nf != 0) {
        ev = run_step(m, g, st, G, u.w[1]);
        if (ev == 0 && st.nf != 0) {
            ev = run_step(m, g, st, G, u.w[2]);
            if (ev == 0 && st.nf != 0)
                ev = run_step(m, g, st, G, u.w[3]);
        }
    }
    return event_of(ev);
}

// The wave's last running lane `t` to the end of its run, by the whole wave: the
// grid in registers, lane W/16 y + x/16 with 16 cells of row y (frontier bits and
// PEND nibbles), everything else uniform.  Called by the whole wave, with lane
// t's run between groups of four steps and not over; returns its event.
//
// A lone lane's step is a chain of 200 (16 x 16) to 250 (32 x 32) instructions
// and three LDS round trips, 0.7 us, and where every wave has few runs the
// longest one is the call's time.  Here the frontier site's row comes from a
// prefix sum over the lanes and a ballot instead of from two levels of words, its
// neighbours by reading lanes, and 64 Philox blocks are computed at once: about
// 170 instructions and no LDS, 0.48 us.  A GA generation of 65,536 three-tile
// genotypes at G = 32, whose longest run has 462 steps, 0.40 -> 0.32 ms; 1,000
// two-tile genotypes 53 -> 43 us.  Two running lanes are faster side by side in
// their own grids.
template <class Grid, class Src>
__device__ __forceinline__ int lone_run(const Src& src, Grid& g, RunState& st, int grid,
                                        const RunKey& key, uint32_t t)
{
    static_assert(Grid::kLean, "the layout of LeanGrid");
    constexpr uint32_t W = Grid::kW, R = W / 16;
    const uint32_t lane = __lane_id();
    auto of = [](uint32_t v, uint32_t l) -> uint32_t {
        return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
    };
    wave_lds_sync();
    uint32_t* const col = g.base - lane + t;
    const bool mine = lane < (W - 1) * R;   // row W-1 is not the run's
    uint32_t f = 0, plo = 0, phi = 0;
    if (mine) {
        f = (col[(Grid::kFr + lane / 2) * 64] >> (16 * (lane & 1))) & 0xFFFFu;
        plo = col[(Grid::kPend + 2 * lane) * 64];
        phi = col[(Grid::kPend + 2 * lane + 1) * 64];
    }
    Src m = src;
    m.t0 = of(src.t0, t);
    m.t1 = of(src.t1, t);
    if constexpr (Src::kManyIds) {
        m.t2 = of(src.t2, t);
        m.t3 = of(src.t3, t);
    }
    m.lo = of(src.lo, t);
    m.hi = of(src.hi, t);
    if constexpr (BondsTraits<Src>::kWide) {
        m.lo2 = of(src.lo2, t);
        m.hi2 = of(src.hi2, t);
    }
    const int G = (int)of((uint32_t)grid, t);
    const uint32_t rid_lo = of(key.rid_lo, t), rid_hi = of(key.rid_hi, t);
    const uint32_t run = of((uint32_t)key.run, t);
    uint32_t nf = of(st.nf, t), lost = of(st.lost, t);
    uint32_t steps = of((uint32_t)st.steps, t);
    uint32_t choice = of(st.choice ? 2u : 0u, t);
    const uint32_t limit = (uint32_t)((G - 1) * (G - 1));

    // one step, as run_step
    auto step = [&](uint32_t u) -> uint32_t {
        const uint32_t j = __umulhi(u, nf);
        choice |= nf & ~1u;
        // inclusive prefix sums of the lanes' frontier sites
        uint32_t sum = (uint32_t)__popc(f);
        sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x111, 0xf, 0xf, false);
        sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x112, 0xf, 0xf, false);
        sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x114, 0xf, 0xf, false);
        sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x118, 0xf, 0xf, false);
        if constexpr (W == 32) {
            sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x142, 0xa, 0xf, false);
            sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x143, 0xc, 0xf, false);
        }
        const uint64_t above = __ballot(sum > j);
        if (above == 0)
            return 1u;   // corrupt: never, the frontier's count is nf
        const uint32_t L = (uint32_t)__builtin_ctzll(above);
        uint32_t rest = of(f, L);
        for (uint32_t rank = j - (of(sum, L) - (uint32_t)__popc(rest)); rank > 0; --rank)
            rest &= rest - 1u;
        const uint32_t xi = (uint32_t)__builtin_ctz(rest | 0x10000u) & 15u;
        // the cells around as (lane, index): N and S share the cell's index; E and W
        // may lie in the next lane, or outside (a lane without cells, then)
        const uint32_t at = 16 * L + xi, x = at % W, y = at / W;
        const uint32_t up = (L - R) & 63u, down = (L + R) & 63u;
        const uint32_t at_e = at + 1, at_w = at - 1;
        const uint32_t le = (at_e >> 4) & 63u, lw = (at_w >> 4) & 63u;
        const uint32_t xe = at_e & 15u, xw = at_w & 15u;
        // every lane's PEND nibble at an index, with bit 7 set if on the frontier
        const uint64_t pend64 = ((uint64_t)phi << 32) | plo;
        const uint32_t f7 = f << 7;
        const uint32_t cells = ((uint32_t)(pend64 >> (4 * xi)) & 15u) | ((f7 >> xi) & 0x80u);
        const uint32_t cells_e = ((uint32_t)(pend64 >> (4 * xe)) & 15u) | ((f7 >> xe) & 0x80u);
        const uint32_t cells_w = ((uint32_t)(pend64 >> (4 * xw)) & 15u) | ((f7 >> xw) & 0x80u);
        const uint32_t around = of(cells, up) | (of(cells_e, le) << 8) | (of(cells, down) << 16) |
                                (of(cells_w, lw) << 24);
        const uint32_t own = of(cells, L) & 15u;
        const uint32_t pend = around & 0x0F0F0F0Fu, fr = around & 0x80808080u;
        const uint32_t occ = (pend + 0x7F7F7F7Fu) & ~fr;
        const uint32_t codes =
            (uint32_t)__builtin_amdgcn_readfirstlane((int)m.codes(m.oriented(own - 1u)));
        const uint32_t tags = codes + 0x01010101u;
        uint32_t fresh;
        const uint32_t ev = check_sites(codes, inside_box(x, y, G), occ, fr, pend, tags, fresh);
        const uint32_t ones = fresh >> 7, ids = tags & ((ones << 4) - ones);
        // the cell leaves the frontier, fresh sites join
        const bool is_n = lane == up, is_s = lane == down, is_e = lane == le, is_w = lane == lw;
        f ^= ((is_n ? ones & 1u : is_s ? (ones >> 16) & 1u : lane == L ? 1u : 0u) << xi) |
             (is_e ? ((ones >> 8) & 1u) << xe : 0u) | (is_w ? (ones >> 24) << xw : 0u);
        uint32_t id = is_n ? ids & 15u : is_s ? (ids >> 16) & 15u : 0u;
        if constexpr (Src::kManyIds) {   // id 15: see LeanGrid
            const uint32_t mark = (own - 1u) >> 31;
            lost |= mark;
            id |= lane == L ? mark : 0u;
        }
        const uint64_t id_e = (uint64_t)((ids >> 8) & 15u) << (4 * xe);
        const uint64_t id_w = (uint64_t)(ids >> 24) << (4 * xw);
        const uint64_t id_v = (uint64_t)id << (4 * xi);
        plo |= (uint32_t)id_v | (is_e ? (uint32_t)id_e : 0u) | (is_w ? (uint32_t)id_w : 0u);
        phi |= (uint32_t)(id_v >> 32) | (is_e ? (uint32_t)(id_e >> 32) : 0u) |
               (is_w ? (uint32_t)(id_w >> 32) : 0u);
        nf = nf + (uint32_t)__popc(fresh) - 1u;
        steps += 1;
        return ev;
    };

    uint32_t ev = 0;
    while (ev == 0 && nf != 0 && steps < limit) {
        // the words of the next 256 steps, four a lane
        const Words4 u = philox4x32_10((steps >> 2) + lane, run, rid_lo, rid_hi, key.key0, key.key1);
        for (uint32_t block = 0; block < 64 && ev == 0 && nf != 0 && steps < limit; ++block) {
            ev = step(of(u.w[0], block));
            if (ev == 0 && nf != 0)
                ev = step(of(u.w[1], block));
            if (ev == 0 && nf != 0)
                ev = step(of(u.w[2], block));
            if (ev == 0 && nf != 0)
                ev = step(of(u.w[3], block));
        }
    }
    if (mine) {
        col[(Grid::kPend + 2 * lane) * 64] = plo;
        col[(Grid::kPend + 2 * lane + 1) * 64] = phi;
    }
    const uint32_t pair = f | ((uint32_t)__shfl((int)f, (int)(lane + 1) & 63) << 16);
    if ((lane & 1u) == 0 && lane < (W == 16 ? 16u : 62u))
        col[(Grid::kFr + lane / 2) * 64] = pair;
    // what the run's state says of its grid: the words with a cell, and the cells
    // in the window at the seed (all occupied unless the run met an event)
    // (every lane takes part in the exchange)
    const int any = __shfl((int)(plo | phi), (int)(2 * lane) & 63) |
                    __shfl((int)(plo | phi), (int)(2 * lane + 1) & 63);
    const uint32_t touched = (uint32_t)__ballot(any != 0);
    uint64_t v = ((uint64_t)phi << 32) | plo;
    v |= v >> 2;
    v = (v | (v >> 1)) & 0x1111111111111111ull;
    v = (v | (v >> 3)) & 0x0303030303030303ull;
    v = (v | (v >> 6)) & 0x000F000F000F000Full;
    v = (v | (v >> 12)) & 0x000000FF000000FFull;
    const uint32_t cells = (uint32_t)(v | (v >> 24)) & 0xFFFFu;
    uint64_t near = 0;
#pragma unroll
    for (uint32_t r = 0; r < 8; ++r) {
        const uint32_t first = ((uint32_t)(G / 2 - 4) + r) * R;
        uint32_t row = of(cells, first);
        if constexpr (R == 2)
            row |= of(cells, first + 1) << 16;
        near |= (uint64_t)((row >> (G / 2 - 4)) & 0xFFu) << (8 * r);
    }
    if (lane == t) {
        st.nf = nf;
        st.osum |= touched;
        st.lost = lost;
        st.steps = (int)steps;
        st.choice = choice != 0;
        st.near = near;
    }
    wave_lds_sync();
    return event_of(ev);
}

// One run from the seed to completion or to an event.
template <class Grid, class Src>
__device__ __forceinline__ int run_assembly(const Src& m, Grid& g, RunState& st, int G,
                                            const RunKey& k)
{
    int ev = run_start(m, g, st, G);
    while (!run_over(ev, st, G))
        ev = run_four(m, g, st, G, k);
    return ev;
}

// True if the shape held in OCC (tiles in PEND) is forced: at every occupied
// cell, the tiles that its occupied neighbours bond to are exactly that
// cell's own tile.  For the final shape of a run that ended without an
// event this means every growth order places the same tile in every cell
// of the shape and nowhere else (a site outside the shape that any shape
// cell bonds to would have stayed on the frontier, or ended the run as
// UNBOUND), and never meets an ambiguous site: every run ends in this shape.
// The seed cell's id is 0, the unrotated seed tile's.
template <class Grid, class Src>
__device__ __forceinline__ bool shape_is_forced(const Src& m, Grid& g, int G)
{
    constexpr int W = Grid::kW, kMask = W * W - 1;
    bool forced = true;
    for (int y = 0; y < G - 1 && forced; ++y) {
        for (uint32_t cells = g.row(y); cells != 0 && forced; cells &= cells - 1) {
            const int p = y * W + __builtin_ctz(cells);
            // the site of this cell's tile in direction d: the neighbour q
            const uint32_t codes = m.codes(m.oriented(g.tile_id(p)));
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int q = (p + (d == 0 ? -W : d == 1 ? 1 : d == 2 ? W : -1)) & kMask;
                const SiteOpts o = split_code(codes >> (8 * d));
                if (g.occupied(q) && o.has && (o.multi || o.id != g.tile_id(q)))
                    forced = false;
            }
        }
    }
    return forced;
}

// Bounding box of the shape held in OCC (cropping, App. F.6).
struct ShapeBox {
    int xmin, ymin, w, h;
};

template <class Grid>
__device__ __forceinline__ ShapeBox crop(Grid& g, int G)
{
    int ymin = Grid::kW, ymax = -1;
    uint32_t cols = 0;
    for (int y = 0; y < G - 1; ++y) {
        const uint32_t r = g.row(y);
        if (r) {
            ymin = y < ymin ? y : ymin;
            ymax = y;
            cols |= r;
        }
    }
    const int xmin = __builtin_ctz(cols);
    const int xmax = 31 - __builtin_clz(cols);
    return ShapeBox{xmin, ymin, xmax - xmin + 1, ymax - ymin + 1};
}

// True if the shape held in OCC (tiles in PEND), left by a run that ended
// without an event, is guarded: every run ends in it.  Call an edge from an
// occupied cell q to an occupied neighbour p good when q's tile admits
// exactly p's tile at p, and a conflict when it admits anything else there.
// The shape is guarded when, for every conflict q -> p with p not the seed,
// every path of good edges from the seed to q passes through p.
//
// Why that suffices: in any growth order a tile is placed only from the
// frontier, where it arrived over an edge from a tile placed before it.  By
// induction over the placements, every tile so far is the shape's own tile
// in a cell of the shape, reached from the seed over good edges through
// cells placed before it; so a conflicting q is never placed while p is
// empty, and q's wrong option at p never counts.  No site outside the shape
// can be bonded to (run 0 would have grown there or met an event), so the
// run places the shape exactly, never meets an event, and places all of it
// (every cell of the shape has a good edge from a cell placed before it in
// run 0).  With no conflicts this is shape_is_forced.
//
// This test takes the shape as an anchored 8 x 8 bitmap and the tile ids by
// cell; the flood fills run on 64-bit bitmaps.  A larger shape is tested with
// shape_is_forced instead.
template <class Src, class IdOf>
__device__ __forceinline__ bool bitmap_is_guarded(const Src& src, uint64_t shape,
                                                  uint64_t seed_bit, const IdOf& id_of)
{
    // good_d / conf_d: bit of cell p set for the edge into p from its
    // neighbour in direction d
    uint64_t good0 = 0, good1 = 0, good2 = 0, good3 = 0;
    uint64_t conf0 = 0, conf1 = 0, conf2 = 0, conf3 = 0;
    int k = 0;
    for (uint64_t cells = shape; cells != 0; cells &= cells - 1, ++k) {
        const int b = __builtin_ctzll(cells);
        const uint32_t codes = src.codes(src.oriented(id_of(b, k)));
        const int x = b & 7, y = b >> 3;
        // the edges from this cell into its neighbour p in direction d, which
        // it enters from direction d + 2
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const bool inside = d == 0 ? y > 0 : d == 1 ? x < 7 : d == 2 ? y < 7 : x > 0;
            const int pb = b + (d == 0 ? -8 : d == 1 ? 1 : d == 2 ? 8 : -1);
            if (!inside || ((shape >> (pb & 63)) & 1ull) == 0ull)
                continue;
            const uint64_t bit = 1ull << pb;
            const SiteOpts o = split_code(codes >> (8 * d));
            const bool good =
                o.has & !o.multi & (o.id == id_of(pb, __popcll(shape & (bit - 1))));
            const bool conf = o.has & !good;
            const uint64_t gb = good ? bit : 0ull, cb = conf ? bit : 0ull;
            if (d == 2) { good0 |= gb; conf0 |= cb; }
            else if (d == 3) { good1 |= gb; conf1 |= cb; }
            else if (d == 0) { good2 |= gb; conf2 |= cb; }
            else { good3 |= gb; conf3 |= cb; }
        }
    }
    // conflicts into the seed never count: the seed is placed first
    uint64_t todo = (conf0 | conf1 | conf2 | conf3) & ~seed_bit;
    bool guarded = true;
    for (; todo != 0 && guarded; todo &= todo - 1) {
        const uint64_t pb = todo & (~todo + 1);
        // the conflicting neighbours of p: N is 8 bits down, S 8 up, E 1 up, W 1 down
        const uint64_t from = ((conf0 & pb) >> 8) | ((conf2 & pb) << 8) | ((conf1 & pb) << 1) |
                              ((conf3 & pb) >> 1);
        const uint64_t allowed = shape & ~pb;
        uint64_t reach = seed_bit, prev = 0;
        while (reach != prev && (reach & from) == 0) {
            prev = reach;
            reach |= (((reach << 8) & good0) | ((reach >> 1) & good1) | ((reach >> 8) & good2) |
                      ((reach << 1) & good3)) & allowed;
        }
        guarded = (reach & from) == 0;
    }
    return guarded;
}

// One-at-a-time hash of the cropped shape in orientation k of the dihedral
// group: bit 2 transposes, bit 0 mirrors x, bit 1 mirrors y.  Cells are
// listed in row-major order of the oriented frame, each as the bytes x, y
// (§3.3, App. F.4).
template <class Grid>
__device__ __forceinline__ uint32_t orientation_hash(Grid& g, const ShapeBox& bx, int k)
{
    const bool transpose = k & 4, flip_x = k & 1, flip_y = k & 2;
    const int wt = transpose ? bx.h : bx.w, ht = transpose ? bx.w : bx.h;
    uint32_t hv = 0;
    for (int yp = 0; yp < ht; ++yp) {
        for (int xp = 0; xp < wt; ++xp) {
            int u = transpose ? yp : xp;
            int v = transpose ? xp : yp;
            u = flip_x ? bx.w - 1 - u : u;
            v = flip_y ? bx.h - 1 - v : v;
            if ((g.row(bx.ymin + v) >> (bx.xmin + u)) & 1u) {
                hv = oaat_add(hv, (uint32_t)xp);
                hv = oaat_add(hv, (uint32_t)yp);
            }
        }
    }
    return oaat_finish(hv);
}

// D4 hashes of the monomer and the domino, which have one shape each up to D4.
constexpr uint32_t oaat_add_c(uint32_t h, uint32_t byte)
{
    h += byte;
    h += h << 10;
    return h ^ (h >> 6);
}
constexpr uint32_t oaat_finish_c(uint32_t h)
{
    h += h << 3;
    h ^= h >> 11;
    return h + (h << 15);
}
// One orientation of n cells in a row from (0, 0), along x or y.
constexpr uint32_t line_hash_c(int n, bool along_x)
{
    uint32_t h = 0;
    for (int i = 0; i < n; ++i) {
        h = oaat_add_c(h, along_x ? (uint32_t)i : 0u);
        h = oaat_add_c(h, along_x ? 0u : (uint32_t)i);
    }
    return oaat_finish_c(h);
}
// Of a line's eight images four lie along x and four along y.
constexpr uint32_t line_shape_hash_c(int n)
{
    const uint32_t x = line_hash_c(n, true), y = line_hash_c(n, false);
    const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
    uint32_t h = 0;
    for (int i = 0; i < 8; ++i)
        for (int b = 0; b < 4; ++b)
            h = oaat_add_c(h, ((i < 4 ? lo : hi) >> (8 * b)) & 0xFFu);
    return oaat_finish_c(h);
}
constexpr uint32_t kMonomerHash = line_shape_hash_c(1), kDominoHash = line_shape_hash_c(2);

// The 8 orientation hashes sorted ascending, hashed again as 32
// little-endian bytes: the same value for every image of the shape.
__device__ __forceinline__ uint32_t combine_orientations(uint32_t hs[8])
{
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) {
#pragma unroll
        for (int i = pass & 1; i + 1 < 8; i += 2) {
            const uint32_t a = hs[i], b = hs[i + 1];
            hs[i] = a < b ? a : b;
            hs[i + 1] = a < b ? b : a;
        }
    }
    uint32_t hv = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            hv = oaat_add(hv, (hs[i] >> (8 * b)) & 0xFFu);
    return oaat_finish(hv);
}

// ---------------------------------------------------------------------------
// Register-only D4 hash for shapes whose bounding box fits 8 x 8: the cropped
// shape is a 64-bit bitmap, bit 8*y + x, so row-major cell order is ascending
// bit order.  The 8 images are the 4 mirror combinations of the shape and of
// its transpose, each re-anchored at (0, 0).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t bytes_reversed(uint64_t v)
{
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    return ((uint64_t)__builtin_bswap32(lo) << 32) | __builtin_bswap32(hi);
}

// Mirror x: reverse the bits of every byte, then shift the shape back to x=0.
__device__ __forceinline__ uint64_t mirror_x8(uint64_t v, int w)
{
    const uint32_t lo = __builtin_bitreverse32((uint32_t)v);
    const uint32_t hi = __builtin_bitreverse32((uint32_t)(v >> 32));
    // bit-reversing each half also reversed byte order: undo that
    const uint64_t r = ((uint64_t)__builtin_bswap32(hi) << 32) | __builtin_bswap32(lo);
    return r >> (8 - w);
}

// Mirror y: reverse the row order, then shift the shape back to y=0.
__device__ __forceinline__ uint64_t mirror_y8(uint64_t v, int h)
{
    return bytes_reversed(v) >> (8 * (8 - h));
}

// Transpose of an 8 x 8 bit matrix (bit 8*y + x -> bit 8*x + y).
__device__ __forceinline__ uint64_t transpose8(uint64_t x)
{
    uint64_t t;
    t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x = x ^ t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x = x ^ t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    x = x ^ t ^ (t << 28);
    return x;
}

// OAAT over (x, y) of every set cell in ascending bit (row-major) order.
__device__ __forceinline__ uint32_t bitmap_hash8(uint64_t v)
{
    uint32_t h = 0;
    while (v != 0) {
        const uint32_t b = (uint32_t)__builtin_ctzll(v);
        v &= v - 1;
        h = oaat_add(h, b & 7u);
        h = oaat_add(h, b >> 3);
    }
    return oaat_finish(h);
}

// Image k (0..7) of the w x h shape m: bit 2 transposes, bit 0 mirrors x,
// bit 1 mirrors y (in the transposed frame when transposed).
__device__ __forceinline__ uint64_t image8(uint64_t m, int w, int h, int k)
{
    uint64_t v = m;
    int ww = w, hh = h;
    if (k & 4) {
        v = transpose8(v);
        ww = h;
        hh = w;
    }
    if (k & 1)
        v = mirror_x8(v, ww);
    if (k & 2)
        v = mirror_y8(v, hh);
    return v;
}

// The cropped shape held in OCC as an 8 x 8 bitmap; false if it does not fit.
template <class Grid>
__device__ __forceinline__ bool shape_bitmap8(Grid& g, int G, uint64_t& m, int& w, int& h,
                                              int& x0, int& y0)
{
    const ShapeBox bx = crop(g, G);
    w = bx.w;
    h = bx.h;
    x0 = bx.xmin;
    y0 = bx.ymin;
    if (bx.w > 8 || bx.h > 8)
        return false;
    m = 0;
    for (int y = 0; y < bx.h; ++y)
        m |= (uint64_t)((g.row(bx.ymin + y) >> bx.xmin) & 0xFFu) << (8 * y);
    return true;
}

template <class Grid>
__device__ __forceinline__ bool shape_bitmap8(Grid& g, int G, uint64_t& m, int& w, int& h)
{
    int x0, y0;
    return shape_bitmap8(g, G, m, w, h, x0, y0);
}

// Width and height of an anchored 8 x 8 bitmap (not empty).
__device__ __forceinline__ void bitmap8_dims(uint64_t m, int& w, int& h)
{
    uint32_t x = (uint32_t)m | (uint32_t)(m >> 32);
    x |= x >> 16;
    x |= x >> 8;
    w = 32 - __builtin_clz(x & 0xFFu);
    h = (63 - __builtin_clzll(m)) / 8 + 1;
}

// The cropped shape as an anchored 8 x 8 bitmap for W = 16, from the 8 OCC
// words at once: row masks and the column union give the bounding box; each
// word (two rows) is shifted to xmin and packed to two bytes; the 8-row
// window at ymin is cut from the 16 packed rows.  False if the box exceeds
// 8 x 8.
template <int B>
__device__ __forceinline__ bool shape_bitmap8_w16(LaneGrid<16, B>& g, uint64_t& m, int& x0,
                                                  int& y0)
{
    uint32_t o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        o[k] = g.occ(k);
    uint32_t rows = 0, cols = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        rows |= (uint32_t)((o[k] & 0xFFFFu) != 0) << (2 * k);
        rows |= (uint32_t)((o[k] >> 16) != 0) << (2 * k + 1);
        cols |= o[k];
    }
    cols = (cols | (cols >> 16)) & 0xFFFFu;
    const int ymin = __builtin_ctz(rows), ymax = 31 - __builtin_clz(rows);
    const int xmin = __builtin_ctz(cols), xmax = 31 - __builtin_clz(cols);
    x0 = xmin;
    y0 = ymin;
    if (xmax - xmin >= 8 || ymax - ymin >= 8)
        return false;
    uint32_t r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t a = (o[2 * q] >> xmin) & 0x00FF00FFu;
        const uint32_t b = (o[2 * q + 1] >> xmin) & 0x00FF00FFu;
        r[q] = ((a | (a >> 8)) & 0xFFFFu) | (((b | (b >> 8)) & 0xFFFFu) << 16);
    }
    // bytes ymin .. ymin+7 of r[0..3] (rows past 15 are empty)
    const int q = ymin >> 2, sh = 8 * (ymin & 3);
    const uint32_t a0 = q == 0 ? r[0] : q == 1 ? r[1] : q == 2 ? r[2] : r[3];
    const uint32_t a1 = q == 0 ? r[1] : q == 1 ? r[2] : q == 2 ? r[3] : 0u;
    const uint32_t a2 = q == 0 ? r[2] : q == 1 ? r[3] : 0u;
    const uint32_t lo = (uint32_t)((((uint64_t)a1 << 32) | a0) >> sh);
    const uint32_t hi = (uint32_t)((((uint64_t)a2 << 32) | a1) >> sh);
    m = ((uint64_t)hi << 32) | lo;
    return true;
}

// A bitmap v of an 8 x 8 window (not empty), anchored at its first row and
// column, which start at (wx, wy) of the grid.
__device__ __forceinline__ uint64_t anchor8(uint64_t v, int wx, int wy, int& x0, int& y0)
{
    const int rows = __builtin_ctzll(v) & ~7;
    uint32_t cols = (uint32_t)v | (uint32_t)(v >> 32);
    cols |= cols >> 16;
    cols |= cols >> 8;
    const int left = __builtin_ctz(cols);
    x0 = wx + left;
    y0 = wy + rows / 8;
    return v >> (rows + left);
}

// The cropped shape of a finished run as an anchored 8 x 8 bitmap and where it
// starts; false if its box exceeds 8 x 8.  Nearly every shape lies in an 8 x 8
// window around the seed, and does so exactly if all of its cells are counted
// there: the lean grid keeps that window in a register; in the 16 x 16 layout
// it is four words (from an even row), shifted to its first column and packed
// to bytes, about 30 instructions against 110 for a box anywhere.
template <class Grid>
__device__ __forceinline__ bool shape_key8(Grid& g, const RunState& st, int G, int size,
                                           uint64_t& m, int& x0, int& y0)
{
    const int s = G / 2 - 1;
    if constexpr (Grid::kLean) {
        if (__popcll(st.near) == size) {
            m = anchor8(st.near, s - 3, s - 3, x0, y0);
            return true;
        }
    } else if constexpr (Grid::kW == 16) {
        const int wx = s - 3, wy = (s - 3) & ~1;
        uint32_t r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            r[q] = g.occ(wy / 2 + q) >> wx;
        const uint32_t lo = __builtin_amdgcn_perm(r[1], r[0], 0x06040200u);
        const uint32_t hi = __builtin_amdgcn_perm(r[3], r[2], 0x06040200u);
        const uint64_t v = ((uint64_t)hi << 32) | lo;
        if (__popcll(v) == size) {
            m = anchor8(v, wx, wy, x0, y0);
            return true;
        }
        return shape_bitmap8_w16(g, m, x0, y0);
    }
    int w, h;
    return shape_bitmap8(g, G, m, w, h, x0, y0);
}

// Whether two finished runs' grids hold the same cells (lean grids of one wave).
template <int W>
__device__ __forceinline__ bool same_cells(LeanGrid<W>& g, LeanGrid<W>& h, int G)
{
    bool same = true;
    for (int k = 0; k < (G - 1) * (W / 8); ++k) {
        // nibbles: set exactly where occupied
        uint32_t v = g.word(LeanGrid<W>::kPend + k), u = h.word(LeanGrid<W>::kPend + k);
        v |= v >> 2;
        u |= u >> 2;
        same = same && (((v | (v >> 1)) ^ (u | (u >> 1))) & 0x11111111u) == 0;
    }
    return same;
}

// ---------------------------------------------------------------------------
// A run's final shape packed into 16 bytes, for the proof stage to check
// without replaying the run: .x/.y the anchored 8 x 8 bitmap (bit 8y + x),
// .z/.w a 64-bit word holding the tile nibble of every cell in ascending bit
// order (at most kPackedCells cells) and, in bits 58..63, the seed's bit.
// All ones in .z/.w: no packed shape (larger box, more cells or, with .x set, tiles'
// ids lost).
// ---------------------------------------------------------------------------
constexpr int kPackedCells = 14;

__device__ __forceinline__ bool packed_shape_valid(const uint4& v)
{
    return !(v.z == 0xFFFFFFFFu && v.w == 0xFFFFFFFFu);
}

// No packed shape.
__device__ __forceinline__ uint4 packed_none(bool lost = false)
{
    return make_uint4(lost ? 1u : 0u, 0u, 0xFFFFFFFFu, 0xFFFFFFFFu);
}

__device__ __forceinline__ bool packed_shape_lost(const uint4& v)
{
    return !packed_shape_valid(v) && v.x != 0u;
}

// What a clean run's grid says of its tiles' ids: with `known`, the id of a cell is
// tile_id's, or 15 in the cells of `last` (anchored 8 x 8 bitmap).
struct TileIds {
    bool known;
    uint64_t last;

    template <class Grid>
    __device__ __forceinline__ uint32_t at(Grid& g, int x0, int y0, int b) const
    {
        return ((last >> b) & 1ull) != 0 ? 15u
                                         : g.tile_id((y0 + (b >> 3)) * Grid::kW + x0 + (b & 7));
    }
};

// The ids of the shape (shape_key8, if it `fits`) that a run without an event left.
// Only a lean grid of a run that placed the sixteenth oriented tile is in doubt, in
// the cells with id 0's tag.  Such a cell was placed because a neighbour placed before
// it admits its tile there, and nothing else: so if its neighbours, each with any id
// that it may have itself, admit only one of the two, that one it is.  (Not for
// shapes beyond 8 x 8, which stay unproven with such a tile.)
template <class Grid, class Src>
__device__ __forceinline__ TileIds shape_ids(const Src& m, Grid& g, const RunState& st, int G,
                                             bool fits, uint64_t shape, int x0, int y0)
{
    TileIds ids{true, 0ull};
    if constexpr (Grid::kLean && Src::kManyIds) {
        if (st.lost != 0) {
            const int s = G / 2 - 1;
            uint64_t doubt = 0;
            if (fits)
                for (uint64_t cells = shape & ~(1ull << ((s - y0) * 8 + (s - x0))); cells != 0;
                     cells &= cells - 1) {
                    const int b = __builtin_ctzll(cells);
                    doubt |= (uint64_t)(ids.at(g, x0, y0, b) == 0u ? 1u : 0u) << b;
                }
            ids.known = fits;
            const uint32_t zero = m.codes(m.oriented(0u)), last = m.codes(m.oriented(15u));
            for (uint64_t cells = doubt; cells != 0; cells &= cells - 1) {
                const int b = __builtin_ctzll(cells);
                bool is_zero = false, is_last = false;
                auto admits = [&](uint32_t code) {   // one tile only
                    const bool one = (code & 0xC0u) == 0x80u;
                    is_zero = is_zero | (one & ((code & 15u) == 0u));
                    is_last = is_last | (one & ((code & 15u) == 15u));
                };
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const bool inside = d == 0   ? b >= 8
                                        : d == 1 ? (b & 7) < 7
                                        : d == 2 ? b < 56
                                                 : (b & 7) > 0;
                    const int q = (b + (d == 0 ? -8 : d == 1 ? 1 : d == 2 ? 8 : -1)) & 63;
                    const int from = 8 * ((d + 2) & 3);   // the neighbour's side
                    if (inside && ((doubt >> q) & 1ull) != 0) {
                        admits(zero >> from);
                        admits(last >> from);
                    } else if (inside && ((shape >> q) & 1ull) != 0) {
                        admits(m.codes(m.oriented(TileIds{true, 0ull}.at(g, x0, y0, q))) >> from);
                    }
                }
                ids.known = ids.known && is_zero != is_last;
                ids.last |= (uint64_t)(is_last ? 1u : 0u) << b;
            }
        }
    }
    return ids;
}

// Packs the shape m (shape_key8) whose box starts at (x0, y0).
template <class Grid>
__device__ __forceinline__ uint4 pack_shape(Grid& g, const RunState& st, int G, int size,
                                            uint64_t m, int x0, int y0)
{
    const bool lost = Grid::kLean && st.lost != 0;
    if (size > kPackedCells || lost)
        return packed_none(lost);
    uint64_t tiles = 0;
    int k = 0;
    for (uint64_t cells = m; cells != 0; cells &= cells - 1, k += 4) {
        const int b = __builtin_ctzll(cells);
        const int p = (y0 + (b >> 3)) * Grid::kW + x0 + (b & 7);
        tiles |= (uint64_t)g.tile_id(p) << k;
    }
    const int sc = G / 2 - 1;
    tiles |= (uint64_t)((sc - y0) * 8 + (sc - x0)) << 58;
    return make_uint4((uint32_t)m, (uint32_t)(m >> 32), (uint32_t)tiles,
                      (uint32_t)(tiles >> 32));
}

// bitmap_is_guarded for a packed shape, from registers: the k-th cell's tile is
// nibble k of the tile word.
template <class Src>
__device__ __forceinline__ bool packed_shape_is_guarded(const Src& src, const uint4& v)
{
    const uint64_t shape = ((uint64_t)v.y << 32) | v.x;
    const uint64_t tiles = ((uint64_t)v.w << 32) | v.z;
    return bitmap_is_guarded(src, shape, 1ull << (int)(tiles >> 58),
                             [tiles](int, int k) { return (uint32_t)(tiles >> (4 * k)) & 15u; });
}

// Whether the shape left by a finished run is guarded; false, too, if its tiles' ids
// are not known.  key, x0, y0: shape_key8's, if it `fits`.
template <class Grid, class Src>
__device__ __forceinline__ bool shape_is_guarded(const Src& m, Grid& g, const TileIds& ids, int G,
                                                 bool fits, uint64_t key, int x0, int y0)
{
    if (!ids.known)
        return false;
    if (!fits)
        return shape_is_forced(m, g, G);
    const int s = G / 2 - 1;
    return bitmap_is_guarded(m, key, 1ull << ((s - y0) * 8 + (s - x0)),
                             [&](int b, int) { return ids.at(g, x0, y0, b); });
}

// D4 hash of a shape given as an anchored 8 x 8 bitmap, by one lane.
__device__ __forceinline__ uint32_t bitmap8_shape_hash(uint64_t m)
{
    int w, h;
    bitmap8_dims(m, w, h);
    uint32_t hs[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        hs[k] = bitmap_hash8(image8(m, w, h, k));
    return combine_orientations(hs);
}

// Per-wave cache of D4 hashes in LDS, keyed by the exact anchored 8 x 8
// bitmap of a shape (which determines the shape, so a hit returns exactly
// the hash the shape has).  N entries {bitmap lo, bitmap hi, hash, 0},
// direct mapped; an all-zero key marks an empty entry (no shape is empty).
// Lanes read it freely; entries are written one lane at a time.  For
// workgroups of one wave (insert synchronises the workgroup).  With a shape
// table, an entry's last word counts the DET records of its bitmap that the
// table does not have yet, small_count those of one and two cells, and kOther
// entries {hash, size, count, 0} those without a bitmap or an entry of their own.
// (These often share one shape, and an atomic each on its word of the table,
// 12 ns one after the other, took most of the time where they are many: 2^25
// three-tile genotypes from 2^33 on, 75,000 of them nine cells in a row, 8.3 ms
// instead of the 2.6 of a tally only.)
template <int N>
struct ShapeCache {
    static_assert((N & (N - 1)) == 0, "N must be a power of two");
    static constexpr uint32_t kOther = 8;
    uint4* e;
    uint32_t* small_count = nullptr;
    uint4* other = nullptr;

    __device__ __forceinline__ static uint32_t slot(uint64_t m)
    {
        const uint32_t x = (uint32_t)m * 0x9E3779B1u ^ (uint32_t)(m >> 32) * 0x85EBCA77u;
        return (x ^ (x >> 15)) & (N - 1);
    }
    __device__ __forceinline__ void clear(int lane)
    {
        for (int i = lane; i < N; i += 64)
            e[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ __forceinline__ bool lookup(uint64_t m, uint32_t& hash) const
    {
        const uint4 v = e[slot(m)];
        hash = v.z;
        return v.x == (uint32_t)m && v.y == (uint32_t)(m >> 32);
    }
    // Called by the whole wave of a one-wave workgroup: every lane with
    // `want` stores its entry, in lane order (a later lane with the same
    // slot overwrites), then the wave's later lookups see the entries.
    __device__ __forceinline__ void insert(bool want, uint64_t m, uint32_t hash, int lane,
                                           const ShapeTable& table = ShapeTable{})
    {
        uint64_t pending = __ballot(want);
        if (pending == 0)
            return;
        if (table.entries != nullptr) {
            // the counts of the entries that go, all lanes at once; the first of a
            // slot's lanes takes them
            wave_lds_sync();
            if (want)
                flush_entry(slot(m), table);
            wave_lds_sync();
        }
        for (; pending != 0; pending &= pending - 1)
            if (lane == __builtin_ctzll(pending))
                e[slot(m)] = make_uint4((uint32_t)m, (uint32_t)(m >> 32), hash, 0u);
        wave_lds_sync();
    }
    // Counts a DET record of bitmap m in its entry; false if it has none.
    __device__ __forceinline__ bool count(uint64_t m)
    {
        uint4& v = e[slot(m)];
        if (v.x != (uint32_t)m || v.y != (uint32_t)(m >> 32))
            return false;
        atomicAdd(&v.w, 1u);
        return true;
    }
    __device__ __forceinline__ void flush_entry(uint32_t i, const ShapeTable& table)
    {
        const uint4 v = e[i];
        const uint32_t n = atomicExch(&e[i].w, 0u);
        if (n != 0)
            table.add(shape_key(v.z, __popc(v.x) + __popc(v.y)), n);
    }
    // Counts the DET records of lanes with `want` among the other shapes; called by
    // the whole wave.
    __device__ __forceinline__ void count_other(bool want, uint32_t hash, int size, int lane,
                                                const ShapeTable& table)
    {
        for (uint64_t todo = __ballot(want); todo != 0;) {
            const int lead = __builtin_ctzll(todo);
            const bool same = want && hash == (uint32_t)__shfl((int)hash, lead) &&
                              size == __shfl(size, lead);
            const uint64_t mates = __ballot(same);
            if (lane == lead) {
                uint4& v = other[(hash ^ (hash >> 16)) % kOther];
                if (v.x != hash || v.y != (uint32_t)size) {
                    if (v.z != 0)
                        table.add(shape_key(v.x, (int32_t)v.y), v.z);
                    v = make_uint4(hash, (uint32_t)size, 0u, 0u);
                }
                v.z += (uint32_t)__popcll(mates);
            }
            wave_lds_sync();
            todo &= ~mates;
        }
    }
    // Every count to the table, at the wave's end.
    __device__ __forceinline__ void flush(const ShapeTable& table, int lane)
    {
        if (table.entries == nullptr)
            return;
        wave_lds_sync();
        for (int i = lane; i < N; i += 64)
            flush_entry((uint32_t)i, table);
        if (lane < 2 && small_count[lane] != 0)
            table.add(shape_key(lane == 0 ? kMonomerHash : kDominoHash, lane + 1),
                      small_count[lane]);
        if (lane < (int)kOther && other[lane].z != 0)
            table.add(shape_key(other[lane].x, (int32_t)other[lane].y), other[lane].z);
    }
};

// The 4 rotation hashes sorted ascending, hashed again as 16 little-endian
// bytes (§3.3's rotation-invariant hash).
__device__ __forceinline__ uint32_t combine_rotations(uint32_t hs[4])
{
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
#pragma unroll
        for (int i = pass & 1; i + 1 < 4; i += 2) {
            const uint32_t a = hs[i], b = hs[i + 1];
            hs[i] = a < b ? a : b;
            hs[i + 1] = a < b ? b : a;
        }
    }
    uint32_t hv = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            hv = oaat_add(hv, (hs[i] >> (8 * b)) & 0xFFu);
    return oaat_finish(hv);
}

// C4-invariant hash of the shape held in OCC: orientations 0 (identity),
// 3 (both mirrors: the half turn), 5 and 6 (a transpose and one mirror: the
// quarter turns) of the dihedral images, computed by one lane.
template <int W, int B>
__device__ uint32_t shape_hash_c4(LaneGrid<W, B>& g, int G)
{
    constexpr int kRot[4] = {0, 3, 5, 6};
    uint32_t hs[4];
    uint64_t m;
    int w, h;
    if (shape_bitmap8(g, G, m, w, h)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            hs[k] = bitmap_hash8(image8(m, w, h, kRot[k]));
    } else {
        const ShapeBox bx = crop(g, G);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            hs[k] = orientation_hash(g, bx, kRot[k]);
    }
    return combine_rotations(hs);
}

// ---------------------------------------------------------------------------
// The movelist traversal (§3.2): the frontier sites on a LIFO stack of cell
// indices (bytes, after the lane's grid words, 16 x 16 layout only).  A site
// that joins the frontier (directions N, E, S, W of each update) goes to slot
// floor(u (len + 1) / 2^32) counted from the bottom of the len sites on the
// stack, u the run's next word (word d for its d-th draw; none while the
// stack is empty); every step places the site on top.
// ---------------------------------------------------------------------------
constexpr int kStackWords = 64;   // 256 one-byte entries >= the 225 cells of the box

template <int B>
struct LaneStack {
    uint32_t* base;   // the lane's first stack word (word k at base[k * B])

    __device__ __forceinline__ uint8_t* byte(int i)
    {
        return reinterpret_cast<uint8_t*>(base + (i >> 2) * B) + (i & 3);
    }
    __device__ __forceinline__ int get(int i) { return *byte(i); }
    __device__ __forceinline__ void set(int i, int v) { *byte(i) = (uint8_t)v; }
};

// The movelist's words, one Philox block kept.  Scalars, never an array: an
// array picked by a run-time index ends up in scratch memory.
struct DrawCache {
    uint32_t block = 0xFFFFFFFFu;
    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;

    // random word s of the run: word s mod 4 of counter block s / 4
    __device__ __forceinline__ uint32_t draw(uint32_t s, const RunKey& k)
    {
        const uint32_t blk = s >> 2;
        if (blk != block) {
            const Words4 v = philox4x32_10(blk, (uint32_t)k.run, k.rid_lo, k.rid_hi, k.key0,
                                           k.key1);
            w0 = v.w[0];
            w1 = v.w[1];
            w2 = v.w[2];
            w3 = v.w[3];
            block = blk;
        }
        const uint32_t lo = (s & 1u) ? w1 : w0, hi = (s & 1u) ? w3 : w2;
        return (s & 2u) ? hi : lo;
    }
};

// Pushes the sites of the directions in `added` (in order N, E, S, W) next to
// p; len is the stack's length before them.  Returns the new length.
template <int W, int B>
__device__ __forceinline__ uint32_t movelist_push(LaneStack<B>& stk, uint32_t len, int p,
                                                  uint32_t added, DrawCache& dc, uint32_t& draws,
                                                  bool& choice, const RunKey& k)
{
    constexpr int kMask = W * W - 1;
    for (int d = 0; d < 4; ++d) {
        if (((added >> d) & 1u) == 0u)
            continue;
        const int delta = d == 0 ? -W : d == 1 ? 1 : d == 2 ? W : -1;
        const int q = (p + delta) & kMask;
        uint32_t pos = 0;
        if (len > 0u) {
            pos = __umulhi(dc.draw(draws, k), len + 1u);
            draws += 1;
            choice = true;
        }
        for (uint32_t i = len; i > pos; --i)
            stk.set((int)i, stk.get((int)i - 1));
        stk.set((int)pos, q);
        len += 1;
    }
    return len;
}

// One run with the movelist traversal, from the seed to completion or an
// event (st.nf is the stack's length throughout).
template <int W, int B, class Src>
__device__ __forceinline__ int run_assembly_lifo(const Src& m, LaneGrid<W, B>& g,
                                                 LaneStack<B>& stk, RunState& st, int G,
                                                 const RunKey& k)
{
    DrawCache dc;
    const int seed_pos = run_clear(g, st, G);
    uint32_t draws = 0, added = 0;
    bool choice = false;
    int ev = update_site(m, g, st, G, seed_pos, m.seed(), &added);
    movelist_push<W>(stk, 0u, seed_pos, added, dc, draws, choice, k);
    while (ev == kEvNone && st.nf > 0 && st.steps < (G - 1) * (G - 1)) {
        const int p = stk.get((int)st.nf - 1);
        st.nf -= 1;
        const int w = p >> 5;
        g.fr(w) = g.fr(w) & ~(1u << (p & 31));
        const uint32_t pw = g.pend_word(p);
        const uint32_t sh = ((uint32_t)p & 7u) * 4u;
        const uint32_t tuple = m.oriented((pw >> sh) & 15u);
        set_bits(g.occ(w), 1u << (p & 31));
        st.osum |= 1u << w;
        st.steps += 1;
        const uint32_t len = st.nf;
        added = 0;
        ev = update_site(m, g, st, G, p, tuple, &added);
        movelist_push<W>(stk, len, p, added, dc, draws, choice, k);
    }
    st.choice = choice;
    return ev;
}

// D4-invariant hash of the shape held in OCC, computed by one lane.
template <class Grid>
__device__ uint32_t shape_hash(Grid& g, int G)
{
    uint32_t hs[8];
    uint64_t m;
    int w, h;
    if (shape_bitmap8(g, G, m, w, h)) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            hs[k] = bitmap_hash8(image8(m, w, h, k));
    } else {
        const ShapeBox bx = crop(g, G);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            hs[k] = orientation_hash(g, bx, k);
    }
    return combine_orientations(hs);
}

}  // namespace jatam
