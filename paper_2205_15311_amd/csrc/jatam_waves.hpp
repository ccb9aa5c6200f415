// jatam_waves.hpp - what the classification kernels' waves share: the call's
// inputs, the screen of a genotype's seed, the hand-out of input chunks, class
// and shape counts, and the repeat runs of candidates.
#pragma once

#include "jatam_assembly.hpp"
#include "jatam_internal.hpp"
#include "jatam_shapes.hpp"

namespace jatam {

// ---------------------------------------------------------------------------
// Inputs: a range, an array of genomes, or an array of mixed items.
// ---------------------------------------------------------------------------
struct Geno {
    uint64_t genome;
    uint64_t rng_id;
    int t;
    int grid;
    bool valid;
    bool windowed;   // run in a window of its own grid (run_geno)
};

// Input modes: a range (genome = first + i, no loads), a genome list or items, as a
// compile-time choice where the kernel is compiled for each, else by the arguments.
// With the mode fixed, a range call has no global loads in its loop, and so no waits
// (the vector memory counter also counts the loop's record stores).
enum { kInRange = 0, kInList = 1, kInItems = 2, kInRuntime = 3 };

// Input i.  `first`: the range mode's first genotype of this call (a.first, moved by
// the slice counter of a replayed enumeration).
template <int kIn>
__device__ __forceinline__ Geno fetch_geno(const BatchArgs& a, uint64_t first, uint32_t i)
{
    Geno g;
    if (kIn == kInItems || (kIn == kInRuntime && a.items != nullptr)) {
        const jatam_item_t it = a.items[i];
        g.genome = it.genome;
        g.rng_id = it.rng_id;
        g.t = it.t;
        g.grid = it.grid;
        const int gbits = 4 * g.t * a.bits;
        g.valid = g.t >= 1 && g.t <= 4 && gbits <= 64 && g.grid >= 8 && g.grid <= 32 &&
                  (g.grid & 1) == 0 && (gbits == 64 || (g.genome >> gbits) == 0);
    } else {
        const bool list = kIn == kInList || (kIn == kInRuntime && a.genomes != nullptr);
        g.genome = list ? a.genomes[i] : first + (uint64_t)i;
        g.t = a.t;
        g.grid = a.grid;
        g.rng_id = g.genome | ((uint64_t)(uint32_t)a.t << 56);
        const int gbits = 4 * a.t * a.bits;
        g.valid = gbits == 64 || (g.genome >> gbits) == 0;
    }
    return g;
}

// The genotype as the kernels of a grid class run it: in the 16 x 16 layout
// an item of G > 16 runs in a window of G = 16 around the seed.  Up to the
// first placement that exposes a bondable site on the window's ring, such a
// run is the run in its own G x G grid (same cells relative to the seed,
// same row-major order, same draws); a run that reaches the window's ring
// ends UNBOUND here, without a record: the item is listed to run again in its
// own grid (DeviceWorkspace::overflow).
template <int W, int kIn = kInRuntime>
__device__ __forceinline__ Geno run_geno(const BatchArgs& a, uint64_t first, uint32_t i)
{
    Geno g = fetch_geno<kIn>(a, first, i);
    g.windowed = W == 16 && g.grid > 16;
    if constexpr (W == 16)
        g.grid = g.grid < 16 ? g.grid : 16;
    return g;
}

// A graph-replayed enumeration reads its slice s from the device: the call
// covers genotypes first + s*n .. and writes records at out + s*n if asked.
// (The kernel argument block is left untouched: a modified copy would live
// in scratch memory.)
__device__ __forceinline__ uint64_t slice_first(const BatchArgs& a)
{
    return a.slice != nullptr ? a.first + (uint64_t)*a.slice * (uint64_t)a.n : a.first;
}

__device__ __forceinline__ jatam_result_t* slice_out(const BatchArgs& a)
{
    return a.slice != nullptr && a.out_per_slice ? a.out + (uint64_t)*a.slice * (uint64_t)a.n
                                                 : a.out;
}

__device__ __forceinline__ RunKey run_key(const BatchArgs& a, const Geno& gd, int run)
{
    return RunKey{a.key0, a.key1, (uint32_t)gd.rng_id, (uint32_t)(gd.rng_id >> 32), run};
}

// Grid class of a genotype: 0 = the 16 x 16 layout, 1 = the 32 x 32 layout.
__device__ __forceinline__ int grid_class(const BatchArgs& a, int grid)
{
    return grid <= a.narrow_max ? 0 : 1;
}

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

__device__ __forceinline__ uint64_t lanes_below() { return (1ull << lane_id()) - 1; }

// Per-wave class counts, added at the wave's end to one of kTallySlots sets of
// counters in blocks of their own (tally_kernel adds them to the caller's): four
// atomics a wave on the caller's four words serialised, 0.1 ms a call over
// S_{2,8}.
struct WaveTally {
    uint32_t n[4];
    __device__ __forceinline__ void add(bool done, int cls)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            n[k] += (uint32_t)__popcll(__ballot(done && cls == k));
    }
    __device__ __forceinline__ void add_to(unsigned long long* to) const
    {
        if (to != nullptr && lane_id() == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (n[k])
                    atomicAdd(&to[k], (unsigned long long)n[k]);
    }
    __device__ __forceinline__ void flush(const BatchArgs& a) const
    {
        if (a.tally != nullptr)
            add_to(a.ws.tally_slots + (blockIdx.x % kTallySlots) * kTallyStride);
    }
};

// LDS entries of the per-wave shape-hash cache.
constexpr int kShapeCache = 32;
using WaveShapeCache = ShapeCache<kShapeCache>;

// D4 hash of a shape of `size` cells given as its anchored 8 x 8 bitmap (`fits`),
// else the one in the lane's OCC, for lanes with `want` (called by the whole
// wave).  A monomer and a domino have one shape each up to D4, so constant
// hashes.  Bitmaps go through the wave's cache; a miss hashes the bitmap and
// fills it.
template <class Grid>
__device__ __forceinline__ uint32_t det_hash(Grid& g, WaveShapeCache& cache, bool want,
                                             int size, int grid, bool fits, uint64_t key,
                                             const ShapeTable& table = ShapeTable{})
{
    uint32_t h = 0;
    bool miss = false;
    if (want) {
        if (size <= 2) {
            h = size <= 1 ? kMonomerHash : kDominoHash;
        } else if (!fits) {
            h = shape_hash(g, grid);
        } else if (!cache.lookup(key, h)) {
            h = bitmap8_shape_hash(key);
            miss = true;
        }
    }
    cache.insert(miss, key, h, lane_id(), table);
    return h;
}

// Adds the DET shapes of lanes with `want` to the call's shape table, if it has
// one (called by the whole wave after det_hash): a bitmap that the cache holds
// is counted in its entry, to be added when the entry goes or the wave ends.
__device__ __forceinline__ void count_shapes(const ShapeTable& table, WaveShapeCache& cache,
                                             bool want, int size, bool fits, uint64_t key,
                                             uint32_t hash)
{
    if (table.entries == nullptr)
        return;
    // (monomers and dominoes have bitmaps like the rest)
    const bool small = size <= 2;
    if (want && small)
        atomicAdd(&cache.small_count[size - 1], 1u);
    cache.count_other(want && !small && (!fits || !cache.count(key)), hash, size, lane_id(), table);
}

// ---------------------------------------------------------------------------
// Screen of a genotype's seed (§3.2: what the seed decides).
// ---------------------------------------------------------------------------
constexpr int kRing = 128;   // LDS survivor ring per wave (>= 2 chunks)

constexpr int kScreenKeep = 100;   // not decided by the seed
constexpr int kScreenSkip = 101;   // nothing to do at this queue position

// Queue position pos (`in_range`: it has an item): the item's index i; its
// class and record if the seed decides it (the return value), else
// kScreenKeep and its seed's site codes.
template <class M, int kIn>
__device__ __forceinline__ bool screen_item(const BatchArgs& a, uint64_t first, int klass,
                                            uint32_t pos, bool in_range, uint32_t& i,
                                            uint32_t& opts, int& cls, jatam_result_t& rec)
{
    i = pos;
    opts = 0;
    cls = kScreenSkip;
    rec = jatam_result_t{JATAM_INVALID, 0, 0u, 0};
    if (in_range && a.order != nullptr) {
        i = a.order[pos];
        in_range = i < (uint64_t)a.n;   // an entry out of range is skipped
    }
    if (!in_range)
        return false;
    const Geno s = fetch_geno<kIn>(a, first, i);
    if (!s.valid) {
        // exactly one launched pass reports an invalid item: its grid's class,
        // or with the window on (the 32 x 32 class then reruns listed items
        // only) the 16 x 16 class
        if (a.narrow_max > 16 ? klass == 0 : grid_class(a, s.grid) == klass) {
            cls = JATAM_INVALID;
            return true;
        }
    } else if (grid_class(a, s.grid) == klass) {
        const M sm = build_bonds<M>(s.genome, s.t, a.bits, a.c);
        opts = sm.codes(sm.seed());
        if ((opts & kSiteMulti) != 0) {
            cls = JATAM_ND_SITE;
            rec = jatam_result_t{JATAM_ND_SITE, 1, 0u, 0};
            return true;
        }
        if (opts == 0) {   // nothing bonds to the seed
            cls = JATAM_DET;
            rec = jatam_result_t{JATAM_DET, 1, kMonomerHash, 0};
            return true;
        }
        cls = kScreenKeep;
    }
    return false;
}

// ---------------------------------------------------------------------------
// Input chunks.  Those below static_end are dealt out: a wave owns its index +
// k * nwaves.  The rest are claimed a few at a time by the waves that run out
// of work first, which evens out the waves' end times.  They are split into
// eight contiguous parts with a counter each (one atomic per claim on one
// address from every wave serialises): a wave starts at part (wave mod 8),
// its XCD's under the round-robin dispatch of workgroups, and moves on to the
// next part when one runs dry, so the parts even out among themselves too.
// Claims are made only where every wave gets at least 16 chunks (with a chunk
// or two per wave there is nothing to even out), of up to claim_chunks chunks,
// fewer while a large claim would leave most waves without one.
// ---------------------------------------------------------------------------
struct ChunkSource {
    uint32_t nchunks, static_end, claim_size, next_chunk, claim_next, claim_end;
    uint32_t claim_blocks, part_blocks, part, parts_dry;
    uint32_t* counters;
    bool claims_left;

    __device__ __forceinline__ void init(const BatchArgs& a, int klass, uint32_t chunks)
    {
        const uint32_t nwaves = gridDim.x, wave = blockIdx.x;
        nchunks = chunks;
        const uint32_t per_wave = nchunks / (16u * nwaves);
        static_end = per_wave < 1u
                         ? nchunks
                         : nchunks - (uint32_t)((uint64_t)nchunks * (uint32_t)a.dyn16 / 16u);
        claim_size = per_wave < (uint32_t)a.claim_chunks ? per_wave : (uint32_t)a.claim_chunks;
        next_chunk = wave;
        claim_next = claim_end = 0;   // chunks claimed, not yet taken
        claims_left = static_end < nchunks;
        claim_blocks = claim_size == 0 ? 0u : (nchunks - static_end + claim_size - 1) / claim_size;
        part_blocks = (claim_blocks + kClaimCounters - 1) / kClaimCounters;
        counters = a.ws.run_claim + klass * kClaimCounters * kClaimStride;
        part = wave % (uint32_t)kClaimCounters;
        parts_dry = 0;
    }

    // The wave's next chunk (wave-uniform); false if there is none, or if the
    // next would have to be claimed and may_claim is not set.
    __device__ __forceinline__ bool take(uint32_t& chunk, bool may_claim)
    {
        if (next_chunk < static_end) {
            chunk = next_chunk;
            next_chunk += gridDim.x;
            return true;
        }
        if (claim_next == claim_end) {
            if (!claims_left || !may_claim)
                return false;
            uint32_t base = nchunks;
            while (parts_dry < (uint32_t)kClaimCounters) {
                uint32_t q = 0;
                if (lane_id() == 0)
                    q = atomicAdd(counters + part * kClaimStride, 1u);
                const uint32_t blk = part * part_blocks + (uint32_t)__shfl((int)q, 0);
                if (blk < min((part + 1u) * part_blocks, claim_blocks)) {
                    base = static_end + blk * claim_size;
                    break;
                }
                part = (part + 1u) % (uint32_t)kClaimCounters;
                ++parts_dry;
            }
            if (base >= nchunks) {
                claims_left = false;
                return false;
            }
            claim_next = base;
            claim_end = min(base + claim_size, nchunks);
        }
        chunk = claim_next++;
        return true;
    }
};

// ---------------------------------------------------------------------------
// The 16 x 16 window (items of G > 16 classified in the 16 x 16 layout, see
// run_geno).  An item that comes out UNBOUND there exposed a bondable site on
// the window's ring in some run up to the deciding one; every other item's
// record is exact: no run up to the deciding one left the window, so those
// runs equal the runs in the item's own grid.  The items that left get no
// record but are listed for a rerun of the pipeline in 32 x 32 grids: those of
// the first runs behind their wave's staged candidates, moved to the list with
// the size sort, those of the repeat runs appended to it here.  (Finding them
// by a pass over all items' records took 0.86 of 7.0 ms on 2^26 mixed items.)
// Called by the whole wave.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void append_overflow(const BatchArgs& a, bool leaves, uint32_t idx)
{
    const uint64_t m = __ballot(leaves);
    if (m == 0)
        return;
    uint32_t at = 0;
    if (lane_id() == 0)
        at = atomicAdd(a.ws.counters + kCntOverflow, (uint32_t)__popcll(m));
    at = (uint32_t)__shfl((int)at, 0);
    if (leaves)
        a.ws.overflow[at + (uint32_t)__popcll(m & lanes_below())] = idx;
}

// ---------------------------------------------------------------------------
// repeat<W>: all R runs of a candidate at once, one lane per run.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_inclusive_sum(int v)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(v, off);
        v += lane_id() >= off ? u : 0;
    }
    return v;
}

//
// With rpass < R (the first of two passes) a group of rpass lanes makes runs
// 0 .. rpass-1 of its candidate: a witness among them decides the record as
// above; a candidate without one goes to queue_out (count_out counts them)
// for the second pass, rpass = R, which makes the rest of its runs.  Most
// non-deterministic candidates are decided by run 1, 2 or 3, so the first
// pass spares most of the runs a single pass would make.
//
// A candidate left undecided by runs 0 .. k-1 ended all of them in run 0's
// occupancy, with size0 - 1 placements each.  In the 16 x 16 layout the
// first pass stores that occupancy at the candidate's queue_out position: its
// bitmap near the seed and its size in cand_shape (free after the size sort)
// if all of it lies there, else eight words, 0-3 in cand_shape and 4-7 in
// occ_hi.  The second pass (skip = k) then makes runs k .. R-1 only, each
// compared with what is stored.
constexpr uint32_t kStoredNear = 0xFFFFFFFFu;   // as word 3: columns 15 are never occupied

// Occupancy word w (rows 2w and 2w + 1) of a finished run in the 16 x 16 layout;
// row 15, never occupied, holds the wave's own data.
__device__ __forceinline__ uint32_t occ_word(LeanGrid<16>& g, int w)
{
    return g.row(2 * w) | (w < 7 ? g.row(2 * w + 1) << 16 : 0u);
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int lane)
{
    return ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(v >> 32), lane) << 32) |
           (uint32_t)__shfl((int)(uint32_t)v, lane);
}

// The LDS and the per-lane layout of the R-lanes-per-candidate repeat runs:
// runs skip .. rpass-1 of each candidate, lane jr of group grp making run
// skip + jr.  round() runs one candidate per group (active groups only) to
// its record, or (a first pass without a witness) to the second queue.
// kSolo: the second queue is a list of indices in LDS (queue_out, its length
// in `kept`), orient has kSoloGroups columns, `out` may be null, DET records are
// counted in `table` if it has one, and a pass of run 0 alone proves the shapes
// that it can (those whose tiles' ids were lost had no proof before).
constexpr int kSoloGroups = 32;   // candidates per round at two lanes each

template <int W, class M, bool kSolo>
struct RepeatWave {
    static constexpr int kGroups = kSolo ? kSoloGroups : 64;
    const BatchArgs& a;
    uint64_t first;
    jatam_result_t* out;
    LeanGrid<W> g;           // this lane's grid
    LeanGrid<W> g0;          // the group's lead lane's grid
    uint32_t* orient;        // hash k of group grp at [k * kGroups + grp]
    WaveShapeCache& cache;
    RunState& st;
    WaveTally& tally;
    int skip;
    bool store_occ, all_runs;
    int R, groups, lane, grp, jr, run, lead, tail;
    uint64_t gmask;
    uint32_t* queue_out;
    uint32_t* count_out;
    ShapeTable table;
    uint32_t kept = 0;       // kSolo: entries of queue_out

    __device__ RepeatWave(const BatchArgs& a_, uint32_t* smem, uint32_t* orient_,
                          WaveShapeCache& cache_, RunState& st_, WaveTally& tally_, int rpass,
                          int skip_, bool store_occ_, uint32_t* queue_out_, uint32_t* count_out_,
                          const ShapeTable& table_ = ShapeTable{})
        : a(a_), first(slice_first(a_)), out(slice_out(a_)), g{smem + threadIdx.x},
          g0{smem}, orient(orient_), cache(cache_), st(st_), tally(tally_), skip(skip_),
          store_occ(store_occ_), all_runs(rpass >= a_.runs), R(rpass - skip_),
          groups(kSolo && rpass - skip_ < 2 ? kSoloGroups : 64 / (rpass - skip_)), lane((int)threadIdx.x), grp(0), jr(0), run(0), lead(0),
          tail(0), gmask(0), queue_out(queue_out_), count_out(count_out_), table(table_)
    {
        grp = lane / R;
        jr = lane - grp * R;
        run = skip + jr;
        lead = grp * R;            // lane making run `skip`
        tail = lead + R - 1;       // lane making run rpass-1
        gmask = R == 64 ? ~0ull : ((1ull << R) - 1);
        g0 = LeanGrid<W>{smem + lead};
    }

    // `active`: this lane's group has candidate idx (wave-uniform per group);
    // `slot`: its position in the input queue (where a first pass stored
    // run 0's occupancy, read when skip > 0).  Called by the whole wave.
    __device__ void round(bool active, uint32_t idx, uint32_t slot)
    {
        Geno gd{};
        int ev = kEvNone;
        bool proven = false;
        if (active) {
            gd = run_geno<W>(a, first, idx);
            const M src = build_bonds<M>(gd.genome, gd.t, a.bits, a.c);
            ev = run_assembly(src, g, st, gd.grid, run_key(a, gd, run));
            if constexpr (kSolo && M::kManyIds) {
                if (R == 1 && ev == kEvNone) {
                    uint64_t shape = 0;
                    int x0 = 0, y0 = 0;
                    const bool fits = shape_key8(g, st, gd.grid, st.size(), shape, x0, y0);
                    const TileIds ids = shape_ids(src, g, st, gd.grid, fits, shape, x0, y0);
                    proven = shape_is_guarded(src, g, ids, gd.grid, fits, shape, x0, y0);
                }
            }
        }
        wave_lds_sync();   // every run's grid is final
        // a witness is a later run that hit an event or ended in another
        // shape than run 0 (the lead lane's, or the stored one): compared by
        // the bitmaps near the seed where run 0's holds all of its cells,
        // else cell by cell
        bool same = true;
        int size0 = __shfl(st.size(), lead);          // run 0's (skip = 0: the lead's)
        uint64_t near0 = shfl64(st.near, lead);
        if (W == 16 && !kSolo && skip > 0 && active) {
            const uint4 lo = a.ws.cand_shape[slot];
            if (lo.w == kStoredNear) {
                near0 = ((uint64_t)lo.y << 32) | lo.x;
                size0 = (int)lo.z;
            } else {
                const uint4 hi = a.ws.occ_hi[slot];
                const uint32_t o[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                size0 = 0;
                near0 = 0;
#pragma unroll
                for (int w = 0; w < 8; ++w) {
                    size0 += __popc(o[w]);
                    if constexpr (W == 16)
                        same = same && (ev != kEvNone || occ_word(g, w) == o[w]);
                }
            }
        }
        const bool near_all = __popcll(near0) == size0;
        if (active && near_all)
            same = st.near == near0 && st.size() == size0;
        else if (active && skip == 0 && ev == kEvNone)
            same = same_cells(g, g0, gd.grid);
        const bool witness = active && (skip > 0 || jr > 0) && (ev != kEvNone || !same);
        const uint64_t wm = (__ballot(witness) >> lead) & gmask;
        const int fw = wm ? (int)__builtin_ctzll(wm) : R;      // R: no witness
        const int wl = lead + (fw < R ? fw : 0);
        const int w_ev = __shfl(ev, wl);
        const int w_size = __shfl(st.size(), wl);
        const int lead_ev = __shfl(ev, lead);
        int cls;
        if (lead_ev == kEvCorrupt || (fw < R && w_ev == kEvCorrupt))
            cls = JATAM_INVALID;
        else if (fw == R)
            cls = JATAM_DET;
        else
            cls = w_ev == kEvUnbound ? JATAM_UNBOUND
                : w_ev == kEvAmbig   ? JATAM_ND_SITE
                                     : JATAM_ND_RUNS;
        // placements summed over runs 0..first witness (all R runs if DET);
        // the skipped runs made size0 - 1 each
        const int last = fw < R ? fw : R - 1;
        const int incl = wave_inclusive_sum(active && jr <= last ? st.steps : 0);
        int steps = __shfl(incl, tail) - __shfl(incl, lead) + __shfl(st.steps, lead) +
                    skip * (size0 - 1);
        if (proven)
            steps = (size0 - 1) * a.runs;
        // without a witness in a first pass the candidate waits for the second
        const bool undecided = active && fw == R && !all_runs && cls == JATAM_DET && !proven;
        const uint64_t um = __ballot(undecided && jr == 0);
        if (um != 0) {
            uint32_t at = kept;
            if constexpr (!kSolo) {
                if (lane == 0)
                    at = atomicAdd(count_out, (uint32_t)__popcll(um));
                at = (uint32_t)__shfl((int)at, 0);
            }
            kept += (uint32_t)__popcll(um);
            const uint32_t qslot = at + (uint32_t)__popcll(um & lanes_below());
            if (undecided && jr == 0)
                queue_out[qslot] = idx;
            if constexpr (W == 16 && !kSolo) {
                if (store_occ && undecided && jr == 0) {
                    if (near_all) {
                        a.ws.cand_shape[qslot] = make_uint4((uint32_t)near0,
                                                            (uint32_t)(near0 >> 32),
                                                            (uint32_t)size0, kStoredNear);
                    } else {
                        a.ws.cand_shape[qslot] = make_uint4(occ_word(g, 0), occ_word(g, 1),
                                                            occ_word(g, 2), occ_word(g, 3));
                        a.ws.occ_hi[qslot] = make_uint4(occ_word(g, 4), occ_word(g, 5),
                                                        occ_word(g, 6), occ_word(g, 7));
                    }
                }
            }
        }
        const bool det = active && cls == JATAM_DET && !undecided;
        // run 0's shape: from the wave's cache, else the group's lanes share
        // its 8 orientation hashes
        uint64_t key = 0;
        bool small = false, hit = false;
        uint32_t cached = 0;
        if (det && size0 > 2) {
            int x0, y0;
            RunState run0{};
            run0.near = near0;
            small = shape_key8(g0, run0, gd.grid, size0, key, x0, y0);
            hit = small && cache.lookup(key, cached);
            if (!hit) {
                if (small) {
                    int w8, h8;
                    bitmap8_dims(key, w8, h8);
                    for (int k = jr; k < 8; k += R)
                        orient[k * kGroups + grp] = bitmap_hash8(image8(key, w8, h8, k));
                } else {
                    const ShapeBox bx = crop(g0, gd.grid);
                    for (int k = jr; k < 8; k += R)
                        orient[k * kGroups + grp] = orientation_hash(g0, bx, k);
                }
            }
        }
        wave_lds_sync();
        const bool leaves =
            W == 16 && active && jr == 0 && cls == JATAM_UNBOUND && gd.windowed;
        if constexpr (W == 16 && !kSolo)
            append_overflow(a, leaves, idx);
        const bool done = active && jr == 0 && !undecided && !leaves;
        uint32_t h = 0;
        if (done) {
            jatam_result_t rec;
            if (det) {
                if (size0 <= 2) {
                    h = size0 <= 1 ? kMonomerHash : kDominoHash;
                } else if (hit) {
                    h = cached;
                } else {
                    uint32_t hs[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        hs[k] = orient[k * kGroups + grp];
                    h = combine_orientations(hs);
                }
                rec = jatam_result_t{JATAM_DET, size0, h, steps};
            } else if (cls == JATAM_INVALID) {
                rec = jatam_result_t{JATAM_INVALID, 0, 0u, 0};
            } else {
                rec = jatam_result_t{cls, w_size, 0u, steps};
            }
            if (!kSolo || out != nullptr)
                out[idx] = rec;
        }
        tally.add(done, cls);
        cache.insert(done && det && small && !hit, key, h, lane, table);
        if constexpr (kSolo)
            count_shapes(table, cache, done && det, size0, small, key, h);
        wave_lds_sync();   // orientation slots and grids reused next round
    }
};

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
// One-wave workgroups of `kernel` that are resident on a CU at once.  The
// runtime's answer is capped by the CU's LDS as it is handed out on gfx950:
// in granules of 1,280 bytes, 128 per CU.  (Measured with spinning
// workgroups of a given dynamic LDS size: eleven of 14,080 bytes run
// together, eleven of 14,336 do not, nor ten of 15,744, while four of
// 39,680 and three of 52,480 do; the runtime reports eleven, eleven and ten
// for the first three.  A persistent grid sized above the true count leaves
// its last workgroups waiting for the first ones to finish.)
template <class K>
int resident_per_cu(K kernel)
{
    constexpr size_t kLdsGranule = 1280, kLdsGranules = 128;
    int occ = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, 64, 0) != hipSuccess || occ < 1)
        occ = 1;
    hipFuncAttributes attr;
    if (hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(kernel)) == hipSuccess &&
        attr.sharedSizeBytes > 0) {
        const size_t granules = (attr.sharedSizeBytes + kLdsGranule - 1) / kLdsGranule;
        const int fit = (int)(kLdsGranules / granules);
        occ = fit < occ ? (fit < 1 ? 1 : fit) : occ;
    }
    return occ;
}

}  // namespace jatam
