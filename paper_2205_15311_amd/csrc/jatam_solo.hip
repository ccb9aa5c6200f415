// jatam_solo.hip - the whole classification in one launch: every wave takes
// genotypes from the seed's screen to their records by itself, without queues in
// device memory.
//
// A wave screens chunks of its input and keeps each lane busy with first runs
// (as first_run_kernel does).  What a clean first run leaves open goes through
// two lists in LDS: packed shapes, proven 64 at a time by all lanes together
// (the proof of one candidate by its own lane would leave the others idle),
// and the candidates that are not proven, whose repeat runs the wave makes in
// rounds (RepeatWave) when its first runs are done, or before if the list fills
// up: runs 0-3 of sixteen candidates at a time, above 32 runs then runs 0-15 of
// four, then all R runs of those without a witness; all R at once where R is at
// most eight.  Up to four runs at G <= 16 it makes them without a proof.
//
// Against the pipeline of jatam_batched.hip it needs one launch instead of
// eight, no workspace and no staging (150 bytes a candidate through HBM), and no
// wave waits for another's first runs; it pays with proofs of mixed sizes and
// with repeat rounds that no other wave shares.
//
// The same kernel makes the first stage of the true class (kOpen): run 0 of every
// genotype and the proof, and what these leave open to a list in device memory.
#include "jatam_waves.hpp"

namespace jatam {

constexpr int kSoloPend = 128;    // unproven candidates: drained above 64
constexpr int kSoloShapes = 64;   // packed shapes waiting for a proof
constexpr int kSecondRuns = 16;   // runs of a second pass of three, and candidates for it
// An unproven candidate (positions are below 2^31) whose tiles' ids were lost, so that
// it has had no proof; from this many of them in a wave's list on they get one, with a
// run 0 of their own.  (Uniform four-tile lists have a few a wave: 2^20 of them 200
// instead of 163 us with a proof for each.  Lists of such shapes only: 2^20 at G = 16
// 189 us, 934 with all runs made.)
constexpr uint32_t kLost = 1u << 31;
constexpr uint32_t kLostProof = 16;

// Three waves a SIMD in the 16 x 16 layout: twelve a CU, where LDS holds eleven
// (with 177 registers two: an enumeration of S_{2,8} 1.27 instead of 1.21 ms).
template <int W, class M, int kIn, bool kOpen>
__global__ __launch_bounds__(64, W == 16 ? 3 : 1) void solo_kernel(const BatchArgs a, int klass,
                                                  uint32_t chunk_items, bool direct_tally,
                                                  ShapeTable table, OpenList open)
{
    using Grid = LeanGrid<W>;
    const uint64_t first = a.first;
    jatam_result_t* const out = a.out;
    __shared__ __attribute__((aligned(16))) uint32_t smem[Grid::kLaneWords * 64];
    __shared__ uint4 shapes[kSoloShapes];
    __shared__ uint32_t shape_idx[kSoloShapes];
    __shared__ uint32_t pend[kSoloPend];
    __shared__ uint32_t orient[8 * kSoloGroups];
    __shared__ uint4 cache_mem[kShapeCache];
    __shared__ uint32_t small_count[2];
    __shared__ uint4 other_shapes[WaveShapeCache::kOther];
    uint32_t* const ring = smem + Grid::kSpare;   // survivor indices
    // the second list of a drain: the shapes are all proven then
    uint32_t* const undecided = reinterpret_cast<uint32_t*>(shapes);
    static_assert(kRing <= 64 * (W / 8), "the ring fits row W-1's PEND words");
    static_assert(kSoloPend * 4 <= sizeof(shapes), "the undecided list fits the shapes'");
    const uint32_t lane = (uint32_t)lane_id();
    Grid g{smem + threadIdx.x};
    g.clear_all();
    WaveShapeCache cache{cache_mem, small_count, other_shapes};
    cache.clear((int)lane);
    if (lane < 2)
        small_count[lane] = 0;
    if (lane < WaveShapeCache::kOther)
        other_shapes[lane] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    RunState st{};
    WaveTally tally{{0, 0, 0, 0}};
    const uint32_t n_items = (uint32_t)a.n;
    ChunkSource chunks;
    chunks.init(a, klass, (n_items + chunk_items - 1) / chunk_items);
    // In the 16 x 16 layout up to four runs cost less than the proof: 2^20 genotypes at
    // R = 2, G = 16, uniform two-tile ones 215 -> 177 us, deterministic ones 393 -> 324,
    // some that run 0 calls deterministic and run 1 may not 542 -> 390.  At G = 32, where
    // runs are longer, 2^20 uniform two-tile ones would take 955 instead of 602.
    constexpr bool direct_runs = W == 16 && !kOpen;
    uint32_t head = 0, queued = 0, nshapes = 0, npend = 0, nlost = 0;   // wave-uniform
    bool busy = false, starved = false;
    uint32_t idx = 0;
    Geno gd{};
    M m{};
    int ev = kEvNone;

    // Records of the waiting shapes that are guarded; the rest to the list of
    // unproven candidates.
    auto prove_shapes = [&]() {
        wave_lds_sync();
        const bool active = lane < nshapes;
        bool forced = false;
        int size = 0;
        uint32_t i = 0;
        uint64_t key = 0;
        if (active) {
            i = shape_idx[lane];
            const uint4 sh = shapes[lane];
            const Geno s = run_geno<W, kIn>(a, first, i);
            forced = packed_shape_is_guarded(build_bonds<M>(s.genome, s.t, a.bits, a.c), sh);
            key = ((uint64_t)sh.y << 32) | sh.x;
            size = __popcll(key);
        }
        const uint32_t h = det_hash(g, cache, forced, size, 0, true, key, table);
        if (forced && out != nullptr)
            out[i] = jatam_result_t{JATAM_DET, size, h, kOpen ? 0 : (size - 1) * a.runs};
        count_shapes(table, cache, forced, size, true, key, h);
        tally.add(forced, JATAM_DET);
        const uint64_t km = __ballot(active && !forced);
        if (active && !forced)
            pend[npend + (uint32_t)__popcll(km & lanes_below())] = i;
        npend += (uint32_t)__popcll(km);
        nshapes = 0;
        wave_lds_sync();
    };
    // kOpen: the unproven candidates to the call's list.
    auto hand_over = [&]() {
        wave_lds_sync();
        uint32_t at = 0;
        if (lane == 0 && npend != 0)
            at = atomicAdd(open.count, npend);
        at = (uint32_t)__shfl((int)at, 0);
        for (uint32_t j = lane; j < npend; j += 64)
            open.items[at + j] = open.base + (pend[j] & ~kLost);
        npend = 0;
        wave_lds_sync();
    };
    // Repeat rounds over the unproven candidates, in passes of ever more lanes each.
    // A pass lists the candidates it leaves undecided for the next one, in the second
    // list, which can be the one it reads: a round's candidates are read before it
    // appends any, and are no fewer.
    auto drain = [&]() {
        uint32_t* list = pend;
        uint32_t count = npend, kept = 0;
        // runs 0-3 first; above 32 runs, where a round of all runs takes one candidate
        // only, 16 if many are left.  (2^20 two-tile genotypes that run 0 calls
        // deterministic and later runs do not, R = 64: 1.79 -> 1.06 ms; for few the
        // pass does not pay, 2^20 uniform four-tile ones 180 -> 198 us.)
        auto pass_after = [&](int runs) {
            return runs < kRepeatFirstRuns && a.runs > 2 * kRepeatFirstRuns ? kRepeatFirstRuns
                   : runs < kSecondRuns && a.runs > 32 && count >= (uint32_t)kSecondRuns
                       ? kSecondRuns
                       : a.runs;
        };
        int rpass = pass_after(0);
        if (M::kManyIds && nlost >= kLostProof) {
            wave_lds_sync();
            uint32_t lost = 0;
            for (uint32_t at = 0; at < npend; at += 64) {
                const uint32_t i = at + lane < npend ? pend[at + lane] : 0u;
                const bool there = at + lane < npend, is_lost = (i & kLost) != 0u;
                const uint64_t lm = __ballot(is_lost), om = __ballot(there && !is_lost);
                if (is_lost)
                    pend[lost + (uint32_t)__popcll(lm & lanes_below())] = i;
                else if (there)
                    undecided[kept + (uint32_t)__popcll(om & lanes_below())] = i;
                lost += (uint32_t)__popcll(lm);
                kept += (uint32_t)__popcll(om);
                wave_lds_sync();
            }
            rpass = 1;
            count = lost;
        }
        for (;;) {
            RepeatWave<W, M, true> rw(a, smem, orient, cache, st, tally, rpass, 0, false, undecided,
                                      nullptr, table);
            rw.kept = kept;
            const uint32_t groups = (uint32_t)rw.groups, grp = (uint32_t)rw.grp;
            for (uint32_t at = 0; at < count; at += groups) {
                const bool active = grp < groups && at + grp < count;
                rw.round(active, active ? list[at + grp] & ~kLost : 0u, 0u);
            }
            wave_lds_sync();
            if (rpass >= a.runs)
                break;
            list = undecided;
            count = rw.kept;
            kept = 0;
            rpass = pass_after(rpass);
        }
        npend = nlost = 0;
    };

    for (;;) {
        // -- lanes whose first run is over ------------------------------------
        const bool finish = busy && run_over(ev, st, gd.grid);
        if (__ballot(finish) != 0) {
            bool done = false, candidate = false, det = false, pack = false, lost = false;
            int cls = 0, steps = st.steps;
            jatam_result_t rec{0, 0, 0u, 0};
            if (finish) {
                done = true;
                if (ev == kEvCorrupt) {
                    rec = jatam_result_t{JATAM_INVALID, 0, 0u, 0};
                    cls = JATAM_INVALID;
                } else if (ev != kEvNone) {
                    cls = ev == kEvUnbound && !kOpen ? JATAM_UNBOUND : JATAM_ND_SITE;
                    rec = kOpen ? jatam_result_t{cls, 0, 0u, 0}
                                : jatam_result_t{cls, st.size(), 0u, st.steps};
                } else if (!st.choice || (!kOpen && a.runs == 1)) {
                    // no random word was drawn: every run would be this run
                    det = true;
                } else {
                    done = false;
                    candidate = true;
                }
            }
            uint64_t key = 0;
            int x0 = 0, y0 = 0;
            bool fits = false;
            uint4 packed = packed_none();
            if (det || candidate)
                fits = shape_key8(g, st, gd.grid, st.size(), key, x0, y0);
            if (candidate && (!direct_runs || a.runs > kRepeatFirstRuns)) {
                if (fits)
                    packed = pack_shape(g, st, gd.grid, st.size(), key, x0, y0);
                pack = packed_shape_valid(packed);
                lost = M::kManyIds && st.lost != 0;
                // a shape too large to wait for the others is checked at once
                if (!pack && !lost &&
                    shape_is_guarded(m, g, TileIds{true, 0ull}, gd.grid, fits, key, x0, y0)) {
                    candidate = false;
                    det = true;
                    steps = st.steps * a.runs;
                }
            }
            if (__ballot(det) != 0) {
                const uint32_t h =
                    det_hash(g, cache, det, st.size(), gd.grid, fits, key, table);
                count_shapes(table, cache, det, st.size(), fits, key, h);
                if (det) {
                    done = true;
                    cls = JATAM_DET;
                    rec = jatam_result_t{JATAM_DET, st.size(), h, kOpen ? 0 : steps};
                }
            }
            if (done && out != nullptr)
                out[idx] = rec;
            busy = busy && !finish;
            tally.add(done, cls);
            const uint64_t pm = __ballot(candidate && pack);
            if (nshapes + (uint32_t)__popcll(pm) > (uint32_t)kSoloShapes)
                prove_shapes();
            if (candidate && pack) {
                const uint32_t at = nshapes + (uint32_t)__popcll(pm & lanes_below());
                shapes[at] = packed;
                shape_idx[at] = idx;
            }
            nshapes += (uint32_t)__popcll(pm);
            const uint64_t um = __ballot(candidate && !pack);
            if (candidate && !pack)
                pend[npend + (uint32_t)__popcll(um & lanes_below())] = idx | (lost ? kLost : 0u);
            npend += (uint32_t)__popcll(um);
            if constexpr (M::kManyIds && !kOpen)
                nlost += (uint32_t)__popcll(__ballot(candidate && !pack && lost));
        }
        // -- refill idle lanes once enough of them wait, unless the list of
        // unproven candidates has to be worked off first: every waiting shape
        // and every busy lane may add one to it, and after a refill 64 lanes
        // are busy ------------------------------------------------------------
        const uint64_t idle = __ballot(!busy);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (npend + nshapes + 64u > (uint32_t)kSoloPend && nshapes != 0)
            prove_shapes();
        if (kOpen && npend + 64u > (uint32_t)kSoloPend)
            hand_over();
        const bool full = !kOpen && npend + 64u > (uint32_t)kSoloPend;
        if (!full && (nidle >= (uint32_t)a.refill || nidle == 64)) {
            starved = false;
            while (queued < nidle) {
                uint32_t chunk;
                if (!chunks.take(chunk, true)) {
                    starved = true;
                    break;
                }
                uint32_t i, opts;
                int cls;
                jatam_result_t rec;
                const uint32_t pos = chunk * chunk_items + lane;
                const bool wrote = screen_item<M, kIn>(
                    a, first, klass, pos, lane < chunk_items && pos < n_items, i, opts, cls, rec);
                const bool keep = cls == kScreenKeep;
                if (kOpen && cls == JATAM_ND_SITE)
                    rec.size = 0;
                if (wrote && out != nullptr)
                    out[i] = rec;
                count_shapes(table, cache, wrote && cls == JATAM_DET, 1, true, 1ull, kMonomerHash);
                tally.add(wrote && cls != JATAM_INVALID, cls);
                const uint64_t km = __ballot(keep);
                if (keep)
                    ring[(head + queued + (uint32_t)__popcll(km & lanes_below())) % kRing] = i;
                queued += (uint32_t)__popcll(km);
            }
            wave_lds_sync();   // ring writes visible to the whole wave
            const uint32_t take = queued < nidle ? queued : nidle;
            if (!busy) {
                const uint32_t rank = (uint32_t)__popcll(idle & lanes_below());
                if (rank < take) {
                    idx = ring[(head + rank) % kRing];
                    gd = run_geno<W, kIn>(a, first, idx);
                    m = build_bonds<M>(gd.genome, gd.t, a.bits, a.c);
                    ev = run_start_known(g, st, gd.grid, m.codes(m.seed()));
                    busy = true;
                }
            }
            head = (head + take) % kRing;
            queued -= take;
            wave_lds_sync();   // ring slots read before they are refilled
        }
        if (__ballot(busy) == 0) {
            const bool over = queued == 0 && starved;
            if (full || over) {
                prove_shapes();
                if constexpr (kOpen)
                    hand_over();
                else
                    drain();
            }
            if (over)
                break;
            continue;
        }
        // -- groups of four steps until enough lanes wait (every lane, once no
        // chunk is left or a drain is due), at least one group ----------------
        const uint32_t enough = full || (queued == 0 && starved) ? 65u : (uint32_t)a.refill;
        for (;;) {
            const bool stepping = busy && !run_over(ev, st, gd.grid);
            const uint64_t still = __ballot(stepping);
            if (still == 0)
                break;
            if (enough > 64u && (still & (still - 1)) == 0) {
                const uint32_t last = (uint32_t)__builtin_ctzll(still);
                const int end = lone_run(m, g, st, gd.grid, run_key(a, gd, 0), last);
                if (stepping)
                    ev = end;
                break;
            }
            if (stepping)
                ev = run_four(m, g, st, gd.grid, run_key(a, gd, 0));
            const uint64_t waiting = __ballot(!busy || run_over(ev, st, gd.grid));
            if ((uint32_t)__popcll(waiting) >= enough)
                break;
        }
    }
    if constexpr (kOpen)
        return;
    cache.flush(table, (int)lane);
    if (direct_tally)
        tally.add_to(a.tally);
    else
        tally.flush(a);
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
void solo_occupancy(int solo[2][kGenoKinds])
{
    solo[0][kGenoTwo] = resident_per_cu(solo_kernel<16, Bonds2, kInRange, false>);
    solo[0][kGenoFour] = resident_per_cu(solo_kernel<16, Bonds4, kInRange, false>);
    solo[0][kGenoC16] = resident_per_cu(solo_kernel<16, BondsC16, kInRange, false>);
    solo[1][kGenoTwo] = resident_per_cu(solo_kernel<32, Bonds2, kInRange, false>);
    solo[1][kGenoFour] = resident_per_cu(solo_kernel<32, Bonds4, kInRange, false>);
    solo[1][kGenoC16] = resident_per_cu(solo_kernel<32, BondsC16, kInRange, false>);
}

template <int W, class M, bool kOpen>
static void launch_solo_t(const BatchArgs& a, int klass, uint32_t blocks, uint32_t chunk_items,
                          bool direct, const ShapeTable& table, const OpenList& open,
                          hipStream_t stream)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64), 0, stream, a, klass, chunk_items,
                           direct, table, open);
    };
    if (a.genomes != nullptr)
        go(solo_kernel<W, M, kInList, kOpen>);
    else if (kOpen || a.items == nullptr)
        go(solo_kernel<W, M, kInRange, kOpen>);
    else
        go(solo_kernel<W, M, kOpen ? kInRange : kInItems, kOpen>);
}

// Waves and chunk size for n items on at most `waves` waves: every wave some
// items, so chunks shrink to one item each where there are fewer items than
// lanes.
static uint32_t solo_blocks(uint64_t n, int waves, uint32_t& chunk)
{
    const uint64_t per = (n + (uint64_t)waves - 1) / (uint64_t)waves;
    chunk = per < 64 ? (uint32_t)per : 64u;
    const uint64_t nchunks = (n + chunk - 1) / chunk;
    return nchunks < (uint64_t)waves ? (uint32_t)nchunks : (uint32_t)waves;
}

template <bool kOpen>
static void launch_solo_class(const BatchArgs& a, int klass, int geno, uint32_t blocks,
                              uint32_t chunk, bool direct, const ShapeTable& table,
                              const OpenList& open, hipStream_t stream)
{
    if (klass == 0) {
        if (geno == kGenoTwo)
            launch_solo_t<16, Bonds2, kOpen>(a, 0, blocks, chunk, direct, table, open, stream);
        else if (geno == kGenoFour)
            launch_solo_t<16, Bonds4, kOpen>(a, 0, blocks, chunk, direct, table, open, stream);
        else
            launch_solo_t<16, BondsC16, kOpen>(a, 0, blocks, chunk, direct, table, open, stream);
    } else {
        if (geno == kGenoTwo)
            launch_solo_t<32, Bonds2, kOpen>(a, 1, blocks, chunk, direct, table, open, stream);
        else if (geno == kGenoFour)
            launch_solo_t<32, Bonds4, kOpen>(a, 1, blocks, chunk, direct, table, open, stream);
        else
            launch_solo_t<32, BondsC16, kOpen>(a, 1, blocks, chunk, direct, table, open, stream);
    }
}

void launch_first_open(const BatchArgs& a, int waves, int geno, const OpenList& open,
                       hipStream_t stream)
{
    uint32_t chunk;
    const uint32_t blocks = solo_blocks((uint64_t)a.n, waves, chunk);
    launch_solo_class<true>(a, a.grid <= 16 ? 0 : 1, geno, blocks, chunk, true, ShapeTable{},
                            open, stream);
}

int launch_solo(const BatchArgs& a, const bool classes[2], const int waves[2], int geno,
                jatam_shape_count_t* shapes, int log2cap, hipStream_t stream)
{
    if (a.n <= 0)
        return JATAM_OK;
    const ShapeTable table{shapes, log2cap};
    uint32_t blocks[2], chunk[2], most = 0;
    for (int k = 0; k < 2; ++k) {
        blocks[k] = solo_blocks((uint64_t)a.n, waves[k], chunk[k]);
        if (classes[k])
            most = blocks[k] > most ? blocks[k] : most;
    }
    // few waves add to the caller's tally themselves (their atomics on its four
    // words serialise, about 12 ns each); more go through the counter sets
    const bool direct = a.tally == nullptr || most <= 1024;
    bool cleared = false;
    for (int k = 0; k < 2; ++k) {
        if (!classes[k])
            continue;
        const bool slots = !direct && !cleared;
        if (a.dyn16 > 0 || slots)
            launch_clear(a.ws.run_claim + k * kClaimCounters * kClaimStride,
                         slots ? a.ws.tally_slots : nullptr, stream);
        cleared = true;
        launch_solo_class<false>(a, k, geno, blocks[k], chunk[k], direct, table, OpenList{},
                                 stream);
    }
    if (!direct)
        launch_tally(a.ws.tally_slots, a.tally, stream);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam
