// jatam_batched.hip - pipelined classification without global queues.
//
// With a whole genotype to each lane a wave lasts as long as its slowest
// genotype: on S_{2,8} the sum over waves of the slowest lane's
// work is ~7x the total work.  Here the classification is split by what the
// work actually is, into three stages per grid class (W = 16 or 32):
//
//   first_run<W>  persistent waves over 64-genotype input chunks: a share of
//                 the chunks is dealt out (chunk k to wave k mod the grid),
//                 the rest are claimed a few at a time from device counters
//                 by the waves that run out of work first.  A wave screens a
//                 chunk (decode, bond options of the seed: an ambiguous seed
//                 neighbour is ND_SITE, a seed with nothing to bond is a DET
//                 monomer; ~61% of S_{2,8}) and keeps the survivors in an LDS
//                 ring.  Each lane runs the
//                 first run of one survivor; a lane that finishes takes the
//                 next survivor at once, so lanes stay busy while run lengths
//                 differ.  A first run ending in an event or without ever
//                 drawing a random word is final; one that drew and ended
//                 cleanly makes the genotype a DET candidate, staged with its
//                 size and its packed run-0 shape in the wave's own segment.
//   size sort     a counting sort of the candidates by run-0 size, largest
//                 first (all runs of a deterministic genotype have that size,
//                 so this orders the later work by its exact cost): per
//                 segment histograms counted in LDS by the first-run waves
//                 as they stage, one scan, scatter with LDS cursors that
//                 moves each packed shape beside its candidate.
//   prove<W>      one lane per candidate checks whether its run-0 shape is
//                 guarded (every growth order ends in it), from the packed
//                 shape or, where the shape did not pack, a replay: then the
//                 record is final.
//   repeat<W>     R lanes per candidate, lane r making run r; the first
//                 witness in run order (an event or a shape different from
//                 run 0's) is found in LDS, and for DET genotypes the 8
//                 orientation hashes are split across the group's lanes.
//                 By default in two passes (runs 0-3, then the rest for the
//                 candidates without a witness); then the proof and the
//                 first pass share one kernel (prove_repeat), each wave
//                 claiming chunks of the sorted queue one at a time and
//                 running the repeat rounds of the candidates it failed to
//                 prove.  Or in one pass, or (repeat_seq) one lane per
//                 candidate making its runs in turn and stopping at the
//                 first witness, both after a separate proof and compaction.
//
// Global atomics on shared counters are few: the first-run claims, a few
// chunks at a time by waves that have finished their dealt-out share, and
// the fused kernel's chunk claims, one atomic per chunk, each spread over
// eight counters in separate 256-byte blocks (atomics on one address from
// every wave serialise); and the second repeat queue's counter, one atomic
// per wave and round of the first pass.  Every other queue is a per-wave
// segment or a scan.  Records are identical
// on every route: each is a pure function of the genotype, never of
// the schedule.
#include "jatam_waves.hpp"

namespace jatam {

__global__ void slice_reset_kernel(uint32_t* counter) { counter[0] = 0; }
__global__ void slice_advance_kernel(uint32_t* counter) { counter[0] += 1; }

int launch_slice_reset(uint32_t* counter, hipStream_t stream)
{
    hipLaunchKernelGGL(slice_reset_kernel, dim3(1), dim3(1), 0, stream, counter);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

int launch_slice_advance(uint32_t* counter, hipStream_t stream)
{
    hipLaunchKernelGGL(slice_advance_kernel, dim3(1), dim3(1), 0, stream, counter);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// The counter sets' sums to the caller's tally: wave k sums class k.
__global__ __launch_bounds__(256) void tally_kernel(const unsigned long long* __restrict__ slots,
                                                    unsigned long long* tally)
{
    static_assert(kTallySlots == 64, "one slot a lane");
    const int k = (int)(threadIdx.x >> 6);
    unsigned long long v = slots[lane_id() * kTallyStride + k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off);
    if (lane_id() == 0 && v != 0)
        atomicAdd(&tally[k], v);
}


// ---------------------------------------------------------------------------
// first_run<W>: screen + first runs with lane refill.
// ---------------------------------------------------------------------------
// Size-sort bucket of a run-0 size: 64 buckets, exact up to 47 cells, then
// 64 cells wide; the largest sizes get the smallest keys.
__device__ __forceinline__ uint32_t size_key(uint32_t size)
{
    const uint32_t b = size < 48 ? size : 48 + min(15u, (size - 48) >> 6);
    return kSizeBuckets - 1 - b;
}

template <int W, class M, int kIn>
__global__ __launch_bounds__(64) void first_run_kernel(const BatchArgs a, int klass)
{
    using Grid = LeanGrid<W>;
    const uint64_t first = slice_first(a);
    jatam_result_t* const out = slice_out(a);
    // The wave's survivor ring, seed codes, hash cache and size counts, as far
    // as they fit in the grid's spare words: 11,520 bytes of LDS in all for
    // W = 16 (9 granules of 1,280: 14 waves a CU) and 40,960 for W = 32
    // (4 waves), where the seed codes are worked out again at the start.
    constexpr bool kKeepCodes = W == 16;
    constexpr int kOwnWords = W == 16 ? kRing + 4 * kShapeCache + kSizeBuckets : 1;
    __shared__ __attribute__((aligned(16))) uint32_t smem[Grid::kLaneWords * 64];
    __shared__ __attribute__((aligned(16))) uint32_t own_words[kOwnWords];
    uint32_t* const ring = smem + Grid::kSpare;   // survivor indices
    uint32_t* const ring_opt = own_words;         // their seeds' site codes (kKeepCodes)
    uint4* const cache_mem =
        reinterpret_cast<uint4*>(W == 16 ? own_words + kRing : smem + Grid::kSpare + kRing);
    // sizes this wave staged, by bucket
    uint32_t* const size_hist =
        W == 16 ? own_words + kRing + 4 * kShapeCache : smem + Grid::kSpareFr;
    static_assert(W == 32 || kRing <= 64 * (W / 8), "the ring fits row 15's PEND words");
    static_assert(W == 16 || (kRing + 4 * kShapeCache <= 64 * (W / 8) && kSizeBuckets <= 64),
                  "ring and cache fit row 31's PEND words, the counts its FR words");
    Grid g{smem + threadIdx.x};
    g.clear_all();
    __syncthreads();
    WaveShapeCache cache{cache_mem};
    cache.clear(lane_id());
    static_assert(kSizeBuckets == 64, "one bucket per lane");
    size_hist[lane_id()] = 0;
    __syncthreads();
    RunState st{};

    const uint32_t wave = blockIdx.x, nwaves = gridDim.x;
    if (wave == 0) {
        // counters of the later stages of this class (the previous call's
        // kernels are done, and these are first used after the size sort)
        if (lane_id() == 0)
            a.ws.counters[kCntRepeat2 + klass] = 0;   // the second repeat queue, empty
        if (lane_id() < kClaimCounters)               // the fused kernel's chunk claims
            a.ws.queue_claim[(klass * kClaimCounters + lane_id()) * kClaimStride] = 0;
    }
    const uint32_t n_items = a.n_dev != nullptr ? *a.n_dev : (uint32_t)a.n;
    // A claim is made only while the wave's candidate segment can hold every
    // item it has in flight plus the claim (a wave that cannot claim with
    // nothing in flight has staged more than its dealt share of slots, so not
    // all waves can be in that state while chunks are left; any wave can take
    // any part's chunks).
    ChunkSource chunks;
    chunks.init(a, klass, (n_items + 63) / 64);
    uint32_t head = 0, queued = 0;            // survivor ring (wave-uniform)
    uint32_t staged = 0;                      // candidates in this wave's segment
    uint32_t left = 0;                        // items that left the window, from its end
    uint32_t* seg_idx = a.ws.cand_idx[klass] + (size_t)wave * a.seg_cap;
    uint16_t* seg_size = a.ws.cand_size[klass] + (size_t)wave * a.seg_cap;
    uint4* seg_shape = a.ws.cand_shape + (size_t)wave * a.seg_cap;
    WaveTally tally{{0, 0, 0, 0}};

    bool busy = false;
    bool starved = false;                     // the last refill found no chunk left
    uint32_t idx = 0;
    Geno gd{};
    M m{};
    int ev = kEvNone;

    for (;;) {
        // -- lanes whose first run is over: records, hashes, staging ----------
        const bool finish = busy && run_over(ev, st, gd.grid);
        if (__ballot(finish) != 0) {
            bool done = false, candidate = false, det = false, leaves = false;
            int cls = 0;
            jatam_result_t rec{0, 0, 0u, 0};
            if (finish) {
                done = true;
                if (W == 16 && ev == kEvUnbound && gd.windowed) {
                    done = false;
                    leaves = true;
                } else if (ev == kEvCorrupt) {
                    rec = jatam_result_t{JATAM_INVALID, 0, 0u, 0};
                    cls = JATAM_INVALID;
                } else if (ev != kEvNone) {
                    cls = ev == kEvUnbound ? JATAM_UNBOUND : JATAM_ND_SITE;
                    rec = jatam_result_t{cls, st.size(), 0u, st.steps};
                } else if (!st.choice || a.runs == 1) {
                    // no random word was drawn: every run would be this run
                    cls = JATAM_DET;
                    det = true;
                    rec = jatam_result_t{JATAM_DET, st.size(), 0u, st.steps};
                } else {
                    done = false;
                    candidate = true;
                }
            }
            // the shape's bitmap, for the hash or for the proof stage
            uint64_t key = 0;
            int x0 = 0, y0 = 0;
            bool fits = false;
            if (det || candidate)
                fits = shape_key8(g, st, gd.grid, st.size(), key, x0, y0);
            if (__ballot(det) != 0)
                rec.hash = det_hash(g, cache, det, st.size(), gd.grid, fits, key);
            if (finish) {
                if (done)
                    out[idx] = rec;
                busy = false;
            }
            tally.add(done, cls);
            const uint64_t cm = __ballot(candidate);
            if (candidate) {
                const uint32_t pos = staged + (uint32_t)__popcll(cm & lanes_below());
                seg_idx[pos] = idx;
                seg_size[pos] = (uint16_t)st.size();
                // the shape, for the proof stage to check without a replay
                seg_shape[pos] =
                    fits ? pack_shape(g, st, gd.grid, st.size(), key, x0, y0) : packed_none();
                atomicAdd(&size_hist[size_key((uint32_t)st.size())], 1u);
            }
            staged += (uint32_t)__popcll(cm);
            if constexpr (W == 16) {
                const uint64_t lm = __ballot(leaves);
                if (leaves)
                    seg_idx[a.seg_cap - 1u - left - (uint32_t)__popcll(lm & lanes_below())] = idx;
                left += (uint32_t)__popcll(lm);
            }
        }
        // -- refill idle lanes once enough of them wait -----------------------
        const uint64_t idle = __ballot(!busy);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (nidle >= (uint32_t)a.refill || nidle == 64) {
            starved = false;
            while (queued < nidle) {
                const uint32_t in_flight = staged + left + (64u - nidle) + queued;
                uint32_t chunk;
                if (!chunks.take(chunk, in_flight + chunks.claim_size * 64u <= a.seg_cap)) {
                    starved = true;
                    break;
                }
                // screen one chunk of the input (§3.2: what the seed decides)
                uint32_t i, opts;
                int cls;
                jatam_result_t rec;
                const uint32_t pos = chunk * 64 + (uint32_t)lane_id();
                const bool wrote = screen_item<M, kIn>(a, first, klass, pos, pos < n_items, i, opts,
                                                       cls, rec);
                const bool done = wrote && cls != JATAM_INVALID, keep = cls == kScreenKeep;
                if (wrote)
                    out[i] = rec;
                tally.add(done, cls);
                const uint64_t km = __ballot(keep);
                if (keep) {
                    const uint32_t slot = (head + queued + (uint32_t)__popcll(km & lanes_below())) % kRing;
                    ring[slot] = i;
                    if constexpr (kKeepCodes)
                        ring_opt[slot] = opts;
                }
                queued += (uint32_t)__popcll(km);
            }
            wave_lds_sync();   // ring writes visible to the whole wave
            const uint32_t take = queued < nidle ? queued : nidle;
            if (!busy) {
                const uint32_t rank = (uint32_t)__popcll(idle & lanes_below());
                if (rank < take) {
                    const uint32_t slot = (head + rank) % kRing;
                    idx = ring[slot];
                    gd = run_geno<W, kIn>(a, first, idx);
                    m = build_bonds<M>(gd.genome, gd.t, a.bits, a.c);
                    ev = run_start_known(g, st, gd.grid,
                                         kKeepCodes ? ring_opt[slot] : m.codes(m.seed()));
                    busy = true;
                }
            }
            head = (head + take) % kRing;
            queued -= take;
            wave_lds_sync();   // ring slots read before they are refilled
        }
        if (__ballot(busy) == 0) {
            // with every lane idle the refill took the whole ring, so the
            // ring is empty exactly when no chunk was left to screen
            if (queued == 0 && starved)
                break;
            continue;
        }
        // -- groups of four steps until enough lanes wait for a refill (every
        // lane, once no chunk is left), at least one group: finished lanes
        // keep their run's state until the finish pass above takes them, so
        // records, hashes and staging are done once per refill rather than at
        // every step.  Lanes start runs between groups only, so the groups of
        // all lanes coincide ----------------------------------------------
        const uint32_t enough = queued == 0 && starved ? 65u : (uint32_t)a.refill;
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
    if (lane_id() == 0) {
        a.ws.seg_count[klass][wave] = staged;
        if constexpr (W == 16)
            a.ws.seg_left[wave] = left;
    }
    wave_lds_sync();   // every staged size counted
    a.ws.seg_hist[klass][(uint32_t)lane_id() * nwaves + wave] = size_hist[lane_id()];
    tally.flush(a);
}

// ---------------------------------------------------------------------------
// Size sort: 64 buckets, exact up to 47 cells, then 64 cells wide; largest
// first.  Each first-run wave counts the sizes it stages (its segment's
// histogram, stored bucket-major); the sort scans the histograms and
// scatters.
// ---------------------------------------------------------------------------

// Exclusive scan of the bucket-major histogram in three coalesced passes:
// each block scans kScanBlock entries in place and writes its total; one
// block scans the totals (and stores the candidate count); the scatter adds
// the block offsets.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(v, off);
        v += lane_id() >= off ? u : 0u;
    }
    return v;
}

// Exclusive scan of kScanBlock values across a 1024-thread block; *total
// receives their sum.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum,
                                                         uint32_t* total)
{
    const uint32_t w = threadIdx.x >> 6, l = lane_id();
    const uint32_t incl = wave_inclusive_scan(v);
    if (l == 63)
        wsum[w] = incl;
    __syncthreads();
    if (w == 0) {
        const uint32_t x = l < kScanBlock / 64 ? wsum[l] : 0u;
        const uint32_t xi = wave_inclusive_scan(x);
        if (l < kScanBlock / 64)
            wsum[l] = xi - x;
        if (l == kScanBlock / 64 - 1)
            wsum[kScanBlock / 64] = xi;
    }
    __syncthreads();
    *total = wsum[kScanBlock / 64];
    return wsum[w] + incl - v;
}

// In-place exclusive scan of h[0..total) in blocks of kScanBlock; block b's
// total goes to sums[b].  With `items` given, only the first
// ceil(*items / 64) entries (the chunks of *items queue positions) are read
// and scanned; the rest count as zero.
__global__ __launch_bounds__(kScanBlock) void scan_blocks_kernel(uint32_t* h, uint32_t total,
                                                                 uint32_t* sums,
                                                                 const uint32_t* items)
{
    __shared__ uint32_t wsum[kScanBlock / 64 + 1];
    const uint32_t n = items != nullptr ? min(total, (*items + 63u) / 64u) : total;
    const uint32_t i = blockIdx.x * kScanBlock + threadIdx.x;
    const uint32_t v = i < n ? h[i] : 0u;
    uint32_t sum;
    const uint32_t excl = block_exclusive_scan(v, wsum, &sum);
    if (i < n)
        h[i] = excl;
    if (threadIdx.x == 0)
        sums[blockIdx.x] = sum;
}

// In-place exclusive scan of the block totals (one block, any count: each
// thread takes a run of them); *total_out receives their sum.
__device__ __forceinline__ void scan_one_block(uint32_t* wsum, uint32_t* sums, uint32_t nblocks,
                                               uint32_t* total_out)
{
    const uint32_t per = (nblocks + kScanBlock - 1) / kScanBlock;
    const uint32_t lo = threadIdx.x * per, hi = min(nblocks, lo + per);
    uint32_t v = 0;
    for (uint32_t b = lo; b < hi; ++b)
        v += sums[b];
    uint32_t total;
    uint32_t run = block_exclusive_scan(v, wsum, &total);
    for (uint32_t b = lo; b < hi; ++b) {
        const uint32_t x = sums[b];
        sums[b] = run;
        run += x;
    }
    if (threadIdx.x == 0)
        *total_out = total;
}

// With `left` given, its nleft entries are scanned too, their sum to *left_out.
__global__ __launch_bounds__(kScanBlock) void scan_sums_kernel(uint32_t* sums, uint32_t nblocks,
                                                               uint32_t* total_out,
                                                               uint32_t* left, uint32_t nleft,
                                                               uint32_t* left_out)
{
    __shared__ uint32_t wsum[kScanBlock / 64 + 1];
    scan_one_block(wsum, sums, nblocks, total_out);
    if (left != nullptr) {
        __syncthreads();
        scan_one_block(wsum, left, nleft, left_out);
    }
}

static void exclusive_scan(uint32_t* h, uint32_t total, uint32_t* sums, uint32_t* total_out,
                           hipStream_t stream, const uint32_t* items = nullptr,
                           uint32_t* left = nullptr, uint32_t nleft = 0,
                           uint32_t* left_out = nullptr)
{
    const uint32_t blocks = (total + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(scan_blocks_kernel, dim3(blocks), dim3(kScanBlock), 0, stream, h, total,
                       sums, items);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kScanBlock), 0, stream, sums, blocks,
                       total_out, left, nleft, left_out);
}

// One block per segment: place its candidates with LDS cursors per bucket, and
// (`left`) list its items that left the window.
__global__ __launch_bounds__(256) void sort_scatter_kernel(BatchArgs a, int klass, bool left)
{
    __shared__ uint32_t cursor[kSizeBuckets];
    const uint32_t seg = blockIdx.x, nseg = gridDim.x;
    if (threadIdx.x < kSizeBuckets) {
        const uint32_t e = threadIdx.x * nseg + seg;
        cursor[threadIdx.x] = a.ws.seg_hist[klass][e] + a.ws.scan_sums[klass][e / kScanBlock];
    }
    __syncthreads();
    const uint32_t n = a.ws.seg_count[klass][seg];
    const uint16_t* sz = a.ws.cand_size[klass] + (size_t)seg * a.seg_cap;
    const uint32_t* ix = a.ws.cand_idx[klass] + (size_t)seg * a.seg_cap;
    const uint4* sh = a.ws.cand_shape + (size_t)seg * a.seg_cap;
    for (uint32_t i = threadIdx.x; i < n; i += 256) {
        const uint32_t pos = atomicAdd(&cursor[size_key(sz[i])], 1u);
        a.ws.sorted[klass][pos] = ix[i];
        a.ws.sorted_shape[pos] = sh[i];
    }
    if (left) {
        // the segment's last entries; seg_left holds the exclusive scan now
        const uint32_t from = a.ws.seg_left[seg];
        const uint32_t to = seg + 1 < nseg ? a.ws.seg_left[seg + 1] : a.ws.counters[kCntOverflow];
        for (uint32_t i = threadIdx.x; i < to - from; i += 256)
            a.ws.overflow[from + i] = ix[a.seg_cap - 1u - i];
    }
}

// ---------------------------------------------------------------------------
// prove<W>: one lane per candidate (in size order) takes its run-0 shape as
// the first-run stage packed it (the sort moved it beside the candidate), or
// replays run 0 where it did not fit (or, from kLostReplay of a wave's candidates
// on, its ids were lost), and checks whether the shape is guarded
// (shape_is_guarded; forced shapes are the case without conflicts): then
// every run ends in it and the record is final without the repeat runs --
// DET, run 0's size and hash, (size - 1) * R placements.  The other
// candidates are kept,
// in queue order, for the repeat runs: keep[pos] holds the candidate or
// kNoCandidate, and chunk_cnt[c] the kept count of queue chunk c (64
// positions; every chunk that holds a candidate is written, and the scan
// and the compaction read no other).
// ---------------------------------------------------------------------------
constexpr uint32_t kNoCandidate = 0xFFFFFFFFu;

// Candidates whose tiles' ids were lost (LeanGrid) that make a wave replay and prove
// them, if the queue gives every wave a chunk.  With fewer, or in a short queue, whose
// time is one wave's chain and not the work, their repeat runs cost less.  1.3 x 10^6
// uniform four-tile genotypes at G = 8, R = 20 (500 chunks) 217 us, with the proofs 276;
// 2^22 of nothing else at G = 16 5.4 ms, with them 0.44.
constexpr int kLostReplay = 32;

// The proof of the candidate at queue position pos of the size-sorted queue
// (lanes with `active`): a guarded shape gets its record here; otherwise
// the candidate is kept (the return value) for the repeat runs.  Called by
// the whole wave.
template <int W, class M>
__device__ __forceinline__ bool prove_one(const BatchArgs& a, uint64_t first,
                                          jatam_result_t* out, LeanGrid<W>& g, RunState& st,
                                          WaveShapeCache& cache, WaveTally& tally, int klass,
                                          bool full_queue, bool active, uint32_t pos,
                                          uint32_t& idx)
{
    bool forced = false, packed = false;
    int size = 0;
    uint64_t key = 0;
    Geno gd{};
    idx = 0;
    const uint4 sh = active ? a.ws.sorted_shape[pos] : packed_none();
    bool replay = true;
    if constexpr (M::kManyIds) {
        const bool lost = packed_shape_lost(sh);
        replay = !lost || (full_queue && __popcll(__ballot(lost)) >= kLostReplay);
    }
    if (active) {
        idx = a.ws.sorted[klass][pos];
        gd = run_geno<W>(a, first, idx);
        const M src = build_bonds<M>(gd.genome, gd.t, a.bits, a.c);
        packed = packed_shape_valid(sh);
        if (packed) {
            // the first-run stage packed the shape: no replay
            key = ((uint64_t)sh.y << 32) | sh.x;
            size = __popcll(key);
            forced = packed_shape_is_guarded(src, sh);
        } else if (replay) {
            const int ev = run_assembly(src, g, st, gd.grid, run_key(a, gd, 0));
            size = st.size();
            int x0 = 0, y0 = 0;
            packed = ev == kEvNone && shape_key8(g, st, gd.grid, size, key, x0, y0);
            forced = ev == kEvNone &&
                     shape_is_guarded(src, g, shape_ids(src, g, st, gd.grid, packed, key, x0, y0),
                                      gd.grid, packed, key, x0, y0);
        }
    }
    // the hash of a packed or replayed shape from its bitmap, if it has one
    const uint32_t h =
        det_hash(g, cache, forced, size, gd.grid, packed, key);
    if (forced)
        out[idx] = jatam_result_t{JATAM_DET, size, h, (size - 1) * a.runs};
    tally.add(forced, JATAM_DET);
    return active && !forced;
}

template <int W, class M>
__global__ __launch_bounds__(64) void prove_kernel(const BatchArgs a, int klass)
{
    const uint64_t first = slice_first(a);
    jatam_result_t* const out = slice_out(a);
    __shared__ uint32_t smem[LeanGrid<W>::kLaneWords * 64];
    __shared__ uint4 cache_mem[kShapeCache];
    LeanGrid<W> g{smem + threadIdx.x};
    g.clear_all();
    WaveShapeCache cache{cache_mem};
    cache.clear(lane_id());
    __syncthreads();
    RunState st{};
    WaveTally tally{{0, 0, 0, 0}};
    const uint32_t count = a.ws.counters[kCntCand + klass];
    uint32_t* keep = a.ws.cand_idx[klass];
    uint32_t* chunk_cnt = a.ws.chunk_cnt[klass];
    const uint32_t qchunks = (count + 63) / 64;   // queue chunks holding candidates
    for (uint32_t c = blockIdx.x; c < qchunks; c += gridDim.x) {
        const uint32_t pos = c * 64 + (uint32_t)lane_id();
        const bool active = pos < count;
        uint32_t idx;
        const bool kept =
            prove_one<W, M>(a, first, out, g, st, cache, tally, klass, qchunks >= gridDim.x, active,
                            pos, idx);
        if (active)
            keep[pos] = kept ? idx : kNoCandidate;
        const uint32_t kc = (uint32_t)__popcll(__ballot(kept));
        if (lane_id() == 0)
            chunk_cnt[c] = kc;
    }
    if (blockIdx.x == 0 && lane_id() == 0) {
        // the candidate count, kept for the compaction (the scan of the kept
        // counts overwrites kCntCand)
        a.ws.counters[kCntCandAll + klass] = count;
    }
    tally.flush(a);
}

// Kept candidates to the front of the queue, in order: a grid-stride loop
// over the queue chunks that hold candidates, a wave per chunk at a time.
__global__ __launch_bounds__(256) void compact_kernel(const BatchArgs a, int klass)
{
    const uint32_t count = a.ws.counters[kCntCandAll + klass];
    const uint32_t span = (count + 63) / 64 * 64;   // whole chunks: every wave ballots
    for (uint32_t pos = blockIdx.x * 256 + threadIdx.x; pos < span; pos += gridDim.x * 256) {
        const uint32_t c = pos >> 6;
        const uint32_t v = pos < count ? a.ws.cand_idx[klass][pos] : kNoCandidate;
        const bool kept = v != kNoCandidate;
        const uint64_t m = __ballot(kept);
        if (kept) {
            const uint32_t base =
                a.ws.chunk_cnt[klass][c] + a.ws.chunk_sums[klass][c / kScanBlock];
            a.ws.sorted[klass][base + (uint32_t)__popcll(m & lanes_below())] = v;
        }
    }
}

template <int W, class M>
__global__ __launch_bounds__(64) void repeat_kernel(const BatchArgs a, int klass, int rpass,
                                                    int skip, bool store_occ,
                                                    const uint32_t* queue_in,
                                                    const uint32_t* count_in,
                                                    uint32_t* queue_out, uint32_t* count_out)
{
    __shared__ uint32_t smem[LeanGrid<W>::kLaneWords * 64];
    __shared__ uint32_t orient[8][64];
    __shared__ uint4 cache_mem[kShapeCache];
    LeanGrid<W> lg{smem + threadIdx.x};
    lg.clear_all();
    WaveShapeCache cache{cache_mem};
    cache.clear(lane_id());
    __syncthreads();
    RunState st{};
    WaveTally tally{{0, 0, 0, 0}};
    RepeatWave<W, M, false> rw(a, smem, &orient[0][0], cache, st, tally, rpass, skip, store_occ,
                               queue_out, count_out);
    const uint32_t count = *count_in;
    const uint32_t groups = (uint32_t)rw.groups, grp = (uint32_t)rw.grp;
    const uint32_t stride = gridDim.x * groups;

    // static round-robin over the size-sorted queue; the next entry is
    // fetched one iteration ahead
    uint32_t base = blockIdx.x * groups;
    uint32_t next_idx = 0;
    if (grp < groups && base + grp < count)
        next_idx = queue_in[base + grp];
    for (; base < count; base += stride) {
        const bool active = grp < groups && base + grp < count;
        const uint32_t idx = next_idx;
        if (grp < groups && base + stride + grp < count)
            next_idx = queue_in[base + stride + grp];
        rw.round(active, idx, base + grp);
    }
    tally.flush(a);
}

// ---------------------------------------------------------------------------
// prove_repeat<W>: the proof and the first repeat pass in one kernel.  A
// wave proves 64 positions of the size-sorted queue at a time (prove_one)
// and keeps its unproven candidates in LDS; whenever they fill its repeat
// groups (64 / rpass of them) it makes their runs 0 .. rpass-1
// (RepeatWave::round).  The proof's steady integer work and the runs'
// latency-bound steps share the CUs, and no compaction or launch sits
// between them.  With rpass < R the candidates without a witness go to the
// second queue (count_out, cleared by the first-run kernel), in the 16 x 16 layout
// with run 0's occupancy stored.
// ---------------------------------------------------------------------------
template <int W, class M>
__global__ __launch_bounds__(64) void prove_repeat_kernel(const BatchArgs a, int klass,
                                                          int rpass, uint32_t* queue_out,
                                                          uint32_t* count_out)
{
    __shared__ uint32_t smem[LeanGrid<W>::kLaneWords * 64];
    __shared__ uint32_t orient[8][64];
    __shared__ uint4 cache_mem[kShapeCache];
    // unproven candidates waiting for a round, in the grid's spare words
    uint32_t* const pend = smem + LeanGrid<W>::kSpare;
    LeanGrid<W> lg{smem + threadIdx.x};
    lg.clear_all();
    WaveShapeCache cache{cache_mem};
    cache.clear(lane_id());
    __syncthreads();
    RunState st{};
    WaveTally tally{{0, 0, 0, 0}};
    RepeatWave<W, M, false> rw(a, smem, &orient[0][0], cache, st, tally, rpass, 0, W == 16,
                               queue_out, count_out);
    const uint32_t count = a.ws.counters[kCntCand + klass];
    const uint32_t qchunks = (count + 63) / 64;
    const uint32_t groups = (uint32_t)rw.groups, grp = (uint32_t)rw.grp;
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t npend = 0;   // wave-uniform, below groups between chunks
    // one round on the first k waiting candidates, the rest moved down
    auto round_of = [&](uint32_t k) {
        const uint32_t pidx = grp < k ? pend[grp] : 0u;
        rw.round(grp < k, pidx, 0u);
        const uint32_t rest = npend - k;   // < 64
        const uint32_t v = lane < rest ? pend[k + lane] : 0u;
        wave_lds_sync();
        if (lane < rest)
            pend[lane] = v;
        wave_lds_sync();
        npend = rest;
    };
    // Chunks are claimed one at a time, so that waves end together however
    // the proofs and rounds of their chunks differ: counter x (x = the
    // block's index mod 8, its XCD under the round-robin dispatch of
    // workgroups) hands out chunks x, x + 8, x + 16, ... of the queue, so
    // each counter serves an even share of every part of the size-sorted
    // queue.  The counters are cleared by the first-run kernel.
    const uint32_t claimer = blockIdx.x % (uint32_t)kClaimCounters;
    uint32_t* const claim_ctr =
        a.ws.queue_claim + (klass * kClaimCounters + claimer) * kClaimStride;
    auto claim = [&]() -> uint32_t {
        uint32_t q = 0;
        if (lane == 0)
            q = atomicAdd(claim_ctr, 1u);
        return claimer + (uint32_t)kClaimCounters * (uint32_t)__shfl((int)q, 0);
    };
    for (uint32_t c = claim(); c < qchunks; c = claim()) {
        const uint32_t pos = c * 64 + lane;
        uint32_t idx;
        const bool kept = prove_one<W, M>(a, rw.first, rw.out, lg, st, cache, tally, klass,
                                          qchunks >= gridDim.x, pos < count, pos, idx);
        const uint64_t km = __ballot(kept);
        if (kept)
            pend[npend + (uint32_t)__popcll(km & lanes_below())] = idx;
        npend += (uint32_t)__popcll(km);
        wave_lds_sync();
        while (npend >= groups)
            round_of(groups);
    }
    while (npend > 0)
        round_of(npend < groups ? npend : groups);
    tally.flush(a);
}

// ---------------------------------------------------------------------------
// repeat_seq<W>: one lane per candidate, its runs made in turn.  Run 0 is
// replayed and its occupancy kept beside the lane's grid (OCC0, the words it
// touched); each later run is compared with it as soon as it ends, and the
// first witness in run order (an event, or another occupancy) decides, so a
// non-deterministic candidate makes only the runs up to its first witness.
// A lane that is done takes the wave's next queue position: the wave owns
// chunks k, k + grid, ... of 64 positions of the size-sorted queue, handed to
// idle lanes in order once at least kSeqRefill of them wait.
// ---------------------------------------------------------------------------
constexpr int kSeqRefill = 8;

template <int W, class M>
__global__ __launch_bounds__(64) void repeat_seq_kernel(const BatchArgs a, int klass)
{
    using Geo = Geometry<W>;
    const uint64_t first = slice_first(a);
    jatam_result_t* const out = slice_out(a);
    __shared__ uint32_t smem[Geo::kLaneWords * 64];
    __shared__ uint32_t occ0_mem[Geo::kWords * 64];   // lane j's word w at [w * 64 + j]
    __shared__ uint4 cache_mem[kShapeCache];
    LaneGrid<W, 64> g{smem + threadIdx.x};
    uint32_t* const occ0 = occ0_mem + threadIdx.x;
    g.clear_all();
    WaveShapeCache cache{cache_mem};
    cache.clear(lane_id());
    __syncthreads();
    RunState st{};
    WaveTally tally{{0, 0, 0, 0}};

    const int R = a.runs;
    const uint32_t count = a.ws.counters[kCntCand + klass];
    const uint32_t* queue = a.ws.sorted[klass];
    const uint32_t nwaves = gridDim.x;
    uint32_t chunk = blockIdx.x, off = 0;   // the wave's next queue position (wave-uniform)
    bool busy = false;
    uint32_t idx = 0, osum0 = 0;
    int run = 0, ev = kEvNone, steps_sum = 0, size0 = 0;
    Geno gd{};
    M src{};

    for (;;) {
        const uint64_t idle = __ballot(!busy);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        const bool left = chunk * 64u + off < count;
        if (left && (nidle >= (uint32_t)kSeqRefill || nidle == 64)) {
            if (!busy) {
                // idle lane of rank k takes the k-th next position (at most
                // one chunk ahead: off + k < 128)
                const uint32_t o = off + (uint32_t)__popcll(idle & lanes_below());
                const uint32_t pos = (o < 64u ? chunk : chunk + nwaves) * 64u + (o & 63u);
                if (pos < count) {
                    idx = queue[pos];
                    gd = run_geno<W>(a, first, idx);
                    src = build_bonds<M>(gd.genome, gd.t, a.bits, a.c);
                    run = 0;
                    steps_sum = 0;
                    ev = run_start(src, g, st, gd.grid);
                    busy = true;
                }
            }
            const uint32_t o = off + nidle;
            chunk = o < 64u ? chunk : chunk + nwaves;
            off = o & 63u;
        }
        if (__ballot(busy) == 0) {
            if (!left)
                break;
            continue;
        }
        if (busy && !run_over(ev, st, gd.grid))
            ev = run_four(src, g, st, gd.grid, run_key(a, gd, run));
        const bool ended = busy && run_over(ev, st, gd.grid);
        bool done = false, det = false;
        int cls = 0;
        jatam_result_t rec{0, 0, 0u, 0};
        if (ended) {
            steps_sum += st.steps;
            if (ev == kEvCorrupt) {
                rec = jatam_result_t{JATAM_INVALID, 0, 0u, 0};
                cls = JATAM_INVALID;
                done = true;
            } else if (run == 0 && ev != kEvNone) {
                // (a candidate's run 0 ended cleanly in the first-run stage)
                cls = ev == kEvUnbound ? JATAM_UNBOUND : JATAM_ND_SITE;
                rec = jatam_result_t{cls, st.size(), 0u, steps_sum};
                done = true;
            } else if (run == 0) {
                // keep run 0's occupancy: only its nonzero words are ever read
                for (uint32_t sw = st.osum; sw != 0; sw &= sw - 1) {
                    const int w = __builtin_ctz(sw);
                    occ0[w * 64] = g.occ(w);
                }
                osum0 = st.osum;
                size0 = st.size();
                run = 1;
                ev = run_start(src, g, st, gd.grid);
            } else {
                // occupancy only grows within a run, so osum is exactly the
                // set of nonzero words
                bool same = ev == kEvNone && st.osum == osum0 && st.size() == size0;
                for (uint32_t sw = osum0; same && sw != 0; sw &= sw - 1) {
                    const int w = __builtin_ctz(sw);
                    same = g.occ(w) == occ0[w * 64];
                }
                if (!same) {
                    cls = ev == kEvUnbound ? JATAM_UNBOUND
                        : ev == kEvAmbig   ? JATAM_ND_SITE
                                           : JATAM_ND_RUNS;
                    rec = jatam_result_t{cls, st.size(), 0u, steps_sum};
                    done = true;
                } else if (run == R - 1) {
                    cls = JATAM_DET;
                    det = true;
                    rec = jatam_result_t{JATAM_DET, size0, 0u, steps_sum};
                    done = true;
                } else {
                    run += 1;
                    ev = run_start(src, g, st, gd.grid);
                }
            }
        }
        // the grid holds run R-1's shape, which is run 0's
        if (__ballot(det) != 0) {
            uint64_t key = 0;
            int x0, y0;
            const bool fits = det && shape_key8(g, st, gd.grid, size0, key, x0, y0);
            rec.hash = det_hash(g, cache, det, size0, gd.grid, fits, key);
        }
        const bool leaves = W == 16 && done && cls == JATAM_UNBOUND && gd.windowed;
        if (done) {
            if (!leaves)
                out[idx] = rec;
            busy = false;
        }
        if constexpr (W == 16)
            append_overflow(a, leaves, idx);
        tally.add(done && !leaves, cls);
    }
    tally.flush(a);
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
// Clears the first-run claim counters of one grid class and, if given, the
// tally's counter sets (a kernel rather than a memset: graph-safe).
__global__ __launch_bounds__(256) void clear_kernel(uint32_t* claims, unsigned long long* slots)
{
    if (threadIdx.x < kClaimCounters)
        claims[threadIdx.x * kClaimStride] = 0u;
    if (slots != nullptr && threadIdx.x < 4 * kTallySlots)
        slots[(threadIdx.x >> 2) * kTallyStride + (threadIdx.x & 3u)] = 0ull;
}

void launch_clear(uint32_t* claims, unsigned long long* slots, hipStream_t stream)
{
    hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(256), 0, stream, claims, slots);
}

void launch_tally(const unsigned long long* slots, unsigned long long* tally, hipStream_t stream)
{
    hipLaunchKernelGGL(tally_kernel, dim3(1), dim3(256), 0, stream, slots, tally);
}

template <int W, class M>
static void occupancy_of(int out[3])
{
    out[0] = resident_per_cu(first_run_kernel<W, M, kInRange>);
    // the repeat grid runs the proof + first pass kernel and the second pass
    const int repeat = resident_per_cu(repeat_kernel<W, M>);
    const int fused = resident_per_cu(prove_repeat_kernel<W, M>);
    out[1] = repeat < fused ? repeat : fused;
    out[2] = resident_per_cu(repeat_seq_kernel<W, M>);
}

void batch_occupancy(BatchOccupancy& occ)
{
    occupancy_of<16, Bonds2>(occ.blocks[0][kGenoTwo]);
    occupancy_of<16, Bonds4>(occ.blocks[0][kGenoFour]);
    occupancy_of<16, BondsC16>(occ.blocks[0][kGenoC16]);
    occupancy_of<32, Bonds2>(occ.blocks[1][kGenoTwo]);
    occupancy_of<32, Bonds4>(occ.blocks[1][kGenoFour]);
    occupancy_of<32, BondsC16>(occ.blocks[1][kGenoC16]);
    solo_occupancy(occ.solo);
}

__global__ __launch_bounds__(256) void records_differ_kernel(const int4* __restrict__ x,
                                                             const int4* __restrict__ y,
                                                             uint64_t n, uint32_t* flag)
{
    bool differ = false;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * 256) {
        const int4 u = x[i], v = y[i];
        differ = differ || u.x != v.x || u.y != v.y || u.z != v.z || u.w != v.w;
    }
    if (__ballot(differ) != 0 && lane_id() == 0)
        atomicOr(flag, 1u);
}

int launch_records_differ(const jatam_result_t* x, const jatam_result_t* y, uint64_t n,
                          uint32_t* flag, hipStream_t stream)
{
    if (n == 0)
        return JATAM_OK;
    const uint64_t want = (n + 255) / 256;
    const uint32_t blocks = (uint32_t)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(records_differ_kernel, dim3(blocks), dim3(256), 0, stream,
                       reinterpret_cast<const int4*>(x), reinterpret_cast<const int4*>(y), n,
                       flag);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// The first-run kernel compiled for the call's input mode.
template <int W, class M>
static void launch_first(const BatchArgs& a, uint32_t nb, hipStream_t stream, int klass)
{
    if (a.items != nullptr)
        hipLaunchKernelGGL((first_run_kernel<W, M, kInItems>), dim3(nb), dim3(64), 0, stream, a,
                           klass);
    else if (a.genomes != nullptr)
        hipLaunchKernelGGL((first_run_kernel<W, M, kInList>), dim3(nb), dim3(64), 0, stream, a,
                           klass);
    else
        hipLaunchKernelGGL((first_run_kernel<W, M, kInRange>), dim3(nb), dim3(64), 0, stream, a,
                           klass);
}

// The R-lanes-per-candidate repeat kernel of grid class k for one pass.
template <class M>
static void launch_repeat(const BatchArgs& a, int k, uint32_t rb, int rpass, int skip,
                          bool store_occ, const uint32_t* qin, const uint32_t* cin,
                          uint32_t* qout, uint32_t* cout, hipStream_t stream)
{
    if (k == 0)
        hipLaunchKernelGGL((repeat_kernel<16, M>), dim3(rb), dim3(64), 0, stream, a, 0, rpass,
                           skip, store_occ, qin, cin, qout, cout);
    else
        hipLaunchKernelGGL((repeat_kernel<32, M>), dim3(rb), dim3(64), 0, stream, a, 1, rpass, 0,
                           false, qin, cin, qout, cout);
}

// The proof + first repeat pass kernel of grid class k.
template <class M>
static void launch_prove_repeat(const BatchArgs& a, int k, uint32_t rb, int rpass,
                                uint32_t* qout, uint32_t* cout, hipStream_t stream)
{
    if (k == 0)
        hipLaunchKernelGGL((prove_repeat_kernel<16, M>), dim3(rb), dim3(64), 0, stream, a, 0,
                           rpass, qout, cout);
    else
        hipLaunchKernelGGL((prove_repeat_kernel<32, M>), dim3(rb), dim3(64), 0, stream, a, 1,
                           rpass, qout, cout);
}

template <class M>
static void launch_stages(BatchArgs a, const bool classes[2], const StageLaunch launch[2],
                          hipStream_t stream, hipEvent_t* marks, uint8_t* launched)
{
    auto begin = [&](int s) {
        if (marks)
            (void)hipEventRecord(marks[2 * s], stream);
    };
    auto end = [&](int s) {
        if (marks) {
            (void)hipEventRecord(marks[2 * s + 1], stream);
            launched[s] = 1;
        }
    };
    for (int k = 0; k < 2; ++k) {
        if (!classes[k])
            continue;
        const uint32_t nb = (uint32_t)launch[k].first_blocks;
        const uint32_t rb = (uint32_t)launch[k].repeat_blocks;
        a.refill = launch[k].refill;
        const uint64_t nchunks = (uint64_t)(a.n + 63) / 64;
        a.dyn16 = launch[k].dyn16;
        a.claim_chunks = launch[k].claim_chunks;
        // a wave's segment holds its dealt-out share and one claim (the
        // first-run kernel's claim size, which is 0 where it makes none)
        const uint64_t per_wave = nchunks / (16u * (uint64_t)nb);
        const uint32_t claim = a.dyn16 <= 0 ? 0u
                               : per_wave < (uint64_t)a.claim_chunks ? (uint32_t)per_wave
                                                                      : (uint32_t)a.claim_chunks;
        a.seg_cap = (uint32_t)((nchunks + nb - 1) / nb * 64) + claim * 64u;
        begin(kStageFirst + kStagesPerClass * k);
        if (k == 1 && a.narrow_max > 16) {
            // the 32 x 32 class reruns only the items that left the window
            a.order = a.ws.overflow;
            a.n_dev = a.ws.counters + kCntOverflow;
            a.narrow_max = 16;
        }
        // the call's first class clears the tally's counter sets
        const bool clear_tally = a.tally != nullptr && (k == 0 || !classes[0]);
        if (a.dyn16 > 0 || clear_tally)
            launch_clear(a.ws.run_claim + k * kClaimCounters * kClaimStride,
                         clear_tally ? a.ws.tally_slots : nullptr, stream);
        if (k == 0)
            launch_first<16, M>(a, nb, stream, 0);
        else
            launch_first<32, M>(a, nb, stream, 1);
        end(kStageFirst + kStagesPerClass * k);
        begin(kStageSort + kStagesPerClass * k);
        const bool window = k == 0 && a.narrow_max > 16;
        exclusive_scan(a.ws.seg_hist[k], (uint32_t)kSizeBuckets * nb, a.ws.scan_sums[k],
                       a.ws.counters + kCntCand + k, stream, nullptr,
                       window ? a.ws.seg_left : nullptr, nb, a.ws.counters + kCntOverflow);
        hipLaunchKernelGGL(sort_scatter_kernel, dim3(nb), dim3(256), 0, stream, a, k, window);
        end(kStageSort + kStagesPerClass * k);
        const int mapping = launch[k].repeat_mapping;
        if (mapping == 2 && a.runs > kRepeatFirstRuns) {
            // two passes: the proof and the first pass (runs 0 ..
            // kRepeatFirstRuns-1, a cheap round of 16 candidates per wave)
            // in one kernel on the repeat grid, the undecided candidates to
            // the staging array (free after the sort) for the second pass,
            // which in the 16 x 16 layout makes only runs kRepeatFirstRuns ..
            // R-1 (the 32 x 32 layout remakes all)
            uint32_t* q1 = a.ws.cand_idx[k];
            uint32_t* c1 = a.ws.counters + kCntRepeat2 + k;   // cleared by the first runs
            begin(kStageProve + kStagesPerClass * k);
            launch_prove_repeat<M>(a, k, rb, kRepeatFirstRuns, q1, c1, stream);
            end(kStageProve + kStagesPerClass * k);
            begin(kStageRepeat + kStagesPerClass * k);
            launch_repeat<M>(a, k, rb, a.runs, k == 0 ? kRepeatFirstRuns : 0, false, q1, c1,
                              nullptr, nullptr, stream);
            end(kStageRepeat + kStagesPerClass * k);
        } else {
            // forced shapes are final; the rest are compacted, in queue
            // order, for one pass of all R runs per candidate (mapping 0: a
            // round of 64 / R candidates is too costly to interleave with the
            // proof) or the one-lane-per-candidate repeat runs (mapping 1)
            begin(kStageProve + kStagesPerClass * k);
            if (k == 0)
                hipLaunchKernelGGL((prove_kernel<16, M>), dim3(nb), dim3(64), 0, stream, a, 0);
            else
                hipLaunchKernelGGL((prove_kernel<32, M>), dim3(nb), dim3(64), 0, stream, a, 1);
            const uint32_t qchunks = (uint32_t)nchunks;
            exclusive_scan(a.ws.chunk_cnt[k], qchunks, a.ws.chunk_sums[k],
                           a.ws.counters + kCntCand + k, stream, a.ws.counters + kCntCandAll + k);
            // a grid-stride loop over the candidates' chunks only (the count
            // is on the device)
            hipLaunchKernelGGL(compact_kernel, dim3(nb), dim3(256), 0, stream, a, k);
            end(kStageProve + kStagesPerClass * k);
            begin(kStageRepeat + kStagesPerClass * k);
            if (mapping != 1)
                launch_repeat<M>(a, k, rb, a.runs, 0, false, a.ws.sorted[k],
                                  a.ws.counters + kCntCand + k, nullptr, nullptr, stream);
            else if (k == 0)
                hipLaunchKernelGGL((repeat_seq_kernel<16, M>), dim3(rb), dim3(64), 0, stream, a,
                                   0);
            else
                hipLaunchKernelGGL((repeat_seq_kernel<32, M>), dim3(rb), dim3(64), 0, stream, a,
                                   1);
            end(kStageRepeat + kStagesPerClass * k);
        }
    }
    if (a.tally != nullptr)
        launch_tally(a.ws.tally_slots, a.tally, stream);
}

int launch_batched(const BatchArgs& a, const bool classes[2], const StageLaunch launch[2],
                   int geno, hipStream_t stream, hipEvent_t* marks, uint8_t* launched)
{
    if (launched)
        for (int s = 0; s < kStages; ++s)
            launched[s] = 0;
    if (a.n > 0) {
        if (geno == kGenoTwo)
            launch_stages<Bonds2>(a, classes, launch, stream, marks, launched);
        else if (geno == kGenoFour)
            launch_stages<Bonds4>(a, classes, launch, stream, marks, launched);
        else
            launch_stages<BondsC16>(a, classes, launch, stream, marks, launched);
    }
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam
