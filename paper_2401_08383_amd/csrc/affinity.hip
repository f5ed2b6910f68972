// affinity_histogram and placement_locality: reductions over a routing trace [L,N] (int32,
// layer-major).  Both are bound by the HBM read of the trace (4 bytes per token and layer), so
// both are shaped like a streaming read: about one 1024-thread workgroup per CU, every thread
// keeping several 16-byte loads in flight.
//
// affinity_histogram
//   partial : a workgroup owns a chunk of tokens (< 65536) and a group of g <= 3 consecutive
//             layer pairs.  A thread loads the g+1 trace columns of its tokens at once, then walks
//             the pairs and bins every transition with one LDS atomic.  The g E x E histograms
//             live in LDS as 16-bit counters packed two to a word (a workgroup can never count
//             more than its chunk, so they cannot overflow), replicated when E*E is small so that
//             hot bins do not serialise.  The packed words are stored as per-chunk partials.
//             Workgroups of one token chunk are mapped to one XCD, so the column shared by two
//             neighbouring pair groups is served by that XCD's L2.
//   finalize: one wavefront per (pair, source expert) row sums the partials over the chunks
//             into int64 counts, forms the row sum (a wavefront reduction: no LDS, no barrier), the
//             layer loads and the conditional probabilities; extra workgroups of the same launch
//             derive the loads of the final layer and the invalid tally.
//   Entries outside [0,E) are tallied; a transition touching one is not binned, but the valid
//   end still counts towards its layer's load through small "orphan" histograms.
//
// placement_locality
//   a workgroup owns a chunk of tokens for ALL layers (each trace entry is read exactly once),
//   maps expert -> device through an LDS copy of the placement, asks for the next two layers while
//   it counts the last two, and counts per pair the tokens whose device does not change; per-chunk
//   partial counts are summed by a second kernel.
#include "trace_tile.hpp"

#include <type_traits>

namespace exf {

constexpr int kXcds = 8;
constexpr int kTraceThreads = 1024;
constexpr int kAffMaxGroup = 3;                 // layer pairs per workgroup (4 columns in registers; 3 measured best,
                                                // 29 against 34 us with 6 on a 24 x 1M trace)
constexpr size_t kAffHistBudget = 48 * 1024;    // LDS bytes for the packed pair histograms
constexpr int64_t kAffMaxChunk = 61440;         // tokens per workgroup: 16-bit counters cannot overflow
constexpr int kTargetWorkgroups = 256;          // about one per CU

// Ids per load of a trace column: four, except that a column of fewer has no vector to load.
static int trace_vec(int64_t N) { return N >= 4 ? 4 : 1; }

// The (chunk, group) of a workgroup of the multi-hop counts, numbered chunk by chunk; below zero: none.  Every XCD takes a contiguous eighth of the
// items: the groups of a chunk share its columns in one L2 (two for a chunk on the edge), and 256 items are one workgroup for every compute
// unit.  Dealt by whole chunks, 21 chunks of twelve groups were 36 workgroups for the 32 compute units of five XCDs (8 x 300000 tokens, 64 experts:
// 17.3 us, now 13.5; 10 x 100000 13.9 and 12.0).
static int64_t xcd_items_grid(int C, int Q) { return (static_cast<int64_t>(C) * Q + kXcds - 1) / kXcds * kXcds; }
__device__ __forceinline__ int xcd_item(int C, int Q)
{
    const int items = C * Q, item = static_cast<int>(blockIdx.x % kXcds) * ((items + kXcds - 1) / kXcds) + static_cast<int>(blockIdx.x / kXcds);
    return item < items ? item : -1;
}

// The second launches ask for the partials of so many chunks together: all of them up to 24 (asked for 16 by 16, 17 chunks were two round trips), past that
// up to 32 for as many rows as the chip has SIMDs and else 16 by 16, where the reads are bound by their number (24 x 1M tokens, 64 experts,
// 32 chunks 26.3 us with 32 and 26.0; 24 x 300000, 32 experts 12.8 and 13.4; 3 x 500000, 24 experts, 123 chunks 12.9 and 14.3).
// Trips of equal length: 35 chunks in two of 24 (2 x 142392 tokens, 24 experts 9.25 us in two of 32,
// 8.9; 16 x 265000, 64 experts, 48 chunks 17.75 and 16.6).
static int chunks_ahead(int C, int64_t rows)
{
    if (C > 24 && rows > 4 * kTargetWorkgroups) return 16;
    const int trips = C > 0 ? (C + 31) / 32 : 1;
    return ((C + trips - 1) / trips + 7) / 8 * 8;
}
static int trips_of_chunks(int C, int64_t rows) { return C > 0 ? (C + chunks_ahead(C, rows) - 1) / chunks_ahead(C, rows) : 0; }

struct AffinityPlan {
    int g;           // layer pairs per workgroup
    int Q;           // pair groups
    int copies;      // histogram replicas (power of two)
    int words;       // 32-bit words of one packed E x E histogram
    int64_t chunk;   // tokens per workgroup
    int C;           // token chunks
    int vec;         // ids per trace load
    size_t off_counts, off_orphan_next, off_orphan_last, off_invalid, off_local, total_bytes;
};

static AffinityPlan make_affinity_plan(int L, int64_t N, int E)
{
    AffinityPlan p;
    const int pairs = L > 1 ? L - 1 : 0;
    p.words = (E * E + 1) / 2;
    const size_t hist_bytes = static_cast<size_t>(p.words) * sizeof(uint32_t);
    int g = static_cast<int>(kAffHistBudget / hist_bytes);
    if (g > kAffMaxGroup) g = kAffMaxGroup;
    if (g < 1) g = 1;
    if (pairs > 0 && g > pairs) g = pairs;
    p.g = g;
    p.copies = 1;
    while (p.copies < 16 && hist_bytes * g * (p.copies * 2) <= kAffHistBudget) p.copies *= 2;
    p.Q = pairs > 0 ? (pairs + g - 1) / g : 1;
    p.vec = trace_vec(N);
    // Up to 32 groups, and where the counters do not ask for shorter chunks: at most one workgroup per compute unit of every XCD, which takes whole chunks.  42 chunks of six groups were 36 workgroups for the 32
    // compute units of two XCDs, which began the last four when the others ended (19 x 870535 tokens, 60 experts 32.9 us, in 40 chunks 22.0; 10 x 1M,
    // 64 experts 28.0 and 19.3; 22 x 1M, 32 experts 32.5 and 21.2).  Dealing an eighth of all workgroups to every XCD instead fills
    // it as well, but reads slower: 20.2 and 22.4 there, 24 x 1M, 64 experts 26.8 and 26.0.
    int c_target = kTargetWorkgroups / kXcds / p.Q * kXcds;
    if (c_target < 1) c_target = kTargetWorkgroups / p.Q;
    if (c_target < 1) c_target = 1;
    // at least a sweep (the second launch reads all chunks: 3 x 79098 tokens in chunks of 512 17.0 us, of 4096 9.2), past that whole wavefronts (one
    // cut by the end of its chunk takes the checked path), not sweeps: 24 x 500000 tokens of 52 experts 20.0 us in 31 chunks, 17.9 in 32
    const int64_t sweep = static_cast<int64_t>(kTraceThreads) * p.vec;  // tokens one pass of the workgroup covers
    const int64_t unit = static_cast<int64_t>(kWave) * p.vec;
    int64_t chunk = (N + c_target - 1) / c_target;
    chunk = (chunk + unit - 1) / unit * unit;
    if (chunk < sweep) chunk = sweep;
    // Between one sweep and two, two where so many fewer chunks save the second launch a round trip: the first one gains less by the compute units that it fills
    // (16 x 230004 tokens, 64 experts: 11.0 us in 48 chunks and 12.6 in 29, the second 7.2 and 4.6, together 17.5 and 14.8; 3 x 1.2M 24.5 and 19.3; 10 x 400000
    // of 16 12.0 and 11.5).  Where they save none: 24 x 147000, 16 experts, 9.6 in 32 chunks and 10.7 in 18.
    const int64_t rows = static_cast<int64_t>(pairs) * E;
    if (chunk > sweep && chunk < 2 * sweep &&
        trips_of_chunks(static_cast<int>((N + 2 * sweep - 1) / (2 * sweep)), rows) < trips_of_chunks(static_cast<int>((N + chunk - 1) / chunk), rows))
        chunk = 2 * sweep;
    if (chunk > kAffMaxChunk) chunk = kAffMaxChunk / unit * unit;
    p.chunk = chunk;
    p.C = static_cast<int>(N > 0 ? (N + chunk - 1) / chunk : 0);
    // room for as many chunks as any shorter trace has: a workspace for the longest one does for all
    const int64_t sweeps = N > 0 ? (N + sweep - 1) / sweep : 0;
    const size_t room = p.C > c_target ? p.C : static_cast<size_t>(sweeps < c_target ? sweeps : c_target);
    size_t off = 0;
    p.off_counts = off;
    off += align_up(room * pairs * p.words * sizeof(uint32_t), 256);
    p.off_orphan_next = off;
    off += align_up(room * (pairs > 0 ? pairs : 1) * E * sizeof(uint32_t), 256);
    p.off_orphan_last = off;
    off += align_up(room * E * sizeof(uint32_t), 256);
    p.off_invalid = off;
    off += align_up(room * p.Q * sizeof(uint32_t), 256);
    p.off_local = off;  // per chunk and pair: transitions that stay on their device (affinity_statistics)
    off += align_up(room * (pairs > 0 ? pairs : 1) * sizeof(uint32_t), 256);
    p.total_bytes = off > 0 ? off : 256;
    return p;
}

template <int VEC>
__global__ __launch_bounds__(kTraceThreads) void affinity_partial_kernel(const int32_t* __restrict__ trace, int L, int64_t N, int E,
                                                                          int g, int Q, int copies, int words, int64_t chunk, int C,
                                                                          uint32_t* __restrict__ part_counts,
                                                                          uint32_t* __restrict__ part_orphan_next,
                                                                          uint32_t* __restrict__ part_orphan_last,
                                                                          uint32_t* __restrict__ part_invalid,
                                                                          const int32_t* __restrict__ placement,  // [L,E] or null
                                                                          uint32_t* __restrict__ part_local)      // with placement
{
    extern __shared__ uint32_t lds[];
    uint32_t* hist = lds;                                 // [copies][g][words], two 16-bit counters per word
    uint32_t* orphan_next = hist + copies * g * words;    // [g][E]   valid id whose successor is invalid
    uint32_t* orphan_last = orphan_next + g * E;          // [E]      valid id of the final layer whose predecessor is invalid
    uint32_t* invalid_cnt = orphan_last + E;              // [1]
    uint32_t* stay_cnt = invalid_cnt + 1;                 // [g]      transitions whose two experts share a device
    int32_t* device = reinterpret_cast<int32_t*>(stay_cnt + g);  // [g+1][E] placement rows of this group's layers

    // XCD-aware decomposition: consecutive workgroup ids are dealt round-robin to the XCDs, so
    // the XCD is blockIdx % 8; all pair groups of one token chunk are given to the same XCD.
    const int xcd = blockIdx.x % kXcds;
    const int j = blockIdx.x / kXcds;
    const int c = (j / Q) * kXcds + xcd;
    const int q = j % Q;
    if (c >= C) return;

    const int pairs = L - 1;
    const int l0 = q * g;                                  // first column of this group
    const int l1 = pairs > 0 ? min(l0 + g, pairs) : 0;     // last column (pairs l0 .. l1-1)
    const bool owns_last = (l1 == L - 1);
    const int64_t n_begin = static_cast<int64_t>(c) * chunk;
    const int64_t n_end = min(N, n_begin + chunk);
    uint32_t* my_hist = hist + (threadIdx.x & (copies - 1)) * g * words;
    uint32_t invalid_local = 0;

    // Software pipeline over the sweeps of the chunk: the (up to four) 16-byte column loads of the
    // NEXT sweep are issued before the current sweep is binned, so that the memory system is never
    // idle while the LDS atomics run.
    const int64_t sweep = static_cast<int64_t>(kTraceThreads) * VEC;
    // (columns past the group's last one and sweeps past the chunk's end are clamped, not skipped:
    // the loads stay free of branches, the duplicates are cache hits)
    auto load_cols = [&](int64_t n0, TokVec<VEC>(&col)[kAffMaxGroup + 1]) {
#pragma unroll
        for (int s = 0; s <= kAffMaxGroup; ++s)
            if (s == 0 || s == kAffMaxGroup) {  // read by the neighbouring groups too: not past the L2 (this launch, 24 x 1M tokens: 25.6 us, so 23.1)
                col[s] = load_tokens<VEC, false>(trace + static_cast<int64_t>(min(l0 + s, l1)) * N, n0, n_end);
            } else {
                col[s] = load_tokens<VEC>(trace + static_cast<int64_t>(min(l0 + s, l1)) * N, n0, n_end);
            }
    };
    TokVec<VEC> col[kAffMaxGroup + 1], nxt[kAffMaxGroup + 1];
    const int devices = placement != nullptr ? (l1 - l0 + 1) * E : 0;  // (at most 4 x 64)
    int32_t my_device = 0;
    if (placement != nullptr) my_device = placement[l0 * E + min(static_cast<int>(threadIdx.x), devices - 1)];
    load_cols(n_begin + static_cast<int64_t>(threadIdx.x) * VEC, col);  // (they travel while the counters are cleared)
    const int lds_words = copies * g * words + g * E + E + 1 + g;
    for (int i = threadIdx.x; i < lds_words; i += kTraceThreads) lds[i] = 0u;
    if (static_cast<int>(threadIdx.x) < devices) device[threadIdx.x] = my_device;
    barrier_for_lds();
    const int64_t wave_first = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)) * (kWave * VEC);
    for (int64_t base = n_begin; base + wave_first < n_end; base += sweep) {
        const int64_t n0 = base + static_cast<int64_t>(threadIdx.x) * VEC;
        load_cols(n0 + sweep, nxt);
        // Fast path (the normal case): every id this wavefront holds in the sweep is inside [0,E) and
        // no lane is past the end of the chunk - one multiply-add, a shift and one LDS atomic per
        // transition.  Anything else goes through the fully checked path below.
        bool clean = n0 + VEC <= n_end;
#pragma unroll
        for (int s = 0; s <= kAffMaxGroup; ++s) {
            if (l0 + s > l1 && s != 0) break;
            unsigned m = 0;
#pragma unroll
            for (int u = 0; u < VEC; ++u) m = max(m, static_cast<unsigned>(col[s].v[u]));
            clean = clean && m < static_cast<unsigned>(E);
        }
        const bool all_clean = __ballot(!clean) == 0ull;
        if (!all_clean) {
#pragma unroll
            for (int s = 0; s <= kAffMaxGroup; ++s) cut_vector(col[s], n0, n_end);
        }
        if (all_clean && L > 1) {
#pragma unroll
            for (int s = 1; s <= kAffMaxGroup; ++s) {
                if (l0 + s > l1) break;
                uint32_t* h = my_hist + (s - 1) * words;
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    const int bin = col[s - 1].v[u] * E + col[s].v[u];
                    atomicAdd(&h[bin >> 1], 1u << ((bin & 1) * 16));
                }
            }
        } else {
#pragma unroll
        for (int s = 1; s <= kAffMaxGroup; ++s) {
            const int l = l0 + s;
            if (l > l1) break;
            uint32_t* h = my_hist + (s - 1) * words;
            const bool last = (l == L - 1);
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                if (n0 + u < n_end) {
                    const int a = col[s - 1].v[u];
                    const int b = col[s].v[u];
                    const bool va = static_cast<unsigned>(a) < static_cast<unsigned>(E);
                    const bool vb = static_cast<unsigned>(b) < static_cast<unsigned>(E);
                    if (va && vb) {
                        const int bin = a * E + b;
                        atomicAdd(&h[bin >> 1], (bin & 1) ? 0x10000u : 1u);
                    } else if (va) {
                        atomicAdd(&orphan_next[(s - 1) * E + a], 1u);
                    }
                    if (!va) invalid_local += 1;  // layer l-1 belongs to this group
                    if (last) {
                        if (!vb) invalid_local += 1;
                        else if (!va) atomicAdd(&orphan_last[b], 1u);
                    }
                }
            }
        }
        }
        if (L == 1) {  // no pair at all: the single column only feeds loads and the invalid tally
#pragma unroll
            for (int u = 0; u < VEC; ++u)
                if (n0 + u < n_end) {
                    const int a = col[0].v[u];
                    if (static_cast<unsigned>(a) < static_cast<unsigned>(E)) atomicAdd(&orphan_last[a], 1u);
                    else invalid_local += 1;
                }
        }
#pragma unroll
        for (int s = 0; s <= kAffMaxGroup; ++s) col[s] = nxt[s];
    }
    if (invalid_local) atomicAdd(invalid_cnt, invalid_local);
    __syncthreads();

    // flush: sum the replicas (packed halves cannot carry: a bin holds at most `chunk` < 65536); with a placement, also count per pair the
    // transitions of the bins whose two experts share a device.  A power of two of lanes takes a row, each of them two of its bins (found
    // for every word by itself, with divisions, the devices were 3.6 us of the 22.7 of this launch at 24 x 1M tokens: the call 28.0 us, now
    // 26.0; fewer than 2.75 words a thread gain nothing, 23 x 7452 of 38 experts 10.6 us and 11.2).  An odd number of experts has words of two rows.
    const int my_pairs = l1 - l0;
    if (placement != nullptr && E % 2 == 0 && my_pairs * words > 11 * kTraceThreads / 4) {
        const int row_words = E / 2, log_lanes = row_words > 1 ? 32 - __builtin_clz(row_words - 1) : 0;
        const int w = static_cast<int>(threadIdx.x) & ((1 << log_lanes) - 1);
        uint32_t stay[kAffMaxGroup] = {};
        for (int row = static_cast<int>(threadIdx.x) >> log_lanes; row < my_pairs * E; row += kTraceThreads >> log_lanes) {
            const int pr = row < E ? 0 : (row < 2 * E ? 1 : 2), i = row - pr * E;
            static_assert(kAffMaxGroup == 3, "pairs of a group");
            if (w >= row_words) continue;
            const int at = pr * words + i * row_words + w;
            uint32_t s = 0;
            for (int r = 0; r < copies; ++r) s += hist[r * g * words + at];
            part_counts[(static_cast<size_t>(c) * pairs + l0) * words + at] = s;
            const int32_t here = device[row], even = device[(pr + 1) * E + 2 * w], odd = device[(pr + 1) * E + 2 * w + 1];
            const uint32_t mine = (here == even ? s & 0xffffu : 0u) + (here == odd ? s >> 16 : 0u);
#pragma unroll
            for (int k = 0; k < kAffMaxGroup; ++k) stay[k] += pr == k ? mine : 0u;
        }
#pragma unroll
        for (int pr = 0; pr < kAffMaxGroup; ++pr) {
            const uint32_t sum = wave_sum(stay[pr]);
            if (lane_id() == 0 && sum != 0) atomicAdd(&stay_cnt[min(pr, g - 1)], sum);
        }
    } else {
        for (int i = threadIdx.x; i < my_pairs * words; i += kTraceThreads) {
            uint32_t s = 0;
            for (int r = 0; r < copies; ++r) s += hist[r * g * words + i];
            part_counts[(static_cast<size_t>(c) * pairs + l0) * words + i] = s;
            if (placement != nullptr) {
                const int pr = i / words, wd = i - pr * words;
                const int32_t* here = device + pr * E;
                const int32_t* there = here + E;
                uint32_t stay = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int bin = 2 * wd + h;
                    if (bin < E * E && here[bin / E] == there[bin % E]) stay += (s >> (16 * h)) & 0xffffu;
                }
                if (stay != 0) atomicAdd(&stay_cnt[pr], stay);
            }
        }
    }
    if (placement != nullptr) {
        __syncthreads();
        if (static_cast<int>(threadIdx.x) < my_pairs) part_local[static_cast<size_t>(c) * pairs + l0 + threadIdx.x] = stay_cnt[threadIdx.x];
    }
    for (int i = threadIdx.x; i < my_pairs * E; i += kTraceThreads)
        part_orphan_next[(static_cast<size_t>(c) * pairs + l0) * E + i] = orphan_next[i];
    if (owns_last || L == 1)
        for (int i = threadIdx.x; i < E; i += kTraceThreads) part_orphan_last[static_cast<size_t>(c) * E + i] = orphan_last[i];
    if (threadIdx.x == 0) part_invalid[static_cast<size_t>(c) * Q + q] = *invalid_cnt;
}

// Counts for EVERY ordered layer pair l < m (the appendix statistic), pairs numbered source layer
// first.  What bounds it is the LDS: one atomic per token and pair (24 layers x 1M tokens: 290 million, 64 of them in 8 to
// 12 cycles), so everything else is kept below that.
//   - A workgroup owns a chunk of tokens and a block pair (I, J) of four layers each: eight columns in registers give 16
//     pairs, half a column read per pair (with one source and three targets it was 1.33, and the reads took 200 us).
//   - The six pairs inside a block are handed out to the block pairs it is part of (19 histograms at 24 layers: 152 KB); with
//     fewer than four blocks they have workgroups of their own.  All workgroups then have nearly the same work, and their
//     number is made a whole number of rounds (see make_multihop_plan).
//   - A histogram row starts at an even counter, so the word of a transition is row(a) + b/2 and its half is b%2: both
//     are formed once per token and column, a transition costs one addition and one atomic.
// Transitions with an invalid end are skipped; the packed per-chunk partials go to part_counts[chunk][pair][words].
// 24 x 1M tokens, 64 experts, both launches: 99.0 us with loops over the targets and a second set of registers for the next sweep, 95.3
// now, 85 and 10 in the profiler.  In the first one a workgroup (one a compute unit) spends 3.5 us on clearing and its first loads, 68 on counting - 59 are the
// LDS's for the atomics (7.6 cycles each; 43 without bank conflicts) -, 7 on writing, 79 on the mean; they end between 73 and 87.  Its wavefronts are done
// between 30 and 68 us after the first loads: the LDS serves some before others.
constexpr int kHopBlock = 4;       // layers per block
constexpr int kHopThreads = 1024;
constexpr int kHopInside = 6;      // pairs inside a block
constexpr int kHopShareBlocks = 4; // from so many blocks on the inside pairs are handed out
__host__ __device__ constexpr int hop_inside_source(int k) { return k < 3 ? 0 : (k < 5 ? 1 : 2); }
__host__ __device__ constexpr int hop_inside_target(int k) { return k < 3 ? k + 1 : (k < 5 ? k - 1 : 3); }
// Inside pairs of block b that the block pair (b, other) takes; b == other: all (no handing out).
__host__ __device__ inline unsigned hop_inside_mask(int b, int other, int blocks, int L)
{
    unsigned mask = 0;
    for (int k = 0; k < kHopInside; ++k) {
        const int turn = k < blocks - 1 ? k : k - (blocks - 1);  // (no divisions; blocks - 1 >= 3 where it is used)
        const int partner = b + 1 + turn < blocks ? b + 1 + turn : b + 1 + turn - blocks;
        const bool mine = b == other || (blocks >= kHopShareBlocks && partner == other);
        if (mine && b * kHopBlock + hop_inside_target(k) < L) mask |= 1u << k;
    }
    return mask;
}
// Block pair q: first those with I < J, then (few blocks) the blocks themselves.
__host__ __device__ inline void hop_blocks(int q, int blocks, int& I, int& J)
{
    const int cross = blocks * (blocks - 1) / 2;
    if (q >= cross) {
        I = J = q - cross;
        return;
    }
    for (I = 0; q >= blocks - 1 - I; ++I) q -= blocks - 1 - I;
    J = I + 1 + q;
}

template <int VEC>
__global__ __launch_bounds__(kHopThreads) void multihop_partial_kernel(const int32_t* __restrict__ trace, int L, int64_t N, int E,
                                                                          int blocks, int Q, int copies, int copy_words, int words,
                                                                          int64_t chunk, int C, uint32_t* __restrict__ part_counts)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];  // [copies][copy_words >= slots * words], two 16-bit counters per word
    const int item = xcd_item(C, Q);
    if (item < 0) return;
    const int c = item / Q;
    int I, J;
    hop_blocks(item - c * Q, blocks, I, J);
    const int i0 = I * kHopBlock, j0 = J * kHopBlock;
    const int targets = I == J ? 0 : min(kHopBlock, L - j0);  // (block I is whole where there is a later one)
    const unsigned inside_i = hop_inside_mask(I, J, blocks, L), inside_j = I == J ? 0u : hop_inside_mask(J, I, blocks, L);
    const int64_t n_begin = static_cast<int64_t>(c) * chunk;
    const int64_t n_end = min(N, n_begin + chunk);
    const uint32_t hist_bytes = static_cast<uint32_t>(words) * 4u;
    const uint32_t row_bytes = static_cast<uint32_t>((E + 1) / 2) * 4u;
    const uint32_t my_copy = static_cast<uint32_t>(threadIdx.x & (copies - 1)) * static_cast<uint32_t>(copy_words) * 4u;
    // The transitions of one sweep.  As the source of a pair a token is the byte offset of its row, as the target that of its word and
    // the addend: one addition and one atomic a transition.
    // Clean wavefronts (nearly all): the pairs inside the blocks first, then the tokens of the others as offsets and addends, formed once
    // and indexed statically; the next sweep's loads then go where this one's tokens were.
    auto add_at = [&](uint32_t at, uint32_t one) { atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(lds) + at), one); };
    auto clean_row = [&](int32_t t) { return my_copy + __umul24(static_cast<uint32_t>(t), row_bytes); };
    auto clean_word = [&](int32_t t) { return (static_cast<uint32_t>(t) << 1) & ~3u; };
    auto clean_one = [&](int32_t t) { return 1u << ((static_cast<uint32_t>(t) << 4) & 31u); };
    auto count_clean = [&](TokVec<VEC>(&col)[2 * kHopBlock], auto load_next) {
        uint32_t slot = targets > 0 ? kHopBlock * kHopBlock * hist_bytes : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < kHopInside; ++k)
                if (((h == 0 ? inside_i : inside_j) >> k & 1u) != 0u) {
                    const TokVec<VEC>&from = col[h * kHopBlock + hop_inside_source(k)], &to = col[h * kHopBlock + hop_inside_target(k)];
#pragma unroll
                    for (int u = 0; u < VEC; ++u) add_at(slot + clean_row(from.v[u]) + clean_word(to.v[u]), clean_one(to.v[u]));
                    slot += hist_bytes;
                }
        uint32_t row[kHopBlock][VEC], word[kHopBlock][VEC], one[kHopBlock][VEC];
#pragma unroll
        for (int s = 0; s < kHopBlock; ++s)
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                row[s][u] = clean_row(col[s].v[u]);
                word[s][u] = clean_word(col[kHopBlock + s].v[u]);
                one[s][u] = clean_one(col[kHopBlock + s].v[u]);
            }
        load_next();
        slot = 0;
#pragma unroll
        for (int t = 0; t < kHopBlock; ++t) {
            if (t >= targets) break;
#pragma unroll
            for (int s = 0; s < kHopBlock; ++s) {
#pragma unroll
                for (int u = 0; u < VEC; ++u) add_at(row[s][u] + word[t][u] + slot, one[t][u]);
                slot += hist_bytes;
            }
        }
    };
    // The others, in loops over the targets and over the two blocks (little code): an invalid id adds 0 (to a word of row 0 or
    // column 0); this costs as many vector instructions as the LDS has cycles.
    auto count_checked = [&](const TokVec<VEC>(&col)[2 * kHopBlock], int left) {
        auto valid = [&](const TokVec<VEC>& t, int u) { return static_cast<uint32_t>(t.v[u]) < static_cast<uint32_t>(E) && u < left; };
        auto row_of = [&](const TokVec<VEC>& t, int u) { return valid(t, u) ? my_copy + __umul24(static_cast<uint32_t>(t.v[u]), row_bytes) : 0u; };
        auto word_of = [&](const TokVec<VEC>& t, int u) { return valid(t, u) ? static_cast<uint32_t>(t.v[u]) / 2u * 4u : 0u; };
        auto one_of = [&](const TokVec<VEC>& t, int u) { return valid(t, u) ? 1u << (static_cast<uint32_t>(t.v[u]) % 2u * 16u) : 0u; };
        auto add = [&](uint32_t at, uint32_t one) { atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(lds) + at), one); };
        uint32_t slot = 0;
        {
            uint32_t row[kHopBlock][VEC];
            TokVec<VEC> target[kHopBlock];
#pragma unroll
            for (int s = 0; s < kHopBlock; ++s) {
                target[s] = col[kHopBlock + s];
#pragma unroll
                for (int u = 0; u < VEC; ++u) row[s][u] = row_of(col[s], u);
            }
#pragma unroll 1
            for (int t = 0; t < targets; ++t) {
                uint32_t word[VEC], one[VEC];
#pragma unroll
                for (int u = 0; u < VEC; ++u) {
                    word[u] = slot + word_of(target[0], u);
                    one[u] = one_of(target[0], u);
                }
#pragma unroll
                for (int s = 0; s < kHopBlock; ++s)
#pragma unroll
                    for (int u = 0; u < VEC; ++u) add(s * hist_bytes + row[s][u] + word[u], valid(col[s], u) ? one[u] : 0u);
                slot += kHopBlock * hist_bytes;
#pragma unroll
                for (int s = 0; s + 1 < kHopBlock; ++s) target[s] = target[s + 1];
            }
        }
        slot = targets > 0 ? kHopBlock * kHopBlock * hist_bytes : 0u;
        TokVec<VEC> x[kHopBlock];
#pragma unroll
        for (int s = 0; s < kHopBlock; ++s) x[s] = col[s];
#pragma unroll 1
        for (unsigned mask = inside_i, h = 0; h < 2; ++h, mask = inside_j) {
#pragma unroll
            for (int k = 0; k < kHopInside; ++k)
                if ((mask >> k & 1u) != 0u) {
                    const TokVec<VEC>&from = x[hop_inside_source(k)], &to = x[hop_inside_target(k)];
#pragma unroll
                    for (int u = 0; u < VEC; ++u) add(slot + row_of(from, u) + word_of(to, u), valid(from, u) ? one_of(to, u) : 0u);
                    slot += hist_bytes;
                }
#pragma unroll
            for (int s = 0; s < kHopBlock; ++s) x[s] = col[kHopBlock + s];
        }
    };
    const int64_t sweep = static_cast<int64_t>(kHopThreads) * VEC;
    auto load_cols = [&](int64_t n0, TokVec<VEC>(&col)[2 * kHopBlock]) {  // clamped, never skipped
#pragma unroll
        for (int s = 0; s < 2 * kHopBlock; ++s)
            col[s] = load_tokens<VEC, false>(trace + static_cast<int64_t>(min(s < kHopBlock ? i0 + s : j0 + s - kHopBlock, L - 1)) * N, n0, n_end);
    };
    TokVec<VEC> col[2 * kHopBlock];
    const int64_t wave_first = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)) * (kWave * VEC);
    load_cols(n_begin + static_cast<int64_t>(threadIdx.x) * VEC, col);
    for (int i = threadIdx.x; i < copies * (copy_words / 2); i += kHopThreads) reinterpret_cast<uint2*>(lds)[i] = make_uint2(0u, 0u);
    __syncthreads();
    for (int64_t base = n_begin; base + wave_first < n_end; base += sweep) {
        const int64_t n0 = base + static_cast<int64_t>(threadIdx.x) * VEC;
        auto load_next = [&]() {
            if (base + sweep + wave_first < n_end) load_cols(n0 + sweep, col);
        };
        unsigned m = 0;
#pragma unroll
        for (int s = 0; s < 2 * kHopBlock; ++s)
#pragma unroll
            for (int u = 0; u < VEC; ++u) m = max(m, static_cast<unsigned>(col[s].v[u]));  // (clamped duplicate columns repeat a checked one)
        const int left = static_cast<int>(min(n_end - n0, static_cast<int64_t>(VEC)));  // tokens of this lane
        if (__ballot(left < VEC || m >= static_cast<unsigned>(E)) == 0ull) {
            count_clean(col, load_next);
        } else {
#pragma unroll
            for (int s = 0; s < 2 * kHopBlock; ++s) cut_vector(col[s], n0, n_end);
            count_checked(col, left);
            load_next();
        }
    }
    __syncthreads();

    // flush, replicas summed (packed halves cannot carry: a bin holds at most `chunk` < 65536)
    const size_t total_pairs = static_cast<size_t>(L) * (L - 1) / 2;
    const int cross = targets > 0 ? kHopBlock * kHopBlock : 0;
    const int used = cross + __builtin_popcount(inside_i) + __builtin_popcount(inside_j);
    const unsigned per_slot = static_cast<unsigned>(words / 2), inverse = ((1u << 26) + per_slot - 1u) / per_slot;  // exact below 20 x 1024
    for (int i = threadIdx.x; i < used * (words / 2); i += kHopThreads) {
        const int slot = static_cast<int>(static_cast<unsigned>(i) * inverse >> 26), w = i - slot * (words / 2);
        int l, to;  // layers of the slot's pair
        if (slot < cross) {
            l = i0 + slot % kHopBlock;
            to = j0 + slot / kHopBlock;
            if (slot / kHopBlock >= targets) continue;
        } else {
            unsigned left = inside_i | inside_j << kHopInside;
            for (int r = slot - cross; r > 0; --r) left &= left - 1u;
            const int k = __builtin_ctz(left), first = k < kHopInside ? i0 : j0, kk = k < kHopInside ? k : k - kHopInside;
            l = first + hop_inside_source(kk);
            to = first + hop_inside_target(kk);
        }
        const uint2* from = reinterpret_cast<const uint2*>(lds + static_cast<size_t>(slot) * words) + w;
        uint2 sum = make_uint2(0u, 0u);
#pragma unroll 4
        for (int r = 0; r < copies; ++r) {
            const uint2 v = from[r * (copy_words / 2)];
            sum.x += v.x;
            sum.y += v.y;
        }
        const size_t pair = static_cast<size_t>(l) * (2 * L - l - 1) / 2 + (to - l - 1);
        reinterpret_cast<uint2*>(part_counts + (static_cast<size_t>(c) * total_pairs + pair) * words)[w] = sum;
    }
}

// The same counts by groups of one source layer and up to three targets: four columns in registers for three pairs, 24 KB of
// histograms (two replicas of them) to clear and to write instead of 152, a sixth of the code.  It reads more than twice as many
// columns per pair as the blocks, but starts and ends sooner: short traces and few layers (see multihop_in_groups; 8 layers x
// 100000 tokens, 64 experts: 25.5 us by blocks, 11.4).  Groups are numbered in pair order; histogram rows and partials as above.
template <int VEC>
__global__ __launch_bounds__(kTraceThreads) void multihop_group_kernel(const int32_t* __restrict__ trace, int L, int64_t N, int E, int Q,
                                                                       int copies, int words, int64_t chunk, int C,
                                                                       uint32_t* __restrict__ part_counts)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];  // [copies][kAffMaxGroup][words], two 16-bit counters per word
    const int item = xcd_item(C, Q);
    if (item < 0) return;
    const int c = item / Q;
    int q = item - c * Q, l = 0, pair = 0;  // source layer and number of its first pair
    for (; q >= (L - 2 - l) / kAffMaxGroup + 1; ++l) {
        q -= (L - 2 - l) / kAffMaxGroup + 1;
        pair += L - 1 - l;
    }
    const int m0 = l + 1 + q * kAffMaxGroup;  // first target
    const int my_pairs = min(kAffMaxGroup, L - m0);
    pair += q * kAffMaxGroup;

    const int64_t n_begin = static_cast<int64_t>(c) * chunk;
    const int64_t n_end = min(N, n_begin + chunk);
    const int64_t sweep = static_cast<int64_t>(kTraceThreads) * VEC;
    auto load_cols = [&](int64_t n0, TokVec<VEC>(&col)[kAffMaxGroup + 1]) {  // clamped, never skipped
        col[0] = load_tokens<VEC, false>(trace + static_cast<int64_t>(l) * N, n0, n_end);
#pragma unroll
        for (int s = 1; s <= kAffMaxGroup; ++s) col[s] = load_tokens<VEC, false>(trace + static_cast<int64_t>(min(m0 + s - 1, L - 1)) * N, n0, n_end);
    };
    TokVec<VEC> col[kAffMaxGroup + 1], nxt[kAffMaxGroup + 1];
    load_cols(n_begin + static_cast<int64_t>(threadIdx.x) * VEC, col);
    for (int i = threadIdx.x; i < copies * kAffMaxGroup * words / 2; i += kTraceThreads) reinterpret_cast<uint2*>(lds)[i] = make_uint2(0u, 0u);
    __syncthreads();
    const int row_words = (E + 1) / 2;
    uint32_t* mine = lds + (threadIdx.x & (copies - 1)) * kAffMaxGroup * words;
    for (int64_t base = n_begin; base < n_end; base += sweep) {
        const int64_t n0 = base + static_cast<int64_t>(threadIdx.x) * VEC;
        load_cols(n0 + sweep, nxt);
        unsigned m = 0;
#pragma unroll
        for (int s = 0; s <= kAffMaxGroup; ++s)
#pragma unroll
            for (int u = 0; u < VEC; ++u) m = max(m, static_cast<unsigned>(col[s].v[u]));  // (clamped duplicate columns repeat a checked one)
        const bool clean = __ballot(n0 + VEC > n_end || m >= static_cast<unsigned>(E)) == 0ull;
        if (!clean) {
#pragma unroll
            for (int s = 0; s <= kAffMaxGroup; ++s) cut_vector(col[s], n0, n_end);
        }
#pragma unroll
        for (int s = 1; s <= kAffMaxGroup; ++s) {
            if (s > my_pairs) break;
            uint32_t* h = mine + (s - 1) * words;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                const int a = col[0].v[u], b = col[s].v[u];
                if (clean || (n0 + u < n_end && static_cast<unsigned>(a) < static_cast<unsigned>(E) && static_cast<unsigned>(b) < static_cast<unsigned>(E)))
                    atomicAdd(&h[a * row_words + (b >> 1)], 1u << ((b & 1) * 16));
            }
        }
#pragma unroll
        for (int s = 0; s <= kAffMaxGroup; ++s) col[s] = nxt[s];
    }
    __syncthreads();
    // flush, replicas summed (packed halves cannot carry: a bin holds at most `chunk` < 65536)
    uint32_t* to = part_counts + (static_cast<size_t>(c) * (static_cast<size_t>(L) * (L - 1) / 2) + pair) * words;
    for (int i = threadIdx.x; i < my_pairs * words; i += kTraceThreads) {
        uint32_t sum = 0;
        for (int r = 0; r < copies; ++r) sum += lds[r * kAffMaxGroup * words + i];
        to[i] = sum;
    }
}

template <typename Launch>
static void with_chunks_ahead(int C, int64_t rows, Launch launch)
{
    const int ahead = chunks_ahead(C, rows);
    if (ahead <= 8) launch(std::integral_constant<int, 8>());
    else if (ahead <= 16) launch(std::integral_constant<int, 16>());
    else if (ahead <= 24) launch(std::integral_constant<int, 24>());
    else launch(std::integral_constant<int, 32>());
}

// Half a wavefront per (pair, source expert) row, lane w of it the counters 2w and 2w+1: sums the chunks (up to 32 independent loads
// in flight), the row sum by lane exchanges, the conditional probabilities.  Bound by the read of the partials: a lane per
// counter fetched every word twice (24 layers, 64 experts, 17 chunks: 18 us, now 12).
template <int U>
__global__ __launch_bounds__(256) void multihop_finalize_kernel(const uint32_t* __restrict__ part_counts, int C, int pairs, int E, int words,
                                                                int64_t* __restrict__ counts, float* __restrict__ cond_prob)
{
    const int row = static_cast<int>(blockIdx.x) * (256 / 32) + static_cast<int>(threadIdx.x) / 32;
    const bool live = row < pairs * E;
    const int w = threadIdx.x % 32, row_words = (E + 1) / 2;
    const int r = live ? row : 0;
    const int pair = r / E, i = r % E;
    const uint32_t* src = part_counts + static_cast<size_t>(pair) * words + i * row_words + min(w, row_words - 1);
    const size_t step = static_cast<size_t>(pairs) * words;
    long long even = 0, odd = 0;
    for (int c0 = 0; c0 < C; c0 += U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = src[min(c0 + u, C - 1) * step];  // clamped, never branched around
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lo += c0 + u < C ? v[u] & 0xffffu : 0u;
            hi += c0 + u < C ? v[u] >> 16 : 0u;
        }
        even += lo;
        odd += hi;
    }
    if (w >= row_words) even = odd = 0;
    long long sum = even + odd;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 32);
    if (!live || w >= row_words) return;
    const size_t o = static_cast<size_t>(row) * E + 2 * w;
    auto share = [&](long long cnt) { return sum > 0 ? static_cast<float>(static_cast<double>(cnt) / static_cast<double>(sum)) : 0.0f; };
    if (2 * w + 1 < E) {
        typedef long long i64x2_v __attribute__((vector_size(2 * sizeof(long long)), aligned(8)));
        typedef float f32x2_v __attribute__((vector_size(2 * sizeof(float)), aligned(4)));
        *reinterpret_cast<i64x2_v*>(counts + o) = i64x2_v{even, odd};
        if (cond_prob != nullptr) *reinterpret_cast<f32x2_v*>(cond_prob + o) = f32x2_v{share(even), share(odd)};
    } else {
        counts[o] = even;
        if (cond_prob != nullptr) cond_prob[o] = share(even);
    }
}

// Workgroups of 256 threads.  The first ceil((L-1)*E / 4) give every wavefront one (pair l, source
// expert i) row: lane p sums bin (i, p) over all chunks (up to 32 independent loads in flight), the row sum
// is a wavefront reduction -> counts, load of (l, i), conditional probabilities; nothing goes through
// LDS and no workgroup barrier is needed.  The next E workgroups take one
// expert p of the FINAL layer each: its load is the column sum of the last pair (taken from the
// partials, so that no result of another workgroup is needed) plus the orphans.  One workgroup
// adds up the invalid tally.  With a placement, L-1 more workgroups form the locality numerators.
constexpr int kFinRowsPerWorkgroup = 4;
template <int U>
__global__ __launch_bounds__(256) void affinity_finalize_kernel(const uint32_t* __restrict__ part_counts,
                                                                const uint32_t* __restrict__ part_orphan_next,
                                                                const uint32_t* __restrict__ part_orphan_last,
                                                                const uint32_t* __restrict__ part_invalid, int C, int Q, int L, int E,
                                                                int words, int64_t* __restrict__ counts, int64_t* __restrict__ loads,
                                                                float* __restrict__ cond_prob, int64_t* __restrict__ n_invalid,
                                                                const uint32_t* __restrict__ part_local,  // [C][L-1] or null
                                                                int64_t* __restrict__ local)              // [L-1] (with part_local)
{
    __shared__ long long orphan_red[4];
    const int pairs = L - 1;
    const int p = lane_id();
    const int w = threadIdx.x / kWave;
    const int rows = pairs * E;
    const int row_blocks = (rows + kFinRowsPerWorkgroup - 1) / kFinRowsPerWorkgroup;
    if (static_cast<int>(blockIdx.x) < row_blocks) {
        const int row = static_cast<int>(blockIdx.x) * kFinRowsPerWorkgroup + w;
        if (row >= rows) return;  // (whole wavefronts; no barrier follows)
        const int l = row / E;
        const int i = row % E;
        long long cnt = 0;
        const uint32_t* orphans = part_orphan_next + static_cast<size_t>(l) * E + i;
        const uint32_t first_orphan = *(C > 0 ? orphans + static_cast<size_t>(min(p, C - 1)) * pairs * E : part_counts);  // (travels with the counts;
        // no chunks: any word that is there)
        const int bin = i * E + min(p, E - 1);
        const int shift = (bin & 1) * 16;
        const uint32_t* src = part_counts + static_cast<size_t>(l) * words + (bin >> 1);
        const size_t step = static_cast<size_t>(pairs) * words;
        for (int c0 = 0; c0 < C; c0 += U) {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = src[min(c0 + u, C - 1) * step];  // clamped, never branched around
            uint32_t sum = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) sum += c0 + u < C ? (v[u] >> shift) & 0xffffu : 0u;
            cnt += sum;
        }
        if (p >= E) cnt = 0;
        long long orphan = p < C ? first_orphan : 0u;
        for (int c = p + kWave; c < C; c += kWave) orphan += orphans[static_cast<size_t>(c) * pairs * E];
        orphan = wave_sum(orphan);
        const long long row_sum = wave_sum(cnt);
        if (p < E) {
            const size_t o = (static_cast<size_t>(l) * E + i) * E + p;
            counts[o] = cnt;
            if (cond_prob != nullptr)
                cond_prob[o] = row_sum > 0 ? static_cast<float>(static_cast<double>(cnt) / static_cast<double>(row_sum)) : 0.0f;
        }
        if (loads != nullptr && p == 0) loads[static_cast<size_t>(l) * E + i] = row_sum + orphan;
    } else if (static_cast<int>(blockIdx.x) < row_blocks + E) {
        if (loads == nullptr) return;
        const int pe = blockIdx.x - row_blocks;  // expert of the final layer
        long long s = 0;
        if (pairs > 0) {  // column pe of the last pair: sum over chunks c and source experts i
            const int total = C * E;
            for (int j0 = threadIdx.x; j0 < total; j0 += 256 * 8) {
                uint32_t v[8];
                int sh[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = min(j0 + 256 * u, total - 1);
                    const int c = j / E, i = j - c * E;
                    const int bin = i * E + pe;
                    sh[u] = (bin & 1) * 16;
                    v[u] = part_counts[(static_cast<size_t>(c) * pairs + (pairs - 1)) * words + (bin >> 1)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (j0 + 256 * u < total) s += (v[u] >> sh[u]) & 0xffffu;
            }
        }
        for (int c = threadIdx.x; c < C; c += 256) s += part_orphan_last[static_cast<size_t>(c) * E + pe];
        s = wave_sum(s);
        if (p == 0) orphan_red[w] = s;
        __syncthreads();
        if (threadIdx.x == 0) loads[static_cast<size_t>(L - 1) * E + pe] = orphan_red[0] + orphan_red[1] + orphan_red[2] + orphan_red[3];
    } else if (static_cast<int>(blockIdx.x) == row_blocks + E) {
        if (n_invalid == nullptr) return;
        long long inv = 0;
        for (int i = threadIdx.x; i < C * Q; i += 256) inv += part_invalid[i];
        inv = wave_sum(inv);
        if (p == 0) orphan_red[w] = inv;
        __syncthreads();
        if (threadIdx.x == 0) *n_invalid = orphan_red[0] + orphan_red[1] + orphan_red[2] + orphan_red[3];
    } else {
        // locality numerator of pair l: the per-chunk counts of the first launch added up
        if (part_local == nullptr) return;
        const int l = blockIdx.x - (row_blocks + E + 1);
        long long stay = 0;
        for (int c = threadIdx.x; c < C; c += 256) stay += part_local[static_cast<size_t>(c) * pairs + l];
        stay = wave_sum(stay);
        if (p == 0) orphan_red[w] = stay;
        __syncthreads();
        if (threadIdx.x == 0) local[l] = orphan_red[0] + orphan_red[1] + orphan_red[2] + orphan_red[3];
    }
}

// ------------------------------------------------------------------------------------------
constexpr int kLocAhead = 2;  // trace layers whose loads are in flight together

// HOME: additionally counts, per layer, the tokens whose expert sits on another device than
// home[n] (the device that owns the token's request); the per-chunk partials then hold the L-1 pair
// counts followed by the L away counts.
template <int VEC, bool HOME>
__global__ __launch_bounds__(kTraceThreads) void locality_partial_kernel(const int32_t* __restrict__ trace,
                                                                          const int32_t* __restrict__ placement,
                                                                          const int32_t* __restrict__ home, int L, int64_t N, int E,
                                                                          int64_t chunk, uint32_t* __restrict__ part)
{
    extern __shared__ int32_t lds_i[];
    int32_t* pl = lds_i;                                              // [L][E]
    uint32_t* pair_cnt = reinterpret_cast<uint32_t*>(lds_i + L * E);  // [L-1] pairs, then (HOME) [L] away counts
    uint32_t* away_cnt = pair_cnt + (L - 1);
    const int n_out = (L - 1) + (HOME ? L : 0);
    const int64_t n_begin = static_cast<int64_t>(blockIdx.x) * chunk;
    const int64_t n_end = min(N, n_begin + chunk);
    const int64_t sweep = static_cast<int64_t>(blockDim.x) * VEC;
    const int lane = lane_id();
    auto load_layers = [&](int lb, int64_t n0, TokVec<VEC>(&dst)[kLocAhead]) {
#pragma unroll
        for (int a = 0; a < kLocAhead; ++a)  // layers past the last one are clamped, not skipped: no branch at the loads
            dst[a] = load_tokens<VEC>(trace + static_cast<int64_t>(min(lb + a, L - 1)) * N, n0, n_end);
    };
    TokVec<VEC> hm, first, cur[kLocAhead], nxt[kLocAhead];
    auto begin_sweep = [&](int64_t n0) {
        if constexpr (HOME) hm = load_tokens<VEC>(home, n0, n_end);
        first = load_tokens<VEC>(trace, n0, n_end);
        load_layers(1, n0, cur);
    };
    // the placement, and behind it the first tokens: they travel together (24 x 999983 tokens with home devices 25.05 us one after
    // the other, 24.3 now; 6 x 2000001 15.2 and 14.7)
    constexpr int kPlacementAhead = 2;
    const int entries = L * E;
    int32_t entry[kPlacementAhead];
#pragma unroll
    for (int k = 0; k < kPlacementAhead; ++k) entry[k] = placement[min(static_cast<int>(threadIdx.x + k * blockDim.x), entries - 1)];
    begin_sweep(n_begin + static_cast<int64_t>(threadIdx.x) * VEC);
    for (int i = threadIdx.x; i < n_out; i += blockDim.x) pair_cnt[i] = 0u;
#pragma unroll
    for (int k = 0; k < kPlacementAhead; ++k)
        if (static_cast<int>(threadIdx.x + k * blockDim.x) < entries) pl[threadIdx.x + k * blockDim.x] = entry[k];
    for (int i = threadIdx.x + kPlacementAhead * blockDim.x; i < entries; i += blockDim.x) pl[i] = placement[i];
    barrier_for_lds();

    for (int64_t base = n_begin; base < n_end; base += sweep) {
        const int64_t n0 = base + static_cast<int64_t>(threadIdx.x) * VEC;
        int dev_prev[VEC];
        bool ok_prev[VEC];
        const bool in_range = n0 + VEC <= n_end;  // all tokens of this lane exist
        bool prev_clean;                           // all ids of the previous layer valid (and in range)
        {
            TokVec<VEC> t = first;
            if (__ballot(!in_range) != 0ull) {
                cut_vector(t, n0, n_end);
                if constexpr (HOME) cut_vector(hm, n0, n_end);
            }
            prev_clean = in_range;
            int away = 0;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                ok_prev[u] = (n0 + u < n_end) && static_cast<unsigned>(t.v[u]) < static_cast<unsigned>(E);
                dev_prev[u] = ok_prev[u] ? pl[t.v[u]] : 0;
                prev_clean = prev_clean && ok_prev[u];
                if constexpr (HOME) away += __popcll(__ballot(ok_prev[u] && dev_prev[u] != hm.v[u]));
            }
            if constexpr (HOME)
                if (lane == 0 && away != 0) atomicAdd(&away_cnt[0], static_cast<uint32_t>(away));
        }
        // software pipeline over batches of kLocAhead layers: the next batch is requested before the
        // current one is counted
        for (int lb = 1; lb < L; lb += kLocAhead) {
            load_layers(lb + kLocAhead, n0, nxt);
#pragma unroll
            for (int a = 0; a < kLocAhead; ++a) {
                const int l = lb + a;
                if (l >= L) break;
                unsigned m = 0;
#pragma unroll
                for (int u = 0; u < VEC; ++u) m = max(m, static_cast<unsigned>(cur[a].v[u]));
                const bool clean = in_range && m < static_cast<unsigned>(E);
                // wavefront total of "device unchanged" flags by ballot + popcount (scalar unit)
                int same = 0, away = 0;
                if (__ballot(!(clean && prev_clean)) == 0ull) {
                    // fast path: every id of this wavefront is valid in both layers - one table
                    // look-up and one compare per transition
#pragma unroll
                    for (int u = 0; u < VEC; ++u) {
                        const int dev = pl[l * E + cur[a].v[u]];
                        same += __popcll(__ballot(dev == dev_prev[u]));
                        if constexpr (HOME) away += __popcll(__ballot(dev != hm.v[u]));
                        dev_prev[u] = dev;
                    }
                } else {
                    cut_vector(cur[a], n0, n_end);
#pragma unroll
                    for (int u = 0; u < VEC; ++u) {
                        const bool ok = (n0 + u < n_end) && static_cast<unsigned>(cur[a].v[u]) < static_cast<unsigned>(E);
                        const int dev = ok ? pl[l * E + cur[a].v[u]] : 0;
                        same += __popcll(__ballot(ok && ok_prev[u] && dev == dev_prev[u]));
                        if constexpr (HOME) away += __popcll(__ballot(ok && dev != hm.v[u]));
                        ok_prev[u] = ok;
                        dev_prev[u] = dev;
                    }
                }
                if constexpr (HOME)
                    if (lane == 0 && away != 0) atomicAdd(&away_cnt[l], static_cast<uint32_t>(away));
                if (clean) {  // the flags the checked path would have produced
#pragma unroll
                    for (int u = 0; u < VEC; ++u) ok_prev[u] = true;
                }
                prev_clean = clean;
                if (lane == 0 && same != 0) atomicAdd(&pair_cnt[l - 1], static_cast<uint32_t>(same));
            }
#pragma unroll
            for (int a = 0; a < kLocAhead; ++a) cur[a] = nxt[a];
        }
        if (base + sweep < n_end) begin_sweep(n0 + sweep);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_out; i += blockDim.x) part[static_cast<size_t>(blockIdx.x) * n_out + i] = pair_cnt[i];
}

// One wavefront per output element j: the first `pairs` elements go to local_per_pair, the rest
// (present with home devices only) to away_per_layer.  The sums of up to 256 chunks are asked for at once; in a loop that leaves
// one lane after the other they were awaited one by one (transfers of 6 x 1000000 tokens, 245 chunks: 12.3 us, now 10.7).
__global__ __launch_bounds__(kWave) void locality_finalize_kernel(const uint32_t* __restrict__ part, int C, int pairs, int n_out,
                                                                   int64_t* __restrict__ local_per_pair,
                                                                   int64_t* __restrict__ away_per_layer)
{
    const int j = blockIdx.x;
    long long s = 0;
    for (int c0 = threadIdx.x; c0 - static_cast<int>(threadIdx.x) < C; c0 += 4 * kWave) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = part[static_cast<size_t>(min(c0 + u * kWave, C - 1)) * n_out + j];  // clamped, never branched around
#pragma unroll
        for (int u = 0; u < 4; ++u) s += c0 + u * kWave < C ? v[u] : 0u;
    }
    s = wave_sum(s);
    if (threadIdx.x == 0) {
        if (j < pairs) local_per_pair[j] = s;
        else away_per_layer[j - pairs] = s;
    }
}

// A thread walks all layers of its tokens, one after the other: a short trace is spread as thin as possible, one token a thread up
// to a token for every thread of the chip, and in workgroups of four wavefronts as long as these give at most one set of
// partial counts per compute unit (1000 sets cost the second launch 4 us).  Transfers of 24 layers x 250000
// tokens: four tokens a thread in workgroups of 1024 23.8 us, one token a thread 15.7.
struct LocalityPlan {
    int vec, threads, C;
    int64_t chunk;
};
static LocalityPlan locality_plan(int64_t N)
{
    LocalityPlan p;
    constexpr int64_t chip = static_cast<int64_t>(kTraceThreads) * kTargetWorkgroups;
    p.vec = N > chip ? 4 : 1;
    p.threads = N <= 256ll * kTargetWorkgroups ? 256 : kTraceThreads;
    const int64_t sweep = static_cast<int64_t>(p.threads) * p.vec;
    p.chunk = (N + kTargetWorkgroups - 1) / kTargetWorkgroups;  // about one workgroup per compute unit
    p.chunk = (p.chunk + sweep - 1) / sweep * sweep;
    if (p.chunk < sweep) p.chunk = sweep;
    const int64_t cap = (1ll << 31) / sweep * sweep;  // 32-bit partial counters
    if (p.chunk > cap) p.chunk = cap;
    p.C = static_cast<int>(N > 0 ? (N + p.chunk - 1) / p.chunk : 0);
    return p;
}

static int validate_trace_args(const char* fn, int L, int64_t N, int E)
{
    if (L < 1 || L > EXF_MAX_TRACE_LAYERS) return fail(EXF_ERR_BAD_SHAPE, "%s: L = %d outside [1,%d]", fn, L, EXF_MAX_TRACE_LAYERS);
    if (N < 0) return fail(EXF_ERR_BAD_SHAPE, "%s: N = %lld < 0", fn, static_cast<long long>(N));
    if (E < 1 || E > EXF_MAX_EXPERTS) return fail(EXF_ERR_BAD_SHAPE, "%s: E = %d outside [1,%d]", fn, E, EXF_MAX_EXPERTS);
    if (N >= (1ll << 40)) return fail(EXF_ERR_BAD_SHAPE, "%s: N must be below 2^40", fn);
    return EXF_OK;
}

// LDS of locality_partial_kernel at most: the placement of all layers and the counts
constexpr size_t kLocMaxLdsBytes = (EXF_MAX_TRACE_LAYERS * EXF_MAX_EXPERTS + 2 * EXF_MAX_TRACE_LAYERS) * sizeof(int32_t);
template <int VEC, bool HOME>
static int launch_locality(const char* fn, const LocalityPlan& p, const int32_t* trace, const int32_t* placement, const int32_t* home, int L,
                           int64_t N, int E, uint32_t* part, hipStream_t stream)
{
    auto kern = locality_partial_kernel<VEC, HOME>;
    const size_t lds = (static_cast<size_t>(L) * E + (L - 1) + (HOME ? L : 0)) * sizeof(int32_t);
    static std::atomic<uint64_t> allowed{0};
    if (lds > 64 * 1024)
        if (int rc = allow_lds(reinterpret_cast<const void*>(kern), kLocMaxLdsBytes, allowed, fn)) return rc;
    hipLaunchKernelGGL(kern, dim3(p.C), dim3(p.threads), lds, stream, trace, placement, home, L, N, E, p.chunk, part);
    return EXF_OK;
}

}  // namespace exf

extern "C" size_t affinity_histogram_workspace_bytes(int L, int64_t N, int E)
{
    if (L < 1 || N < 0 || E < 1 || E > EXF_MAX_EXPERTS) return 0;
    return exf::make_affinity_plan(L, N, E).total_bytes;
}

namespace exf {

// affinity_histogram and affinity_statistics: the same two launches.  With a placement every
// workgroup of the first launch also counts, per pair, the transitions of its finished histogram whose
// two experts share a device, and the second launch has one more workgroup per pair to add these up.
static int run_affinity(const char* fn, const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int64_t* counts,
                        int64_t* loads, float* cond_prob, int64_t* n_invalid, int64_t* local_per_pair, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    const AffinityPlan p = make_affinity_plan(L, N, E);
    if (workspace_bytes < p.total_bytes) return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "%s: workspace %zu < %zu bytes", fn, workspace_bytes, p.total_bytes);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (statistics_direct(trace, placement, L, N, E, counts, loads, cond_prob, n_invalid, local_per_pair, s)) return check_launch(fn);
    char* ws = static_cast<char*>(workspace);
    uint32_t* part_counts = reinterpret_cast<uint32_t*>(ws + p.off_counts);
    uint32_t* part_orphan_next = reinterpret_cast<uint32_t*>(ws + p.off_orphan_next);
    uint32_t* part_orphan_last = reinterpret_cast<uint32_t*>(ws + p.off_orphan_last);
    uint32_t* part_invalid = reinterpret_cast<uint32_t*>(ws + p.off_invalid);
    uint32_t* part_local = placement != nullptr ? reinterpret_cast<uint32_t*>(ws + p.off_local) : nullptr;
    if (p.C > 0) {
        const int c_pad = (p.C + kXcds - 1) / kXcds * kXcds;
        const unsigned grid = static_cast<unsigned>(c_pad) * p.Q;
        const size_t lds = (static_cast<size_t>(p.copies) * p.g * p.words + static_cast<size_t>(p.g) * E + E + 1 + p.g +
                            static_cast<size_t>(p.g + 1) * E) * sizeof(uint32_t);
        static_assert(kAffHistBudget + ((2 * kAffMaxGroup + 2) * EXF_MAX_EXPERTS + 1 + kAffMaxGroup) * sizeof(uint32_t) <= 64 * 1024,
                      "within the LDS that a launch may use without asking");
        auto kern = p.vec == 4 ? affinity_partial_kernel<4> : affinity_partial_kernel<1>;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kTraceThreads), lds, s, trace, L, N, E, p.g, p.Q, p.copies, p.words, p.chunk, p.C, part_counts,
                           part_orphan_next, part_orphan_last, part_invalid, placement, part_local);
    }
    // rows of all pairs, then the loads of the final layer, the invalid tally and (with a placement) the
    // locality numerators of all pairs
    const unsigned fin_grid = static_cast<unsigned>(((L - 1) * E + kFinRowsPerWorkgroup - 1) / kFinRowsPerWorkgroup + E + 1 +
                                                   (placement != nullptr ? L - 1 : 0));
    with_chunks_ahead(p.C, static_cast<int64_t>(L - 1) * E, [&](auto ahead) {
        hipLaunchKernelGGL(affinity_finalize_kernel<decltype(ahead)::value>, dim3(fin_grid), dim3(256), 0, s, part_counts, part_orphan_next, part_orphan_last,
                           part_invalid, p.C, p.Q, L, E, p.words, counts, loads, cond_prob, n_invalid, part_local, local_per_pair);
    });
    return check_launch(fn);
}

}  // namespace exf

extern "C" int affinity_histogram(const int32_t* trace, int L, int64_t N, int E, int64_t* counts, int64_t* loads,
                                  float* cond_prob, int64_t* n_invalid, void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace exf;
    if (int rc = validate_trace_args("affinity_histogram", L, N, E)) return rc;
    if (N > 0) EXF_REQUIRE_PTR(trace);
    if (L > 1) EXF_REQUIRE_PTR(counts);
    EXF_REQUIRE_PTR(workspace);
    return run_affinity("affinity_histogram", trace, nullptr, L, N, E, counts, loads, cond_prob, n_invalid, nullptr, workspace,
                        workspace_bytes, stream);
}

extern "C" size_t affinity_statistics_workspace_bytes(int L, int64_t N, int E) { return affinity_histogram_workspace_bytes(L, N, E); }

extern "C" int affinity_statistics(const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int G, int64_t* counts,
                                   int64_t* loads, float* cond_prob, int64_t* n_invalid, int64_t* local_per_pair, void* workspace,
                                   size_t workspace_bytes, void* stream)
{
    using namespace exf;
    if (int rc = validate_trace_args("affinity_statistics", L, N, E)) return rc;
    if (G < 1) return fail(EXF_ERR_BAD_SHAPE, "affinity_statistics: G = %d < 1", G);
    if (N > 0) EXF_REQUIRE_PTR(trace);
    EXF_REQUIRE_PTR(placement);
    if (L > 1) {
        EXF_REQUIRE_PTR(counts);
        EXF_REQUIRE_PTR(local_per_pair);
    }
    EXF_REQUIRE_PTR(workspace);
    return run_affinity("affinity_statistics", trace, placement, L, N, E, counts, loads, cond_prob, n_invalid, local_per_pair,
                        workspace, workspace_bytes, stream);
}

namespace exf {
struct MultihopPlan {
    bool groups;  // multihop_group_kernel instead of blocks of four by four layers
    int blocks, Q, copies, copy_words, words, C, vec, pairs;
    int64_t chunk;
    size_t lds_bytes, total_bytes;
};
constexpr int kHopLdsBytes = 160 * 1024;
constexpr int kHopBanks = 64;
constexpr int64_t kHopMaxChunk = 65280;  // 16-bit counters cannot overflow; whole wavefronts of four tokens a lane
constexpr int64_t kHopMinChunk = 1024;
constexpr int64_t kHopPartialWords = 4 << 20;  // partials that are written and added up within a few microseconds
static size_t multihop_partial_bytes(const MultihopPlan& p)
{
    return align_up(static_cast<size_t>(p.C > 0 ? p.C : 1) * (p.pairs > 0 ? p.pairs : 1) * p.words * sizeof(uint32_t), 256);
}
// Groups of three pairs or blocks of sixteen: the blocks read fewer columns per pair and their workgroups clear and write far larger
// histograms, so they pay for long traces of many layers.  Where both take the same time, in millions of transitions (pairs times
// tokens), by layers and experts, measured at 4 to 24 layers x 8, 24, 40 and 64 experts x 2000 to 800000 tokens.  Groups and blocks, us:
// 4 x 300000, 64 experts 13.0 and 26.7; 8 x 100000, 64 experts 11.4 and 25.5; 12 x 150000, 8 experts 12.2 and 13.9; 12 x 250001, 8
// experts 19.3 and 15.8; 18 x 9787, 64 experts 17 and 24; 16 x 450000, 64 experts 40.8 and 38.3; 24 x 1000000, 64 experts 126 and 90.
static bool multihop_in_groups(int L, int64_t N, int E)
{
    if (N > kAffMaxChunk * kTargetWorkgroups) return false;  // (more chunks than the blocks cut, each with partials of its own)
    const double most = L <= 17 ? 8.0 + 0.32 * E : (L <= 19 ? 4.0 + 0.3 * E : (L <= 22 ? 0.6 * (E - 40) : 0.0));
    return 1e-6 * (0.5 * L * (L - 1)) * static_cast<double>(N) <= most;
}
static void plan_multihop_groups(MultihopPlan& p, int L, int64_t N)
{
    p.Q = 0;
    for (int l = 0; l + 1 < L; ++l) p.Q += (L - 2 - l) / kAffMaxGroup + 1;
    if (p.Q < 1) p.Q = 1;
    p.copies = 1;
    while (p.copies < 16 && sizeof(uint32_t) * p.words * kAffMaxGroup * (p.copies * 2) <= kAffHistBudget) p.copies *= 2;
    p.lds_bytes = sizeof(uint32_t) * p.words * kAffMaxGroup * p.copies;
    const int64_t sweep = static_cast<int64_t>(kTraceThreads) * p.vec;
    const int64_t c_target = kTargetWorkgroups / p.Q > 1 ? kTargetWorkgroups / p.Q : 1;
    p.chunk = ((N + c_target - 1) / c_target + sweep - 1) / sweep * sweep;
    if (p.chunk < sweep) p.chunk = sweep;
    if (p.chunk > kAffMaxChunk) p.chunk = kAffMaxChunk / sweep * sweep;
    p.C = static_cast<int>(N > 0 ? (N + p.chunk - 1) / p.chunk : 0);
    p.total_bytes = multihop_partial_bytes(p);
}
static MultihopPlan make_multihop_plan(int L, int64_t N, int E)
{
    MultihopPlan p{};
    p.pairs = L * (L - 1) / 2;
    p.words = (E * ((E + 1) / 2) + 1) / 2 * 2;
    p.vec = trace_vec(N);
    p.groups = multihop_in_groups(L, N, E);
    if (p.groups) {
        plan_multihop_groups(p, L, N);
        return p;
    }
    p.blocks = (L + kHopBlock - 1) / kHopBlock;
    const int cross = p.blocks * (p.blocks - 1) / 2;
    p.Q = cross + (p.blocks < kHopShareBlocks ? p.blocks : 0);
    int slots = p.blocks >= 8 ? kHopBlock * kHopBlock + 2 : 1;  // (at least seven partners: one inside pair of each block)
    for (int q = 0; q < p.Q && p.blocks < 8; ++q) {
        int I, J;
        hop_blocks(q, p.blocks, I, J);
        const int inside = __builtin_popcount(hop_inside_mask(I, J, p.blocks, L)) + (I == J ? 0 : __builtin_popcount(hop_inside_mask(J, I, p.blocks, L)));
        const int need = inside + (I == J ? 0 : kHopBlock * kHopBlock);
        if (need > slots) slots = need;
    }
    // replicas of small histograms, so that hot bins do not serialise, each beginning on the LDS banks after the previous one's
    p.copy_words = slots * p.words;
    if (p.words < kHopBanks) p.copy_words += ((p.words - p.copy_words) % kHopBanks + kHopBanks) % kHopBanks;
    p.copies = 1;
    while (p.copies < 32 && p.copy_words * 4 * (p.copies * 2) <= kHopLdsBytes / 2) p.copies *= 2;
    p.lds_bytes = static_cast<size_t>(p.copy_words) * p.copies * sizeof(uint32_t);
    // As few chunks as the counters allow (each costs a pass over its histograms), but a whole number of rounds of one workgroup
    // per compute unit
    int64_t c_least = (N + kHopMaxChunk - 1) / kHopMaxChunk;
    if (c_least < 1) c_least = 1;
    const int64_t rounds = (c_least * p.Q + kTargetWorkgroups - 1) / kTargetWorkgroups;
    int64_t c_target = rounds * kTargetWorkgroups / p.Q;
    // (two tokens a counter word at least, or clearing and writing the histograms takes longer than filling them - unless these are few)
    const int64_t few = kHopPartialWords / (static_cast<int64_t>(p.pairs > 0 ? p.pairs : 1) * p.words);
    int64_t c_most = N / (2 * p.words) > few ? N / (2 * p.words) : few;
    if (c_most > N / kHopMinChunk) c_most = N / kHopMinChunk;
    if (c_target > c_most) c_target = c_most;
    if (c_target < c_least) c_target = c_least;
    p.chunk = ((N + c_target - 1) / c_target + 255) / 256 * 256;  // (a wavefront cut by the end of its chunk takes the checked path)
    if (p.chunk < 256) p.chunk = 256;
    p.C = static_cast<int>(N > 0 ? (N + p.chunk - 1) / p.chunk : 0);
    p.total_bytes = multihop_partial_bytes(p);
    return p;
}
}  // namespace exf

extern "C" size_t affinity_multihop_workspace_bytes(int L, int64_t N, int E)
{
    if (L < 1 || N < 0 || E < 1 || E > EXF_MAX_EXPERTS) return 0;
    return exf::make_multihop_plan(L, N, E).total_bytes;
}

extern "C" int affinity_multihop(const int32_t* trace, int L, int64_t N, int E, int64_t* counts, float* cond_prob, void* workspace,
                                 size_t workspace_bytes, void* stream)
{
    using namespace exf;
    if (int rc = validate_trace_args("affinity_multihop", L, N, E)) return rc;
    if (L == 1) return EXF_OK;  // no pair, no output element
    if (N > 0) EXF_REQUIRE_PTR(trace);
    EXF_REQUIRE_PTR(counts);
    EXF_REQUIRE_PTR(workspace);
    const MultihopPlan p = make_multihop_plan(L, N, E);
    if (workspace_bytes < p.total_bytes)
        return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "affinity_multihop: workspace %zu < %zu bytes", workspace_bytes, p.total_bytes);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (multihop_direct(trace, L, N, E, counts, cond_prob, s)) return check_launch("affinity_multihop");
    uint32_t* part_counts = static_cast<uint32_t*>(workspace);
    if (p.C > 0 && p.groups) {
        const int64_t grid = xcd_items_grid(p.C, p.Q);
        if (grid >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "affinity_multihop: too many workgroups");
        auto kern = p.vec == 4 ? multihop_group_kernel<4> : multihop_group_kernel<1>;
        hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(kTraceThreads), p.lds_bytes, s, trace, L, N, E, p.Q, p.copies, p.words,
                           p.chunk, p.C, part_counts);
    } else if (p.C > 0) {
        const int64_t grid = xcd_items_grid(p.C, p.Q);
        if (grid >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "affinity_multihop: too many workgroups");
        auto kern = p.vec == 4 ? multihop_partial_kernel<4> : multihop_partial_kernel<1>;
        static std::atomic<uint64_t> allowed4{0}, allowed1{0};
        if (int rc = allow_lds(reinterpret_cast<const void*>(kern), kHopLdsBytes, p.vec == 4 ? allowed4 : allowed1, "affinity_multihop")) return rc;
        hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(kHopThreads), p.lds_bytes, s, trace, L, N, E, p.blocks, p.Q,
                           p.copies, p.copy_words, p.words, p.chunk, p.C, part_counts);
    }
    const int64_t fin_grid = (static_cast<int64_t>(p.pairs) * E + 256 / 32 - 1) / (256 / 32);
    with_chunks_ahead(p.C, static_cast<int64_t>(p.pairs) * E, [&](auto ahead) {
        hipLaunchKernelGGL(multihop_finalize_kernel<decltype(ahead)::value>, dim3(static_cast<unsigned>(fin_grid)), dim3(256), 0, s, part_counts, p.C, p.pairs, E,
                           p.words, counts, cond_prob);
    });
    return check_launch("affinity_multihop");
}

extern "C" size_t placement_locality_workspace_bytes(int L, int64_t N)
{
    if (L < 1 || N < 0) return 0;
    const int C = exf::locality_plan(N).C;
    return exf::align_up(static_cast<size_t>(C > 0 ? C : 1) * static_cast<size_t>(L > 1 ? L - 1 : 1) * sizeof(uint32_t), 256);
}

extern "C" int placement_locality(const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int G,
                                  int64_t* local_per_pair, void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace exf;
    if (int rc = validate_trace_args("placement_locality", L, N, E)) return rc;
    if (G < 1) return fail(EXF_ERR_BAD_SHAPE, "placement_locality: G = %d < 1", G);
    if (L == 1) return EXF_OK;  // no transition, no output element
    EXF_REQUIRE_PTR(placement);
    EXF_REQUIRE_PTR(local_per_pair);
    EXF_REQUIRE_PTR(workspace);
    if (N > 0) EXF_REQUIRE_PTR(trace);
    if (workspace_bytes < placement_locality_workspace_bytes(L, N))
        return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "placement_locality: workspace %zu < %zu bytes", workspace_bytes,
                    placement_locality_workspace_bytes(L, N));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (locality_direct(trace, placement, nullptr, L, N, E, local_per_pair, nullptr, s)) return check_launch("placement_locality");
    const LocalityPlan p = locality_plan(N);
    const int C = p.C;
    uint32_t* part = static_cast<uint32_t*>(workspace);
    if (C > 0) {
        const int rc = p.vec == 4 ? launch_locality<4, false>("placement_locality", p, trace, placement, nullptr, L, N, E, part, s)
                                  : launch_locality<1, false>("placement_locality", p, trace, placement, nullptr, L, N, E, part, s);
        if (rc != EXF_OK) return rc;
    }
    hipLaunchKernelGGL(locality_finalize_kernel, dim3(L - 1), dim3(kWave), 0, s, part, C, L - 1, L - 1, local_per_pair, nullptr);
    return check_launch("placement_locality");
}

extern "C" size_t routing_transfers_workspace_bytes(int L, int64_t N)
{
    if (L < 1 || N < 0) return 0;
    const int C = exf::locality_plan(N).C;
    return exf::align_up(static_cast<size_t>(C > 0 ? C : 1) * static_cast<size_t>(2 * L - 1) * sizeof(uint32_t), 256);
}

extern "C" int routing_transfers(const int32_t* trace, const int32_t* placement, const int32_t* home, int L, int64_t N, int E, int G,
                                 int64_t* local_per_pair, int64_t* away_per_layer, void* workspace, size_t workspace_bytes,
                                 void* stream)
{
    using namespace exf;
    if (int rc = validate_trace_args("routing_transfers", L, N, E)) return rc;
    if (G < 1) return fail(EXF_ERR_BAD_SHAPE, "routing_transfers: G = %d < 1", G);
    EXF_REQUIRE_PTR(placement);
    EXF_REQUIRE_PTR(away_per_layer);
    if (L > 1) EXF_REQUIRE_PTR(local_per_pair);
    EXF_REQUIRE_PTR(workspace);
    if (N > 0) {
        EXF_REQUIRE_PTR(trace);
        EXF_REQUIRE_PTR(home);
    }
    if (workspace_bytes < routing_transfers_workspace_bytes(L, N))
        return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "routing_transfers: workspace %zu < %zu bytes", workspace_bytes,
                    routing_transfers_workspace_bytes(L, N));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (locality_direct(trace, placement, home, L, N, E, local_per_pair, away_per_layer, s)) return check_launch("routing_transfers");
    const LocalityPlan p = locality_plan(N);
    const int C = p.C;
    uint32_t* part = static_cast<uint32_t*>(workspace);
    const int n_out = 2 * L - 1;
    if (C > 0) {
        const int rc = p.vec == 4 ? launch_locality<4, true>("routing_transfers", p, trace, placement, home, L, N, E, part, s)
                                  : launch_locality<1, true>("routing_transfers", p, trace, placement, home, L, N, E, part, s);
        if (rc != EXF_OK) return rc;
    }
    hipLaunchKernelGGL(locality_finalize_kernel, dim3(n_out), dim3(kWave), 0, s, part, C, L - 1, n_out, local_per_pair, away_per_layer);
    return check_launch("routing_transfers");
}
