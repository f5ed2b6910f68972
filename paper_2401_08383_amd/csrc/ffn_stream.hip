// Grouped expert GEMM for few rows per expert (bf16), and for any number of rows in fp32.
//
// bf16: with a handful of rows per expert the contraction is a stream of weights (r rows: r flop per weight byte;
// HBM and the matrix cores balance at about 270).  What counts is how many bytes are in flight on every compute
// unit all the time, not operand reuse:
//   - 256 persistent workgroups (one per compute unit), each with a contiguous range of the work items (expert, row tile of
//     at most 64 rows, block of 8 to 64 columns), all ranges of about the same cost.  The blocks of one row tile are one continuous stream: the loads
//     of the next block are in flight while the current one is summed and stored.
//   - the W wavefronts of a workgroup deal the 128-byte pieces ("units") of the reduction among themselves
//     (wavefront w takes units w, w + W, ..: neighbouring lines of a row are requested at the same time) and add
//     their sums through LDS once per block.
//   - every wavefront owns a ring of R slots in LDS and fills it with direct-to-LDS loads, eight rows of 128 bytes
//     per load.  Nobody else reads its slots, so no barrier is needed between units, only its own count of
//     outstanding loads.  (Loading the operands straight into registers in the lane layout of the matrix cores makes
//     every load touch 64 pieces of 16 bytes: 5.3 TB/s where this streams 6.4.)
//   - the slot of a block's last unit is free until the block is stored: it carries the sums (at most eight rows have a place of
//     their own for them).
//   - the weights are read once: loaded with the streaming hint they leave the L2 to the activations (64 experts of
//     4096 x 16384, 256 tokens top-2, both contractions: 3.08 ms without, 2.66 with, 2.89 as 64-row tiles of ffn_tiles.hpp).
//   - row ids and gate weights travel through LDS as well, so that no load result is awaited through a register (the
//     compiler would wait for every load in flight).
// fp32 (the exact path, small layers): operands straight from global memory into registers, no LDS but for the sums.
#include <cmath>

#include "ffn_common.hpp"
#include "gate_tile.hpp"

#include <type_traits>

namespace exf {

// ---------------------------------------------------------------------------- shared
// The sorted copy of the operand rows, sorted row s by workgroup s % gridDim.x (list[s] / a_div: its row): behind everything else, where
// the loads of nothing wait for it.
template <int THREADS, typename ST>
__device__ __forceinline__ void copy_sorted_rows(const StreamGemm& p, const int* list, int kept, int a_div)
{
    const int vec_per_row = p.K * static_cast<int>(sizeof(ST)) / 16;
    for (int s = static_cast<int>(blockIdx.x); s < kept; s += static_cast<int>(gridDim.x)) {
        int row = list[s];
        if (a_div > 1) row = static_cast<int>(static_cast<unsigned>(row) / static_cast<unsigned>(a_div));
        const uint4* from = reinterpret_cast<const uint4*>(p.act) + static_cast<size_t>(row) * vec_per_row;
        uint4* to = reinterpret_cast<uint4*>(p.sorted_act) + static_cast<size_t>(s) * vec_per_row;
        for (int c = threadIdx.x; c < vec_per_row; c += THREADS) to[c] = from[c];
    }
}

// The two rows of a token of a top-2 layer come from different workgroups of the second contraction.  Eight bytes of either (four bf16, two
// floats) meet in a word of p.exchange: an atomic exchange puts a row's there and returns what was; who gets kNoRow came first and leaves,
// who gets the other row's bytes adds both up, in the order of the combine.  Nobody waits and the data travel inside the atomics, so no
// store has to be made visible to another XCD's L2.  The launch of the combine is gone.
//   kNoRow is eight bytes of NaN: a row with these leaves others.  (fp32 rows do have them, where a weight has every bit set; the bf16 conversion makes
// 0xffc0 of such a NaN, so that no bf16 row is known to.)
constexpr unsigned long long kRowOfNans = 0x7fff7fff7fff7fffull;
__host__ __device__ constexpr unsigned long long word_of_row(unsigned long long mine) { return mine == kNoRow ? kRowOfNans : mine; }
static_assert(word_of_row(kNoRow) != kNoRow && word_of_row(~1ull) == ~1ull && word_of_row(0) == 0, "only the word that stands for no row is another one");
__device__ __forceinline__ unsigned long long meet(unsigned long long* word, unsigned long long mine)
{
    return __hip_atomic_exchange(word, word_of_row(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// By the first contraction, behind everything else.
template <int THREADS, typename ST>
__device__ __forceinline__ void clear_exchange(const StreamGemm& p)
{
    const uint32_t none = static_cast<uint32_t>(kNoRow);
    const int64_t vecs = static_cast<int64_t>(p.max_rows / 2) * (p.K * static_cast<int>(sizeof(ST)) / 16);
    for (int64_t i = blockIdx.x * THREADS + threadIdx.x; i < vecs; i += gridDim.x * THREADS)
        reinterpret_cast<uint4*>(p.exchange)[i] = make_uint4(none, none, none, none);
}

// The stable counting sort of moe_dispatch for at most kInlineDispatchMax assignments, by one workgroup into LDS.  Loading
// the ids costs the same memory round trip as loading finished offsets would, and the sort itself about a third of
// the launch it replaces.  Segments (round, wavefront) are ascending assignment order.
// offs[e]: first sorted position of expert e, offs[E_local] = number kept; list[s]: assignment at position s.
constexpr int kInlineSegments = kInlineDispatchMax / kWave;
struct InlineDispatch {
    int list[kInlineDispatchMax];
    int offs[EXF_MAX_EXPERTS + 1];
    unsigned short seg[kInlineSegments][EXF_MAX_EXPERTS];  // count, then start inside its expert's bucket
};
// each(a, dropped): of every assignment and, to fill its wavefront, of some past the end (not dropped), by all lanes of the wavefront that has it.
template <int THREADS, typename Each>
__device__ __forceinline__ void sort_assignments(const StreamGemm& p, InlineDispatch& d, bool publish, Each each)
{
    constexpr int WAVES = THREADS / kWave, R = kInlineDispatchMax / THREADS;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int A = p.max_rows, rounds = (A + THREADS - 1) / THREADS;
    int e[R], rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) e[r] = p.topk_idx[min(r * THREADS + static_cast<int>(threadIdx.x), A - 1)];
    for (int i = threadIdx.x; i < rounds * WAVES * (EXF_MAX_EXPERTS / 2); i += THREADS) reinterpret_cast<uint32_t*>(d.seg)[i] = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool ok = r * THREADS + static_cast<int>(threadIdx.x) < A && e[r] >= 0 && e[r] < p.E;
        int local = e[r];
        if (p.expert_map != nullptr) local = p.expert_map[ok ? e[r] : 0];
        e[r] = (ok && local >= 0 && local < p.E_local) ? local : -1;
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= rounds) break;
        const unsigned long long m = same_expert_lanes(e[r], p.E_local);
        rank[r] = __popcll(m & below);
        if (e[r] >= 0 && (m & below) == 0ull) d.seg[r * WAVES + wave][e[r]] = static_cast<unsigned short>(__popcll(m));
    }
    __syncthreads();
    if (wave == 0) {  // lane = expert
        int run = 0;
        constexpr int AHEAD = kInlineSegments < 8 ? kInlineSegments : 8;  // segments read together: they do not wait for one another's store
        for (int s0 = 0; s0 < rounds * WAVES; s0 += AHEAD) {
            int c[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) c[i] = d.seg[min(s0 + i, kInlineSegments - 1)][lane];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (s0 + i >= rounds * WAVES) break;
                d.seg[s0 + i][lane] = static_cast<unsigned short>(run);
                run += c[i];
            }
        }
        const int incl = wave_inclusive_scan(run);
        d.offs[lane] = incl - run;
        if (lane == kWave - 1) d.offs[kWave] = incl;
        if (publish) {
            if (lane < p.E_local) {
                p.expert_counts[lane] = run;
                p.expert_offsets[lane] = incl - run;
            }
            if (lane == p.E_local - 1) p.expert_offsets[p.E_local] = incl;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= rounds) break;
        const int a = r * THREADS + static_cast<int>(threadIdx.x);
        int pos = -1;
        if (e[r] >= 0) {
            pos = d.offs[e[r]] + d.seg[r * WAVES + wave][e[r]] + rank[r];
            d.list[pos] = a;
            if (publish) p.src_of_sorted[pos] = a;
        }
        if (publish && a < A) p.sorted_of_src[a] = pos;
        each(a, a < A && pos < 0);
    }
    __syncthreads();
}

// Row ranges and row tiles of the experts (lane e = expert e), running sum and total of the tiles.
struct ExpertTiles {
    int lo, hi, tiles, incl, total;
};
__device__ __forceinline__ void count_tiles(ExpertTiles& t, int tile_rows)
{
    t.tiles = (t.hi - t.lo + tile_rows - 1) / tile_rows;
    t.incl = wave_inclusive_scan(t.tiles);
    t.total = wave_read_lane(t.incl, kWave - 1);
}
__device__ __forceinline__ ExpertTiles scan_row_tiles(const StreamGemm& p, const int32_t* offsets, int tile_rows)
{
    ExpertTiles t;
    const int lane = lane_id();
    t.lo = 0;
    t.hi = 0;
    if (lane < p.E_local) {  // clamped so that a corrupt offsets array can never index past the buffers
        t.lo = min(max(offsets[lane], 0), p.max_rows);
        t.hi = min(max(offsets[lane + 1], t.lo), p.max_rows);
    }
    count_tiles(t, tile_rows);
    return t;
}

// Sorting at most kFewAssignments: lane = assignment, every wavefront for itself, no barrier and no memory but the ids and the
// expert map, which are asked for together (with the output rows' gate weights in the second contraction).  sorted[s]: token at
// position s; in the second contraction of a top-1 layer the gate weight of position s at sorted[64 + s].  Neither contraction then
// waits for maps in memory, which themselves wait for offsets.
// The gate of at most 16 tokens joins in (first contraction, p.w_gate): each workgroup needs its result anyway, and computing it in all
// of them takes 1.9 us where its own launch, of one workgroup, took 3.1 and the gap behind it.  These kernels are chains of
// instructions and memory round trips (a wavefront issues one instruction in about five cycles), so what a launch of at most
// eight rows does not need is compiled out (EIGHT).  One token, 8 experts of 1024 x 4096: 15.2 us in three launches, 12.2 in
// two; one GPU's 2 of 8 experts with the routing given 15.6 and 12.1; 16 tokens, 8 experts 32.1 and 29.7.
template <int W, int LDS, bool EIGHT, bool SECOND, bool PAIRS>
__device__ __forceinline__ ExpertTiles route_few(const StreamGemm& p, unsigned char* smem, int* sorted, int tile_rows)
{
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int A = p.max_rows;
    const int at = min(lane, A - 1);
    const bool gated = !SECOND && p.w_gate != nullptr && (blockIdx.x == 0 || p.topk_idx == p.gate_idx);  // (the same in all wavefronts)
    const int local_of = p.expert_map != nullptr ? p.expert_map[min(lane, p.E - 1)] : lane;  // lane = expert
    int id = 0;
    if (SECOND || p.w_gate == nullptr || p.topk_idx != p.gate_idx) id = p.topk_idx[at];
    float scale = 1.0f;
    if (SECOND && p.out_row != nullptr) scale = p.out_scale[at];
    float mate_scale = 0.0f;
    if constexpr (PAIRS) mate_scale = p.out_scale[at ^ 1];
    if (gated) {
        const int T = A / p.k;
        Route r;
        auto gate = [&](auto nt, auto sums) {
            constexpr int NT = decltype(nt)::value, P = decltype(sums)::value;
            r = gate_few<NT, P, W, LDS>(p.act, p.w_gate, T, p.K, p.E, p.k, p.renormalize, smem);
        };
        const int nt = (p.E + 15) / 16;
        const bool eight = gate_sums(nt, p.K) == 8;
        typedef std::integral_constant<int, 4> Four;
        typedef std::integral_constant<int, 8> Eight;
        if (nt == 1 && eight) gate(std::integral_constant<int, 1>(), Eight());
        else if (nt == 1) gate(std::integral_constant<int, 1>(), Four());
        else if (nt == 2 && eight) gate(std::integral_constant<int, 2>(), Eight());
        else if (nt == 2) gate(std::integral_constant<int, 2>(), Four());
        else if (nt == 3) gate(std::integral_constant<int, 3>(), Four());
        else gate(std::integral_constant<int, 4>(), Four());
        const int first = __shfl(r.i0, p.k == 1 ? lane : lane >> 1, kWave), second = __shfl(r.i1, lane >> 1, kWave);
        const int mine = p.k == 1 || (lane & 1) == 0 ? first : second;
        if (p.topk_idx == p.gate_idx) id = mine;
        if (blockIdx.x == 0 && wave == 0 && lane < T) store_route(r, lane, p.k, p.gate_idx, p.gate_w);
    }
    const bool ok = lane < A && id >= 0 && id < p.E;
    int e = __shfl(local_of, ok ? id : 0, kWave);
    e = ok && e >= 0 && e < p.E_local ? e : -1;
    int pos = 0, below = 0, count = 0;  // (the last two: lane = expert)
    if (A <= 4) {
        for (int b = 0; b < A; ++b) {
            const int other = wave_read_lane(e, b);
            if (other < 0) continue;
            pos += other < e || (other == e && b < lane) ? 1 : 0;
            below += other < lane ? 1 : 0;
            count += other == lane ? 1 : 0;
        }
    } else {
        // assignments of this one's expert; its first one tells the expert's lane how many (`sorted` is scratch so far)
        const unsigned long long like = same_expert_lanes(e, p.E_local);
        sorted[lane] = 0;
        __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS accesses are done in order)
        const int rank = static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(like >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(like), 0u)));
        if (e >= 0 && rank == 0) sorted[e] = __popcll(like);
        __builtin_amdgcn_wave_barrier();
        count = sorted[lane];
        below = wave_inclusive_scan(count) - count;
        pos = __shfl(below, max(e, 0), kWave) + rank;
        __builtin_amdgcn_wave_barrier();
    }
    if (e >= 0) {
        sorted[pos] = p.k == 2 && !PAIRS ? lane >> 1 : lane;
        if (SECOND) reinterpret_cast<float*>(sorted)[kWave + pos] = scale;
    }
    const int mate = PAIRS ? __shfl_xor(e, 1, kWave) : -1;  // local expert of the token's other assignment
    if (PAIRS && e >= 0) {
        reinterpret_cast<float*>(sorted)[2 * kWave + pos] = mate_scale;
        sorted[3 * kWave + pos] = mate;
    }
    if (!SECOND && blockIdx.x == 0 && wave == 0) {
        if (lane < p.E_local) {
            p.expert_counts[lane] = count;
            p.expert_offsets[lane] = below;
        }
        if (lane == p.E_local - 1) p.expert_offsets[p.E_local] = below + count;
        if (lane < A) p.sorted_of_src[lane] = e >= 0 ? pos : -1;
        if (e >= 0) p.src_of_sorted[pos] = lane;
    }
    if (SECOND && p.unrouted != nullptr) {  // output rows nobody writes, dealt to the workgroups
        unsigned long long todo = __ballot(lane < A && e < 0 && mate < 0 && !(PAIRS && (lane & 1) != 0));
        for (int n = 0; todo != 0ull; ++n, todo &= todo - 1ull) {
            if (n != static_cast<int>(blockIdx.x)) continue;
            uint4* row = reinterpret_cast<uint4*>(p.out) + static_cast<size_t>(__builtin_ctzll(todo) >> (PAIRS ? 1 : 0)) * (p.N / 8);
            for (int c = threadIdx.x; c < p.N / 8; c += W * kWave) row[c] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    ExpertTiles t;
    t.lo = below;
    t.hi = below + count;
    if constexpr (EIGHT) {  // one tile an expert
        const unsigned long long some = __ballot(count > 0);
        t.tiles = count > 0 ? 1 : 0;
        t.incl = t.tiles + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(some >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(some), 0u)));
        t.total = __popcll(some);
    } else {
        count_tiles(t, tile_rows);
    }
    return t;
}

// ---------------------------------------------------------------------------- bf16
constexpr int kStreamGrid = 256;     // workgroups: one per compute unit
constexpr int kStreamIdBytes = 1024;  // per wavefront and row of a tile: its id, its gate weight, that of its token's other row, whether there is one
// C8: columns of a block / 8.  A row tile has at most 8 * stream_max_ar(C8) rows (narrow blocks have shorter tiles: the
// activations would fill the ring).
__host__ __device__ constexpr int stream_max_ar(int C8) { return C8 == 8 ? 8 : 4; }

// Ring slots of a wavefront for row tiles of 8 AR rows: what fits 144 KiB, at most eight (with four the second contraction of a single
// row, 8 units a wavefront, was two round trips to memory).
__host__ __device__ constexpr int stream_slot_bytes(int C8, int AR) { return (8 * C8 + 8 * AR) * 128; }
__host__ __device__ constexpr int stream_ring(int C8, int AR, int W)
{
    const int fit = 144 * 1024 / (W * stream_slot_bytes(C8, AR));
    return fit > 8 ? 8 : fit;
}
__host__ __device__ constexpr int stream_ring_bytes(int C8, int W)
{
    int most = 0;
    for (int ar = 1; ar <= stream_max_ar(C8); ar *= 2) {
        const int b = W * stream_ring(C8, ar, W) * stream_slot_bytes(C8, ar);
        most = b > most ? b : most;
    }
    return most;
}

// Sums of a block of eight rows of kRowsEight: behind the row ids.
__host__ __device__ constexpr int stream_sums_at(int C8, int W) { return stream_ring_bytes(C8, W) + W * kStreamIdBytes; }
__host__ __device__ constexpr int stream_sums_bytes(int C8) { return 8 * 8 * C8 * 4; }

// What a block of a row tile of 8 AR rows costs, in tenths of its weights: the activations are read again by every block and weigh
// more the more of the ring they take.  Dealing ranges of equal cost instead of equal numbers of blocks keeps the tall tiles of
// the experts that many tokens chose from being what the launch waits for, both contractions, rows falling on the experts as
// 1/rank^1.1: 290 rows, 57 experts of 1024 x 4096 180 us before, 144 now; 400 rows, 32 of 2048 x 8192 489 and 379; 655
// rows, 29 of 2560 x 10240 755 and 593 (64-row tiles of ffn_tiles.hpp: 164, 423, 557); evenly spread rows as before or up to 6 %
// less.  Coefficients of 3 and 5 instead of 4 give 601 and 586 there, but 290 instead of 284 with 5 for 128 rows, 8 of 4096 x 14336.
__host__ __device__ constexpr uint32_t stream_cost(int C8, int AR) { return static_cast<uint32_t>((10 * C8 + 8 * AR) / C8); }

// Waits until at most `units` units of LPU loads each are outstanding.
template <int LPU, int R>
__device__ __forceinline__ void wait_units(int units)
{
    static_assert((R - 1) * LPU < 64, "outstanding loads must fit the vmcnt counter");
    if constexpr (R <= 1) {
        wait_vmcnt<0>();
    } else {
        if (units >= R - 1) wait_vmcnt<(R - 1) * LPU>();
        else wait_units<LPU, R - 1>(units);
    }
}

// Where the rows of a contraction come from: sorted (maps in memory), sorted by the workgroup, sorted by every wavefront.
enum StreamRows { kRowsSorted, kRowsInline, kRowsFew, kRowsEight };  // (the last: as kRowsFew, at most eight)

// The sorted rows that are wanted besides the result: none, p.sorted_act (a contraction that sorts), p.sorted_out (one that scales).  Instances
// of their own: what a handful of rows does not need costs them 0.6 us of 12.
// The last: the two rows of a token meet in p.exchange (bf16: p.sorted_out as well if it is given; fp32 layers that keep their sorted rows have a combine).
enum StreamKeep { kKeepNone, kKeepAct, kKeepOut, kKeepPairs };

// Column blocks [block_begin, block_end) of one row tile (rows [row_begin, row_end), at most 8 AR).
template <int C8, int AR, int W, StreamKeep KEEP, StreamRows ROWS, bool SECOND>
__device__ __forceinline__ void stream_segment(const StreamGemm& p, int e, int row_begin, int row_end, int block_begin, int block_end,
                                               int rotate, const int* list, unsigned char* smem)
{
    constexpr bool KEEP_OUT = KEEP == kKeepOut, PAIRS = KEEP == kKeepPairs;
    constexpr bool FEW_ROWS = ROWS == kRowsEight, FEW = FEW_ROWS || ROWS == kRowsFew;  // FEW: `list` holds tokens, not assignments
    const bool listed_out = FEW && SECOND && p.out_row != nullptr;
    constexpr int C = (C8 + 1) / 2, M = (AR + 1) / 2;  // MFMA tiles along the columns and the rows (eight of either are read twice)
    constexpr int R = stream_ring(C8, AR, W);
    constexpr int SLOT = stream_slot_bytes(C8, AR);
    constexpr int LW = C8, LA = AR, LPU = LW + LA;  // loads of a unit: eight rows each
    constexpr int COLS = 8 * C8, QUADS = 2 * C8;     // columns of a block, and fours of them
    constexpr int STEP = AR == 1 && C8 == 1 ? 4 : (AR == 1 && C8 == 2 ? 2 : 1);  // units read at once: a few rows wait for the LDS, unit by unit
    static_assert(STEP < R, "loads go on while a step is read");
    static_assert(R >= 2, "a ring of one slot cannot overlap anything");
    static_assert(8 * AR * COLS * 4 <= SLOT, "a block's sums must fit the slot of its last unit");
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t smem_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem));
    const uint32_t ring_addr = smem_addr + wave * (R * SLOT);
    unsigned char* ring = smem + wave * (R * SLOT);
    constexpr int kIds = stream_ring_bytes(C8, W);
    const uint32_t ids_addr = smem_addr + kIds + wave * kStreamIdBytes;
    // output rows and their gate weights: of the tile, or of all sorted rows (listed_out)
    const int* ids = reinterpret_cast<const int*>(smem + kIds + wave * kStreamIdBytes) + (listed_out ? row_begin : 0);
    const float* gate = reinterpret_cast<const float*>(ids + kWave);
    const uint32_t row_bytes = static_cast<uint32_t>(p.K) * 2u;

    const int units = static_cast<int>(static_cast<unsigned>(p.K) / 64u);
    const int cnt = static_cast<int>(static_cast<unsigned>(max(units - wave + W - 1, 0)) / W);  // units of a block this wavefront sums
    const int total = (block_end - block_begin) * cnt;
    const int start = cnt == 0 ? 0 : ((cnt & (cnt - 1)) == 0 ? rotate & (cnt - 1) : rotate % cnt);  // the unit a block begins with (see stream_gemm_kernel)

    // LDS row r of a slot (8 C8 weight rows, then 8 AR activation rows) holds 16-byte piece c at position c ^ ((r / 2) % 8)
    const int r8 = lane >> 3, c8 = lane & 7;
    const uint32_t off_even = static_cast<uint32_t>(r8) * row_bytes + ((c8 ^ (r8 >> 1)) * 16);      // rows 8 i + r8, i even
    const uint32_t off_odd = static_cast<uint32_t>(r8) * row_bytes + ((c8 ^ (r8 >> 1) ^ 4) * 16);   //   i odd
    const unsigned char* w_block = uniform_ptr(static_cast<const unsigned char*>(p.weight) +
                                               (static_cast<size_t>(e) * p.N + static_cast<size_t>(block_begin) * COLS) * row_bytes);
    const unsigned char* act = uniform_ptr(static_cast<const unsigned char*>(p.act));
    const size_t block_bytes = static_cast<size_t>(COLS) * row_bytes;

    auto issue_w = [&](int slot, int u) {
        const int at = u + start < cnt ? u + start : u + start - cnt;
        const unsigned char* base = w_block + static_cast<size_t>(wave + at * W) * 128;
#pragma unroll
        for (int i = 0; i < LW; ++i)
            lds_dma_16B_stream(base + static_cast<size_t>(i * 8) * row_bytes, (i & 1) ? off_odd : off_even, ring_addr + slot * SLOT + i * 1024);
    };
    uint32_t off_a[LA];
    auto issue_a = [&](int slot, int u) {
        const int at = u + start < cnt ? u + start : u + start - cnt;
        const unsigned char* base = act + static_cast<size_t>(wave + at * W) * 128;
#pragma unroll
        for (int i = 0; i < LA; ++i) lds_dma_16B(base, off_a[i], ring_addr + slot * SLOT + (LW + i) * 1024);
    };

    // ---- start: row ids, the weights of the first units, then (ids known) their activations -------------------
    const int32_t* id_list = FEW || ROWS == kRowsInline ? nullptr : (SECOND ? p.out_row : p.a_row);
    const bool known = id_list == nullptr;  // no row ids to wait for: units are asked for whole, as later on
    auto place_rows = [&]() {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int r = i * 8 + r8;
            int row = min(row_begin + r, row_end - 1);  // rows past the end repeat the last one
            if (ROWS == kRowsInline || (FEW && !SECOND)) row = list[row];
            else if (ROWS == kRowsSorted && !SECOND && p.a_row != nullptr) row = ids[r];
            if (!FEW && !SECOND && p.a_div > 1) row = static_cast<int>(static_cast<unsigned>(row) / static_cast<unsigned>(p.a_div));
            off_a[i] = static_cast<uint32_t>(row) * row_bytes + ((c8 ^ ((r >> 1) & 7)) * 16);
        }
    };
    if (known) place_rows();
    const int first = min(total, R);
    if (!known)
        lds_dma_4B(uniform_ptr(reinterpret_cast<const unsigned char*>(id_list)), static_cast<uint32_t>(min(row_begin + lane, row_end - 1)) * 4u, ids_addr);
    int next_u = 0, next_slot = 0;  // the unit of the block at w_block, and the slot, the next load goes to
    int q_issued = 0;
    int u_of[R];
#pragma unroll
    for (int s = 0; s < R; ++s) {
        u_of[s] = 0;
        if (s < first) {
            issue_w(s, next_u);
            if (known) issue_a(s, next_u);
            u_of[s] = next_u;
            next_u += 1;
            q_issued += 1;
            if (next_u == cnt) {
                next_u = 0;
                w_block += block_bytes;
            }
        }
    }
    next_slot = first == R ? 0 : first;
    if (!known) {  // loads land in order: the ids are there once only the weights are outstanding
        wait_units<LW, R + 1>(first);
    }
    if (!known) place_rows();
    if (!FEW && SECOND && p.out_row != nullptr) lds_dma_4B(uniform_ptr(reinterpret_cast<const unsigned char*>(p.out_scale)), static_cast<uint32_t>(ids[lane]) * 4u, ids_addr + 256);
    if constexpr (!FEW && PAIRS) {
        lds_dma_4B(uniform_ptr(reinterpret_cast<const unsigned char*>(p.out_scale)), static_cast<uint32_t>(ids[lane] ^ 1) * 4u, ids_addr + 512);
        lds_dma_4B(uniform_ptr(reinterpret_cast<const unsigned char*>(p.unrouted)), static_cast<uint32_t>(ids[lane] ^ 1) * 4u, ids_addr + 768);
    }
    if (!known) {
#pragma unroll
        for (int s = 0; s < R; ++s)
            if (s < first) issue_a(s, u_of[s]);
        wait_vmcnt<0>();
    }

    // ---- stream -----------------------------------------------------------------------------------------------
    const int r16 = lane & 15, g = lane >> 4;
    const int rw = C8 == 1 ? r16 & 7 : r16, ra = AR == 1 ? r16 & 7 : r16;  // eight rows have no second half: read it twice
    int frag[2], frag_a[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        frag[h] = rw * 128 + (((4 * h + g) ^ (rw >> 1)) * 16);
        frag_a[h] = LW * 1024 + ra * 128 + (((4 * h + g) ^ (ra >> 1)) * 16);
    }
    auto refill = [&]() {
        if (q_issued < total) {
            issue_w(next_slot, next_u);
            issue_a(next_slot, next_u);
            q_issued += 1;
            next_u += 1;
            if (next_u == cnt) {
                next_u = 0;
                w_block += block_bytes;
            }
            next_slot = next_slot + 1 == R ? 0 : next_slot + 1;
        }
    };
    const int cnt_hi = (units + W - 1) / W, w_hi = units - (cnt_hi - 1) * W;  // wavefronts below w_hi sum cnt_hi units, the others one less
    int last_hi = R - 1, last_lo = R - 1;  // ring position of the last unit of a block, for either kind of wavefront
    int slot = 0, q = 0;
    for (int block = block_begin; block < block_end; ++block) {
        f32x4_t acc[C][M];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int m = 0; m < M; ++m) acc[c][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int u = 0; u < cnt; u += STEP) {
            const int n = min(STEP, cnt - u);
            wait_units<LPU, R>(q_issued - q - n);
            bf16x8_t fw[STEP][C][2], fa[STEP][M][2];
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                if (i > 0 && i >= n) break;
                const unsigned char* s = ring + slot * SLOT;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int c = 0; c < C; ++c) fw[i][c][h] = *reinterpret_cast<const bf16x8_t*>(s + c * 2048 + frag[h]);
#pragma unroll
                    for (int m = 0; m < M; ++m) fa[i][m][h] = *reinterpret_cast<const bf16x8_t*>(s + m * 2048 + frag_a[h]);
                }
                slot = slot + 1 == R ? 0 : slot + 1;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slots have been read: they may be filled again
#pragma unroll
            for (int i = 0; i < STEP; ++i)
                if (FEW_ROWS ? i < n : u + i + 1 < cnt) refill();
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                if (i > 0 && i >= n) break;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < C; ++c)
#pragma unroll
                        for (int m = 0; m < M; ++m)
                            acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i][c][h], fa[i][m][h], acc[c][m], 0, 0, 0);
            }
            q += n;
        }
        // sums -> the slot of this block's last unit; float4 of row r, columns 4 j .. at position j ^ (r % QUADS)
        if constexpr (!FEW_ROWS) {
            last_hi = (last_hi + cnt_hi) % R;
            last_lo = (last_lo + cnt_hi - 1) % R;
        }
        {
            unsigned char* red = FEW_ROWS ? smem + stream_sums_at(C8, W) + wave * stream_sums_bytes(C8) : ring + (wave < w_hi ? last_hi : last_lo) * SLOT;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int r = m * 16 + r16, j = c * 4 + g;
                    if ((AR == 1 && r16 >= 8) || (C8 == 1 && g >= 2)) continue;
                    *reinterpret_cast<f32x4_t*>(red + (r * QUADS + (j ^ (r & (QUADS - 1)))) * 16) = acc[c][m];
                }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int n0 = block * COLS;
        for (int i = threadIdx.x; i < (row_end - row_begin) * QUADS; i += W * kWave) {
            const int r = i / QUADS, j = i % QUADS;
            const int at = (r * QUADS + (j ^ (r & (QUADS - 1)))) * 16;
            f32x4_t z = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w)
                z += *reinterpret_cast<const f32x4_t*>((FEW_ROWS ? smem + stream_sums_at(C8, W) + w * stream_sums_bytes(C8)
                                                                 : smem + w * (R * SLOT) + (w < w_hi ? last_hi : last_lo) * SLOT) +
                                                       at);
            int dst = row_begin + r;
            float scale = 1.0f;
            if (SECOND && p.out_row != nullptr) {
                dst = ids[r];
                scale = gate[r];
            }
            const int n = n0 + j * 4;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = z[k];
            if (p.bias != nullptr) {
                const bf16_t* bias = static_cast<const bf16_t*>(p.bias) + static_cast<size_t>(e) * p.N + n;
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] += bf16_to_f32(bias[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (!SECOND) v[k] = p.epi == kEpiGeluErf ? gelu_erf_fast(v[k]) : gelu_tanh_fast(v[k]);
                else if constexpr (!KEEP_OUT && !PAIRS) v[k] *= scale;
            }
            if constexpr (PAIRS) {
                const uint2 y = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                if (p.sorted_out != nullptr) *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.sorted_out) + static_cast<size_t>(row_begin + r) * p.N + n) = y;
                const bool second = (dst & 1) != 0, mated = ids[3 * kWave + r] >= 0;
                dst >>= 1;
                uint2 other = make_uint2(0u, 0u);
                if (mated) {
                    const unsigned long long got = meet(p.exchange + (static_cast<size_t>(dst) * p.N + n) / 4, static_cast<unsigned long long>(y.y) << 32 | y.x);
                    if (got == kNoRow) continue;  // the other row's thread finds this one
                    other = make_uint2(static_cast<uint32_t>(got), static_cast<uint32_t>(got >> 32));
                }
                const uint2 y0 = second ? other : y, y1 = second ? y : other;
                const float mate_scale = mated ? gate[kWave + r] : 0.0f, w0 = second ? mate_scale : scale, w1 = second ? scale : mate_scale;
                const uint32_t b0[2] = {y0.x, y0.y}, b1[2] = {y1.x, y1.y};
#pragma unroll
                for (int k = 0; k < 4; ++k) {  // (the combine's bits)
                    const uint32_t f0 = (k & 1) != 0 ? b0[k / 2] & 0xffff0000u : b0[k / 2] << 16, f1 = (k & 1) != 0 ? b1[k / 2] & 0xffff0000u : b1[k / 2] << 16;
                    v[k] = fmaf(w1, __uint_as_float(f1), fmaf(w0, __uint_as_float(f0), 0.0f));
                }
            }
            if constexpr (KEEP_OUT) {
                const uint2 y = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.sorted_out) + static_cast<size_t>(row_begin + r) * p.N + n) = y;
                const uint32_t w[4] = {y.x << 16, y.x & 0xffff0000u, y.y << 16, y.y & 0xffff0000u};
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = fmaf(scale, __uint_as_float(w[k]), 0.0f);  // (the combine's bits)
            }
            *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.out) + static_cast<size_t>(dst) * p.N + n) =
                make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();  // everybody has read the sums: the slots may be filled again
        asm volatile("" ::: "memory");
        if (!FEW_ROWS && cnt > 0) refill();
    }
}

// SECOND: a second contraction, which has no activation but may scale and scatter its rows.
template <int C8, int W, StreamRows ROWS, StreamKeep KEEP, bool SECOND>
__global__ __launch_bounds__(W * 64) void stream_gemm_kernel(const StreamGemm p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    touch_arguments<sizeof(StreamGemm)>();
    constexpr int MAX_AR = stream_max_ar(C8), TILE_ROWS = 8 * MAX_AR, COLS = 8 * C8;
    constexpr bool FEW = ROWS == kRowsFew || ROWS == kRowsEight;
    constexpr bool PAIRS = KEEP == kKeepPairs;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int* list = nullptr;
    ExpertTiles et;
    if constexpr (FEW) {
        int* sorted = reinterpret_cast<int*>(smem + stream_ring_bytes(C8, W) + wave * kStreamIdBytes);
        et = route_few<W, stream_ring_bytes(C8, W), ROWS == kRowsEight, SECOND, PAIRS>(p, smem, sorted, TILE_ROWS);
        list = sorted;
    } else {
        const int32_t* offsets = p.offsets;
        if constexpr (ROWS == kRowsInline) {
            InlineDispatch* d = reinterpret_cast<InlineDispatch*>(smem + stream_ring_bytes(C8, W) + W * kStreamIdBytes);
            sort_assignments<W * kWave>(p, *d, blockIdx.x == 0, [](int, bool) {});
            list = d->list;
            offsets = d->offs;
        }
        et = scan_row_tiles(p, offsets, TILE_ROWS);
        if (SECOND && p.unrouted != nullptr && wave_read_lane(et.hi, p.E_local - 1) < p.max_rows)  // (else every assignment is kept)
            clear_unrouted_rows<false, PAIRS>(p.unrouted, p.n_unrouted, static_cast<uint4*>(p.out), p.N / 8, W);
    }
    const uint32_t n_blocks = static_cast<uint32_t>(p.N / COLS);
    // Every workgroup begins its blocks at another place of the reduction: rows a power of two bytes apart put the same
    // columns of all rows on few memory channels, and workgroups that walk the reduction in step all ask these
    // (rows of 8 and 32 KiB, 256 workgroups: 5.3 and 4.8 TB/s in step, 6.1 rotated; rows of 4.5 KiB 6.0 either way).
    // items (expert, row tile, column block); consecutive workgroup ids are on different XCDs: an XCD's workgroups
    // take neighbouring ranges, so an expert's rows meet in one L2.  The ranges have the same number of blocks, or the same cost
    // where that is expected to end earlier: by the dearest block at most above the mean, against a whole number of dearest blocks.
    const int cnt = et.hi - et.lo;
    const uint32_t whole = static_cast<uint32_t>(cnt) / TILE_ROWS;
    const int rest = cnt - static_cast<int>(whole) * TILE_ROWS;
    constexpr uint32_t kWholeCost = stream_cost(C8, MAX_AR);
    uint32_t whole_cost = 1u, rest_cost = rest != 0 ? 1u : 0u, cost_incl = static_cast<uint32_t>(et.incl);  // cost of a block
    if (ROWS != kRowsEight && et.total > 1 && __ballot(cnt > 16) != 0ull) {  // (else all blocks cost nearly the same)
        const uint32_t c = rest == 0 ? 0u : (rest <= 8 ? stream_cost(C8, 1) : (rest <= 16 ? stream_cost(C8, 2) : (rest <= 32 ? stream_cost(C8, 4) : kWholeCost)));
        const uint32_t incl = static_cast<uint32_t>(wave_inclusive_scan(static_cast<int>(whole * kWholeCost + c)));
        const uint32_t dearest = __ballot(cnt > 32) != 0ull ? kWholeCost : stream_cost(C8, 4);
        const uint32_t even = (static_cast<uint32_t>(et.total) * n_blocks + kStreamGrid - 1) / kStreamGrid * dearest;
        const float all = static_cast<float>(wave_read_lane(static_cast<int>(incl), kWave - 1)) * static_cast<float>(n_blocks);
        if (all < 2e9f && all * (1.0f / kStreamGrid) + static_cast<float>(dearest) < static_cast<float>(even)) {  // (32-bit products below)
            whole_cost = kWholeCost;
            rest_cost = c;
            cost_incl = incl;
        }
    }
    const uint32_t cost = whole * whole_cost + rest_cost;
    const uint32_t total = static_cast<uint32_t>(ROWS == kRowsEight ? et.total : wave_read_lane(static_cast<int>(cost_incl), kWave - 1)) * n_blocks;
    constexpr int per_xcd = kStreamGrid / kXcdCount;
    const int lin = static_cast<int>(blockIdx.x % kXcdCount) * per_xcd + static_cast<int>(blockIdx.x / kXcdCount);
    // total * lin / kStreamGrid and the next one's begin, in 32 bits and scalar registers
    const uint32_t t_hi = __builtin_amdgcn_readfirstlane(total / kStreamGrid), t_lo = __builtin_amdgcn_readfirstlane(total % kStreamGrid);
    uint32_t at = __builtin_amdgcn_readfirstlane(t_hi * lin + t_lo * lin / kStreamGrid);
    const uint32_t end = __builtin_amdgcn_readfirstlane(t_hi * (lin + 1) + t_lo * (lin + 1) / kStreamGrid);
    while (at < end) {
        if constexpr (ROWS == kRowsEight) {  // an expert with rows has one tile
            const uint32_t t = uniform_udiv(at, n_blocks);
            const int e = __builtin_ctzll(__ballot(cnt > 0 && et.incl == static_cast<int>(t) + 1));
            const int row_begin = wave_read_lane(et.lo, e), row_end = wave_read_lane(et.hi, e);
            const int b0 = static_cast<int>(at - t * n_blocks);
            at = min(end, (t + 1) * n_blocks);
            stream_segment<C8, 1, W, KEEP, ROWS, SECOND>(p, e, row_begin, row_end, b0, static_cast<int>(at - t * n_blocks), lin, list, smem);
            continue;
        }
        const int e = __builtin_ctzll(__ballot(at < cost_incl * n_blocks));
        const uint32_t e_cost = static_cast<uint32_t>(wave_read_lane(static_cast<int>(cost), e));
        const uint32_t e_begin = (static_cast<uint32_t>(wave_read_lane(static_cast<int>(cost_incl), e)) - e_cost) * n_blocks;
        const uint32_t e_whole = static_cast<uint32_t>(wave_read_lane(static_cast<int>(whole), e));
        uint32_t tile = 0, c = whole_cost;
        if (e_whole != 0) tile = (at - e_begin) / (whole_cost * n_blocks);  // (a division by a run-time value takes a quarter of a microsecond)
        if (tile >= e_whole) {
            tile = e_whole;
            c = e_cost - e_whole * whole_cost;
        }
        const uint32_t tile_begin = e_begin + tile * whole_cost * n_blocks;
        // the blocks that begin inside the range
        uint32_t block = at - tile_begin, block_end = end - tile_begin;
        if (c != 1u) {
            block = (block + c - 1) / c;
            block_end = (block_end + c - 1) / c;
        }
        block_end = min(n_blocks, block_end);
        const int row_begin = __builtin_amdgcn_readfirstlane(wave_read_lane(et.lo, e) + static_cast<int>(tile) * TILE_ROWS);
        const int row_end = __builtin_amdgcn_readfirstlane(min(row_begin + TILE_ROWS, wave_read_lane(et.hi, e)));
        const int b0 = __builtin_amdgcn_readfirstlane(static_cast<int>(block)), b1 = __builtin_amdgcn_readfirstlane(static_cast<int>(block_end));
        at = __builtin_amdgcn_readfirstlane(tile_begin + c * n_blocks);
        if (b0 >= b1) continue;
        const int rows = row_end - row_begin;
        if (rows <= 8) stream_segment<C8, 1, W, KEEP, ROWS, SECOND>(p, e, row_begin, row_end, b0, b1, lin, list, smem);
        else if (rows <= 16) stream_segment<C8, 2, W, KEEP, ROWS, SECOND>(p, e, row_begin, row_end, b0, b1, lin, list, smem);
        else if (rows <= 32) stream_segment<C8, 4, W, KEEP, ROWS, SECOND>(p, e, row_begin, row_end, b0, b1, lin, list, smem);
        else stream_segment<C8, MAX_AR, W, KEEP, ROWS, SECOND>(p, e, row_begin, row_end, b0, b1, lin, list, smem);
    }
    if constexpr (KEEP == kKeepAct) copy_sorted_rows<W * kWave, bf16_t>(p, list, wave_read_lane(et.hi, p.E_local - 1), FEW ? 1 : p.a_div);
    if (!SECOND && ROWS != kRowsSorted && p.exchange != nullptr) clear_exchange<W * kWave, bf16_t>(p);
}

template <int C8, int W, StreamRows ROWS, StreamKeep KEEP, bool SECOND>
static int launch_stream_as(const StreamGemm& p, hipStream_t stream)
{
    constexpr size_t lds = static_cast<size_t>(stream_ring_bytes(C8, W)) + W * kStreamIdBytes + (ROWS == kRowsInline ? sizeof(InlineDispatch) : (ROWS == kRowsEight ? W * stream_sums_bytes(C8) : 0));
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    auto kern = stream_gemm_kernel<C8, W, ROWS, KEEP, SECOND>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_expert_ffn")) return rc;
    hipLaunchKernelGGL(kern, dim3(kStreamGrid), dim3(W * kWave), lds, stream, p);
    return EXF_OK;
}

enum StreamWant { kWantResult, kWantSorted, kWantPairs };  // the last: rows that meet in p.exchange
template <int C8, int W, StreamRows ROWS, StreamWant WANT>
static int launch_stream_rows(const StreamGemm& p, hipStream_t stream)
{
    const bool second = p.epi == kEpiNone;
    if constexpr (WANT == kWantResult) {
        if constexpr (ROWS != kRowsInline) {  // (a first contraction)
            if (second) return launch_stream_as<C8, W, ROWS, kKeepNone, true>(p, stream);
        }
        return launch_stream_as<C8, W, ROWS, kKeepNone, false>(p, stream);
    } else {
        if constexpr (WANT == kWantSorted && ROWS != kRowsSorted) {  // (rows that are there in sorted order are not wanted again)
            if (!second && p.sorted_act != nullptr) return launch_stream_as<C8, W, ROWS, kKeepAct, false>(p, stream);
        }
        if constexpr (WANT == kWantSorted && ROWS != kRowsInline) {
            if (second && p.sorted_out != nullptr) return launch_stream_as<C8, W, ROWS, kKeepOut, true>(p, stream);
        }
        if constexpr (WANT == kWantPairs && ROWS != kRowsInline) return launch_stream_as<C8, W, ROWS, kKeepPairs, true>(p, stream);
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: sorted rows of a contraction that has none");
    }
}
template <int C8, int W, StreamWant WANT>
static int launch_stream(const StreamGemm& p, hipStream_t stream)
{
    if (p.topk_idx == nullptr) return launch_stream_rows<C8, W, kRowsSorted, WANT>(p, stream);
    if (p.max_rows <= 8) return launch_stream_rows<C8, W, kRowsEight, WANT>(p, stream);
    return p.max_rows <= kFewAssignments ? launch_stream_rows<C8, W, kRowsFew, WANT>(p, stream) : launch_stream_rows<C8, W, kRowsInline, WANT>(p, stream);
}

// Columns per block, by a model of the launch (blocks of 8 columns: one row of 4096 x 1024 has 128 of them for 256 workgroups
// instead of 64 of 16, the layer of one token 14.2 us and 13.6): a workgroup has ceil(q) blocks, and the activations, which every block
// reads again, weigh about 0.6 of as many bytes of weights (fitted to 9 shapes of 1 to 617 tokens: it picks the fastest or one within
// 5 %).  A single expert's row tiles are known and counted: blocks of up to 32 columns have tiles of 32 rows, so more rows are twice the
// blocks (one expert of 2048 x 8192, 40 to 64 rows 45.5 us without them - its second contraction in 512 blocks of 8 columns - and
// 40.3; of 512 x 2048 15.3 and 14.3).  Among several, blocks of 8 columns only where an expert's rows hardly exceed a tile: up to
// kFewAssignments in all (four experts of 512 x 2048, 120 rows 20.7 us with them and 18.5) and 28 an expert (two of 768 x 3072, 60
// rows 23.0 and 20.4; 48 rows 16.4 and 16.9).
template <StreamWant WANT>
static int launch_stream_bf16(const StreamGemm& p, hipStream_t stream)
{
    const double A = p.max_rows, E = p.E_local;
    const double touched = E * (1.0 - exp(A * log1p(-1.0 / E)));  // experts with rows, if A rows fall on E experts at random
    const bool one = p.E_local == 1 && p.max_rows <= kFewAssignments;
    int best = 8;
    double best_cost = 1e300;
    for (int c = 8; c >= (one || (p.max_rows <= kFewAssignments && 1.125 * A / touched <= 8 * stream_max_ar(1)) ? 1 : 2); c /= 2) {  // (in eights)
        const double tiles = one ? ceil(A / (8 * stream_max_ar(c))) : 1.0;
        const double act_rows = 8.0 * ceil((one ? A / tiles : 1.3 * A / touched) / 8.0);
        const double q = touched * tiles * (p.N / (8 * c)) / kStreamGrid;
        const double cost = ceil(q) * (8 * c + 0.6 * act_rows);
        if (cost < best_cost) {
            best_cost = cost;
            best = c;
        }
    }
    if (best == 8) return launch_stream<8, 4, WANT>(p, stream);
    if (best == 4) return launch_stream<4, 4, WANT>(p, stream);
    if (best == 2) return launch_stream<2, 8, WANT>(p, stream);
    return launch_stream<1, 8, WANT>(p, stream);
}

// ---------------------------------------------------------------------------- fp32
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t reg128_t;
constexpr int kExactUnit = 32;  // reduction elements per step: 128 bytes of every row

// Sums of this wavefront's units [u_begin, u_end) for 16 C columns x 16 M rows, written to red[row][column] (row
// stride RS floats).  A lane loads two 16-byte pieces of one weight row and the same pieces of one activation row per
// unit; they are the operands of eight 16x16x4 MFMAs as they lie (the order in which the reduction index is dealt
// to the lanes is free as long as both operands agree).  Loads run D units ahead; units past the end are clamped.
//   Whatever the kernel, a reduction is kExactParts sums of its own, added in order: short chains for the precision's sake, and the same bits from all of
// them.  A wavefront that takes SUB parts adds them up as it goes (the first one of its item) or leaves each in a slot of its own.
constexpr int kExactParts = 4;
template <int C, int M, int D, int RS, int SUB>
__device__ __forceinline__ void exact_units(const float* __restrict__ wexp, const float* __restrict__ act, const int32_t* __restrict__ a_row,
                                            int a_div, int row_begin, int row_end, int n0, int K, int N, int part, float* __restrict__ red, int slot_floats)
{
    const int units = (K + kExactUnit - 1) / kExactUnit;
    const int u_begin = part * SUB * units / kExactParts, u_end = (part + 1) * SUB * units / kExactParts;
    const bool first_parts = SUB == kExactParts || part == 0;
    if (!first_parts) red += (1 + (part - 1) * SUB) * slot_floats;
    const int lane = lane_id();
    const int r16 = lane & 15, g = lane >> 4;
    const float *row_w[C], *row_a[M];
#pragma unroll
    for (int c = 0; c < C; ++c) row_w[c] = wexp + static_cast<size_t>(min(n0 + c * 16 + r16, N - 1)) * K;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        int r = min(row_begin + m * 16 + r16, row_end - 1);  // rows past the end repeat the last one
        if (a_row != nullptr) r = a_row[r];
        if (a_row != nullptr && a_div > 1) r = static_cast<int>(static_cast<unsigned>(r) / static_cast<unsigned>(a_div));
        row_a[m] = act + static_cast<size_t>(r) * K;
    }
    f32x4_t acc[C][M];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[c][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    f32x4_t w[D][C][2], a[D][M][2];
    auto load = [&](int u, int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = u * kExactUnit + h * 16 + g * 4;  // K % 4 == 0: a piece is inside or outside as a whole
            const bool in = k < K;
            const int at = in ? k : 0;
#pragma unroll
            for (int c = 0; c < C; ++c) w[s][c][h] = *reinterpret_cast<const f32x4_t*>(row_w[c] + at);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(row_a[m] + at);
                a[s][m][h] = in ? v : f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    // a lane holds four consecutive columns of one row
    auto store = [&](const f32x4_t(&sum)[C][M]) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int m = 0; m < M; ++m) *reinterpret_cast<f32x4_t*>(red + (m * 16 + r16) * RS + c * 16 + g * 4) = sum[c][m];
    };
    f32x4_t earlier[C][M];  // parts that are complete (a single wavefront, or the first one of an item)
    if constexpr (SUB > 1) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int m = 0; m < M; ++m) earlier[c][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    int ends[SUB];
#pragma unroll
    for (int i = 0; i + 1 < SUB; ++i) ends[i] = (part * SUB + i + 1) * units / kExactParts;
    auto behind = [&](int u) {  // all units below u are in acc: on to the next part?
        if constexpr (SUB > 1) {
            static_assert(SUB == 2 || SUB == kExactParts, "one slot a part");
            bool next = false;
#pragma unroll
            for (int i = 0; i + 1 < SUB; ++i) next = next || u == ends[i];
            if (!next) return;
            if (SUB == kExactParts || first_parts) {
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int m = 0; m < M; ++m) earlier[c][m] += acc[c][m];
            } else {
                store(acc);
                red += slot_floats;
            }
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int m = 0; m < M; ++m) acc[c][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto compute = [&](int u, int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int m = 0; m < M; ++m)
                        acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][c][h][j], a[s][m][h][j], acc[c][m], 0, 0, 0);
        behind(u + 1);
    };
    behind(u_begin);
    if (u_begin < u_end) {
#pragma unroll
        for (int s = 0; s < D; ++s) load(min(u_begin + s, u_end - 1), s);
        int u = u_begin;
        for (; u + D < u_end; u += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                compute(u + s, s);
                __builtin_amdgcn_sched_barrier(0);
                load(min(u + D + s, u_end - 1), s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (u + s < u_end) compute(u + s, s);
    }
    if constexpr (SUB > 1) {
        if (SUB == kExactParts || first_parts) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int m = 0; m < M; ++m) acc[c][m] = earlier[c][m] + acc[c][m];
        }
    }
    store(acc);
}

// WI items per workgroup, WK wavefronts per item (they share its parts).
__host__ __device__ constexpr int exact_slots(int WK) { return 1 + (WK - 1) * (kExactParts / WK); }
template <int C, int M, int WK, int WI, int D, bool INLINE, StreamKeep KEEP>
__global__ __launch_bounds__(WK* WI * 64) void exact_gemm_kernel(const StreamGemm p)
{
    constexpr int COLS = 16 * C, RS = COLS + 4;  // (padded: the 16 rows of a float4 column store hit distinct banks)
    constexpr int TILE_ROWS = 16 * M;
    extern __shared__ float red[];  // [WI][exact_slots(WK)][TILE_ROWS][RS]
    constexpr int SLOTS = exact_slots(WK);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (p.unrouted != nullptr) clear_unrouted_rows<true, KEEP == kKeepPairs>(p.unrouted, p.n_unrouted, static_cast<uint4*>(p.out), p.N / 4, WK * WI);
    const int32_t *a_row = p.a_row, *offsets = p.offsets;
    if constexpr (INLINE) {
        InlineDispatch* d = reinterpret_cast<InlineDispatch*>(red + WI * SLOTS * TILE_ROWS * RS);
        sort_assignments<WK * WI * kWave>(p, *d, blockIdx.x == 0, [](int, bool) {});
        a_row = d->list;
        offsets = d->offs;
    }

    // work items are numbered (expert, column block, row tile); every XCD takes a contiguous share, so the row
    // tiles of a weight block and the column blocks of an expert's rows meet in one L2
    const int n_blocks = (p.N + COLS - 1) / COLS;
    const ExpertTiles et = scan_row_tiles(p, offsets, TILE_ROWS);
    const int total = et.total * n_blocks;
    const int xcd = static_cast<int>(blockIdx.x % kXcdCount), pos = static_cast<int>(blockIdx.x / kXcdCount);
    const int first_item = static_cast<int>(static_cast<int64_t>(total) * xcd / kXcdCount);
    const int last_item = static_cast<int>(static_cast<int64_t>(total) * (xcd + 1) / kXcdCount);
    const int item = first_item + pos * WI + wave / WK;
    const bool valid = item < last_item;  // (the same for the wavefronts of an item)
    const unsigned long long owner = __ballot(item < et.incl * n_blocks);
    const int e = valid ? __builtin_ctzll(owner) : 0;  // (item < total: some lane owns it)
    const int e_tiles = max(wave_read_lane(et.tiles, e), 1);
    const int in_expert = item - (wave_read_lane(et.incl, e) - e_tiles) * n_blocks;
    const int block = in_expert / e_tiles, tile = in_expert - block * e_tiles;
    const int row_begin = __builtin_amdgcn_readfirstlane(wave_read_lane(et.lo, e) + tile * TILE_ROWS);
    const int row_end = __builtin_amdgcn_readfirstlane(min(row_begin + TILE_ROWS, wave_read_lane(et.hi, e)));
    const int n0 = __builtin_amdgcn_readfirstlane(block * COLS);

    // the output row and its weight, where this thread stores four columns of one row below: two dependent loads, begun in front
    // of the sums (behind them they were 0.9 us of a small layer's 14.2)
    constexpr int GROUPS = COLS / 4;
    constexpr bool ONE = TILE_ROWS * GROUPS <= WK * kWave;
    const int thread = threadIdx.x % (WK * kWave);
    int one_dst = 0;
    float one_scale = 1.0f, one_mate_scale = 0.0f;
    bool one_mated = false;
    if (ONE && valid && p.out_row != nullptr) {
        one_dst = p.out_row[min(row_begin + thread / GROUPS, row_end - 1)];
        one_scale = p.out_scale[one_dst];
        if constexpr (KEEP == kKeepPairs) {
            one_mate_scale = p.out_scale[one_dst ^ 1];
            one_mated = p.unrouted[one_dst ^ 1] >= 0;
        }
    }

    float* item_red = red + static_cast<size_t>(wave / WK) * (SLOTS * TILE_ROWS * RS);
    if (valid) {
        const float* wexp = static_cast<const float*>(p.weight) + static_cast<size_t>(e) * p.N * p.K;
        const float* act = static_cast<const float*>(p.act);
        const int m_used = (row_end - row_begin + 15) / 16;
#define EXF_EXACT_UNITS(MU) \
    exact_units<C, MU, D, RS, kExactParts / WK>(wexp, act, a_row, p.a_div, row_begin, row_end, n0, p.K, p.N, wave % WK, item_red, TILE_ROWS* RS)
        if constexpr (M == 1) {
            EXF_EXACT_UNITS(1);
        } else {
            if (m_used == 1) EXF_EXACT_UNITS(1);
            else if (m_used == 2) EXF_EXACT_UNITS(2);
            else EXF_EXACT_UNITS(4);
        }
#undef EXF_EXACT_UNITS
    }
    __syncthreads();
    if constexpr (INLINE && KEEP == kKeepAct) copy_sorted_rows<WK * WI * kWave, float>(p, a_row, offsets[p.E_local], p.a_div);
    if (INLINE && p.exchange != nullptr) clear_exchange<WK * WI * kWave, float>(p);
    if (!valid) return;

    // four columns of one row per thread: the parts' sums in a fixed order, bias, activation, scale
    const float* bias = p.bias != nullptr ? static_cast<const float*>(p.bias) + static_cast<size_t>(e) * p.N : nullptr;
    for (int i = thread; i < (row_end - row_begin) * GROUPS; i += WK * kWave) {
        const int r = i / GROUPS, q = i % GROUPS;
        const int n = n0 + q * 4;
        f32x4_t z = *reinterpret_cast<const f32x4_t*>(item_red + r * RS + q * 4);
#pragma unroll
        for (int slot = 1; slot < SLOTS; ++slot) z += *reinterpret_cast<const f32x4_t*>(item_red + (slot * TILE_ROWS + r) * RS + q * 4);
        if (n >= p.N) continue;  // N % 4 == 0: the four columns are inside or outside together
        int dst = row_begin + r;
        float scale = 1.0f;
        if (p.out_row != nullptr) {
            dst = ONE ? one_dst : p.out_row[dst];
            scale = ONE ? one_scale : p.out_scale[dst];
        }
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = z[j];
            if (bias != nullptr) v[j] += bias[n + j];
            if (p.epi == kEpiGeluErf) v[j] = gelu_erf_exact(v[j]);
            else if (p.epi == kEpiGeluTanh) v[j] = gelu_tanh_exact(v[j]);
            if constexpr (KEEP != kKeepOut && KEEP != kKeepPairs) v[j] *= scale;
        }
        if constexpr (KEEP == kKeepPairs) {
            const bool second = (dst & 1) != 0, mated = ONE ? one_mated : p.unrouted[dst ^ 1] >= 0;
            const float mate_scale = !mated ? 0.0f : (ONE ? one_mate_scale : p.out_scale[dst ^ 1]);
            const float w0 = second ? mate_scale : scale, w1 = second ? scale : mate_scale;
            dst >>= 1;
            const size_t at = static_cast<size_t>(dst) * p.N + n;
            unsigned long long other[2] = {0ull, 0ull};
            if (mated) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    other[h] = meet(p.exchange + at / 2 + h, static_cast<unsigned long long>(__float_as_uint(v[2 * h + 1])) << 32 | __float_as_uint(v[2 * h]));
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (other[h] == kNoRow) continue;  // the other row's thread finds this one
                float o[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {  // (the combine's bits)
                    const float theirs = __uint_as_float(static_cast<uint32_t>(other[h] >> (32 * j))), ours = v[2 * h + j];
                    o[j] = fmaf(w1, second ? ours : theirs, fmaf(w0, second ? theirs : ours, 0.0f));
                }
                *reinterpret_cast<float2*>(static_cast<float*>(p.out) + at + 2 * h) = make_float2(o[0], o[1]);
            }
            continue;
        }
        if constexpr (KEEP == kKeepOut) {
            *reinterpret_cast<float4*>(static_cast<float*>(p.sorted_out) + static_cast<size_t>(row_begin + r) * p.N + n) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = fmaf(scale, v[j], 0.0f);  // (the combine's bits)
        }
        *reinterpret_cast<float4*>(static_cast<float*>(p.out) + static_cast<size_t>(dst) * p.N + n) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

template <int C, int M, int WK, int WI, int D, bool INLINE, StreamKeep KEEP>
static int launch_exact_as(const StreamGemm& p, hipStream_t stream)
{
    constexpr int TILE_ROWS = 16 * M;
    constexpr size_t lds = static_cast<size_t>(exact_slots(WK) * WI) * TILE_ROWS * (16 * C + 4) * sizeof(float) + (INLINE ? sizeof(InlineDispatch) : 0);
    auto kern = exact_gemm_kernel<C, M, WK, WI, D, INLINE, KEEP>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_expert_ffn")) return rc;
    // row tiles: whole ones and at most one partial tile per expert with rows
    const int64_t A = p.max_rows;
    const int64_t row_tiles = A / TILE_ROWS + (A < p.E_local ? A : p.E_local);
    const int64_t share = row_tiles * ((p.N + 16 * C - 1) / (16 * C)) / kXcdCount + 1;  // items of an XCD at most
    const int64_t grid = (share + WI - 1) / WI * kXcdCount;
    if (grid >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: too many tiles");
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(WK * WI * kWave), lds, stream, p);
    return EXF_OK;
}

template <int C, int M, int WK, int WI, int D>
static int launch_exact(const StreamGemm& p, hipStream_t stream)
{
    if (p.topk_idx != nullptr) {
        if (p.sorted_act != nullptr) return launch_exact_as<C, M, WK, WI, D, true, kKeepAct>(p, stream);
        return launch_exact_as<C, M, WK, WI, D, true, kKeepNone>(p, stream);
    }
    if (p.exchange != nullptr) {
        if (p.sorted_out != nullptr) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: sorted rows of a contraction that keeps none");
        return launch_exact_as<C, M, WK, WI, D, false, kKeepPairs>(p, stream);
    }
    if (p.sorted_out != nullptr) return launch_exact_as<C, M, WK, WI, D, false, kKeepOut>(p, stream);
    return launch_exact_as<C, M, WK, WI, D, false, kKeepNone>(p, stream);
}

// Enough tiles of 64 columns x 16 M rows for the chip: one wavefront per tile of 64 rows where the reduction is short (nothing to
// add up), two per 32 columns of 16 rows (7688 rows, 5 experts of 132 x 396, both contractions 54.3 us, with one per 64 columns 62.7; 3017, 6 of 96 x 284
// 19.1 and 22.5), four for long reductions.  A smaller problem is cut into 16 x 16 tiles with four wavefronts along the reduction
// (512 tokens x 8 experts x 64 x 256: 36 workgroups of 64 rows took 8.3 us in the second contraction, 4 now).
constexpr int64_t kExactFewTiles = 384;
constexpr int kExactShortReduction = 1024;
static int64_t exact_tiles(int64_t A, int N, int E_local, int rows) { return ((A < E_local ? A : E_local) + A / rows) * ((N + 63) / 64); }
template <int M>
static int launch_exact_rows(const StreamGemm& p, hipStream_t stream)
{
    if (exact_tiles(p.max_rows, p.N, p.E_local, 16 * M) < kExactFewTiles) return launch_exact<1, 1, 4, 1, 2>(p, stream);
    if (p.K > kExactShortReduction) return launch_exact<4, M, 4, 1, 2>(p, stream);
    if constexpr (M == 1) return launch_exact<2, 1, 2, 2, 2>(p, stream);
    else return launch_exact<4, M, 1, 4, 2>(p, stream);
}

// What an fp32 contraction [A,K] x [N,K] takes in launch_exact_rows<tall ? 4 : 1>, us.  Fitted to both contractions of 1540 lists (1025 to 100000 rows,
// 1 to 64 experts, 16 x 64 to 1024 x 4096) in every combination of the kernels: within 5 % for half of them, 15 for nine tenths.  Wavefronts per SIMD (w)
// run side by side until the operands' way from the L2 bounds them; tiles of 64 rows take their registers, one wavefront a SIMD, so that theirs come in rounds.
static double exact_cost(int64_t A, int K, int N, int E_local, bool gelu, bool tall)
{
    const double experts = static_cast<double>(A < E_local ? A : E_local), written = static_cast<double>(A) * N * 4e-6;  // MB
    const double simds = 4.0 * 256, row_tiles = A / 16.0 + experts / 2, col_tiles = (N + 63) / 64;  // (on the mean half a tile more per expert)
    if (exact_tiles(A, N, E_local, tall ? 64 : 16) < kExactFewTiles)
        return 2.7 + K / 4 * (0.0166 + 0.0106 * row_tiles * ((N + 15) / 16) * 4 / simds) + 1.15 * written;
    if (tall) {
        const bool parts = K > kExactShortReduction;
        const double w = (A / 64.0 + experts / 2) * col_tiles * (parts ? 4 : 1) / simds, whole = floor(w);
        const double begun = w < 2 ? 0.7 : 0.45, rounds = w <= 1 ? 1 : whole + (w > whole ? begun + (1 - begun) * (w - whole) : 0);
        return parts ? 2.3 + rounds * (0.0203 * K + 2.3) + 1.1 * written : 3.1 + rounds * (0.0806 * K + (gelu ? 9.1 : 6.6)) + 0.41 * written;
    }
    if (K > kExactShortReduction) return K / 4 * (0.0298 + 0.0259 * row_tiles * col_tiles * 4 / simds) + 5.0 * written;
    return 3.0 + K / 2 * (0.0115 + 0.0176 * row_tiles * ((N + 31) / 32) * 2 / simds) + 0.52 * written;
}

// Do the tiles of 64 rows nearly fill whole rounds of wavefronts?  Then they beat tiles of 16 by more than the model knows, but for reductions of 96 to 128 and
// below 48: 32000 rows of 256 x 256, both contractions, 180 us in 16 rows and 144 in 64 (1.96 rounds); 8000 of 512 x 512 178 and 114 (0.99), of 16
// experts (1.04) 178 and 206; 2000 of 64 x 4096 84.7 and 77.8 with the first in 64; first contraction of 16000 of 128 x 2048 22 more of 340.
static bool whole_rounds(int64_t A, int K, int N, int E_local)
{
    if (A <= 16ll * E_local || !(K >= 240 || (K >= 48 && K <= 64)) || exact_tiles(A, N, E_local, 64) < kExactFewTiles) return false;
    const int64_t half_tiles = (A / 32 + E_local) * ((N + 63) / 64) * (K > kExactShortReduction ? 4 : 1);
    return 10 * half_tiles >= 9 * 2048 * ((half_tiles + 2047) / 2048);
}

// Tiles of 64 rows, else 16: for the weights' sake where these do not lie in the L2s (2^18 floats an expert; 3544 rows, 4 experts of 232 x 524, which do, both
// contractions 61.1 us in 64 rows, 47.6 in 16), else where they fill their rounds or cost less.  Layers that were always in 16 rows and
// now: 20000 rows, 8 experts of 512 x 512 454 and 337 us; 40000, 64 of 64 x 4096 1445 and 1186; 20000, 8 of 128 x 2048 444 and 388.
static bool tall_exact_tiles(int64_t A, int K, int N, int E_local, bool gelu)
{
    if (A <= 16ll * E_local) return false;
    if (static_cast<int64_t>(K) * N > 1 << 18) return true;
    if (exact_tiles(A, N, E_local, 64) < kExactFewTiles) return false;
    return whole_rounds(A, K, N, E_local) || exact_cost(A, K, N, E_local, gelu, true) < 0.95 * exact_cost(A, K, N, E_local, gelu, false);
}

// ---------------------------------------------------------------------------- fp32, both contractions at once
// A workgroup takes a tile of 16 sorted rows through both contractions: the hidden activations stay in LDS, and the second launch goes with
// what it waits for (the first one's last workgroup, row ranges, row ids, a round trip for the weights; those of the second contraction
// are asked for behind the first one's products).  What it cannot do is spread a tile over compute units: one takes the expert's weights
// in at some 40 bytes a cycle, 0.2 us for 1000 d f, so it is for layers whose tiles fill the chip (see exact_pair_fits).
// Every sum is that of exact_gemm_kernel<1, 1, 4, 1>: the reduction in four parts, added in order.  Two launches and one, us: 3724 rows, 10 experts
// of 120 x 444 26.0 and 17.6; 3333, 9 of 92 x 192 16.0 and 10.1; 2692, 2 of 56 x 256 14.8 and 9.1; 7688, 5 of 132 x 396 54.3 and 37.6.
constexpr int kPairRows = 16, kPairWaves = 16, kPairParts = kExactParts;
constexpr int kPairAhead = 2;  // units of 32 asked for ahead (two workgroups share a compute unit: 64 registers)
struct PairWeights {
    f32x4_t w[kPairAhead][2];
    const float* row;
    int K;
    __device__ __forceinline__ void load(int u, int s)
    {
        const int g = lane_id() >> 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = u * kExactUnit + h * 16 + g * 4;
            w[s][h] = *reinterpret_cast<const f32x4_t*>(row + (k < K ? k : 0));
        }
    }
    __device__ __forceinline__ void begin(const float* weight, int n0, int N, int K_, int u_begin, int u_end)
    {
        row = weight + static_cast<size_t>(min(n0 + (lane_id() & 15), N - 1)) * K_;
        K = K_;
        if (u_begin >= u_end) return;
#pragma unroll
        for (int s = 0; s < kPairAhead; ++s) load(min(u_begin + s, u_end - 1), s);
    }
    // Units [u_begin, u_end) (behind begin()); act: 16 rows of `stride` floats in LDS.  `after(u)`: unit u is in acc.
    template <typename After>
    __device__ __forceinline__ void sum(const float* act, int stride, int u_begin, int u_end, f32x4_t& acc, After after)
    {
        const int g = lane_id() >> 4;
        const float* row_a = act + (lane_id() & 15) * stride;
        auto compute = [&](int u, int s) {
            f32x4_t a[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = u * kExactUnit + h * 16 + g * 4;  // K % 4 == 0: a piece is inside or outside as a whole
                a[h] = *reinterpret_cast<const f32x4_t*>(row_a + (k < K ? k : 0));
                if (k >= K) a[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][h][j], a[h][j], acc, 0, 0, 0);
            after(u);
        };
        int u = u_begin;
        for (; u + kPairAhead < u_end; u += kPairAhead) {
#pragma unroll
            for (int s = 0; s < kPairAhead; ++s) {
                compute(u + s, s);
                __builtin_amdgcn_sched_barrier(0);
                load(min(u + kPairAhead + s, u_end - 1), s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < kPairAhead; ++s)
            if (u + s < u_end) compute(u + s, s);
    }
};
__host__ __device__ constexpr size_t pair_floats(int d, int f) { return static_cast<size_t>(kPairRows) * (f + 4) + static_cast<size_t>(kPairParts) * kPairRows * (d + 4); }

// INLINE: of a list that is sorted on the way (p.topk_idx): gate and this are the whole layer.
template <bool INLINE>
__global__ __launch_bounds__(kPairWaves * 64, 8) void exact_pair_kernel(const StreamGemm p, const StreamGemm q)
{
    extern __shared__ __attribute__((aligned(16))) float pair_smem[];
    touch_arguments<2 * sizeof(StreamGemm)>();
    const int lane = lane_id(), r16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int d = p.K, f = p.N;
    const int act_stride = d + 4, hid_stride = f + 4;  // (padded: 16 rows lie in distinct banks)
    float* hid = pair_smem;                     // [16][f + 4]
    float* act = hid + kPairRows * hid_stride;  // [16][d + 4], later the sums of the parts: [4][16][d + 4]
    const int32_t *a_row = p.a_row, *out_row = q.out_row, *offsets = p.offsets;
    if constexpr (INLINE) {
        InlineDispatch* sort = reinterpret_cast<InlineDispatch*>(pair_smem + pair_floats(d, f));
        // Every workgroup clears its share of the rows that are dropped, a wavefront a row (by the one thread that has the
        // assignment 1000 tokens, 2 of 16 experts of 64 x 256 took 15.9 us and take 14.7; 1024 without an expert here, 468 x 564 19.2 and 10.8).
        sort_assignments<kPairWaves * kWave>(p, *sort, blockIdx.x == 0, [&](int a, bool dropped) {
            if (q.unrouted == nullptr) return;
            unsigned long long todo = __ballot(dropped && static_cast<unsigned>(a) % gridDim.x == blockIdx.x);
            while (todo != 0) {
                uint4* row = reinterpret_cast<uint4*>(q.out) + static_cast<size_t>(a - lane + __builtin_ctzll(todo)) * (d / 4);
                todo &= todo - 1;
                for (int c = lane; c < d / 4; c += kWave) row[c] = make_uint4(0u, 0u, 0u, 0u);
            }
        });
        a_row = sort->list;
        if (out_row != nullptr) out_row = sort->list;
        offsets = sort->offs;
    } else if (q.unrouted != nullptr) {
        clear_unrouted_rows<false, false>(q.unrouted, q.n_unrouted, static_cast<uint4*>(q.out), d / 4, kPairWaves);
    }
    // every XCD takes a contiguous share of the tiles: those of an expert meet in one L2
    const ExpertTiles et = scan_row_tiles(p, offsets, kPairRows);
    const int xcd = static_cast<int>(blockIdx.x % kXcdCount);
    const int item = static_cast<int>(static_cast<int64_t>(et.total) * xcd / kXcdCount) + static_cast<int>(blockIdx.x / kXcdCount);
    if (item >= static_cast<int>(static_cast<int64_t>(et.total) * (xcd + 1) / kXcdCount)) return;
    const int e = __builtin_ctzll(__ballot(item < et.incl));  // (item < total: some lane owns it)
    const int tile = item - (wave_read_lane(et.incl, e) - wave_read_lane(et.tiles, e));
    const int row_begin = wave_read_lane(et.lo, e) + tile * kPairRows, rows = min(kPairRows, wave_read_lane(et.hi, e) - row_begin);

    // a wavefront brings one row and stores it; the first weights travel with the rows
    const float* w1 = static_cast<const float*>(p.weight) + static_cast<size_t>(e) * f * d;
    const float* w2 = static_cast<const float*>(q.weight) + static_cast<size_t>(e) * d * f;
    const int units1 = (d + kExactUnit - 1) / kExactUnit, units2 = (f + kExactUnit - 1) / kExactUnit;
    const int sorted = row_begin + min(wave, rows - 1);  // (rows past the end repeat the last one)
    int from = sorted;
    if (a_row != nullptr) from = p.a_div > 1 ? static_cast<int>(static_cast<unsigned>(a_row[sorted]) / static_cast<unsigned>(p.a_div)) : a_row[sorted];
    int dst = sorted;
    float scale = 1.0f;
    if (out_row != nullptr) {
        dst = out_row[sorted];
        scale = q.out_scale[dst];
    }
    PairWeights pw;
    pw.begin(w1, wave * 16, f, d, 0, units1);
    for (int c = lane; c < d / 4; c += kWave) {
        const float4 v = reinterpret_cast<const float4*>(static_cast<const float*>(p.act) + static_cast<size_t>(from) * d)[c];
        reinterpret_cast<float4*>(act + wave * act_stride)[c] = v;
        if (INLINE && p.sorted_act != nullptr && wave < rows) reinterpret_cast<float4*>(static_cast<float*>(p.sorted_act) + static_cast<size_t>(sorted) * d)[c] = v;
    }
    __syncthreads();

    // ---- hidden activations: 16 columns by a wavefront, all four parts
    const int part_end[3] = {units1 / kPairParts, 2 * units1 / kPairParts, 3 * units1 / kPairParts};
    for (int n0 = wave * 16; n0 < f; n0 += kPairWaves * 16) {
        f32x4_t z = f32x4_t{0.f, 0.f, 0.f, 0.f}, acc = z;
        pw.sum(act, act_stride, 0, units1, acc, [&](int u) {
            if (u + 1 == part_end[0] || u + 1 == part_end[1] || u + 1 == part_end[2]) {
                z += acc;
                acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        });
        z += acc;
        if (n0 + kPairWaves * 16 < f) pw.begin(w1, n0 + kPairWaves * 16, f, d, 0, units1);
        const int n = n0 + g * 4;
        if (n < f) {  // f % 4 == 0: the four columns are inside or outside together
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = z[j];
                if (p.bias != nullptr) v[j] += static_cast<const float*>(p.bias)[static_cast<size_t>(e) * f + n + j];
                v[j] = p.epi == kEpiGeluErf ? gelu_erf_exact(v[j]) : gelu_tanh_exact(v[j]);
            }
            *reinterpret_cast<float4*>(hid + r16 * hid_stride + n) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }

    // ---- outputs: (16 columns, part) by a wavefront
    const int items2 = (d + 15) / 16 * kPairParts;
    auto begin2 = [&](int i) {
        const int part = i % kPairParts;
        pw.begin(w2, i / kPairParts * 16, d, f, part * units2 / kPairParts, (part + 1) * units2 / kPairParts);
    };
    if (wave < items2) begin2(wave);
    __syncthreads();
    float* red = act;
    for (int i = wave; i < items2; i += kPairWaves) {
        const int part = i % kPairParts, n = i / kPairParts * 16 + g * 4;
        f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
        pw.sum(hid, hid_stride, part * units2 / kPairParts, (part + 1) * units2 / kPairParts, acc, [](int) {});
        if (i + kPairWaves < items2) begin2(i + kPairWaves);
        if (n < d) *reinterpret_cast<f32x4_t*>(red + (part * kPairRows + r16) * act_stride + n) = acc;
    }
    __syncthreads();
    if (wave >= rows) return;
    const float* bias = q.bias != nullptr ? static_cast<const float*>(q.bias) + static_cast<size_t>(e) * d : nullptr;
    for (int c = lane; c < d / 4; c += kWave) {
        f32x4_t z = *reinterpret_cast<const f32x4_t*>(red + wave * act_stride + c * 4);
#pragma unroll
        for (int part = 1; part < kPairParts; ++part) z += *reinterpret_cast<const f32x4_t*>(red + (part * kPairRows + wave) * act_stride + c * 4);
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = bias != nullptr ? z[j] + bias[c * 4 + j] : z[j];
        if (q.sorted_out != nullptr) {
            reinterpret_cast<float4*>(static_cast<float*>(q.sorted_out) + static_cast<size_t>(sorted) * d)[c] = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = fmaf(scale, v[j], 0.0f);  // (the combine's bits)
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] *= scale;
        }
        reinterpret_cast<float4*>(static_cast<float*>(q.out) + static_cast<size_t>(dst) * d)[c] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// What the launch takes, us: rounds of tiles, one or (LDS) two on a compute unit.  In a tile the wavefronts wait for their operands (in units of 32
// by 16 columns, all 16 wavefronts at once) and for the first ones of every 16 hidden columns and every quarter of 16 output columns; rows
// of a multiple of 128 bytes begin on the same channels.  Fitted to 1000 lists as exact_cost: within 4 % for half of them, 9 for nine tenths.
static double exact_pair_cost(int64_t A, int d, int f, int E_local)
{
    const int units1 = (d + 31) / 32, units2 = (f + 31) / 32, passes1 = (f + 255) / 256, passes2 = ((d + 15) / 16 * kPairParts + kPairWaves - 1) / kPairWaves;
    const bool even1 = d % 32 == 0, even2 = f % 32 == 0;
    const double operands = 0.455 * units1 * ((f + 15) / 16) / kPairWaves * (even1 ? 1.475 : 1.0) + 0.775 * units2 * ((d + 15) / 16) / kPairWaves * (even2 ? 1.1 : 1.0);
    const double waits = passes1 * (0.47 + 0.093 * units1) + passes2 * (0.6 + 0.146 * ((units2 + 3) / 4)) * (even2 ? 1.1 : 1.0);
    const double one = 2.0 + operands + waits, two = 2.0 + 1.9 * operands + 1.675 * waits;
    const int64_t tiles = A / kPairRows + (A < E_local ? A : E_local) / 2;
    if (pair_floats(d, f) * sizeof(float) > 80 * 1024) return 1.75 + (tiles + 255) / 256 * one;
    const int64_t rest = tiles % 512;
    return 1.75 + tiles / 512 * two + (rest == 0 ? 0 : (rest <= 256 ? one : two));
}

// The line: not where two launches would cost a twentieth less, nor where both contractions fill whole rounds of tiles of 64 rows.  Two launches and one, us:
// 1500 rows, 4 experts of 256 x 256 18.0 and 19.4; 1100, 16 of 96 x 400 11.4 and 14.3; 1100, 64 of 256 x 1024 47 and 62; 1500, 4 of 64 x 1024 24.5 and
// 19.1; 4000, 16 of 512 x 128 33.5 and 49.9; 64000 of 512 x 128 299 and 398; 32000 of 256 x 512 255 and 264; 8000 of 256 x 1024 156 and 126.  Over 1540 lists the choice
// costs 1.5 % more than the best one (one launch wherever it fits 3.8).  Shorter lists are sorted on the way, see below.
static double exact_both_cost(int64_t A, int d, int f, int E_local)
{
    return exact_cost(A, d, f, E_local, true, tall_exact_tiles(A, d, f, E_local, true)) + exact_cost(A, f, d, E_local, false, tall_exact_tiles(A, f, d, E_local, false));
}
bool exact_pair_fits(int64_t A, int d, int f, int E_local)
{
    if (A <= kInlineDispatchMax || pair_floats(d, f) * sizeof(float) > 160 * 1024) return false;
    if (d >= 240 && whole_rounds(A, d, f, E_local) && whole_rounds(A, f, d, E_local)) return false;
    return exact_both_cost(A, d, f, E_local) >= 0.95 * exact_pair_cost(A, d, f, E_local);
}

// Lists that are sorted on the way: sorting takes the same time in either, and so few tiles leave most compute units idle, so where the model has this launch
// ahead.  Whole layers with two and one, us: 1024 tokens, 8 experts of 64 x 256 15.6 and 13.5; 512, 8 of 64 x 128 12.7 and 11.3; 512, 4 of 32 x 128
// 12.2 and 10.6; 700, 14 of 44 x 300, separate calls 15.3 and 14.1; 900, 29 of 468 x 564 74.7 and 69.6; not 512, 8 of 64 x 256 13.3 and 13.4; 100 of
// these 11.9 and 13.2; 512, 8 of 128 x 256 15.3 and 16.3; 512, 8 of 256 x 512 20.9 and 37.3.
// With a share of the experts nobody here knows how many rows are kept.  Fewer rows shorten two launches and not the one, whose tiles take as long each, but two
// have the other rows cleared by a few wavefronts in front of the second one's products, which takes at least kClearing.  So the model has to have the
// one ahead with all rows kept and, but for that, with the experts' share of them: 1000 tokens, 2 of 16 of 64 x 256 18.4 and 14.7; 512, 2 of 8 of 32 x 128 15.0 and
// 10.7; 900, 16 of 32 of 92 x 252 19.1 and 17.7; 700, 7 of 56 of 44 x 300, separate calls 23.1 and 19.2; not 900, 29 of 58 of 468 x 564 59.7 and 75.9.
constexpr double kClearing = 2.0;
bool exact_pair_routed_fits(int64_t A, int d, int f, int E, int E_local)
{
    if (A > kInlineDispatchMax || pair_floats(d, f) * sizeof(float) + sizeof(InlineDispatch) > 160 * 1024) return false;
    if (exact_both_cost(A, d, f, E_local) < exact_pair_cost(A, d, f, E_local)) return false;
    const int64_t share = A * E_local >= E ? A * E_local / E : 1;
    return share >= A || exact_both_cost(share, d, f, E_local) + kClearing >= exact_pair_cost(share, d, f, E_local);
}

template <bool INLINE>
static int launch_exact_pair_as(const StreamGemm& first, const StreamGemm& second, hipStream_t stream)
{
    auto kern = exact_pair_kernel<INLINE>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), 160 * 1024, allowed, "moe_expert_ffn")) return rc;
    const int64_t A = first.max_rows;
    const int64_t share = (A / kPairRows + (A < first.E_local ? A : first.E_local)) / kXcdCount + 1;  // tiles of an XCD at most
    const size_t lds = pair_floats(first.K, first.N) * sizeof(float) + (INLINE ? sizeof(InlineDispatch) : 0);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(share * kXcdCount)), dim3(kPairWaves * kWave), lds, stream, first, second);
    return EXF_OK;
}
int launch_exact_pair(const StreamGemm& first, const StreamGemm& second, hipStream_t stream)
{
    return first.topk_idx != nullptr ? launch_exact_pair_as<true>(first, second, stream) : launch_exact_pair_as<false>(first, second, stream);
}

// ---------------------------------------------------------------------------- host
// With the routing given only the first workgroup is the gate, and its launch is saved whatever it takes (8 of 8 x 4096 to 64 x 16384
// 3 to 14 us less).  Otherwise every workgroup is, in front of its own weights, which costs more than the launch where a wavefront
// has many units of the reduction to walk, each with 16 rows of tokens and those of the experts: separate minus joined, mean over 1 to 16
// tokens and f from 64 to 2048, us, by these rows in sixteens: 32 x 2048 (12) 0.4, 64 x 1024 (20) 0.4, 32 x 4096 (24) 0.25, 64 x 1536 (30)
// 0.1, 8 x 8192 (32) 0.2, 48 x 2048 (32) 0.0, 64 x 2048 (40) -0.3, 32 x 8192 (48) -0.8, 8 x 16384 (64) -0.8, 64 x 4096 (80) -0.6, 64 x 16384 -2.2.
bool gate_joins_layer(int64_t T, int d, int E, int dt, bool routed)
{
    const int nt = (E + 15) / 16;
    return dt == EXF_BF16 && T <= kGateFewTokens && (routed || d / 64 * (nt + 1) <= 32 * gate_sums(nt, d));
}

// bf16: the weights are streamed where few rows use them, on the mean at most 28 an expert: 24 rows of 64 experts of 1024 x 4096 take
// 222 us against 219 with the tiles of ffn_tiles.hpp, 32 rows of 8 experts of 2048 x 8192 both 114.  With few experts the
// tiles also wait for their K loops, a quarter of a microsecond for 64 elements of d + f, while streaming costs 35 ns per row and
// million weights: up to 256 rows in all the lower of the two (three experts of 1024 x 4096: 21.2 us against 27.2 with 87 rows, 27.6
// against 27.3 with 117).  Up to 128 rows of a single expert are known to fill 32, 64 or 128 of a row tile's, which is what they
// cost (1024 x 4096: 24.8 against 27.4 with 117 rows; 2048 x 8192: 37.1 against 44.9 with 58, 53.2 against 45.6 with 65; 4096 x
// 14336: 52.7 against 74.0 with 30, 83.4 against 74.2 with 33).
bool stream_path_fits(int64_t A, int d, int f, int E_local, int dt)
{
    if (dt == EXF_F32 || A <= 28ll * E_local) return true;
    if (A > 256) return false;
    const int64_t rows = E_local > 1 || A > 128 ? A : (A <= 32 ? 32 : (A + 63) / 64 * 64);
    return rows * d * f <= 120000ll * (static_cast<int64_t>(d) + f);
}

int launch_stream_gemm(const StreamGemm& p, int dt, hipStream_t stream)
{
    if (dt == EXF_BF16) {
        if (p.epi == kEpiNone && p.exchange != nullptr) return launch_stream_bf16<kWantPairs>(p, stream);
        if (p.sorted_act == nullptr && p.sorted_out == nullptr) return launch_stream_bf16<kWantResult>(p, stream);
        return launch_stream_bf16<kWantSorted>(p, stream);
    }
    return tall_exact_tiles(p.max_rows, p.K, p.N, p.E_local, p.epi != kEpiNone) ? launch_exact_rows<4>(p, stream) : launch_exact_rows<1>(p, stream);
}

}  // namespace exf
