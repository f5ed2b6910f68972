// The grouped bf16 contraction in tiles, a workgroup a tile (see ffn.hip, ffn_keep.hip, which instantiate it).
//
// gfx950 matrix cores, one workgroup per compute unit:
//   - a tile is H x NT outputs in 16x16 accumulators (v_mfma_f32_16x16x32_bf16).  On random operands the chip is held by its
//     power limit, and what draws least is fastest: the 16x16x32 instruction instead of the 32x32x16 one, and four
//     wavefronts of 128 x 128 outputs, which fetch a third less from LDS than eight of 128 x 64 (8192 x 4096 x 4096, K loops
//     alike: 1285 TFLOP/s eight wavefronts 32x32, 1370 eight 16x16, 1334 four 32x32, 1465 four 16x16; with all-zero
//     operands 1705 / 1610 / 1812 / 1822).  128 x 128 accumulators are the whole accumulator half of a wavefront's registers:
//     they are named as such ("a" registers) in inline assembly; left to the compiler they are copied to and fro.
//   - the second contraction runs four wavefronts, the first one eight: a single wavefront per SIMD issues vector
//     instructions at half rate, and GELU on a 256 x 256 tile then takes 8.4 us instead of 4 - more than a K loop of 16
//     tiles gains.
//   - global -> LDS with direct-to-LDS 16-byte loads (no staging registers), a ring of K tiles of 64,
//     one workgroup barrier per K tile, placed in the middle of the last K step so that MFMAs are in
//     flight on both sides of it.  A direct-to-LDS load writes 64 lanes x 16 B contiguously, so
//     the LDS layout is fixed; bank conflicts on the MFMA operand reads are avoided by choosing
//     WHICH 16-byte chunk of a row each lane fetches (XOR swizzle applied on the global side).
//   - the K loop's steady state has no branch: first, last and refill-free K tiles are instances of their own.
//   - the weight tile feeds the MFMA row axis and the activation tile the column axis, so a lane
//     ends up with 4 consecutive output columns of one row; one swap between rows of 16 lanes makes that 8,
//     and a 16-byte store needs no transposition through LDS.
#pragma once

#include <type_traits>

#include "ffn_common.hpp"

namespace exf {

constexpr int kLdsBytes = 160 * 1024;  // LDS of a compute unit
constexpr int kComputeUnits = 256;
constexpr int kTallestTile = 320;      // rows
constexpr int kKTile = 64;             // reduction elements of a stage: 128 bytes of every row

// Optional row indirections of the bf16 grouped GEMM; all members null / zero = sorted rows on both sides.
// They let the contraction read the tokens where they lie (no sorted copy of the activations) and
// let the second contraction of a top-1 layer write the gate-weighted result straight to the
// token's own row (no sorted copy of the outputs, no separate combine pass).
// (No padding between the members: all arguments and the size of the grid, which lies behind them, are two lines.)
struct RowMap {
    const int32_t* a_row;     // operand row of sorted row s is a_row[s] / a_div        (null: row s)
    const int32_t* out_row;   // output row of sorted row s is out_row[s]; every output row is the
    const float* out_scale;   //   target of at most one s and is scaled by out_scale[out_row[s]] in
                              //   fp32 before the single rounding to bf16              (null: row s, no scale)
    const int32_t* unrouted;  // [n_unrouted]: output row t with unrouted[t] < 0 is set to zero
    // Measurement only (exf_probe_ffn_timeline; null in every other call): workgroup b < timeline_cap
    // writes eight 64-bit words - [0] start, [1] tile located, [2] first K tile landed, [3] K loop done,
    // [4] end (all on the constant 100 MHz clock), [5] hardware id, [6] tile kind / expert / column tile /
    // rows / K tiles, [7] the experts' row ranges have arrived (between [0] and [1]).
    unsigned long long* timeline;
    // With out_row and kEpiKeepSorted: sorted row s is the result in bf16, and what is scaled and rounded again is that, as the combine does it.
    bf16_t* sorted_out;
    int a_div, n_unrouted, timeline_cap;
};
static_assert(sizeof(RowMap) == 64, "with the other arguments 120 bytes");

// The hidden activations between the two contractions live in a layout of their own (nobody else reads them): the
// 16-byte pieces (8 columns) of 32 consecutive rows are contiguous, and every expert starts on a 32-row boundary: sorted
// row m of expert e is hidden row m + 32 e - (first row of e) % 32.  The first contraction stores its accumulators 256 bytes
// at a time that way (row-major they are 64-byte segments: the epilogue of a 256 x 256 tile took 8 us, and up to 23 when
// all compute units wrote), and the 4 KiB of a K tile of 32 rows do not meet on the few memory channels that rows a
// power of two apart share.
constexpr int kHiddenRowBlock = 32;
__host__ __device__ inline uint32_t hidden_offset(uint32_t h, uint32_t piece, uint32_t pieces)
{
    return (h / kHiddenRowBlock * pieces + piece) * (kHiddenRowBlock * 16) + (h % kHiddenRowBlock) * 16;
}

__device__ __forceinline__ void timeline_stamp(const RowMap& map, int slot)
{
    if (map.timeline != nullptr && threadIdx.x == 0 && static_cast<int>(blockIdx.x) < map.timeline_cap)
        map.timeline[static_cast<size_t>(blockIdx.x) * 8 + slot] = wall_clock64();
}

// A first contraction that is the dispatch as well: every workgroup counts all assignments, finds its tile by that and collects the tile's
// rows; the tiles of the first output columns write the maps, and every tile its share of the columns of the sorted rows.
struct TileRouting {
    const int32_t* topk_idx;    // [A]
    const int32_t* expert_map;  // [E] or null
    int32_t *src_of_sorted, *sorted_of_src, *expert_counts, *expert_offsets;
    bf16_t* sorted_act;         // [A,K]
    int E, k;
};
constexpr int kRoutedRounds = kRoutedTilesMax / (8 * kWave);  // assignments of a thread
constexpr int kRoutedCopies = 8;  // of a counter, so that few experts do not meet at one address
struct RoutedSort {
    uint32_t count[EXF_MAX_EXPERTS][kRoutedCopies];
    int wave_rows[8];
    int list[kTallestTile];  // assignments of the tile's rows
};

// ---------------------------------------------------------------------------- row tiles
// The rows of an expert become q = rows / 256 tiles, and what is left over is spread over them in quanta of 32 rows: a tile
// of 288 rows costs an eighth more, one more tile a whole one.  A tile takes at most `most` quanta; where the
// remainder is larger there is one tile more, all of one height.  most = 1, or 2 where the launch then has fewer rounds of
// tiles (see plan_tiles).  An expert of at most 128 rows has one small tile.  Heights of a tile: 64 and 128 (small), 192, 224,
// 256, 288, 320; of a piece of one (see locate_tile) 64, 96, 128 and 160 besides.  160 instead of 192 and
// 224 instead of 256 (`by160`, `by224`) in launches of more tiles than half the compute units: the tallest whole tile of the only round is the
// time (from 136 tiles on all are whole; of 129 to 135 the XCDs that have 17 keep them whole, the others cut theirs in two: 22 layers of 129 to 135 tiles, 150 and 210
// rows an expert, 41 to 66 us, 2 to 6 % faster than with the line at 136).  160 where no expert of a single round has more rows, or in several rounds.  Experts of up to 160 rows in 192 and in 160: 1000 tokens, 8 experts of
// 2048 x 8192 131.9 -> 122.9 us, 1100, 8 of 1536 x 6144 97.4 -> 92.0, 2200, 16 of 2048 x 8192 236 -> 222, 8600, 60 of 2048 x 8192 867 -> 839; with a
// taller one among them 1150, 8 of 2048 x 8192 132.5 and 134.8.  Up to 224 rows in 256 and in 224: 3000, 16 of 1024 x 4096 85.5 -> 82.7; 3360, 8 of
// 2048 x 8192 247 -> 234; 12000, 60 of 2048 x 8192 999 -> 979; 1531 top-2, 16 of 1024 x 4096 96.6 -> 95.8.  In up to half as many tiles as compute
// units, which are cut, the second one of two ends in a piece of a few rows more: 420, one of 2048 x 8192 57.7 and 59.5.  (The exact rule, no tile of the
// only round taller, takes the heights of all experts in front of the look-up: 0.4 to 2 us of 44 to 100.)
constexpr int kTileRows = 256;
constexpr int kQuantum = 32;
constexpr int kSmallRows = 128;

struct TileRows {
    int tiles, height, extra;  // row tiles, their base height, quanta spread over them
};
__device__ __forceinline__ TileRows cut_rows(int cnt, int most, bool by160 = true, bool by224 = true)
{
    TileRows t;
    const int q = cnt / kTileRows, r = cnt - q * kTileRows;
    t.tiles = q;
    t.height = kTileRows;
    t.extra = (r + kQuantum - 1) / kQuantum;
    if (t.extra > q * most) {
        t.tiles = q + 1;
        t.extra = 0;
        // (q is at most 7 here)
        const int even = q == 0 ? cnt : (q == 1 ? (cnt + 1) / 2 : (q == 2 ? (cnt + 2) / 3 : kTileRows));
        t.height = even <= 64 && q == 0 ? 64 : (even <= kSmallRows && q == 0 ? kSmallRows : (even <= 160 && by160 ? 160 : (even <= 192 ? 192 : (even <= 224 && by224 ? 224 : kTileRows))));
    }
    return t;
}

// A tile of `height` rows (`rows` of them there are) in 2^pieces pieces: its columns in 2^cut parts, its rows in 2^row_cut of `height`
// rows.  Every cut goes where it leaves the fewer rows of operands (see locate_tile) and where there is an instance.
struct TileCut {
    int cut, row_cut, height;
};
__host__ __device__ constexpr TileCut cut_tile(int NT, int height, int rows, int pieces)
{
    TileCut t{pieces, 0, height};
    if (t.cut == 3 && rows <= 64) t.cut = 2;  // no instance of an eighth: four pieces
    for (int i = 1; i <= 2; ++i) {
        const int part = ((rows + (kQuantum << i) - 1) >> (i + 5)) * kQuantum;
        const bool too_tall = t.cut == 2 && t.height > NT / 2;  // no instance of that height
        if (t.row_cut == i - 1 && t.cut > 0 && (t.height - part > NT >> t.cut || too_tall)) {
            t.row_cut = i;
            t.cut -= 1;
            t.height = part;
        }
    }
    return t;
}
// The kernel's instances, and the next height there is one of.
__host__ __device__ constexpr bool has_instance(int NT, int height, int cut)
{
    const bool wide = NT == 256;
    if (cut == 0) return height == 64 || (height == 96 && !wide) || height == 128 || height == 160 || height == 192 || height == 224 || height == 256 || height == 288 || height == 320;
    if (cut == 1) return height == 64 || height == 96 || height == 128 || height == 160 || (wide && (height == 192 || height == 256 || height == 320));
    return cut == 2 && (height == 64 || (wide && height == 128));
}
__host__ __device__ constexpr int instance_height(int NT, int height, int cut)
{
    if (height < 64) height = 64;
    if (NT == 256 && height == 96 && cut != 1) height = 128;
    if (height == 224 && cut == 1) height = 256;
    if (height == 288 && cut == 1) height = 320;
    return height;
}
// Every tile, whole or in pieces, has all its rows in pieces that the kernel has an instance for (it writes nothing otherwise).
constexpr bool tiles_are_covered(int NT)
{
    const int heights[] = {64, 128, 160, 192, 224, 256, 288, 320};
    for (int height : heights)
        for (int rows = 1; rows <= height; rows += rows % kQuantum == 1 ? kQuantum - 2 : 1)  // 1, 31, 32, 33, 63, ..
            for (int pieces = 0; pieces <= 3; ++pieces) {
                const TileCut t = pieces > 0 ? cut_tile(NT, height, rows, pieces) : TileCut{0, 0, height};
                const int taken = instance_height(NT, t.height, t.cut);
                if (!has_instance(NT, taken, t.cut) || taken < t.height || t.height << t.row_cut < rows || t.cut < 0 || t.cut + t.row_cut > pieces) return false;
            }
    return true;
}
static_assert(tiles_are_covered(128) && tiles_are_covered(256), "a tile without an instance");

struct TilePlan {  // lane e = expert e; the same in every workgroup
    int lo, hi;
    int tiles;                  // row tiles (0: no rows)
    int big_incl, small_incl;   // running sums of row tiles times column tiles
    int total_big, total_small;
    int most;                   // quanta a tile takes at most
};
struct Tile2D {
    int expert;
    int row_begin, row_end;
    int n0;      // first output column
    int height;
    int cut;     // log2 of the pieces its columns are cut into (height and rows are those of the piece)
    int hid_shift;  // hidden row of sorted row m of this expert: m + hid_shift
    bool through;   // its hidden rows are written through to memory
    bool once;      // nobody else reads its weights (see gemm_tile)
    int turn;       // of kComputeUnits: where it begins the reduction
};

struct RowRange {  // rows [lo, hi) of expert `lane`; the last expert's hi is the number of rows
    int lo, hi;
};
__device__ __forceinline__ RowRange row_range(const int32_t* __restrict__ offsets, int E_local, int max_rows)
{
    RowRange r{0, 0};
    const int lane = lane_id();
    if (lane < E_local) {  // clamped so that a corrupt offsets array can never index past the buffers
        r.lo = min(max(offsets[lane], 0), max_rows);
        r.hi = min(max(offsets[lane + 1], r.lo), max_rows);
    }
    return r;
}

// The same from the assignments.  e[u]: local expert of assignment (wave * rounds + u) * 64 + lane (-1: none); wavefronts have consecutive ones.
__device__ __forceinline__ RowRange count_rows(const TileRouting& r, int E_local, int A, int rounds, int (&e)[kRoutedRounds], RoutedSort& d)
{
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int map = r.expert_map != nullptr ? r.expert_map[min(lane, r.E - 1)] : lane;  // lane = expert
    const int first = wave * rounds * kWave + lane;
#pragma unroll
    for (int u = 0; u < kRoutedRounds; ++u) e[u] = u < rounds ? r.topk_idx[min(first + u * kWave, A - 1)] : -1;
    reinterpret_cast<uint32_t*>(d.count)[threadIdx.x] = 0u;  // (as many counters as threads)
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRoutedRounds; ++u) {
        const bool ok = u < rounds && first + u * kWave < A && e[u] >= 0 && e[u] < r.E;
        const int m = r.expert_map != nullptr ? __shfl(map, ok ? e[u] : 0, kWave) : e[u];
        e[u] = ok && m >= 0 && m < E_local ? m : -1;
        if (e[u] >= 0) atomicAdd(&d.count[e[u]][lane % kRoutedCopies], 1u);
    }
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int c = 0; c < kRoutedCopies; ++c) total += d.count[lane][c];  // (beyond E_local: zero)
    RowRange range;
    range.hi = wave_inclusive_scan(static_cast<int>(total));
    range.lo = range.hi - static_cast<int>(total);
    if (blockIdx.x == 0) {
        if (wave == 0 && lane < E_local) {
            r.expert_counts[lane] = static_cast<int>(total);
            r.expert_offsets[lane] = range.lo;
            if (lane == E_local - 1) r.expert_offsets[E_local] = range.hi;
        }
#pragma unroll
        for (int u = 0; u < kRoutedRounds; ++u)
            if (u < rounds && first + u * kWave < A && e[u] < 0) r.sorted_of_src[first + u * kWave] = -1;
    }
    return range;
}

// Assignments of sorted rows [row_begin, row_end) of `expert`, whose rows begin at `lo`, into d.list (behind the last barrier).
__device__ __forceinline__ void collect_rows(int expert, int lo, int row_begin, int row_end, int rounds, const int (&e)[kRoutedRounds], RoutedSort& d)
{
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    unsigned long long like[kRoutedRounds];
    int mine = 0;
#pragma unroll
    for (int u = 0; u < kRoutedRounds; ++u) {
        like[u] = __ballot(e[u] == expert);
        mine += __popcll(like[u]);
    }
    if (lane == 0) d.wave_rows[wave] = mine;
    __syncthreads();
    int at = lo - row_begin;
#pragma unroll
    for (int w = 0; w < 7; ++w) at += w < wave ? d.wave_rows[w] : 0;
#pragma unroll
    for (int u = 0; u < kRoutedRounds; ++u) {
        const int row = at + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(like[u] >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(like[u]), 0u)));
        if (e[u] == expert && row >= 0 && row < row_end - row_begin) d.list[row] = (wave * rounds + u) * kWave + lane;
        at += __popcll(like[u]);
    }
    __syncthreads();
}

__device__ __forceinline__ TilePlan plan_tiles(const RowRange& range, int n_tiles, const RowMap& probe)
{
    TilePlan p;
    p.lo = range.lo;
    p.hi = range.hi;
    const int cnt = p.hi - p.lo;
    if (probe.timeline != nullptr) {  // measurement only: when did the row ranges arrive?
        if (__ballot(cnt >= 0) != 0ull) timeline_stamp(probe, 7);
    }
    // one quantum per tile, unless two make the launch a round of tiles shorter
    const bool small = cnt <= kSmallRows;
    const int lean = cnt > 0 ? cut_rows(cnt, 1).tiles : 0, tall = cnt > 0 ? cut_rows(cnt, 2).tiles : 0;
    const int lean_incl = wave_inclusive_scan(small ? 0 : lean * n_tiles), tall_incl = wave_inclusive_scan(small ? 0 : tall * n_tiles);
    p.small_incl = wave_inclusive_scan(small ? lean * n_tiles : 0);
    const int lean_total = wave_read_lane(lean_incl, kWave - 1), tall_total = wave_read_lane(tall_incl, kWave - 1);
    const bool use_tall = (tall_total + kComputeUnits - 1) / kComputeUnits < (lean_total + kComputeUnits - 1) / kComputeUnits;
    p.most = use_tall ? 2 : 1;
    p.tiles = use_tall ? tall : lean;
    p.big_incl = use_tall ? tall_incl : lean_incl;
    p.total_big = use_tall ? tall_total : lean_total;
    p.total_small = wave_read_lane(p.small_incl, kWave - 1);
    return p;
}

// Size of XCD `xcd`'s share of n items of one kind; `begin` receives its first item.  An XCD runs the workgroups whose
// id is its own modulo 8, so the map workgroup -> item decides how much work it gets: of the n items of a kind (big,
// small) every XCD takes a contiguous share of n/8, and the n%8 left over go one each to consecutive XCDs, continuing
// where the previous kind stopped.  Contiguous items share an expert's rows and a few weight panels in one L2.
__device__ __forceinline__ int xcd_share(int n, int xcd, int& rot, int& begin)
{
    const int b = static_cast<int>(static_cast<unsigned>(n) / kXcdCount), r = static_cast<int>(static_cast<unsigned>(n) % kXcdCount);
    const int xr = (xcd - rot) & (kXcdCount - 1);
    begin = xr * b + min(xr, r);
    rot = (rot + r) & (kXcdCount - 1);
    return b + (xr < r ? 1 : 0);
}

// Work item of workgroup `wg`: the big tiles of its XCD first, then the small ones, which fill the ragged end.  The tiles of an
// XCD's last (or only) round are cut into two, four or eight pieces where its compute units have room for that: a tile
// runs on one compute unit for as long as its K loop takes, however idle the others are.  (32 skewed experts of
// 2048 x 8192, 16384 tokens, second contraction: 584 tiles of 200 us in 2.3 rounds, 645 -> 545 us with the K loop below.)
//   A compute unit takes in about 25 bytes a cycle of what its XCD's L2 holds, and that bounds a piece, not its MFMAs: every cut
// goes where it leaves the fewer rows of operands, across the rows of the tile as long as these are more than its columns.
// Both contractions, columns only in up to four pieces -> either way in up to eight: four experts of 1024 x 4096, 800 rows
// 63.7 -> 47.8 us; one of 2048 x 8192, 130 rows 75.4 -> 60.0; eight of 1024 x 4096, 2000 rows 92.3 -> 81.5; 16 of them, 3062
// rows (the second contraction alone is cut: 256 x 64 -> 128 x 128) 101.9 -> 96.4.
constexpr int kUnitsPerXcd = kComputeUnits / kXcdCount;
template <bool STREAMS>
__device__ __forceinline__ bool locate_tile(const RowRange& range, int NT, int N, int wg, const RowMap& probe, Tile2D& out)
{
    const int n_tiles = (N + NT - 1) / NT;
    const TilePlan p = plan_tiles(range, n_tiles, probe);
    const int xcd = static_cast<int>(static_cast<unsigned>(wg) % kXcdCount);
    int pos = static_cast<int>(static_cast<unsigned>(wg) / kXcdCount);
    int rot = 0, begin = 0, begin_small = 0;
    const int share = xcd_share(p.total_big, xcd, rot, begin), share_small = xcd_share(p.total_small, xcd, rot, begin_small);
    const int last_round = (share + share_small) % kUnitsPerXcd, whole = share + share_small - last_round;
    int row_cut = 0;
    out.cut = last_round > kUnitsPerXcd / 2 ? 0 : (last_round > kUnitsPerXcd / 4 ? 1 : (last_round > kUnitsPerXcd / 8 ? 2 : 3));
    int piece = 0;
    if (pos < whole) {
        out.cut = 0;
    } else {
        piece = (pos - whole) & ((1 << out.cut) - 1);
        pos = whole + ((pos - whole) >> out.cut);
    }
    const bool small = pos >= share;
    if (small) {
        pos -= share;
        begin = begin_small;
        if (pos >= share_small) return false;
    }
    const int j = begin + pos;
    const unsigned long long owner = __ballot(j < (small ? p.small_incl : p.big_incl));
    const int e = __builtin_ctzll(owner);  // (j is below the total: some lane owns it)
    const int e_lo = wave_read_lane(p.lo, e), e_hi = wave_read_lane(p.hi, e), e_rt = wave_read_lane(p.tiles, e);
    const int r = j - (wave_read_lane(small ? p.small_incl : p.big_incl, e) - e_rt * n_tiles);
    // Order of the expert's tiles.  With many row tiles, consecutive tiles form blocks of 32, up to eight columns wide: the 32
    // workgroups of an XCD that run side by side share 4 activation and 8 weight panels in their L2, against 16 and 2 when the
    // rows of a column simply follow each other.  Four column tiles: blocks of 8 x 4 (32768 tokens, 8 experts of 1024 x 4096:
    // 521 us with rows simply following each other, 511).  Remaining row tiles (and small experts) run row tile fastest.
    const unsigned block_cols = min(static_cast<unsigned>(n_tiles & -n_tiles), 8u), block_rows = 32u / block_cols;  // powers of two
    int row_tile, col_tile;
    const int blocked_rows = block_cols > 1u ? (e_rt & -static_cast<int>(block_rows)) : 0;
    if (r < blocked_rows * n_tiles) {
        const unsigned rbk = uniform_udiv(static_cast<unsigned>(r), block_rows * static_cast<unsigned>(n_tiles));
        const unsigned in_rb = static_cast<unsigned>(r) - rbk * (block_rows * static_cast<unsigned>(n_tiles));
        const unsigned in_b = in_rb % 32u, in_col = uniform_udiv(in_b, block_rows);
        col_tile = static_cast<int>(in_rb / 32u * block_cols + in_col);
        row_tile = static_cast<int>(rbk * block_rows + (in_b - in_col * block_rows));
    } else {
        const unsigned rr = static_cast<unsigned>(r - blocked_rows * n_tiles), rows_left = static_cast<unsigned>(e_rt - blocked_rows);
        const unsigned c = uniform_udiv(rr, rows_left);
        col_tile = static_cast<int>(c);
        row_tile = blocked_rows + static_cast<int>(rr - c * rows_left);
    }
    const int tiles = p.total_big + p.total_small;
    const bool by224 = tiles > kComputeUnits / 2, by160 = tiles > kComputeUnits || (by224 && __ballot(p.hi - p.lo > 160) == 0ull);
    const TileRows t = cut_rows(e_hi - e_lo, p.most, by160, by224);
    // quanta: every tile takes extra / tiles, the first extra % tiles one more
    const int each = t.extra >= 2 * t.tiles ? 2 : (t.extra >= t.tiles ? 1 : 0), more = t.extra - each * t.tiles;
    const int begin_row = e_lo + row_tile * t.height + (row_tile * each + min(row_tile, more)) * kQuantum;
    int height = t.height + (each + (row_tile < more ? 1 : 0)) * kQuantum;
    int row_begin = begin_row, row_end = min(begin_row + height, e_hi);
    if (out.cut > 0) {
        const TileCut t = cut_tile(NT, height, __builtin_amdgcn_readfirstlane(row_end - row_begin), out.cut);
        if (piece >= 1 << (t.cut + t.row_cut)) return false;
        out.cut = t.cut;
        row_cut = t.row_cut;
        height = t.height;
        if (t.row_cut > 0) {
            row_begin += (piece & ((1 << t.row_cut) - 1)) * height;
            row_end = min(row_end, row_begin + height);
            piece >>= t.row_cut;
        }
    }
    const int n0 = col_tile * NT + piece * (NT >> out.cut);
    if (n0 >= N || row_begin >= row_end) return false;  // a piece of a ragged last column tile, or of a tile of few rows
    // every lane holds the same values; readfirstlane tells the compiler so (scalar registers)
    out.expert = __builtin_amdgcn_readfirstlane(e);
    out.n0 = __builtin_amdgcn_readfirstlane(n0);
    out.cut = __builtin_amdgcn_readfirstlane(out.cut);
    out.row_begin = __builtin_amdgcn_readfirstlane(row_begin);
    out.row_end = __builtin_amdgcn_readfirstlane(row_end);
    out.height = __builtin_amdgcn_readfirstlane(instance_height(NT, height, out.cut));
    // Hidden rows of experts with several row tiles in a launch of at most two rounds: nothing overlaps the last stores there, and
    // what they leave in the L2s has to be written back when the kernel ends.  Written through, both contractions: 8192 tokens, 8
    // experts of 1024 x 4096 152.2 -> 147.0 us (two rounds), 4 experts, 2048 tokens 65.9 -> 63.0, one, 6000 tokens 124.3 -> 118.3.  Not in
    // longer launches (32768 tokens, 8 experts: 520 -> 535 us) and not where the weights of experts of one row tile bound the
    // launch (16 experts, 2500 tokens: 87.0 -> 89.7): non-temporal stores.
    out.through = __builtin_amdgcn_readfirstlane(e_rt >= 2 && p.total_big + p.total_small <= 2 * kComputeUnits ? 1 : 0) != 0;
    // Where the reduction begins.  Rows a power of two bytes apart put the same columns of all rows on few memory channels, and compute
    // units that walk the reduction in step all ask these, so the XCDs begin at different places.  The tiles of one XCD, which share
    // panels in their L2, stay in step - but where much weight is streamed for experts of one or two row tiles: their activations fit the L2 as
    // a whole, and every column tile has a place of its own (its row tiles and pieces, which share weights, stay together).  1200 tokens,
    // 16 experts of 4096 x 16384 858 -> 747 us, 4000 1361 -> 1221; two row tiles: 4000 of 8 1064 -> 1042, 5000 of 16 of 2048 x 8192 447 -> 441;
    // less weight: 2500 of 8 of 1024 x 4096 61.5 and 62.2.  The place decides the order of the fp32 sums and so the last bit of some results, not
    // their error: against 64 bits 2.349e-3 of the result with and without (16384 skewed tokens, 32 of 2048 x 8192).
    out.turn = xcd * kUnitsPerXcd;
    if (STREAMS && e_rt <= 2) out.turn += col_tile % kUnitsPerXcd;
    out.turn = __builtin_amdgcn_readfirstlane(out.turn);
    out.once = STREAMS && __builtin_amdgcn_readfirstlane(e_rt == 1 && row_cut == 0 && height <= kTileRows ? 1 : 0) != 0;
    out.hid_shift = __builtin_amdgcn_readfirstlane(kHiddenRowBlock * e - (e_lo & (kHiddenRowBlock - 1)));
    return true;
}

// ---------------------------------------------------------------------------- tile
// D += A * B in accumulator f of a wavefront.  The first 64 accumulators are the accumulator half of the register file;
// a tall tile's others are ordinary registers.
template <bool ACC_HALF>
__device__ __forceinline__ void mfma_16x16x32(bf16x8_t a, bf16x8_t b, f32x4_t& c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (ACC_HALF) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
#else
    (void)a; (void)b; (void)c;
#endif
}

// Ring depths of an H x NT tile (K tiles of 64, activations / weights): as many as fit the LDS, up to eight (small tiles wait
// for memory, not for the matrix cores).  The activations, which fewer compute units share, get the third stage where
// only one operand can have it.
__host__ __device__ constexpr bool ring_fits(int H, int NT, int sa, int sb) { return (sa * H + sb * NT) * kKTile * 2 <= kLdsBytes; }
__host__ __device__ constexpr int both_stages(int H, int NT)
{
    int s = 8;
    while (!ring_fits(H, NT, s, s)) --s;
    return s;
}
__host__ __device__ constexpr int act_stages(int H, int NT) { return both_stages(H, NT) == 2 && ring_fits(H, NT, 3, 2) ? 3 : both_stages(H, NT); }
__host__ __device__ constexpr int wgt_stages(int H, int NT) { return both_stages(H, NT); }
__host__ __device__ constexpr int tile_ring_bytes(int H, int NT) { return (act_stages(H, NT) * H + wgt_stages(H, NT) * NT) * kKTile * 2; }

// Wavefronts side by side over the columns of a tile (the others over its rows): the LDS of a compute unit delivers 128
// bytes a cycle, and a narrow tile waits for the operand fetches of its wavefronts (H/WM + NT/WN rows each), so the
// arrangement with the least of them.
__host__ __device__ constexpr int wave_columns(int H, int NT, int waves)
{
    int best = 0, cost = 1 << 30;
    for (int wn = waves / 2; wn >= 1; wn /= 2) {
        const int wm = waves / wn;
        if (H % (16 * wm) != 0 || NT % (32 * wn) != 0 || wm > 4 || NT / wn > 512 / waves) continue;  // (weight fragments are double: registers)
        if (H / wm + NT / wn < cost) {
            best = wn;
            cost = H / wm + NT / wn;
        }
    }
    return best;
}

template <int H, int NT, int WAVES_, bool ONCE>
struct GemmTile {
    static constexpr int RB = kKTile * 2;           // bytes per tile row
    static constexpr int WAVES = WAVES_;
    static constexpr int WN = wave_columns(H, NT, WAVES), WM = WAVES / WN;
    static constexpr int SA = act_stages(H, NT), SB = wgt_stages(H, NT);
    static constexpr int A_BYTES = H * RB, W_BYTES = NT * RB;  // of a stage
    static constexpr int WTM = H / WM, WTN = NT / WN;  // outputs of a wavefront
    static constexpr int TM = WTM / 16, TN = WTN / 16;
    static constexpr int SLOTS = TM * TN;           // MFMAs of a K step (two K steps of 32 per K tile)
    static constexpr int HALF = SLOTS / 2;          // MFMAs of the last K step in front of the hand-over
    static constexpr int GA = H / 8, GW = NT / 8;   // groups of eight rows: one direct-to-LDS load each
    static constexpr int LA = (GA + WAVES - 1) / WAVES, LW = (GW + WAVES - 1) / WAVES, LPW = LA + LW;  // loads per K tile and wavefront
    static constexpr int LOAD_SLOTS = SLOTS;        // slots over which a K tile's loads are spread
    // loads in flight behind the next K tile at a hand-over: its weights were followed by activations of a later tile (if those
    // run ahead) and by SB - 2 whole refills
    static constexpr int IN_FLIGHT = (SA > SB ? LA : 0) + (SB - 2) * LPW;
    static constexpr int ACC_HALF = 256 / WAVES;  // accumulators in the accumulator half of the registers
    static_assert(H % 32 == 0 && TN % 2 == 0 && SA >= SB && SA - SB <= 1 && SB >= 2 && IN_FLIGHT < 64, "tile shape");
    static_assert(tile_ring_bytes(H, NT) <= kLdsBytes, "LDS of a compute unit");

    f32x4_t acc[TM][TN];
    bf16x8_t fw[2][TN], fa[TM];
    uint32_t off_a[LA], off_w[LW];
    uint32_t frag_w[2], frag_a[2];  // LDS byte offsets of the operand fetches of the two K steps
    const unsigned char *act_b, *wgt_b;
    int64_t a_step, a_back, w_back; // bytes of the activation operand from K tile to K tile, of both from the last one to the first
    int a_left, w_left, nk;         // K tiles behind those the pointers are at, K tiles of the reduction
    unsigned char* smem;            // activation stages, then weight stages
    uint32_t smem_addr;
    int wave;

    // groups of this wavefront: wave, wave + WAVES, ..; past the last one it is loaded once more (every wavefront then has
    // the same number of loads in flight)
    __device__ __forceinline__ int group_a(int i) const { return GA % WAVES == 0 ? i * WAVES + wave : min(i * WAVES + wave, GA - 1); }
    __device__ __forceinline__ int group_w(int i) const { return GW % WAVES == 0 ? i * WAVES + wave : min(i * WAVES + wave, GW - 1); }
    __device__ __forceinline__ void issue_a(uint32_t st, int i) { lds_dma_16B(act_b, off_a[i], smem_addr + st + group_a(i) * 1024); }
    __device__ __forceinline__ void issue_w(uint32_t st, int i)
    {
        const uint32_t at = smem_addr + SA * A_BYTES + st + group_w(i) * 1024;
        if constexpr (ONCE) lds_dma_16B_stream(wgt_b, off_w[i], at);
        else lds_dma_16B(wgt_b, off_w[i], at);
    }

    // On to the next K tile of the reduction; behind the last one follows the first (see gemm_tile).
    // (A loop of few MFMAs is bound by the issue of its other instructions, so the way back is kept and rings of equal depth share a
    // counter: the 64 x 32 tile's K tile had 75 instructions, 58 of them scalar, and has 58.  One expert of 2048 x 8192, 130 rows 61.0 ->
    // 55.4 us; the large tiles gain as well, 32 of them, 16384 rows 1042 -> 1028.)
    __device__ __forceinline__ void step_a()
    {
        const bool wrap = a_left == 0;
        a_left = wrap ? nk - 1 : a_left - 1;
        act_b += wrap ? a_back : a_step;
    }
    __device__ __forceinline__ void step_w()
    {
        const bool wrap = w_left == 0;
        w_left = wrap ? nk - 1 : w_left - 1;
        wgt_b += wrap ? w_back : static_cast<int64_t>(RB);
    }
    __device__ __forceinline__ void step_both()  // SA == SB: behind the first loads both operands are at one K tile
    {
        const bool wrap = a_left == 0;
        a_left = wrap ? nk - 1 : a_left - 1;
        act_b += wrap ? a_back : a_step;
        wgt_b += wrap ? w_back : static_cast<int64_t>(RB);
    }

    // Stages of one operand's ring around a K tile: the one read now, the next one, the one whose refill is being completed.
    struct Stages {
        uint32_t cur, nxt, prev;
        __device__ __forceinline__ void advance(uint32_t bytes, uint32_t ring)
        {
            prev = cur;
            cur = nxt;
            nxt = nxt + bytes == ring ? 0 : nxt + bytes;
        }
    };

    // Flags of a K tile that is not in the steady state: the refill begun at the previous hand-over had activations / weights, the
    // one begun here has; K tiles behind the next one are in flight as in the steady state, or (bits 5 and up) so many.
    static constexpr unsigned kPrevA = 1u, kPrevW = 2u, kThisA = 4u, kThisW = 8u, kFull = 16u;
    __device__ __forceinline__ void wait_tail(unsigned tiles)
    {
        constexpr bool deep = SA == SB;
        if (deep && SA > 5 && tiles >= 4) wait_vmcnt<(SA > 5 ? 4 : 0) * LPW>();
        else if (deep && SA > 4 && tiles == 3) wait_vmcnt<(SA > 4 ? 3 : 0) * LPW>();
        else if (deep && SA > 3 && tiles == 2) wait_vmcnt<(SA > 3 ? 2 : 0) * LPW>();
        else if (deep && SA > 2 && tiles == 1) wait_vmcnt<(SA > 2 ? 1 : 0) * LPW>();
        else wait_vmcnt<0>();
    }

    // MFMAs of one K tile.  Operand fetches run one K step ahead: the weights' registers are double, an activation
    // fragment is fetched into the register its last MFMA has just read.  At the hand-over (everyone's share of the next K
    // tile has landed, everyone is done reading this one) in the middle of the last K step the stages of this tile are
    // free: their refill, weights first, is spread over the slots up to the middle of the next K tile's first K step.
    //   NEXT: there is a next K tile.  STEADY: a refill was begun at the previous hand-over and one begins here, both operands;
    //   otherwise the flags say.
    template <bool NEXT, bool STEADY>
    __device__ __forceinline__ void k_tile(const Stages& sa, const Stages& sw, unsigned flags)
    {
        const unsigned char *ac = smem + sa.cur, *an = smem + sa.nxt;
        const unsigned char *wc = smem + SA * A_BYTES + sw.cur, *wnx = smem + SA * A_BYTES + sw.nxt;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bool last = ks == 1;
#pragma unroll
            for (int m = 0; m < SLOTS; ++m) {
                const int a = m % TN, b = m / TN;
                if (NEXT && last && m == HALF) {
                    if (STEADY || (flags & kFull) != 0u) wait_vmcnt<IN_FLIGHT>();
                    else wait_tail(flags >> 5);
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // my operand fetches from this tile are complete
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    if constexpr (SA == SB) {
                        if (STEADY || (flags & kThisA) != 0u) step_both();
                    } else {
                        if (STEADY || (flags & kThisA) != 0u) step_a();
                        if (STEADY || (flags & kThisW) != 0u) step_w();
                    }
                }
                if (b * TN + a < ACC_HALF) mfma_16x16x32<true>(fw[ks][a], fa[b], acc[b][a]);
                else mfma_16x16x32<false>(fw[ks][a], fa[b], acc[b][a]);
                __builtin_amdgcn_sched_barrier(0);
                if (!last) {
                    if (a == TN - 1) fa[b] = *reinterpret_cast<const bf16x8_t*>(ac + frag_a[1] + b * 16 * RB);
#pragma unroll
                    for (int r = 0; r < TN; ++r)
                        if (m == (r * SLOTS / TN + 1 < SLOTS ? r * SLOTS / TN + 1 : SLOTS - 1)) fw[1][r] = *reinterpret_cast<const bf16x8_t*>(wc + frag_w[1] + r * 16 * RB);
                } else if (NEXT) {
#pragma unroll
                    for (int r = 0; r < TN; ++r) {
                        const int p = HALF + 2 * r < SLOTS ? HALF + 2 * r : SLOTS - 1;
                        if (m == p) fw[0][r] = *reinterpret_cast<const bf16x8_t*>(wnx + frag_w[0] + r * 16 * RB);
                    }
#pragma unroll
                    for (int r = 0; r < TM; ++r) {
                        const int free = r * TN + TN - 1;  // its last MFMA of this K step
                        const int want = HALF + 2 * r + 1 > free ? HALF + 2 * r + 1 : free;
                        const int p = want < SLOTS ? want : SLOTS - 1;
                        if (m == p) fa[r] = *reinterpret_cast<const bf16x8_t*>(an + frag_a[0] + r * 16 * RB);
                    }
                }
                if (last && m >= HALF) {
                    if (NEXT) {
#pragma unroll
                        for (int i = 0; i < LPW; ++i)
                            if (i * LOAD_SLOTS / LPW == m - HALF) {
                                if (i < LW) {
                                    if (STEADY || (flags & kThisW) != 0u) issue_w(sw.cur, i < LW ? i : 0);
                                } else {
                                    if (STEADY || (flags & kThisA) != 0u) issue_a(sa.cur, i >= LW ? i - LW : 0);
                                }
                            }
                    }
                } else {
                    const int p = SLOTS - HALF + ks * SLOTS + m;
#pragma unroll
                    for (int i = 0; i < LPW; ++i)
                        if (i * LOAD_SLOTS / LPW == p) {
                            if (i < LW) {
                                if (STEADY || (flags & kPrevW) != 0u) issue_w(sw.prev, i < LW ? i : 0);
                            } else {
                                if (STEADY || (flags & kPrevA) != 0u) issue_a(sa.prev, i >= LW ? i - LW : 0);
                            }
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
};

// ONCE: the weights are read by this workgroup alone and loaded with the streaming hint, which leaves the L2 to the activations.  Tiles that share
// a panel lose by it (8 experts of 1024 x 4096, 8192 tokens 143.7 -> 159.7 us), and so do weights that lie in the memory-side cache from the call
// before, which such loads do not keep there (see weights_are_streamed).
// ROUTED: the tile's rows are the assignments in RoutedSort::list at the begin of the LDS, which the ring overwrites once they are read.
template <int H, int NT, int WAVES, int EPI, bool ONCE, bool ROUTED>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ act, const bf16_t* __restrict__ wexp, const bf16_t* __restrict__ bias_e,
                                          int row_begin, int row_end, int hid_shift, bool through, int turn, int n0, int K, int N, bf16_t* __restrict__ out,
                                          unsigned char* smem, const RowMap& map, const TileRouting& route)
{
    typedef GemmTile<H, NT, WAVES, ONCE> G;
    constexpr int RB = G::RB, SA = G::SA, SB = G::SB, TM = G::TM, TN = G::TN, LA = G::LA, LW = G::LW;
    G g;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave / G::WN, wn = wave % G::WN;
    g.wave = wave;
    g.smem = smem;
    g.smem_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem));
    constexpr bool HIDDEN_ACT = EPI == kEpiNone || EPI == kEpiKeepSorted, HIDDEN_OUT = !HIDDEN_ACT;  // the first contraction writes what the second reads
    const int r8 = lane >> 3, c8 = lane & 7;
    const int nk = K / kKTile;
    const int k0 = static_cast<int>(static_cast<unsigned>(turn) * static_cast<unsigned>(nk) / kComputeUnits);
    g.nk = nk;
    g.a_left = nk - 1 - k0;
    g.w_left = nk - 1 - k0;
    g.a_step = HIDDEN_ACT ? kKTile / 8 * kHiddenRowBlock * 16 : RB;
    g.a_back = -g.a_step * (nk - 1);
    g.w_back = -static_cast<int64_t>(RB) * (nk - 1);
    g.act_b = uniform_ptr(reinterpret_cast<const unsigned char*>(act) + static_cast<size_t>(k0) * g.a_step);
    g.wgt_b = uniform_ptr(reinterpret_cast<const unsigned char*>(wexp) + static_cast<size_t>(k0) * RB);

    // A stage holds the rows of a K tile of one operand.  One wavefront-wide load covers 8 consecutive rows (1 KiB of LDS): lane ->
    // row lane/8 of the group and the 16-byte chunk (lane%8) ^ (row/2 % 8).  Sources are 32-bit byte offsets from the two
    // (uniform) base pointers.
    const uint32_t row_bytes = static_cast<uint32_t>(K) * 2u;
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int row = g.group_w(i) * 8 + r8;
        g.off_w[i] = static_cast<uint32_t>(min(n0 + row, N - 1)) * row_bytes + ((c8 ^ ((row >> 1) & 7)) * 16);
    }
    // Gathered activation rows need their row ids first - a dependent load in front of the tile's first loads.  The ids of
    // this wavefront's rows are fetched straight into LDS (where its own loads of the last stage will land), the weights of the
    // first K tiles behind them, and the ids are read back once only the weights are outstanding: ids and weights travel
    // together.  (Through a register the id load would be awaited with vmcnt(0), i.e. together with the weights.)
    const bool gather = !ROUTED && map.a_row != nullptr;
    constexpr int ID_LOADS = (LA + 7) / 8;
    const uint32_t ids_at = static_cast<uint32_t>((SA - 1) * G::A_BYTES + wave * 1024);
    static_assert(ID_LOADS * 256 <= 1024, "row ids fit the wavefront's first group of a stage");
    if (gather) {
        const unsigned char* ids_b = uniform_ptr(reinterpret_cast<const unsigned char*>(map.a_row));
#pragma unroll
        for (int i = 0; i < ID_LOADS; ++i) {
            const int row = g.group_a(min(i * 8 + r8, LA - 1)) * 8 + c8;
            lds_dma_4B(ids_b, static_cast<uint32_t>(min(row_begin + row, row_end - 1)) * 4u, g.smem_addr + ids_at + i * 256);
        }
    }
    auto chunk_of = [&](int i) { return static_cast<uint32_t>((c8 ^ (((g.group_a(i) * 8 + r8) >> 1) & 7)) * 16); };
    if constexpr (ROUTED) {
        const RoutedSort& d = *reinterpret_cast<const RoutedSort*>(smem);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            unsigned r = static_cast<unsigned>(d.list[min(g.group_a(i) * 8 + r8, row_end - row_begin - 1)]);
            if (route.k > 1) r /= static_cast<unsigned>(route.k);
            g.off_a[i] = r * row_bytes + chunk_of(i);
        }
        __syncthreads();  // (the list has been read: its place may be written)
    }
    const int first_a = min(nk, SA), first_w = min(nk, SB);
    auto first_weights = [&](int s) {
        if (s > 0) g.step_w();
#pragma unroll
        for (int i = 0; i < LW; ++i) g.issue_w(static_cast<uint32_t>(s * G::W_BYTES), i);
    };
    auto first_activations = [&](int s) {
        if (s > 0) g.step_a();
#pragma unroll
        for (int i = 0; i < LA; ++i) g.issue_a(static_cast<uint32_t>(s * G::A_BYTES), i);
    };
    first_weights(0);
    if (first_w > 1) first_weights(1);
    if (gather) {
        if (first_w > 1) wait_vmcnt<2 * LW>();
        else wait_vmcnt<LW>();
    }
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        if constexpr (HIDDEN_ACT) {
            // consecutive lanes take consecutive rows of one piece (whole lines); the 1 KiB group in LDS is then [piece][row],
            // the pieces of odd groups pairwise exchanged so that the two groups of a fragment sit in different banks
            const int row = g.group_a(i) * 8 + c8;
            const uint32_t h = static_cast<uint32_t>(min(row_begin + row, row_end - 1) + hid_shift);
            g.off_a[i] = hidden_offset(h, static_cast<uint32_t>(r8 ^ (g.group_a(i) & 1)), static_cast<uint32_t>(K) / 8u);
            continue;
        }
        const int row = g.group_a(i) * 8 + r8;
        if constexpr (ROUTED) continue;
        int r = min(row_begin + row, row_end - 1);  // rows past the tile end re-read the last valid row
        if (gather) {
            r = *reinterpret_cast<const int*>(smem + ids_at + i * 32 + r8 * 4);
            if (map.a_div > 1) r = static_cast<int>(static_cast<unsigned>(r) / static_cast<unsigned>(map.a_div));
        }
        g.off_a[i] = static_cast<uint32_t>(r) * row_bytes + ((c8 ^ ((row >> 1) & 7)) * 16);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the ids have been read: their place may be written)
    first_activations(0);
    if (first_a > 1) first_activations(1);
    for (int s = 2; s < first_a; ++s) {
        if (s < first_w) first_weights(s);
        first_activations(s);
    }
    // operand row = base + lane%16; K step ks uses chunk 4 ks + lane/16
    {
        const int row = lane & 15, quad = lane >> 4;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint32_t f = static_cast<uint32_t>(row * RB + (((4 * ks + quad) ^ (row >> 1)) * 16));
            g.frag_a[ks] = static_cast<uint32_t>(wm * G::WTM * RB) +
                           (HIDDEN_ACT ? static_cast<uint32_t>((row >> 3) * 1024 + ((4 * ks + quad) ^ (row >> 3)) * 128 + (row & 7) * 16) : f);
            g.frag_w[ks] = f + static_cast<uint32_t>(wn * G::WTN * RB);
        }
    }
    // first K tile complete: behind it come the activations of the second and whatever fills the rings
    if (first_a == SA) wait_vmcnt<LA + (SA == SB ? SA - 2 : 0) * G::LPW + (SA > SB ? LA : 0)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    timeline_stamp(map, 2);
    const unsigned char* w_smem = smem + SA * G::A_BYTES;
#pragma unroll
    for (int r = 0; r < TN; ++r) g.fw[0][r] = *reinterpret_cast<const bf16x8_t*>(w_smem + g.frag_w[0] + r * 16 * RB);
#pragma unroll
    for (int r = 0; r < TM; ++r) g.fa[r] = *reinterpret_cast<const bf16x8_t*>(smem + g.frag_a[0] + r * 16 * RB);
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int a = 0; a < TN; ++a) g.acc[b][a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // the accumulators have to be there before the first MFMA reads them, and the last MFMA done before they are read below (the
    // compiler sees neither)
#define EXF_PIN_ACC()                                                                        \
    do {                                                                                     \
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");                                   \
        _Pragma("unroll") for (int b = 0; b < TM; ++b) _Pragma("unroll") for (int a = 0; a < TN; ++a) \
        {                                                                                    \
            if (b * TN + a < G::ACC_HALF) asm volatile("" : "+a"(g.acc[b][a]));              \
            else asm volatile("" : "+v"(g.acc[b][a]));                                       \
        }                                                                                    \
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");                                   \
    } while (0)
    EXF_PIN_ACC();

    typename G::Stages sa{0u, static_cast<uint32_t>(G::A_BYTES), 0u}, sw{0u, static_cast<uint32_t>(G::W_BYTES), 0u};
    auto advance = [&]() {
        sa.advance(G::A_BYTES, SA * G::A_BYTES);
        sw.advance(G::W_BYTES, SB * G::W_BYTES);
    };
    auto flags_of = [&](int kt) {
        unsigned flags = (kt + SA < nk ? G::kThisA : 0u) | (kt + SB < nk ? G::kThisW : 0u);
        if (kt > 0) flags |= (kt - 1 + SA < nk ? G::kPrevA : 0u) | (kt - 1 + SB < nk ? G::kPrevW : 0u);
        return flags | (kt + SA <= nk ? G::kFull : static_cast<unsigned>(nk - 2 - kt) << 5);
    };
    int kt = 0;
    if (nk > 1) {
        g.template k_tile<true, false>(sa, sw, flags_of(0));
        advance();
        for (kt = 1; kt + SA < nk; ++kt) {
            g.template k_tile<true, true>(sa, sw, 0u);
            advance();
        }
        for (; kt + 1 < nk; ++kt) {
            g.template k_tile<true, false>(sa, sw, flags_of(kt));
            advance();
        }
    }
    g.template k_tile<false, false>(sa, sw, 0u);
    timeline_stamp(map, 3);
    EXF_PIN_ACC();
#undef EXF_PIN_ACC

    // ---- epilogue -----------------------------------------------------------------------------
    // A lane holds, for the 16 x 16 block (b, a), row lane%16 and columns 4*(lane/16) .. +3.  For two blocks side by side the
    // odd rows of 16 lanes of the first trade with the even ones of the second: every lane then holds eight
    // consecutive columns of one block, 16 bytes.
    const int quad = lane >> 4;
    const int n_lane = n0 + wn * G::WTN + (quad & 1) * 16 + (quad >> 1) * 8;
    int dst[TM];
    float scale[TM];
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        dst[b] = row_begin + wm * G::WTM + b * 16 + (lane & 15);
        scale[b] = 1.0f;
    }
    if constexpr (HIDDEN_ACT) {
        if (map.out_row != nullptr) {
#pragma unroll
            for (int b = 0; b < TM; ++b) dst[b] = map.out_row[min(dst[b], row_end - 1)];
#pragma unroll
            for (int b = 0; b < TM; ++b) scale[b] = map.out_scale[dst[b]];
        }
    }
    auto finish = [&](auto written_through) {
#pragma unroll
        for (int a = 0; a < TN; a += 2) {
            const int n = n_lane + a * 16;
            float bias_v[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) bias_v[q][v] = 0.0f;
            if (bias_e != nullptr) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        bias_v[q][v] = bf16_to_f32(bias_e[min(n0 + wn * G::WTN + (a + q) * 16 + quad * 4 + v, N - 1)]);
            }
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                uint32_t w[2][2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float z = g.acc[b][a + q][r] + bias_v[q][r];
                        if constexpr (EPI == kEpiGeluErf) z = gelu_erf_fast(z);
                        else if constexpr (EPI == kEpiGeluTanh) z = gelu_tanh_fast(z);
                        else if constexpr (EPI == kEpiNone) z *= scale[b];
                        v[r] = z;
                    }
                    w[q][0] = pack_bf16x2(v[0], v[1]);
                    w[q][1] = pack_bf16x2(v[2], v[3]);
                }
                const auto s0 = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
                const int m = row_begin + wm * G::WTM + b * 16 + (lane & 15);
                uint4* to;
                if constexpr (HIDDEN_OUT)
                    to = reinterpret_cast<uint4*>(reinterpret_cast<unsigned char*>(out) +
                                                  hidden_offset(static_cast<uint32_t>(m + hid_shift), static_cast<uint32_t>(n) / 8u, static_cast<uint32_t>(N) / 8u));
                else
                    to = reinterpret_cast<uint4*>(out + static_cast<size_t>(dst[b]) * N + n);
                if (m < row_end && n < N) {  // N % 64 == 0: eight columns are inside or outside together
                    if constexpr (EPI == kEpiKeepSorted) {
                        const uint4 y = make_uint4(s0[0], s1[0], s0[1], s1[1]);
                        store_stream16(reinterpret_cast<uint4*>(map.sorted_out + static_cast<size_t>(m) * N + n), y);
                        const uint32_t p[4] = {y.x, y.y, y.z, y.w};
                        uint32_t o[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) o[c] = pack_bf16x2(fmaf(scale[b], __uint_as_float(p[c] << 16), 0.0f), fmaf(scale[b], __uint_as_float(p[c] & 0xffff0000u), 0.0f));
                        store_stream16(to, make_uint4(o[0], o[1], o[2], o[3]));
                    } else if constexpr (decltype(written_through)::value) store_through16(to, make_uint4(s0[0], s1[0], s0[1], s1[1]));
                    else store_stream16(to, make_uint4(s0[0], s1[0], s0[1], s1[1]));
                }
            }
        }
    };
    if (HIDDEN_OUT && through) finish(std::integral_constant<bool, HIDDEN_OUT>());
    else finish(std::false_type());

    // The columns of the sorted rows that fall to this tile's outputs.  Behind the hidden activations, which the next launch waits for, and past the L2 like these: in
    // front of the epilogue, as ordinary stores, they made that launch longer as well (2500 rows, five experts of 832 x 3328: 30.8 us with a dispatch launch, 35.9 with
    // these; the layer 65.4, 70.8 and now 60.5 to 63.3; 397 top-2, 10 of 1024 x 4096 66.6, 68.1, 64.9).
    if constexpr (ROUTED) {
        const int pieces = K / 8, piece_begin = static_cast<int>(static_cast<int64_t>(n0) * pieces / N);
        const int piece_end = static_cast<int>(static_cast<int64_t>(min(n0 + NT, N)) * pieces / N);
        for (int piece = piece_begin + c8; piece < piece_end; piece += 8) {
            f32x4_t v[LA];  // (16 bytes)
#pragma unroll
            for (int i = 0; i < LA; ++i) v[i] = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const unsigned char*>(act) + (g.off_a[i] - chunk_of(i)) + piece * 16);
#pragma unroll
            for (int i = 0; i < LA; ++i) {
                const int row = row_begin + (i * WAVES + wave) * 8 + r8;
                if (row < row_end) __builtin_nontemporal_store(v[i], reinterpret_cast<f32x4_t*>(route.sorted_act) + static_cast<size_t>(row) * pieces + piece);
            }
        }
    }
}

template <int NT, int WAVES, int EPI, bool STREAMS, bool ROUTED>
__device__ __forceinline__ void run_tile(const Tile2D& tile, const bf16_t* __restrict__ act, const bf16_t* __restrict__ weight, const bf16_t* __restrict__ bias,
                                         int K, int N, bf16_t* __restrict__ out, unsigned char* smem, const RowMap& map, const TileRouting& route)
{
    const bf16_t* wexp = weight + static_cast<size_t>(tile.expert) * N * K;
    const bf16_t* bias_e = bias != nullptr ? bias + static_cast<size_t>(tile.expert) * N : nullptr;
#define EXF_CASE(H, CUT, ONCE)                                                                                                                        \
    case (CUT) * 16 + (H) / kQuantum:                                                                                                                 \
        if constexpr (has_instance(NT, H, CUT) && (!(ONCE) || H <= kTileRows))                                                                        \
            gemm_tile<H, (NT >> CUT), WAVES, EPI, ONCE, ROUTED>(act, wexp, bias_e, tile.row_begin, tile.row_end, tile.hid_shift, tile.through, tile.turn,     \
                                                        tile.n0, K, N, out, smem, map, route);                                                               \
        break
#define EXF_CASES(CUT, ONCE)  \
    EXF_CASE(64, CUT, ONCE);  \
    EXF_CASE(96, CUT, ONCE);  \
    EXF_CASE(128, CUT, ONCE); \
    EXF_CASE(160, CUT, ONCE); \
    EXF_CASE(192, CUT, ONCE); \
    EXF_CASE(224, CUT, ONCE); \
    EXF_CASE(256, CUT, ONCE); \
    EXF_CASE(288, CUT, ONCE); \
    EXF_CASE(320, CUT, ONCE)
    const int instance = tile.cut * 16 + tile.height / kQuantum;
    if (STREAMS && tile.once) {
        switch (instance) {
            EXF_CASES(0, STREAMS);
            EXF_CASES(1, STREAMS);
            EXF_CASES(2, STREAMS);
        }
    } else {
        switch (instance) {
            EXF_CASES(0, false);
            EXF_CASES(1, false);
            EXF_CASES(2, false);
        }
    }
#undef EXF_CASES
#undef EXF_CASE
}

template <int NT, int WAVES, int EPI, bool STREAMS>
__global__ __launch_bounds__(WAVES * kWave, 1) void grouped_gemm_bf16_kernel(const bf16_t* __restrict__ act,     // [A,K]
                                                                            const int32_t* __restrict__ offsets,
                                                                            const bf16_t* __restrict__ weight,  // [E_local,N,K]
                                                                            const bf16_t* __restrict__ bias,    // [E_local,N] or null
                                                                            int max_rows, int K, int N, int E_local,
                                                                            bf16_t* __restrict__ out,           // [A,N]
                                                                            const RowMap map)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    timeline_stamp(map, 0);
    if (map.timeline != nullptr && threadIdx.x == 0 && static_cast<int>(blockIdx.x) < map.timeline_cap)
        map.timeline[static_cast<size_t>(blockIdx.x) * 8 + 4] = 0ull;  // stays zero if this workgroup has no tile
    const RowRange range = row_range(offsets, E_local, max_rows);
    // Where every token is kept nobody has to look for others.  The last expert's end tells, and it has come with the ranges the tile is found by: asked for
    // by itself in front of them it was a second round trip for every tile (5920 tokens of which an eighth is kept, 1024 x 4096 54.1 us, now 53.2; 3000
    // tokens, 8 experts of 768 x 3072 60.9 and 60.5).
    if (map.unrouted != nullptr && wave_read_lane(range.hi, E_local - 1) < map.n_unrouted)
        clear_unrouted_rows<false, false>(map.unrouted, map.n_unrouted, reinterpret_cast<uint4*>(out), N / 8, WAVES);
    Tile2D tile;
    if (!locate_tile<STREAMS>(range, NT, N, static_cast<int>(blockIdx.x), map, tile)) return;
    timeline_stamp(map, 1);
    if (map.timeline != nullptr && threadIdx.x == 0 && static_cast<int>(blockIdx.x) < map.timeline_cap) {
        unsigned hw = 0, xcc = 0;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
#endif
        unsigned long long* rec = map.timeline + static_cast<size_t>(blockIdx.x) * 8;
        rec[5] = static_cast<unsigned long long>(hw) | (static_cast<unsigned long long>(xcc & 0xfu) << 32);
        rec[6] = static_cast<unsigned long long>(tile.height < kTileRows ? 1 : (tile.height > kTileRows ? 2 : 0)) |
                 (static_cast<unsigned long long>(tile.expert) << 8) | (static_cast<unsigned long long>(tile.n0 / NT) << 16) |
                 (static_cast<unsigned long long>(tile.row_end - tile.row_begin) << 32) | (static_cast<unsigned long long>(K / kKTile) << 48);
    }
    run_tile<NT, WAVES, EPI, STREAMS, false>(tile, act, weight, bias, K, N, out, smem, map, TileRouting{});
    timeline_stamp(map, 4);
}

// The first contraction of a layer whose assignments it sorts itself (at most kRoutedTilesMax).
template <int NT, int EPI>
__global__ __launch_bounds__(8 * kWave, 1) void routed_gemm_bf16_kernel(const bf16_t* __restrict__ act, const bf16_t* __restrict__ weight, int A, int K, int N,
                                                                        int E_local, bf16_t* __restrict__ out, const TileRouting route)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    touch_arguments<3 * 8 + 4 * 4 + sizeof(TileRouting)>();
    static_assert(sizeof(RoutedSort::count) == 8 * kWave * 4 && sizeof(RoutedSort) <= 64 * kKTile * 4, "a counter a thread; less than the smallest ring");
    RoutedSort& d = *reinterpret_cast<RoutedSort*>(smem);
    const int rounds = (A + 8 * kWave - 1) / (8 * kWave);
    int e[kRoutedRounds];
    const RowRange range = count_rows(route, E_local, A, rounds, e, d);
    const RowMap map{};
    Tile2D tile;
    if (!locate_tile<false>(range, NT, N, static_cast<int>(blockIdx.x), map, tile)) return;
    collect_rows(tile.expert, wave_read_lane(range.lo, tile.expert), tile.row_begin, tile.row_end, rounds, e, d);
    if (tile.n0 == 0) {
        for (int i = threadIdx.x; i < tile.row_end - tile.row_begin; i += 8 * kWave) {
            const int a = d.list[i];
            route.src_of_sorted[tile.row_begin + i] = a;
            route.sorted_of_src[a] = tile.row_begin + i;
        }
    }
    run_tile<NT, 8, EPI, false, true>(tile, act, weight, nullptr, K, N, out, smem, map, route);
}

// ---------------------------------------------------------------------------- host launchers
template <int NT>
constexpr int gemm_lds_bytes()
{
    int most = 0;
    const int heights[] = {64, 96, 128, 160, 192, 224, kTileRows, kTileRows + kQuantum, kTileRows + 2 * kQuantum};
    for (int h : heights) most = tile_ring_bytes(h, NT) > most ? tile_ring_bytes(h, NT) : most;
    for (int h : heights) most = tile_ring_bytes(h, NT / 2) > most ? tile_ring_bytes(h, NT / 2) : most;
    for (int h : heights) most = tile_ring_bytes(h, NT / 4) > most ? tile_ring_bytes(h, NT / 4) : most;
    return most;
}

// worst case: every expert has one tile more than whole ones (a cut round has at most one workgroup per compute unit); two
// kinds of tiles are shared out over the XCDs, and the last round may be cut
static int64_t tile_grid(int64_t A, int N, int NT, int E_local)
{
    const int64_t items = (A / kTileRows + (A < E_local ? A : E_local)) * ((N + NT - 1) / NT);
    return (items / kXcdCount + 2 + kUnitsPerXcd) * kXcdCount;
}

template <int NT, int WAVES, int EPI, bool STREAMS = false>
static int launch_bf16_as(const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N, int E_local,
                          void* out, hipStream_t stream, const RowMap& map)
{
    constexpr size_t lds = gemm_lds_bytes<NT>();
    const int64_t grid = tile_grid(A, N, NT, E_local);
    if (grid >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: too many tiles");
    auto kern = grouped_gemm_bf16_kernel<NT, WAVES, EPI, STREAMS>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_expert_ffn")) return rc;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(WAVES * kWave), lds, stream, static_cast<const bf16_t*>(act), offsets,
                       static_cast<const bf16_t*>(weight), static_cast<const bf16_t*>(bias), static_cast<int>(A), K, N, E_local,
                       static_cast<bf16_t*>(out), map);
    return EXF_OK;
}

template <int EPI>
static int launch_routed_as(const void* act, const void* weight, int64_t A, int K, int N, int E_local, void* out, hipStream_t stream, const TileRouting& route)
{
    constexpr int NT = 256;
    constexpr size_t lds = gemm_lds_bytes<NT>();
    auto kern = routed_gemm_bf16_kernel<NT, EPI>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_expert_ffn")) return rc;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(tile_grid(A, N, NT, E_local))), dim3(8 * kWave), lds, stream, static_cast<const bf16_t*>(act),
                       static_cast<const bf16_t*>(weight), static_cast<int>(A), K, N, E_local, static_cast<bf16_t*>(out), route);
    return EXF_OK;
}

// The second contraction that leaves its sorted rows besides (ffn_keep.hip): `wide`, 256 columns a tile instead of 128.
int launch_kept_contraction(bool wide, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N,
                            int E_local, void* out, hipStream_t stream, const RowMap& map);
// Contractions whose weights are streamed where one row tile reads them (ffn_once.hip, ffn_once_second.hip); epi: kEpiGeluErf or kEpiGeluTanh.
int launch_once_first(int epi, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N, int E_local,
                      void* out, hipStream_t stream, const RowMap& map);
int launch_once_second(bool wide, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N, int E_local,
                       void* out, hipStream_t stream, const RowMap& map);

// First contractions that sort the assignments (ffn_routed.hip).
int launch_routed_first(int epi, const void* act, const void* weight, int64_t A, int K, int N, int E_local, void* out, hipStream_t stream, const TileRouting& route);

}  // namespace exf
