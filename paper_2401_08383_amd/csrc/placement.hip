// Placement search driven by the co-routing statistic (Design, "Solving Affinity's duality by
// Integer Programming" and "Staged Experts Affinity").
//
// The integer program minimises the crossing transitions  sum_k sum_j R_{k,j}  under load balance
// (every part holds E/P experts of every layer) and exclusivity (every expert on one part).  With
// the E x E counts of affinity_histogram the objective of a map is
//     total - sum_l sum_{i,p} counts[l][i][p] * [part_l(i) == part_{l+1}(p)],
// so it is evaluated from 754 KB of counts instead of the trace.
//
//   placement_locality_from_counts : GPU, scores a BATCH of candidate maps against the counts, as a contraction of
//       the counts' digits with the maps' "same part" matrices on the matrix cores; exact integer arithmetic.
//   exf_placement_search           : host.  The paper names no solver; this one is
//       - exact when the number of balanced partitions of a layer is small: the objective is a
//         chain over layers, so a dynamic programme over (layer, partition) finds the optimum;
//       - otherwise layer by layer greedy (largest regret first) followed by pairwise-swap local
//         search with exact O(1) swap gains from per-expert inflow / outflow tables, over several
//         random restarts.
//       Two stages as in the paper: first experts -> nodes (crossings between nodes), then inside
//       every node its experts -> its GPUs, scored with the transitions that stay in the node.
#include <stdint.h>

#include <algorithm>
#include <numeric>
#include <type_traits>
#include <vector>

#include "common.hpp"

namespace exf {

constexpr int kScoreWaves = 4;
constexpr int kScoreThreads = kScoreWaves * kWave;
constexpr int kScoreWorkgroups = 768;      // three workgroups fill a compute unit's registers
constexpr int kScoreShare = 32;            // of an XCD at least: one per compute unit
constexpr int kDigits = 4, kDigitBits = 7; // of a count, 28 bits of it at a time
constexpr int kCountBits = kDigits * kDigitBits;
constexpr int kSourceRow = kDigits * EXF_MAX_EXPERTS;  // bytes of a source expert in LDS: [digit][target expert]
constexpr int kSetMaps = 16;               // candidates of a set: columns of a matrix operand
constexpr int kMapBytes = EXF_MAX_EXPERTS; // a map's row in LDS: a byte per expert

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4_t;

// LOADS x (WIDE ? 4 : 1) rows of candidates' maps, four part numbers a lane and load (WIDE) or one, on their way to LDS as
// bytes [map][expert].  Columns past the last expert get whatever is there: their counts are zero.
template <int ROWS, bool WIDE>
struct MapRows {
    static constexpr int PER = WIDE ? 4 : 1, LOADS = ROWS / PER;  // rows a load, loads
    typedef typename std::conditional<WIDE, int4, int>::type Piece;
    Piece v[LOADS];
    // Rows `stride` bytes apart (less than 2^32 in all), those past row `most` are that one again.  One scalar address and offsets: with an
    // address of its own for every row these were spilled (4096 maps of 24 x 30: 12.2 us, 9.4 now).
    __device__ __forceinline__ void load(const unsigned char* first, uint32_t stride, int most, int E, int lane)
    {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if constexpr (WIDE) v[i] = *reinterpret_cast<const int4*>(first + (static_cast<uint32_t>(min(4 * i + (lane >> 4), most)) * stride + min(4 * (lane & 15), E - 4) * 4u));
            else v[i] = *reinterpret_cast<const int*>(first + (static_cast<uint32_t>(min(i, most)) * stride + min(lane, E - 1) * 4u));
        }
    }
    // returns all bits of the numbers
    __device__ __forceinline__ uint32_t store(unsigned char* to, int lane) const
    {
        uint32_t any = 0;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if constexpr (WIDE) {
                any |= static_cast<uint32_t>((v[i].x | v[i].y) | (v[i].z | v[i].w));
                const uint32_t lo = __builtin_amdgcn_perm(v[i].y, v[i].x, 0x0c0c0400u), hi = __builtin_amdgcn_perm(v[i].w, v[i].z, 0x04000c0cu);
                *reinterpret_cast<uint32_t*>(to + (4 * i + (lane >> 4)) * kMapBytes + 4 * (lane & 15)) = lo | hi;
            } else {
                any |= static_cast<uint32_t>(v[i]);
                to[i * kMapBytes + lane] = static_cast<unsigned char>(v[i]);
            }
        }
        return any;
    }
    // change(part, the other rows' part at its place)
    template <typename Change>
    __device__ __forceinline__ void each(const MapRows& other, Change change)
    {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if constexpr (WIDE) {
                change(v[i].x, other.v[i].x), change(v[i].y, other.v[i].y);
                change(v[i].z, other.v[i].z), change(v[i].w, other.v[i].w);
            } else {
                change(v[i], other.v[i]);
            }
        }
    }
    // row n, a lane an expert (lanes past the last one get whatever is there)
    __device__ __forceinline__ int row(int n, int lane) const
    {
        if constexpr (WIDE) {
            const int4& x = v[n / 4];
            const int at = 16 * (n % 4) + (lane >> 2);
            const int a = __shfl(x.x, at, kWave), b = __shfl(x.y, at, kWave), c = __shfl(x.z, at, kWave), d = __shfl(x.w, at, kWave);
            return (lane & 2) != 0 ? ((lane & 1) != 0 ? d : c) : ((lane & 1) != 0 ? b : a);
        } else {
            return v[n];
        }
    }
};

// Part numbers that do not fit seven bits (-1 for an expert without a place, the device ids of a large cluster).  Only which parts are
// equal counts, so a wavefront renumbers those of a few maps at a time.  Where their codes differ in at most seven bits, these
// bits are the numbers.  Otherwise the lowest source expert with the same part stands for it (64 for a target whose part no
// source expert has), by the lanes that agree in each differing bit, a lane an expert.  Returns all bits of the numbers, or 128.
// 50 maps of 3 x 64, us (parts below 128: 3.8): parts 128 to 135 4.3, -1 to 63 4.6, 0 to 7 and 256 to 263 4.5, -3 to 100 5.6, any
// 8.7, where rows loaded once more, map by map, and looked at bit by bit in the order of memory took 6.8, 13.0, 7.1, 12.9 and 12.8;
// 4096 of 24 x 64, parts -1 to 7, 27 and 117.
constexpr int kRenumbered = 4;  // maps at a time
template <bool WIDE>
__device__ __forceinline__ uint32_t renumber(MapRows<kRenumbered, WIDE> (&rows)[2], int E, int lane, unsigned char* from, unsigned char* to)
{
    // Gray codes, their top bit moved to the bottom: parts near each other differ in few bits, on either side of zero as well
#pragma unroll
    for (int h = 0; h < 2; ++h)
        rows[h].each(rows[h], [](int& part, int) {
            const uint32_t gray = static_cast<uint32_t>(part) ^ (static_cast<uint32_t>(part) >> 1);
            part = static_cast<int>(gray << 1 | gray >> 31);
        });
    int first;
    if constexpr (WIDE) first = __builtin_amdgcn_readfirstlane(rows[0].v[0].x);
    else first = __builtin_amdgcn_readfirstlane(rows[0].v[0]);
    uint32_t bits = 0;  // in which codes differ
#pragma unroll
    for (int h = 0; h < 2; ++h) rows[h].each(rows[h], [&](int& code, int) { bits |= static_cast<uint32_t>(code ^ first); });
#pragma unroll
    for (int off = 1; off < kWave; off *= 2) bits |= __shfl_xor(bits, off, kWave);
    bits = __builtin_amdgcn_readfirstlane(bits);
    if (__builtin_popcount(bits) <= 7) {
        const MapRows<kRenumbered, WIDE> codes[2] = {rows[0], rows[1]};
#pragma unroll
        for (int h = 0; h < 2; ++h) rows[h].each(codes[h], [](int& number, int) { number = 0; });
#pragma unroll 1
        for (uint32_t left = bits; left != 0u; left &= left - 1u) {
            const int bit = __builtin_ctz(left);
#pragma unroll
            for (int h = 0; h < 2; ++h) rows[h].each(codes[h], [&](int& number, int code) { number = number << 1 | (code >> bit & 1); });
        }
        return rows[0].store(from, lane) | rows[1].store(to, lane);
    }
    int a[kRenumbered], b[kRenumbered];
    uint64_t like_a[kRenumbered], like_b[kRenumbered];  // source experts with the same part
#pragma unroll
    for (int n = 0; n < kRenumbered; ++n) {
        a[n] = rows[0].row(n, lane);
        b[n] = rows[1].row(n, lane);
        like_a[n] = like_b[n] = E == kWave ? ~0ull : (1ull << E) - 1ull;
    }
#pragma unroll 1
    for (uint32_t left = bits; left != 0u; left &= left - 1u) {
        const int bit = __builtin_ctz(left);
#pragma unroll
        for (int n = 0; n < kRenumbered; ++n) {
            const int64_t all_a = static_cast<int>(__builtin_amdgcn_sbfe(a[n], bit, 1));  // the bit in all places
            const int64_t all_b = static_cast<int>(__builtin_amdgcn_sbfe(b[n], bit, 1));
            const uint64_t set = __ballot(all_a != 0);
            like_a[n] &= ~(set ^ static_cast<uint64_t>(all_a));
            like_b[n] &= ~(set ^ static_cast<uint64_t>(all_b));
        }
    }
#pragma unroll
    for (int n = 0; n < kRenumbered; ++n) {
        from[n * kMapBytes + lane] = static_cast<unsigned char>(like_a[n] != 0ull ? __builtin_ctzll(like_a[n]) : kWave + 1);
        to[n * kMapBytes + lane] = static_cast<unsigned char>(like_b[n] != 0ull ? __builtin_ctzll(like_b[n]) : kWave);
    }
    return 128u;
}

// Bytes that say where a target's part is the source's.  FEW (all parts below eight): ones; the source's part picks one of eight
// bytes, and the targets' parts select from them, one byte permutation for four targets.  Otherwise (parts below 128): 128
// minus the difference of the parts has bit 7 set only for equal parts - as a signed byte -128 instead of one.
template <bool FEW>
struct SamePart {
    uint32_t lo, hi;
    __device__ __forceinline__ SamePart(uint32_t word, int byte)
    {
        if constexpr (FEW) {  // (`word` holds eight times the parts)
            const uint64_t lut = 1ull << ((word >> (8 * byte)) & 63u);
            lo = static_cast<uint32_t>(lut), hi = static_cast<uint32_t>(lut >> 32);
        } else {
            lo = __builtin_amdgcn_perm(0u, word, 0x01010101u * static_cast<uint32_t>(byte));
            hi = 0u;
        }
    }
    __device__ __forceinline__ int operator()(uint32_t targets) const
    {
        if constexpr (FEW) return static_cast<int>(__builtin_amdgcn_perm(hi, lo, targets));
        else return static_cast<int>((0x80808080u - (targets ^ lo)) & 0x80808080u);
    }
};

// Digits of the scores of SETS x 16 candidates: sum over source and target experts of digit * [same part].  Lanes of a quarter
// hold the source experts 16 * quarter + j, four of them in a word: the words [word, words).
template <bool FEW, int SETS>
__device__ __forceinline__ void contract(const unsigned char* digits, const unsigned char* from, const unsigned char* to, int word, int words, int chunks,
                                         int lane, i32x4_t (&acc)[SETS])
{
    const int map_at = (lane & 15) * kMapBytes;
    uint32_t target[SETS][16];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint4 x = *reinterpret_cast<const uint4*>(to + s * kSetMaps * kMapBytes + map_at + t * 16);
            target[s][4 * t] = x.x, target[s][4 * t + 1] = x.y, target[s][4 * t + 2] = x.z, target[s][4 * t + 3] = x.w;
        }
    const unsigned char* row = digits + ((lane >> 4) * 16 + word * 4) * kSourceRow + (lane & (kDigits - 1)) * EXF_MAX_EXPERTS;
#pragma unroll 1  // (each instruction is fetched once a pass otherwise)
    for (; word < words; ++word, row += 4 * kSourceRow) {
        uint32_t source[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            source[s] = *reinterpret_cast<const uint32_t*>(from + s * kSetMaps * kMapBytes + map_at + (lane >> 4) * 16 + word * 4);
            if (FEW) source[s] <<= 3;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (t >= chunks) break;
                const i32x4_t a = *reinterpret_cast<const i32x4_t*>(row + j * kSourceRow + t * 16);
#pragma unroll
                for (int s = 0; s < SETS; ++s) {
                    const SamePart<FEW> same(source[s], j);
                    const i32x4_t b = {same(target[s][4 * t]), same(target[s][4 * t + 1]), same(target[s][4 * t + 2]), same(target[s][4 * t + 3])};
                    acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc[s], 0, 0, 0);
                }
            }
        }
    }
}

// score[map] = sum over (i, p) of counts[i][p] * [part_l(i) == part_{l+1}(p)]: a product of the pair's counts, cut into four
// digits of seven bits (four rows of a matrix operand, the other twelve repeat them), with a zero-one matrix of 4096 rows
// (i, p) and a column per map.  The counts' digits lie in LDS in operand order; a lane builds its part of the other operand in
// registers: it holds the parts of 16 source experts (its quarter of the wavefront's) and of all target experts of one map.
// Sums are exact in 32 bits (4096 * 127 * 128 < 2^31).  Counts of 2^28 and more take further rounds over their higher bits, as many as
// they have (333 maps of 6 x 33, counts of up to 28 bits 4.5 us, of up to 56 6.0; 6.3 with the counts loaded again, always three rounds 8.0).
// SPLIT wavefronts share SETS x 16 candidates and take a part of the source experts each (a small batch), or every wavefront
// has its own.
// 4096 maps of 24 layers x 64 experts: 13.3 us for 2, 4 or 8 parts (walking the matching source experts of every target: 58.6,
// 36.8 and 26.7), 17.4 for 64, 6.8 with 8 experts: about half is the loads of the maps and the start of a workgroup.  The rest is
// issue: per 16 candidates and pair 64 matrix instructions and 330 vector ones that build the operand.
template <int SPLIT, int SETS, bool WIDE>
__global__ __launch_bounds__(kScoreThreads, 3) void placement_score_kernel(const int64_t* __restrict__ counts,
                                                                           const int32_t* __restrict__ placements, int B, int L, int E,
                                                                           int passes, int64_t* __restrict__ local)
{
    constexpr int GROUPS = kScoreWaves / SPLIT, GROUP_MAPS = SETS * kSetMaps, MAPS = GROUPS * GROUP_MAPS;  // candidates of a pass
    constexpr int OWN = GROUP_MAPS / SPLIT;  // rows a wavefront loads
    __shared__ __attribute__((aligned(16))) unsigned char digits[EXF_MAX_EXPERTS * kSourceRow];
    __shared__ __attribute__((aligned(16))) unsigned char maps[GROUPS][2][GROUP_MAPS * kMapBytes];  // parts at layers l and l + 1
    __shared__ i32x4_t sums[SPLIT > 1 ? kScoreWaves : 1][SETS * 16];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int group = wave / SPLIT, piece = wave % SPLIT;
    // Workgroups are numbered candidates first, pairs second, and an XCD takes consecutive ones: a row that two pairs share mostly comes
    // from its L2.  Equal shares however few candidates there are, but one per compute unit at least: spread thinner, pairs of the same
    // maps read these from memory once per XCD (16 maps of 12 x 64: 3.9 us, 3.7 now).  (A whole XCD for each group of candidates: one map of
    // 100 x 64 6.1 us, now 4.1; 200 maps of them, parts 0 to 63, 19.8 and 8.7.)
    const int xcd = static_cast<int>(blockIdx.x % 8u), rest = static_cast<int>(blockIdx.x / 8u);
    const int item = xcd * static_cast<int>(gridDim.x / 8u) + rest;
    const int l = item % (L - 1);
    const int64_t first = static_cast<int64_t>(item / (L - 1)) * passes * MAPS;
    if (first >= B) return;
    const int64_t last = min(static_cast<int64_t>(B), first + static_cast<int64_t>(passes) * MAPS);
    // rows of both layers of the maps from the b-th on
    auto load_rows = [&](auto (&some)[2], int64_t b) {
        b = min(b, static_cast<int64_t>(B) - 1);
        const unsigned char* row = reinterpret_cast<const unsigned char*>(placements + (static_cast<size_t>(b) * L + l) * E);
        const int most = static_cast<int>(min(static_cast<int64_t>(B) - 1 - b, static_cast<int64_t>(OWN)));
#pragma unroll
        for (int h = 0; h < 2; ++h) some[h].load(row + h * E * 4, static_cast<uint32_t>(L * E) * 4u, most, E, lane);
    };

    MapRows<OWN, WIDE> rows[2];
    auto load_maps = [&](int64_t pass) { load_rows(rows, pass + group * GROUP_MAPS + piece * OWN); };
    load_maps(first);

    // 28 bits of the pair's counts, from bit `shift`: four targets of a source expert at a time, a byte each in a word per
    // digit.  Returns the bits above.
    const int64_t* src = counts + static_cast<size_t>(l) * E * E;
    constexpr int ITEMS = EXF_MAX_EXPERTS * EXF_MAX_EXPERTS / 4 / kScoreThreads;
    auto load_counts = [&](uint64_t (&c)[ITEMS][4]) {
#pragma unroll
        for (int n = 0; n < ITEMS; ++n) {
            const int item = static_cast<int>(threadIdx.x) + n * kScoreThreads, i = item / (EXF_MAX_EXPERTS / 4), p = item % (EXF_MAX_EXPERTS / 4) * 4;
            if constexpr (WIDE) {
                typedef __attribute__((__vector_size__(4 * sizeof(uint64_t)), __aligned__(16))) uint64_t u64x4_t;
                const u64x4_t x = *reinterpret_cast<const u64x4_t*>(src + min(i, E - 1) * E + min(p, E - 4));
#pragma unroll
                for (int q = 0; q < 4; ++q) c[n][q] = x[q];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) c[n][q] = static_cast<uint64_t>(src[min(i, E - 1) * E + min(p + q, E - 1)]);
            }
        }
    };
    auto cut_counts = [&](const uint64_t (&c)[ITEMS][4], int shift) {
        uint64_t above = 0;
#pragma unroll
        for (int n = 0; n < ITEMS; ++n) {
            const int item = static_cast<int>(threadIdx.x) + n * kScoreThreads, i = item / (EXF_MAX_EXPERTS / 4), p = item % (EXF_MAX_EXPERTS / 4) * 4;
            uint32_t v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t x = i < E && p + q < E ? c[n][q] >> shift : 0ull;
                above |= x >> kCountBits;
                v[q] = static_cast<uint32_t>(x);
            }
#pragma unroll
            for (int d = 0; d < kDigits; ++d) {
                uint32_t word = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) word |= ((v[q] >> (kDigitBits * d)) & ((1u << kDigitBits) - 1u)) << (8 * q);
                *reinterpret_cast<uint32_t*>(digits + i * kSourceRow + d * EXF_MAX_EXPERTS + p) = word;
            }
        }
        return __syncthreads_or(above != 0ull ? 1 : 0) != 0;
    };
    const int chunks = (E + 15) / 16, words = min(4, (E + 3) / 4);
    uint64_t first_counts[ITEMS][4];
    load_counts(first_counts);
    unsigned char *from = maps[group][0], *to = maps[group][1];
    auto store_maps = [&](int64_t pass) {
        unsigned char *own_from = from + piece * OWN * kMapBytes, *own_to = to + piece * OWN * kMapBytes;
        uint32_t any = rows[0].store(own_from, lane) | rows[1].store(own_to, lane);
        if (__builtin_expect(__ballot(any >= 128u) == 0ull, 1)) return any;
        any = 0;  // (a wavefront's LDS accesses are done in order)
        if constexpr (OWN == kRenumbered) {
            any = renumber<WIDE>(rows, E, lane, own_from, own_to);
        } else {  // loaded again, from the L2: holding all rows until here would spill registers of every launch
#pragma unroll 1
            for (int n0 = 0; n0 < OWN; n0 += kRenumbered) {
                MapRows<kRenumbered, WIDE> some[2];
                load_rows(some, pass + group * GROUP_MAPS + piece * OWN + n0);
                any |= renumber<WIDE>(some, E, lane, own_from + n0 * kMapBytes, own_to + n0 * kMapBytes);
            }
        }
        return any;
    };
    uint32_t any = store_maps(first);
    const bool more = cut_counts(first_counts, 0);  // counts of 2^28 or more

    for (int64_t pass = first; pass < last; pass += MAPS) {
        const int64_t b0 = pass + group * GROUP_MAPS;
        const int here = static_cast<int>(max(static_cast<int64_t>(0), min(last - b0, static_cast<int64_t>(GROUP_MAPS))));
        uint64_t score[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) score[s] = 0;
        bool few = true, above = more;  // counts have bits above these
        for (int shift = 0; shift == 0 || (above && shift < 64); shift += kCountBits) {
            if (more && (shift > 0 || pass > first)) {  // (the same in all wavefronts)
                if constexpr (SPLIT > 1) {  // (one pass: the counts are still in registers)
                    __syncthreads();
                    above = cut_counts(first_counts, shift);
                } else {
                    uint64_t c[ITEMS][4];
                    load_counts(c);
                    __syncthreads();  // (others may still read the digits)
                    above = cut_counts(c, shift);
                }
            } else if (SPLIT > 1) {
                __syncthreads();
            }
            if (shift == 0) {
                __builtin_amdgcn_wave_barrier();
                if constexpr (SPLIT == 1) {
                    few = __ballot(any >= 8u) == 0ull;
                } else {  // all parts of the group's maps, not only of the rows loaded here
                    uint32_t seen = 0;
                    for (int n = lane; n < 2 * GROUP_MAPS * kMapBytes / 16; n += kWave) {
                        const uint4 x = *reinterpret_cast<const uint4*>(from + n * 16);
                        seen |= (x.x | x.y) | (x.z | x.w);
                    }
                    few = __ballot((seen & 0xf8f8f8f8u) != 0u) == 0ull;
                }
            }
            i32x4_t acc[SETS];
#pragma unroll
            for (int s = 0; s < SETS; ++s) acc[s] = i32x4_t{0, 0, 0, 0};
            if (here > 0) {
                const int w0 = SPLIT == 1 ? 0 : piece * (4 / SPLIT), w1 = SPLIT == 1 ? words : min(words, w0 + 4 / SPLIT);
                if (few) contract<true, SETS>(digits, from, to, w0, w1, chunks, lane, acc);
                else contract<false, SETS>(digits, from, to, w0, w1, chunks, lane, acc);
            }
            if constexpr (SPLIT > 1) {
                if (lane < 16)
#pragma unroll
                    for (int s = 0; s < SETS; ++s) sums[wave][s * 16 + lane] = acc[s];
                __syncthreads();
                if (piece == 0 && lane < 16)
#pragma unroll
                    for (int w = 1; w < SPLIT; ++w)
#pragma unroll
                        for (int s = 0; s < SETS; ++s) acc[s] += sums[wave + w][s * 16 + lane];
            }
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                int64_t sum = 0;
#pragma unroll
                for (int d = 0; d < kDigits; ++d) sum += static_cast<int64_t>(acc[s][d]) << (kDigitBits * d);
                score[s] += static_cast<uint64_t>(few ? sum : -sum >> 7) << shift;
            }
        }
        if (lane < 16 && piece == 0) {
#pragma unroll
            for (int s = 0; s < SETS; ++s)
                if (s * 16 + lane < here) local[static_cast<size_t>(b0 + s * 16 + lane) * (L - 1) + l] = static_cast<int64_t>(score[s]);
        }
        if (SPLIT > 1 && pass + MAPS < last) __syncthreads();
        if (pass + MAPS < last) {
            load_maps(pass + MAPS);
            any = store_maps(pass + MAPS);
        }
    }
}

template <int SPLIT, int SETS>
static void launch_scores(const int64_t* counts, const int32_t* placements, int B, int L, int E, int64_t* local, hipStream_t stream)
{
    constexpr int MAPS = kScoreWaves / SPLIT * SETS * kSetMaps;
    const int64_t all = (static_cast<int64_t>(B) + MAPS - 1) / MAPS;
    const int passes = static_cast<int>((all * (L - 1) + kScoreWorkgroups - 1) / kScoreWorkgroups);  // of a workgroup
    const int64_t groups = (all + passes - 1) / passes;
    const int64_t share = std::max<int64_t>((groups * (L - 1) + 7) / 8, kScoreShare);  // workgroups of an XCD
    const dim3 grid(static_cast<unsigned>(share * 8));
    if (E % 4 == 0 && aligned16(placements) && aligned16(counts))
        hipLaunchKernelGGL((placement_score_kernel<SPLIT, SETS, true>), grid, dim3(kScoreThreads), 0, stream, counts, placements, B, L, E, passes, local);
    else
        hipLaunchKernelGGL((placement_score_kernel<SPLIT, SETS, false>), grid, dim3(kScoreThreads), 0, stream, counts, placements, B, L, E, passes, local);
}

// ------------------------------------------------------------------------------------ host solver
namespace {

// counts of one sub-problem: n experts per layer, counts[l][i][p] for the L-1 pairs
struct Problem {
    int L, n, P;
    std::vector<int64_t> c;  // [(L-1)][n][n]
    int64_t at(int l, int i, int p) const { return c[(static_cast<size_t>(l) * n + i) * n + p]; }
};

int64_t score(const Problem& pb, const std::vector<int>& part)  // part [L][n]
{
    int64_t s = 0;
    for (int l = 0; l + 1 < pb.L; ++l)
        for (int i = 0; i < pb.n; ++i)
            for (int p = 0; p < pb.n; ++p)
                if (part[l * pb.n + i] == part[(l + 1) * pb.n + p]) s += pb.at(l, i, p);
    return s;
}

// all labelled balanced partitions of n experts into P parts, if there are at most `limit` of them
bool enumerate_partitions(int n, int P, size_t limit, std::vector<std::vector<int>>& out)
{
    const int cap = n / P;
    std::vector<int> cur, left(P, cap);
    bool ok = true;
    auto rec = [&](auto&& self, int e) -> void {
        if (!ok) return;
        if (e == n) {
            if (out.size() >= limit) {
                ok = false;
                return;
            }
            out.push_back(cur);
            return;
        }
        for (int p = 0; p < P; ++p)
            if (left[p] > 0) {
                left[p] -= 1;
                cur.push_back(p);
                self(self, e + 1);
                cur.pop_back();
                left[p] += 1;
            }
    };
    rec(rec, 0);
    return ok;
}

// exact optimum by dynamic programming over the chain of layers; returns false if the state space is too large
bool solve_exact(const Problem& pb, std::vector<int>& part)
{
    std::vector<std::vector<int>> parts;
    if (!enumerate_partitions(pb.n, pb.P, 128, parts)) return false;
    const int S = static_cast<int>(parts.size());
    const int n = pb.n;
    std::vector<int64_t> best(static_cast<size_t>(pb.L) * S, 0);
    std::vector<int> from(static_cast<size_t>(pb.L) * S, 0);
    for (int l = 1; l < pb.L; ++l) {
        for (int t = 0; t < S; ++t) {
            int64_t top = -1;
            int arg = 0;
            for (int s = 0; s < S; ++s) {
                int64_t v = best[static_cast<size_t>(l - 1) * S + s];
                for (int i = 0; i < n; ++i)
                    for (int p = 0; p < n; ++p)
                        if (parts[s][i] == parts[t][p]) v += pb.at(l - 1, i, p);
                if (v > top) {
                    top = v;
                    arg = s;
                }
            }
            best[static_cast<size_t>(l) * S + t] = top;
            from[static_cast<size_t>(l) * S + t] = arg;
        }
    }
    int t = 0;
    for (int s = 1; s < S; ++s)
        if (best[static_cast<size_t>(pb.L - 1) * S + s] > best[static_cast<size_t>(pb.L - 1) * S + t]) t = s;
    part.assign(static_cast<size_t>(pb.L) * n, 0);
    for (int l = pb.L - 1; l >= 0; --l) {
        for (int e = 0; e < n; ++e) part[l * n + e] = parts[t][e];
        t = from[static_cast<size_t>(l) * S + t];
    }
    return true;
}

struct Rng {  // splitmix64: the restarts must not depend on the C library's generator
    uint64_t s;
    uint64_t next()
    {
        uint64_t z = (s += 0x9e3779b97f4a7c15ull);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        return z ^ (z >> 31);
    }
    int below(int n) { return static_cast<int>(next() % static_cast<uint64_t>(n)); }
};

// layer l+1 from layer l: expert p gains  gain[p][g] = sum_{i on part g} counts[l][i][p]  on part g;
// experts are fixed one at a time, the one with the largest regret (best minus second-best open part) first
void greedy_next_layer(const Problem& pb, int l, std::vector<int>& part)
{
    const int n = pb.n, P = pb.P, cap = n / P;
    std::vector<int64_t> gain(static_cast<size_t>(n) * P, 0);
    for (int i = 0; i < n; ++i)
        for (int p = 0; p < n; ++p) gain[static_cast<size_t>(p) * P + part[l * n + i]] += pb.at(l, i, p);
    std::vector<int> left(P, cap);
    std::vector<char> done(n, 0);
    for (int step = 0; step < n; ++step) {
        int pick = -1, pick_part = 0;
        int64_t pick_regret = -1;
        for (int p = 0; p < n; ++p) {
            if (done[p]) continue;
            int64_t b1 = -1, b2 = -1;
            int a1 = 0;
            for (int g = 0; g < P; ++g) {
                if (left[g] == 0) continue;
                const int64_t v = gain[static_cast<size_t>(p) * P + g];
                if (v > b1) {
                    b2 = b1;
                    b1 = v;
                    a1 = g;
                } else if (v > b2) {
                    b2 = v;
                }
            }
            const int64_t regret = b2 < 0 ? b1 : b1 - b2;
            if (regret > pick_regret) {
                pick_regret = regret;
                pick = p;
                pick_part = a1;
            }
        }
        done[pick] = 1;
        left[pick_part] -= 1;
        part[(l + 1) * n + pick] = pick_part;
    }
}

// pairwise swaps inside a layer until none improves.  value[l][e][g] = transitions of expert e of layer
// l that stay local if e sits on part g (inflow from layer l-1 plus outflow to layer l+1); two experts
// of one layer never interact, so the gain of a swap is exact.
void local_search(const Problem& pb, std::vector<int>& part)
{
    const int L = pb.L, n = pb.n, P = pb.P;
    std::vector<int64_t> value(static_cast<size_t>(L) * n * P);
    auto rebuild_layer = [&](int l) {
        for (int e = 0; e < n; ++e)
            for (int g = 0; g < P; ++g) value[(static_cast<size_t>(l) * n + e) * P + g] = 0;
        if (l > 0)
            for (int i = 0; i < n; ++i)
                for (int e = 0; e < n; ++e) value[(static_cast<size_t>(l) * n + e) * P + part[(l - 1) * n + i]] += pb.at(l - 1, i, e);
        if (l + 1 < L)
            for (int e = 0; e < n; ++e)
                for (int p = 0; p < n; ++p) value[(static_cast<size_t>(l) * n + e) * P + part[(l + 1) * n + p]] += pb.at(l, e, p);
    };
    for (int l = 0; l < L; ++l) rebuild_layer(l);
    bool improved = true;
    for (int sweep = 0; improved && sweep < 1000; ++sweep) {
        improved = false;
        for (int l = 0; l < L; ++l) {
            for (int a = 0; a < n; ++a)
                for (int b = a + 1; b < n; ++b) {
                    const int ga = part[l * n + a], gb = part[l * n + b];
                    if (ga == gb) continue;
                    const int64_t* va = &value[(static_cast<size_t>(l) * n + a) * P];
                    const int64_t* vb = &value[(static_cast<size_t>(l) * n + b) * P];
                    const int64_t delta = (va[gb] + vb[ga]) - (va[ga] + vb[gb]);
                    if (delta > 0) {
                        part[l * n + a] = gb;
                        part[l * n + b] = ga;
                        if (l > 0) rebuild_layer(l - 1);
                        if (l + 1 < L) rebuild_layer(l + 1);
                        improved = true;
                    }
                }
        }
    }
}

void solve_heuristic(const Problem& pb, int restarts, uint64_t seed, std::vector<int>& best_part)
{
    const int n = pb.n, P = pb.P, cap = n / P;
    Rng rng{seed};
    int64_t best = -1;
    std::vector<int> part(static_cast<size_t>(pb.L) * n);
    for (int r = 0; r < std::max(restarts, 1); ++r) {
        std::vector<int> order(n);
        std::iota(order.begin(), order.end(), 0);
        if (r > 0)
            for (int i = n - 1; i > 0; --i) std::swap(order[i], order[rng.below(i + 1)]);  // first restart: contiguous
        for (int i = 0; i < n; ++i) part[order[i]] = i / cap;
        for (int l = 0; l + 1 < pb.L; ++l) greedy_next_layer(pb, l, part);
        local_search(pb, part);
        const int64_t s = score(pb, part);
        if (s > best) {
            best = s;
            best_part = part;
        }
    }
}

void solve(const Problem& pb, int restarts, uint64_t seed, std::vector<int>& part)
{
    if (pb.P == 1) {
        part.assign(static_cast<size_t>(pb.L) * pb.n, 0);
        return;
    }
    if (!solve_exact(pb, part)) solve_heuristic(pb, restarts, seed, part);
}

}  // namespace
}  // namespace exf

extern "C" int placement_locality_from_counts(const int64_t* counts, const int32_t* placements, int B, int L, int E,
                                              int64_t* local, void* stream)
{
    using namespace exf;
    if (L < 1 || L > EXF_MAX_TRACE_LAYERS) return fail(EXF_ERR_BAD_SHAPE, "placement_locality_from_counts: L = %d outside [1,%d]", L, EXF_MAX_TRACE_LAYERS);
    if (E < 1 || E > EXF_MAX_EXPERTS) return fail(EXF_ERR_BAD_SHAPE, "placement_locality_from_counts: E = %d outside [1,%d]", E, EXF_MAX_EXPERTS);
    if (B < 0 || B > (1 << 24)) return fail(EXF_ERR_BAD_SHAPE, "placement_locality_from_counts: B = %d outside [0,2^24]", B);
    if (B == 0 || L == 1) return EXF_OK;  // no candidate or no transition: no output element
    EXF_REQUIRE_PTR(counts);
    EXF_REQUIRE_PTR(placements);
    EXF_REQUIRE_PTR(local);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // A batch that one round of workgroups of 16 candidates covers is split over the wavefronts, otherwise every wavefront takes 32
    // (64 candidates of 24 x 64: 3.9 us split, 6.2 not; 1024: 8.1 and 7.3)
    if ((static_cast<int64_t>(B) + kSetMaps - 1) / kSetMaps * (L - 1) <= kScoreWorkgroups) launch_scores<4, 1>(counts, placements, B, L, E, local, s);
    else launch_scores<1, 2>(counts, placements, B, L, E, local, s);
    return check_launch("placement_locality_from_counts");
}

extern "C" int exf_placement_search(const int64_t* counts_host, int L, int E, int G, int nodes, int restarts, uint64_t seed,
                                    int32_t* placement_host)
{
    using namespace exf;
    EXF_REQUIRE_PTR(placement_host);
    if (L < 1 || L > EXF_MAX_TRACE_LAYERS || E < 1 || E > EXF_MAX_EXPERTS)
        return fail(EXF_ERR_BAD_SHAPE, "exf_placement_search: L = %d, E = %d out of range", L, E);
    if (G < 1 || nodes < 1 || E % G != 0 || G % nodes != 0)
        return fail(EXF_ERR_BAD_SHAPE, "exf_placement_search: need nodes | G | E (E=%d G=%d nodes=%d)", E, G, nodes);
    if (L > 1) EXF_REQUIRE_PTR(counts_host);
    for (int l = 0; l + 1 < L; ++l)
        for (int i = 0; i < E * E; ++i)
            if (counts_host[static_cast<size_t>(l) * E * E + i] < 0)
                return fail(EXF_ERR_BAD_SHAPE, "exf_placement_search: negative count in layer pair %d", l);

    // stage 1: experts -> nodes
    Problem top{L, E, nodes, {}};
    top.c.assign(counts_host, counts_host + static_cast<size_t>(L > 1 ? L - 1 : 0) * E * E);
    std::vector<int> node_of;
    solve(top, restarts, seed, node_of);

    // stage 2: inside every node, its experts -> its GPUs, scored with the transitions that stay in the node
    const int per_node = G / nodes, n_sub = E / nodes;
    for (int nd = 0; nd < nodes; ++nd) {
        std::vector<int> members(static_cast<size_t>(L) * n_sub);  // expert ids of this node, per layer, ascending
        for (int l = 0; l < L; ++l) {
            int k = 0;
            for (int e = 0; e < E; ++e)
                if (node_of[l * E + e] == nd) members[l * n_sub + k++] = e;
        }
        Problem sub{L, n_sub, per_node, {}};
        sub.c.resize(static_cast<size_t>(L > 1 ? L - 1 : 0) * n_sub * n_sub);
        for (int l = 0; l + 1 < L; ++l)
            for (int i = 0; i < n_sub; ++i)
                for (int p = 0; p < n_sub; ++p)
                    sub.c[(static_cast<size_t>(l) * n_sub + i) * n_sub + p] =
                        counts_host[(static_cast<size_t>(l) * E + members[l * n_sub + i]) * E + members[(l + 1) * n_sub + p]];
        std::vector<int> gpu_of;
        solve(sub, restarts, seed + 0x1000u * static_cast<uint64_t>(nd + 1), gpu_of);
        for (int l = 0; l < L; ++l)
            for (int i = 0; i < n_sub; ++i) placement_host[static_cast<size_t>(l) * E + members[l * n_sub + i]] = nd * per_node + gpu_of[l * n_sub + i];
    }
    return EXF_OK;
}
