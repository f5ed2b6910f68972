// Short traces in one launch.  The kernels of affinity.hip cut a trace into chunks that fill the chip and add their partial
// counts up in a second launch; where a trace is short, that launch (its start, its gap and its round trip to memory: 4 to 5 us) and
// the clearing and writing of the partials are most of the time.  Here a workgroup takes a whole layer pair (counts) or a
// whole layer (locality, transfers), however little of the chip that fills, and writes final results.
#include <algorithm>

#include "trace_tile.hpp"

namespace exf {

constexpr int kPairThreads = 1024;
constexpr int kPairWaves = kPairThreads / kWave;
constexpr int kPairMaxCopies = 16;
constexpr int kPairHistBytes = 32 * 1024;  // replicas of small histograms, so that hot bins do not serialise

// Sum of a 32-bit count over the wavefront, in all lanes.
__device__ __forceinline__ int wave_total(int v) { return wave_read_lane(wave_inclusive_scan(v), kWave - 1); }

// Counts, probabilities, loads and locality of one layer pair per workgroup.  The histogram has a row and a column for
// invalid ids: an id is its unsigned value or E, whichever is less, and every token is one LDS atomic without a test.
//   HOPS: all ordered pairs, numbered source layer first; counts and probabilities only.  Otherwise the adjacent ones, and one
//   workgroup more that counts the invalid ids of the whole trace where n_invalid is asked for.
template <bool HOPS>
__global__ __launch_bounds__(kPairThreads) void pair_direct_kernel(const int32_t* __restrict__ trace, int L, int64_t N, int E, int copies, int copy_words,
                                                                   const int32_t* __restrict__ placement, int64_t* __restrict__ counts,
                                                                   float* __restrict__ cond_prob, int64_t* __restrict__ loads,
                                                                   int64_t* __restrict__ n_invalid, int64_t* __restrict__ local)
{
    extern __shared__ uint32_t pair_lds[];
    uint32_t* hist = pair_lds;                    // [copies][copy_words >= (E+1)(E+1)]
    uint32_t* column = hist + copies * copy_words;  // [64] tokens of the pair's target layer per expert (final layer)
    uint32_t* tally = column + EXF_MAX_EXPERTS;     // [1]
    constexpr int VEC = 4, AHEAD = 2;
    touch_arguments<88>();
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t sweep = static_cast<int64_t>(kPairThreads) * VEC;
    if (!HOPS && static_cast<int>(blockIdx.x) == L - 1) {
        const int64_t all = N * L;
        if (threadIdx.x == 0) *tally = 0u;
        __syncthreads();
        int bad = 0;
        constexpr int U = 8;
        for (int64_t base = 0; base < all; base += U * sweep) {
            const int64_t n0 = base + static_cast<int64_t>(threadIdx.x) * VEC;
            TokVec<VEC> t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) t[u] = load_tokens<VEC>(trace, n0 + u * sweep, all);  // (past the end: the last vector again)
            uint32_t most = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v) most = max(most, static_cast<uint32_t>(t[u].v[v]));
            if (__ballot(most >= static_cast<uint32_t>(E)) == 0ull) continue;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cut_vector(t[u], n0 + u * sweep, all);
#pragma unroll
                for (int v = 0; v < VEC; ++v) bad += n0 + u * sweep + v < all && static_cast<uint32_t>(t[u].v[v]) >= static_cast<uint32_t>(E) ? 1 : 0;
            }
        }
        bad = wave_total(bad);
        if (lane == 0 && bad != 0) atomicAdd(tally, static_cast<uint32_t>(bad));
        __syncthreads();
        if (threadIdx.x == 0) *n_invalid = *tally;
        return;
    }
    int l = static_cast<int>(blockIdx.x), m = l + 1;
    if constexpr (HOPS) {
        int q = l;
        for (l = 0; q >= L - 1 - l; ++l) q -= L - 1 - l;
        m = l + 1 + q;
    }
    const int32_t *from = trace + static_cast<int64_t>(l) * N, *to = trace + static_cast<int64_t>(m) * N;
    const int64_t first = static_cast<int64_t>(threadIdx.x) * VEC;
    TokVec<VEC> a[AHEAD], b[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        a[s] = load_tokens<VEC, false>(from, first + s * sweep, N);
        b[s] = load_tokens<VEC, false>(to, first + s * sweep, N);
    }
    const bool located = !HOPS && placement != nullptr;
    int there = 0;  // lane = target expert
    if (located) there = placement[static_cast<int64_t>(m) * E + min(lane, E - 1)];
    for (int i = threadIdx.x; i < copies * copy_words + EXF_MAX_EXPERTS + 1; i += kPairThreads) hist[i] = 0u;
    __syncthreads();
    uint32_t* mine = hist + (threadIdx.x & (copies - 1)) * copy_words;
    const uint32_t row = static_cast<uint32_t>(E) + 1u;
    auto count = [&](TokVec<VEC>& x, TokVec<VEC>& y, int64_t n0) {
        if (__ballot(n0 + VEC > N) != 0ull) {
            cut_vector(x, n0, N);
            cut_vector(y, n0, N);
#pragma unroll
            for (int u = 0; u < VEC; ++u)
                if (n0 + u < N) atomicAdd(&mine[__umul24(min(static_cast<uint32_t>(x.v[u]), static_cast<uint32_t>(E)), row) + min(static_cast<uint32_t>(y.v[u]), static_cast<uint32_t>(E))], 1u);
        } else {
#pragma unroll
            for (int u = 0; u < VEC; ++u)
                atomicAdd(&mine[__umul24(min(static_cast<uint32_t>(x.v[u]), static_cast<uint32_t>(E)), row) + min(static_cast<uint32_t>(y.v[u]), static_cast<uint32_t>(E))], 1u);
        }
    };
    for (int64_t base = 0; base < N; base += AHEAD * sweep) {
        const int64_t n0 = base + first;
        const bool more = base + AHEAD * sweep < N;  // (uniform)
        TokVec<VEC> na[AHEAD], nb[AHEAD];
        if (more) {
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) {
                na[s] = load_tokens<VEC, false>(from, n0 + (AHEAD + s) * sweep, N);
                nb[s] = load_tokens<VEC, false>(to, n0 + (AHEAD + s) * sweep, N);
            }
        }
#pragma unroll
        for (int s = 0; s < AHEAD; ++s)
            if (base + s * sweep < N) count(a[s], b[s], n0 + s * sweep);
        if (more) {
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) {
                a[s] = na[s];
                b[s] = nb[s];
            }
        }
    }
    __syncthreads();

    // a wavefront per row of the histogram, lane = target expert
    auto cell = [&](int i, int p) {
        uint32_t c = 0;
        const uint32_t* at = hist + i * static_cast<int>(row) + p;
        if (copies == kPairMaxCopies) {  // all reads in flight together
#pragma unroll
            for (int r = 0; r < kPairMaxCopies; ++r) c += at[r * copy_words];
        } else {
            for (int r = 0; r < copies; ++r) c += at[r * copy_words];
        }
        return static_cast<int>(c);
    };
    const bool final_layer = !HOPS && loads != nullptr && m == L - 1;
    int stay = 0, reach = 0;
    for (int i = wave; i < E; i += kPairWaves) {
        const int c = lane < E ? cell(i, lane) : 0;
        const int sum = wave_total(c);
        if (lane < E) {
            const size_t o = (static_cast<size_t>(blockIdx.x) * E + i) * E + lane;
            counts[o] = c;
            if (cond_prob != nullptr) cond_prob[o] = sum > 0 ? static_cast<float>(static_cast<double>(c) / static_cast<double>(sum)) : 0.0f;
        }
        if constexpr (!HOPS) {
            if (loads != nullptr && lane == 0) loads[static_cast<size_t>(l) * E + i] = sum + cell(i, E);
            if (located && placement[static_cast<int64_t>(l) * E + i] == there) stay += c;
            reach += c;
        }
    }
    if constexpr (!HOPS) {
        if (final_layer) {
            if (wave == 0 && lane < E) reach += cell(E, lane);
            if (lane < E) atomicAdd(&column[lane], static_cast<uint32_t>(reach));
        }
        if (located) {
            stay = wave_total(stay);
            if (lane == 0) atomicAdd(tally, static_cast<uint32_t>(stay));
        }
        __syncthreads();
        if (final_layer && static_cast<int>(threadIdx.x) < E) loads[static_cast<size_t>(m) * E + threadIdx.x] = column[threadIdx.x];
        if (located && threadIdx.x == 0) local[l] = *tally;
    }
}

static bool pair_trace_fits(int L, int64_t N) { return L > 1 && N >= 4 && N < (1ll << 30); }
template <bool HOPS>
static void launch_pairs(int workgroups, const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int64_t* counts, int64_t* loads,
                         float* cond_prob, int64_t* n_invalid, int64_t* local, hipStream_t stream)
{
    const int copy_words = (E + 1) * (E + 1) | 1;  // (odd: replicas begin on different banks)
    int copies = 1;
    while (copies < kPairMaxCopies && copy_words * 4 * (copies * 2) <= kPairHistBytes) copies *= 2;
    const size_t lds = (static_cast<size_t>(copies) * copy_words + EXF_MAX_EXPERTS + 1) * sizeof(uint32_t);
    hipLaunchKernelGGL(pair_direct_kernel<HOPS>, dim3(static_cast<unsigned>(workgroups)), dim3(kPairThreads), lds, stream, trace, L, N, E, copies, copy_words,
                       placement, counts, cond_prob, loads, n_invalid, local);
}

// Two launches and one, us: 24 x 1000, 64 experts 13.1 and 5.5; 24 x 4099 13.0 and 5.7; 12 x 8192, 8 experts 8.3 and 6.5; 4 x 32768, 32
// experts 9.5 and 7.1.  The invalid ids of the whole trace are one workgroup's: 12 x 16384 8.3 and 11.6; and a pair's tokens: 2 x
// 32768, 8 experts 7.8 and 8.1.
constexpr int64_t kStatisticsTokens = 24576, kStatisticsIds = 122880;
bool statistics_direct(const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int64_t* counts, int64_t* loads, float* cond_prob,
                       int64_t* n_invalid, int64_t* local_per_pair, hipStream_t stream)
{
    if (!pair_trace_fits(L, N) || N > kStatisticsTokens || N * L > kStatisticsIds) return false;
    launch_pairs<false>(L - 1 + (n_invalid != nullptr ? 1 : 0), trace, placement, L, N, E, counts, loads, cond_prob, n_invalid, local_per_pair, stream);
    return true;
}

// A pair's workgroup takes 3 to 4 us and 0.1 us for 1000 tokens, and again that for every further set of pairs that the compute units
// hold (253 pairs of 23 layers at once, 276 of 24 two to a unit).  The chunked kernels take longer the more layers and experts there
// are and hardly by tokens, so each range of layers has its line.  Chunked and direct at it, us: 4 x 20000, 32 experts 7.3 and 5.0, 9 x
// 50000, 8 experts 7.7 and 9.1; 13 x 50000, 24 experts 9.4 and 8.6, 13 x 100000, 64 experts 15.8 and 14.4; with 4, 16 and 64 experts 16 x
// 106496 14.8, 19.6, 24.6 and 14.0, 14.4, 16.0, 19 x 106496 15.3, 17.7, 28.2 and 14.1, 14.5, 16.5, 23 x 106496 17.9, 20.6, 38.7 and 14.9,
// 15.3, 17.4; 24 x 49152, 8 experts 14.7 and 12.3, 24 x 90112, 24 experts 23.5 and 21.0, 24 x 131072, 48 experts 34.7 and 30.2; 32 layers
// of these 17.0 and 14.4, 27.2 and 25.4, 38.0 and 37.5.
//   Beyond, every pair costs a workgroup's start while the chunked kernels' cost per pair shrinks with the experts: 64 x 16384, 4, 12
// and 64 experts 20.5, 26.1, 61.8 and 22.8, 24.9, 39.1; 100 x 8192, 4, 24 and 64 experts 35.0, 65.2, 123.3 and 48.0, 59.3, 74.4; shorter
// traces need more of them (80 x 1000, 24 experts a tenth longer, 80 x 4000 a twentieth shorter).  255 x 4000, 32 experts 349 and 591.
static bool few_hop_tokens(int L, int64_t N, int E)
{
    if (L < 12) return N <= 32768;
    if (L < 16) return N <= (E >= 40 ? 81920 : 49152);
    if (L < 24) return N <= 106496;
    if (L > 32) return L <= 100 && N <= 16384 && E >= (N < 2048 ? 1.0 : 0.7) * (L - 48);
    return N <= (E >= 40 ? 131072 : (E >= 24 ? 90112 : 49152));
}
bool multihop_direct(const int32_t* trace, int L, int64_t N, int E, int64_t* counts, float* cond_prob, hipStream_t stream)
{
    if (!pair_trace_fits(L, N) || !few_hop_tokens(L, N, E)) return false;
    launch_pairs<true>(L * (L - 1) / 2, trace, nullptr, L, N, E, counts, nullptr, cond_prob, nullptr, nullptr, stream);
    return true;
}

// Locality of the pair (l, l+1) and (HOME) transfers of layer l by workgroup l.
template <bool HOME>
__global__ __launch_bounds__(kPairThreads) void locality_direct_kernel(const int32_t* __restrict__ trace, const int32_t* __restrict__ placement,
                                                                       const int32_t* __restrict__ home, int L, int64_t N, int E,
                                                                       int64_t* __restrict__ local, int64_t* __restrict__ away)
{
    __shared__ int device[2][EXF_MAX_EXPERTS + 1];  // of an expert at layer l and at l + 1
    __shared__ int sums[2];
    constexpr int VEC = 4, AHEAD = 2;
    const int lane = lane_id();
    const int l = static_cast<int>(blockIdx.x);
    const bool pair = l + 1 < L;
    const int32_t *from = trace + static_cast<int64_t>(l) * N, *to = trace + static_cast<int64_t>(min(l + 1, L - 1)) * N;
    const int64_t sweep = static_cast<int64_t>(kPairThreads) * VEC, first = static_cast<int64_t>(threadIdx.x) * VEC;
    TokVec<VEC> a[AHEAD], b[AHEAD], h[AHEAD];
    auto load = [&](int64_t n0) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            a[s] = load_tokens<VEC, false>(from, n0 + s * sweep, N);
            b[s] = load_tokens<VEC, false>(to, n0 + s * sweep, N);
            if constexpr (HOME) h[s] = load_tokens<VEC, false>(home, n0 + s * sweep, N);
        }
    };
    load(first);
    if (threadIdx.x < 2u * kWave) {
        const int which = threadIdx.x / kWave;
        if (lane < E) device[which][lane] = placement[static_cast<int64_t>(min(l + which, L - 1)) * E + lane];
    }
    if (threadIdx.x < 2) sums[threadIdx.x] = 0;
    __syncthreads();
    int same = 0, gone = 0;
    for (int64_t base = 0; base < N; base += AHEAD * sweep) {
        const int64_t n0 = base + first;
        TokVec<VEC> x[AHEAD], y[AHEAD], z[AHEAD];
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            x[s] = a[s];
            y[s] = b[s];
            if constexpr (HOME) z[s] = h[s];
        }
        if (base + AHEAD * sweep < N) load(n0 + AHEAD * sweep);
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            const int64_t n = n0 + s * sweep;
            if (__ballot(n + VEC > N) != 0ull) {
                cut_vector(x[s], n, N);
                cut_vector(y[s], n, N);
                if constexpr (HOME) cut_vector(z[s], n, N);
            }
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                const bool ok = n + u < N && static_cast<uint32_t>(x[s].v[u]) < static_cast<uint32_t>(E);
                const bool next_ok = static_cast<uint32_t>(y[s].v[u]) < static_cast<uint32_t>(E);
                const int here = device[0][ok ? x[s].v[u] : 0];
                same += ok && next_ok && here == device[1][next_ok ? y[s].v[u] : 0] ? 1 : 0;
                if constexpr (HOME) gone += ok && here != z[s].v[u] ? 1 : 0;
            }
        }
    }
    same = wave_total(same);
    gone = wave_total(gone);
    if (lane == 0) {
        if (same != 0) atomicAdd(&sums[0], same);
        if (HOME && gone != 0) atomicAdd(&sums[1], gone);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (pair) local[l] = sums[0];
        if constexpr (HOME) away[l] = sums[1];
    }
}

// A layer's workgroup takes 3 us and 1.1 for every 8192 tokens after the first ones, with home devices 3.7 and 1.3; the chunked kernels longer
// the more layers there are.  Two launches and one at the line, us: locality 2 x 8192 4.3 and 3.1, 3 x 9792 4.9 and 4.3, 24 x 43392 8.8
// and 8.1, 96 x 158592 36.1 and 22.8, 256 x 414592 167 and 119; transfers 2 x 8192 5.0 and 3.8, 4 x 9792 5.4 and 5.3, 24 x 41792 10.2 and 10.4, 96
// x 156992 44.4 and 28.7 (3 x 9792 5.0 and 5.2, 24 x 43392 9.9 and 10.3: one layer less in the line).
bool locality_direct(const int32_t* trace, const int32_t* placement, const int32_t* home, int L, int64_t N, int E, int64_t* local_per_pair,
                     int64_t* away_per_layer, hipStream_t stream)
{
    if (N < 4 || N > 8192 + 1600ll * (home != nullptr ? std::max(L - 3, 0) : L - 2)) return false;
    if (home != nullptr)
        hipLaunchKernelGGL(locality_direct_kernel<true>, dim3(static_cast<unsigned>(L)), dim3(kPairThreads), 0, stream, trace, placement, home, L, N, E,
                           local_per_pair, away_per_layer);
    else
        hipLaunchKernelGGL(locality_direct_kernel<false>, dim3(static_cast<unsigned>(L - 1)), dim3(kPairThreads), 0, stream, trace, placement, nullptr, L, N,
                           E, local_per_pair, nullptr);
    return true;
}

}  // namespace exf
