// Shared by the grouped expert GEMM kernels: activations and the launch interface of the weight-streaming path.
#pragma once

#include <math.h>

#include "common.hpp"

namespace exf {

constexpr int kXcdCount = 8;

// Quotient of two wavefront-uniform non-negative numbers; the divisors are powers of two in the common shapes
// (column tiles per row), and a division by a run-time value costs some twenty dependent instructions.
__device__ __forceinline__ unsigned uniform_udiv(unsigned a, unsigned d)
{
    if ((d & (d - 1u)) == 0u) return a >> (31 - __builtin_clz(d | 1u));  // d = 2^k (d = 0 never occurs)
    return a / d;
}

// ---------------------------------------------------------------------------- activations
__device__ __forceinline__ float gelu_erf_exact(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_tanh_exact(float z)
{
    return 0.5f * z * (1.0f + tanhf(0.79788456080286535588f * (z + 0.044715f * z * z * z)));
}

// bf16 path: z * Phi(z) with the normal CDF evaluated as a logistic function of an odd
// polynomial,  Phi(z) ~ 1 / (1 + exp(-z (c0 + c1 z^2 + c2 z^4))),  coefficients fitted (minimax
// on [-10,10]) to the exact erf form: max |error| of the GELU value is 2.6e-5, two orders of
// magnitude below the bf16 rounding the result receives next.  z^2 is clamped where the logistic
// has long saturated, so that the quartic term cannot turn the polynomial around.
__device__ __forceinline__ float gelu_erf_fast(float z)
{
    const float t = fminf(z * z, 60.0f);
    // coefficients carry the factor -log2(e): exp(-z p(t)) = 2^(z q(t)), one v_exp_f32
    float q = fmaf(1.01407394e-3f, t, -1.06774916e-1f);
    q = fmaf(q, t, -2.30112032f);
    const float e = __builtin_amdgcn_exp2f(z * q);
    return z * __builtin_amdgcn_rcpf(1.0f + e);  // v_rcp_f32: 1 ulp
}
// z/2 (1 + tanh u) = z / (1 + exp(-2u))
__device__ __forceinline__ float gelu_tanh_fast(float z)
{
    const float u = 0.79788456080286535588f * (z + 0.044715f * z * z * z);
    return z * __builtin_amdgcn_rcpf(1.0f + __expf(-2.0f * u));
}

// Output rows that no sorted row writes (unrouted[t] < 0), dealt evenly to all wavefronts of the launch, at most 64 at a time.  (64 to each of
// the first ones, these cleared them one after the other in front of their share of the product: 98 tokens of which a tenth is kept, one
// expert of 1600 x 6400, 49.1 us, now 41.9; 1759 of which a fifth, 1216 x 4864, 42.7 and 36.6.)  ALL_AT_ONCE: 64 to each of the first ones all
// the same, for launches of a few microseconds that wait for every instruction in front of their loads (fp32, 394 tokens, 4 experts of
// 76 x 492 15.0 us dealt out and 14.7).
template <bool ALL_AT_ONCE, bool PAIRS>
__device__ __forceinline__ void clear_unrouted_rows(const int32_t* __restrict__ unrouted, int n_unrouted, uint4* __restrict__ out, int vec_per_row, int waves)
{
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t all = gridDim.x * static_cast<uint32_t>(waves);
    uint32_t mine = ALL_AT_ONCE ? kWave : 1;
    while (mine < static_cast<uint32_t>(kWave) && static_cast<uint64_t>(mine) * all < static_cast<uint64_t>(n_unrouted)) mine *= 2;  // (a division takes a quarter of a microsecond)
    for (int64_t first = static_cast<int64_t>(blockIdx.x * static_cast<uint32_t>(waves) + wave) * mine; first < n_unrouted; first += static_cast<int64_t>(all) * mine) {
        const int64_t t = first + lane;
        int pos = 0;
        if (lane < static_cast<int>(mine) && t < n_unrouted) pos = PAIRS ? max(unrouted[2 * t], unrouted[2 * t + 1]) : unrouted[t];
        unsigned long long todo = __ballot(pos < 0);
        while (todo != 0) {
            const int b = __builtin_ctzll(todo);
            todo &= todo - 1;
            uint4* row = out + static_cast<size_t>(first + b) * vec_per_row;
            for (int c = lane; c < vec_per_row; c += kWave) row[c] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
}

enum Epilogue { kEpiNone = 0, kEpiGeluErf = 1, kEpiGeluTanh = 2, kEpiKeepSorted = 3 };  // (the last: tiles of ffn_tiles.hpp, RowMap::sorted_out)

// ---------------------------------------------------------------------------- weight-streaming path
// One contraction  out[rows of e, N] = epi(act[rows, K] * weight_e[N, K]^T + bias_e)  (see ffn_stream.hip).
struct StreamGemm {
    const void* act;          // [*,K]
    const void* weight;       // [E_local,N,K]
    const void* bias;         // [E_local,N] or null
    void* out;                // [*,N]
    const int32_t* offsets;   // [E_local+1]
    const int32_t* a_row;     // operand row of sorted row s is a_row[s] / a_div     (null: row s)
    const int32_t* out_row;   // output row of sorted row s is out_row[s], scaled by out_scale[out_row[s]] (null: row s, no scale)
    const float* out_scale;
    const int32_t* unrouted;  // [n_unrouted]: output row t with unrouted[t] < 0 is set to zero (null: none)
    int n_unrouted;
    int a_div;
    int max_rows;             // row capacity A
    int K, N, E_local;
    int epi;                  // Epilogue
    int E, k, renormalize;    // of the routing below (up here no padding is sent along: another line of arguments is 0.2 us of a launch)
    // Routing instead of sorted rows (first contraction of a short batch; null: `offsets` and `a_row` above): every
    // workgroup sorts the assignments for itself, workgroup 0 writes the maps.
    const int32_t* topk_idx;    // [max_rows]
    const int32_t* expert_map;  // [E] or null
    int32_t *src_of_sorted, *sorted_of_src, *expert_counts, *expert_offsets;
    // At most kFewAssignments: both contractions sort, every wavefront for itself; the second one reads rows in sorted order.  With
    // `w_gate` the first one is the gate of act [T,K] as well (workgroup 0 stores gate_idx and gate_w, and the others compute it, too,
    // where topk_idx is gate_idx).
    const void* w_gate;
    int32_t* gate_idx;
    float* gate_w;
    // The sorted rows besides the result (null: not wanted).  With topk_idx: [*,K], the operand rows in sorted order.
    void* sorted_act;
    // With out_row: [*,N], sorted row s before it is scaled, in the storage type; the scaled one is formed from that, as the combine would.
    void* sorted_out;
    // A top-2 layer whose token rows are added up by the second contraction: [T,N] of the storage type in words of eight bytes, see meet() in
    // ffn_stream.hip.  The first contraction fills them with kNoRow.  (Then out_row: assignments, unrouted: of both.)
    unsigned long long* exchange;
};
constexpr unsigned long long kNoRow = ~0ull;
constexpr int kFewAssignments = 64;
constexpr int kInlineDispatchMax = 1024;  // assignments a workgroup sorts for itself
constexpr int kRoutedTilesMax = 4096;     // ... in a contraction in tiles
// Is the path taken for A rows of `dt` spread over E_local experts?
bool stream_path_fits(int64_t A, int d, int f, int E_local, int dt);
int launch_stream_gemm(const StreamGemm& g, int dt, hipStream_t stream);
// fp32: are both contractions one launch, and that launch (out of the first one is not written).
bool exact_pair_fits(int64_t A, int d, int f, int E_local);
bool exact_pair_routed_fits(int64_t A, int d, int f, int E, int E_local);  // (that sorts; its rows do not meet, see StreamGemm::exchange)
int launch_exact_pair(const StreamGemm& first, const StreamGemm& second, hipStream_t stream);
// Bytes [a, a + n) and [b, b + m) have none in common (a null pointer: there are none).
inline bool lie_apart(const void* a, size_t n, const void* b, size_t m)
{
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return a == nullptr || b == nullptr || (p <= q ? q - p >= n : p - q >= m);
}
// One launch writes results while other workgroups of it still read what the first contraction reads, and write what it leaves besides.  Two launches
// may have these in one place (the result of a layer over the sorted copies of its rows, rows that are written where they were read), so one is
// taken only where the results lie apart from all of that.  Sorted rows over the sorted copies of the same rows are no matter: the thread that
// copies a piece of a row writes the result's as well.
inline bool pair_lies_apart(const StreamGemm& first, const StreamGemm& second)
{
    const size_t A = static_cast<size_t>(first.max_rows), rows = A * first.K * 4, weights = static_cast<size_t>(first.E_local) * first.N;
    const struct {
        const void* at;
        size_t bytes;
    } early[] = {{first.act, first.a_div > 1 ? rows / first.a_div : rows}, {first.weight, weights * first.K * 4}, {first.bias, weights * 4}, {first.sorted_act, rows},
                 {first.a_row, A * 4}, {first.topk_idx, A * 4}, {first.expert_map, static_cast<size_t>(first.E) * 4}, {first.src_of_sorted, A * 4},
                 {first.expert_counts, static_cast<size_t>(first.E_local) * 4}};
    auto apart = [&](const void* to, bool sorted) {
        for (const auto& e : early)
            if (!(sorted && to == first.sorted_act && e.at == to) && !lie_apart(to, rows, e.at, e.bytes)) return false;
        return true;
    };
    return apart(second.out, second.out_row == nullptr) && apart(second.sorted_out, true);
}
inline int launch_stream_pair(const StreamGemm& first, const StreamGemm& second, int dt, hipStream_t stream)
{
    if (dt == EXF_F32 && first.exchange == nullptr) {
        const bool fits = first.topk_idx != nullptr ? exact_pair_routed_fits(first.max_rows, first.K, first.N, first.E, first.E_local)
                                                    : exact_pair_fits(first.max_rows, first.K, first.N, first.E_local);
        if (fits && pair_lies_apart(first, second)) return launch_exact_pair(first, second, stream);
    }
    const int rc = launch_stream_gemm(first, dt, stream);
    return rc == EXF_OK ? launch_stream_gemm(second, dt, stream) : rc;
}

// moe_dispatch and the expert FFN as one: the first contraction sorts the assignments itself.  Only where routed_path_fits() says so;
// the maps, and the sorted rows where they are wanted, are written as moe_dispatch and moe_expert_ffn write them.
struct FfnRouting {
    const int32_t *topk_idx, *expert_map;
    int E;
    int32_t *src_of_sorted, *sorted_of_src, *expert_counts, *expert_offsets;
    const void* w_gate;  // the first contraction is the gate as well (null: it has run); only where gate_joins_layer() says so
    int renormalize;
    int32_t* gate_idx;
    float* gate_w;
    void *x_sorted, *y_sorted;  // null: not wanted
};
inline bool routed_path_fits(int64_t A, int d, int f, int E_local, int dt)
{
    return A > 0 && A <= kInlineDispatchMax && stream_path_fits(A, d, f, E_local, dt);
}
// The same in tiles (bf16, separate calls), with all E experts resident.
bool routed_tiles_fit(int64_t A, int d, int f, int E, int E_local, int dt);
// Is a layer on the routed path gated by its first contraction?  routed: its experts are given, the gate's ids are only stored.
bool gate_joins_layer(int64_t T, int d, int E, int dt, bool routed);
// The expert FFN of a top-1 layer and its combine, moe_expert_ffn and moe_combine in two launches: the same results.
int ffn_combined(const void* x_sorted, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w, const int32_t* expert_offsets,
                 const void* w1, const void* w2, int64_t T, int d, int f, int E_local, int act, int dt, void* y_sorted, void* out, void* workspace,
                 void* stream);
int ffn_fused_routed(const FfnRouting& r, const void* x, const float* topk_w, const void* w1, const void* w2, int64_t T, int k, int d, int f,
                     int E_local, int act, int dt, void* out, void* workspace, size_t workspace_bytes, void* stream);

}  // namespace exf
