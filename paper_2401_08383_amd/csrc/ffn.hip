// moe_expert_ffn: grouped expert FFN  y = act(x W1^T + b1) W2^T + b2  over expert-contiguous rows.
//
// Two launches of one grouped "NT" GEMM kernel  C[rows of e, N] = A[rows, K] * B_e[N, K]^T
// (both operands have the reduction dimension contiguous): the first with the bias+GELU
// epilogue writing the hidden activations of the A rows to the workspace, the second writing y.
// The per-expert row ranges are read from expert_offsets ON THE DEVICE: the grid is sized for
// the worst case and every workgroup locates its own (expert, row tile, column tile) with a
// wavefront scan; surplus workgroups exit at once.
//
// bf16: ffn_tiles.hpp; fp32 and few rows per expert: ffn_stream.hip.
#include "ffn_tiles.hpp"

namespace exf {

// Launches in which some experts have a single row tile, whose weights nobody else reads, and are too many to stay in the
// memory-side cache of 256 MB from call to call (268 MB in both contractions): those tiles load them with the streaming hint.
// us without and with it, the same weights from call to call / other ones each time, as in a model of several layers:
//   tokens, experts                    weights
//   1000, 10 of 1024 x 4096             42 M   54.2 and 61.7 / 62.5 and 60.6
//   1500, 15 of 1024 x 4096             63 M   62.1 and 70.2 / 71.5 and 67.8
//   6000, 60 of 512 x 2048              63 M   76.4 and 83.7 / 85.4 and 81.8
//   6400, 64 of 512 x 2048              67 M   80.6 -> 87.3 / 87.8 -> 83.3
//   1600, 16 of 1024 x 4096             67 M   65.4 -> 66.3 / 72.5 -> 68.6
//   2000, 20 of 1024 x 4096             84 M   93.5 -> 96.4 / 95.0 -> 91.3
//   2400, 24 of 1024 x 4096            101 M   109.9 -> 109.6 / 105.8 -> 101.4
//   600, 4 of 2560 x 10240             105 M   161 -> 144 / 162 -> 160
//   1500, 16 of 2048 x 8192            268 M   217 -> 206 / 214 -> 197
//   6000, 64 of 2048 x 8192           1074 M   835 -> 761 / 866 -> 788
//   1200, 16 of 4096 x 16384          1074 M   827 -> 730 / 852 -> 752 (both begin the reduction at different places)
// Other weights each time gain from 33 M on; called again with the same ones, layers below the line lose up to 15 % by it, up to 84 M at most 8 % (the cache still has
// some of them), beyond nothing.
// The line in rows is where nothing is left to gain or lose, routing as uneven as Zipf's (it leaves some experts one row tile far beyond it, which are then a small
// part of the launch).  us without and with the hint by rows an expert on the mean, 16 experts of 1024 x 4096: 256 127.3 -> 124.7, 512 182.5 -> 181.8, 1024
// 307.1 -> 307.4, 1536 446.3 and 447.3, 2048 549.1 and 551.8; 64 of 1024 x 1024: 256 142.1 -> 139.4, 512 201.9 -> 200.0, 1024 355.9 -> 358.6, 1536 520.4
// and 521.1, 2048 674.0 and 676.6.
constexpr int64_t kStreamedWeights = 1ll << 26;
constexpr int64_t kStreamedMeanRows = 1024;
static bool weights_are_streamed(int64_t A, int K, int N, int E_local)
{
    return A <= kStreamedMeanRows * E_local && static_cast<int64_t>(E_local) * K * N >= kStreamedWeights;
}

static int launch_first_contraction(const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N,
                                    int E_local, int epi, void* out, hipStream_t stream, const RowMap& map)
{
    if (weights_are_streamed(A, K, N, E_local)) return launch_once_first(epi, act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    if (epi == kEpiGeluErf) return launch_bf16_as<256, 8, kEpiGeluErf>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    return launch_bf16_as<256, 8, kEpiGeluTanh>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
}

// In tiles the first contraction sorts where the sorted rows are wanted besides, so that the launch that goes had rows to move, where all experts are resident (few
// rows to move otherwise), where their tiles are one round (every round counts again) and where the weights are not streamed (they are asked for later than
// behind finished offsets).  Separate calls, other tensors each time, with a dispatch of its own and without, us:
//   one round: 4000 tokens, 8 experts of 1024 x 4096 101.5 -> 96.5, 2000 top-2, 8 of 576 x 2304 62.3 -> 57.1, 4096, 4 of 512 x 1024 33.8 -> 32.0,
//     300, 4 of 1024 x 4096 36.8 -> 35.6, 1000, 4 of 512 x 2048 32.8 -> 31.4, 1600, 2 of 2560 x 10240 190.5 -> 189.1, 638, 9 of 896 x 3584 46.5 -> 46.3; where
//     the tensors lie decides most about 2500, 5 of 832 x 3328 71.7 -> 63.3 or 64.4 -> 60.5 and 3000, 6 of 768 x 3072 70.0 -> 71.3 or 71.7 -> 67.7 (45
//     such layers twice: the least 0.98, all others 1.002 or more, 1.04 on the mean)
//   more: 2000 top-2, 32 of 1024 x 4096 138 and 143, 850 top-2, 27 of 3072 x 8512 545 and 574, 4000, 40 of 512 x 2048 71.9 and 73.1, 4000, 4 of
//     4096 x 16384 944 and 949; 4096, 14 of 1024 x 4096 130.8 and 128.9
//   a share of the experts: 4000, 8 of 64 of 1024 x 4096 56.7 and 57.4, 3900, 16 of 64 of 960 x 3840 75.1 and 75.5; with many rows of it kept 2000 top-2, 8 of 32
//     of 768 x 3072 50.6 and 48.3
//   no sorted rows (fused): 4000, 8 of 1024 x 4096 79.8 and 82.1, 300, 4 of them 34.6 and 34.8
//   streamed: 600, 8 of 4096 x 8192 189.6 and 201.1, 1531 top-2, 16 of 1024 x 4096 101.5 and 100.7, 2048 top-2, 8 of 4096 x 4096 301 and 294
bool routed_tiles_fit(int64_t A, int d, int f, int E, int E_local, int dt)
{
    if (dt != EXF_BF16 || A <= 0 || A > kRoutedTilesMax || E_local != E || stream_path_fits(A, d, f, E_local, dt) || weights_are_streamed(A, d, f, E)) return false;
    constexpr int kRows = kTileRows + kQuantum;
    return (A + static_cast<int64_t>(E) * kRows - 1) / (static_cast<int64_t>(E) * kRows) * E * ((f + 255) / 256) <= kComputeUnits;
}

// The second contraction has few output columns (N = d).  With 256x128 tiles it offers twice as many
// tiles, which a short batch needs to fill the chip; the 256x256 tile of the first contraction moves
// a third less operand data per flop through the L2s and is taken once it, too, gives every compute
// unit at least kWideRounds tiles.
constexpr int kWideRounds = 2;
static int launch_second_contraction(const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A,
                                     int K, int N, int E_local, void* out, hipStream_t stream, const RowMap& map)
{
    const int64_t wide_tiles = (A / 256) * ((N + 255) / 256);
    const bool wide = wide_tiles >= static_cast<int64_t>(kWideRounds) * kComputeUnits;
    if (weights_are_streamed(A, K, N, E_local)) return launch_once_second(wide, act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    if (map.sorted_out == nullptr) {
        if (wide) return launch_bf16_as<256, 4, kEpiNone>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
        return launch_bf16_as<128, 4, kEpiNone>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    }
    return launch_kept_contraction(wide, act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
}

}  // namespace exf


namespace exf {
// The workspace the entry points ask for, bf16: hidden activations of A rows, of up to 32 more per expert (see
// hidden_offset), and 16 MiB in reserve (the sizes are part of the interface; a top-2 layer of separate calls uses them, see pairs_meet).
constexpr int kReservedRowsPerExpert = kHiddenRowBlock;
constexpr size_t kReservedBytes = 16u << 20;
static size_t hidden_bytes(int64_t A, int f, int E_local, int dt)
{
    size_t rows = static_cast<size_t>(A > 0 ? A : 1);
    if (dt == EXF_BF16)
        rows = (rows + static_cast<size_t>(kReservedRowsPerExpert) * (E_local > 0 ? E_local : 1) + kReservedRowsPerExpert - 1) / kReservedRowsPerExpert *
               kReservedRowsPerExpert;
    return align_up(rows * static_cast<size_t>(f) * (dt == EXF_BF16 ? 2 : 4), 256);
}
}  // namespace exf

extern "C" size_t moe_expert_ffn_workspace_bytes(int64_t A, int d, int f, int E_local, int dt)
{
    (void)d;
    if (A < 0 || f < 1 || (dt != EXF_F32 && dt != EXF_BF16)) return 0;
    return exf::hidden_bytes(A, f, E_local, dt) + (dt == EXF_BF16 ? exf::kReservedBytes : 0);
}

int exf::check_ffn(const void* x_sorted, const int32_t* expert_offsets, const void* w1, const void* w2, int64_t A, int d, int f, int E_local,
                   int act, int dt, const void* y_sorted, const void* workspace, size_t workspace_bytes)
{
    if (dt != EXF_F32 && dt != EXF_BF16) return fail(EXF_ERR_BAD_DTYPE, "moe_expert_ffn: dt = %d", dt);
    if (act != EXF_ACT_GELU_ERF && act != EXF_ACT_GELU_TANH) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: act = %d", act);
    if (A < 0 || A >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: A = %lld outside [0,2^31)", static_cast<long long>(A));
    if (E_local < 1 || E_local > EXF_MAX_EXPERTS)
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: E_local = %d outside [1,%d]", E_local, EXF_MAX_EXPERTS);
    const int gran = dt == EXF_BF16 ? 64 : 4;
    if (d < gran || d % gran != 0 || f < gran || f % gran != 0)
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: d = %d and f = %d must be positive multiples of %d", d, f, gran);
    if (dt == EXF_BF16) {  // the bf16 kernel addresses rows with 32-bit byte offsets
        const unsigned long long widest = static_cast<unsigned long long>(d > f ? d : f);
        const unsigned long long rows = static_cast<unsigned long long>(A) + static_cast<unsigned long long>(kReservedRowsPerExpert) * (E_local + 1);
        if (rows * widest * 2ull >= (1ull << 32) ||
            static_cast<unsigned long long>(d) * static_cast<unsigned long long>(f) * 2ull >= (1ull << 32))
            return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn: (A + 32 (E_local + 1))*max(d,f) and d*f must stay below 2^31 elements (bf16)");
    }
    if (A == 0) return EXF_OK;
    EXF_CHECK_PTR("moe_expert_ffn", x_sorted);
    EXF_CHECK_PTR("moe_expert_ffn", expert_offsets);
    EXF_CHECK_PTR("moe_expert_ffn", w1);
    EXF_CHECK_PTR("moe_expert_ffn", w2);
    EXF_CHECK_PTR("moe_expert_ffn", y_sorted);
    EXF_CHECK_PTR("moe_expert_ffn", workspace);
    EXF_CHECK_ALIGNED("moe_expert_ffn", x_sorted);
    EXF_CHECK_ALIGNED("moe_expert_ffn", w1);
    EXF_CHECK_ALIGNED("moe_expert_ffn", w2);
    EXF_CHECK_ALIGNED("moe_expert_ffn", y_sorted);
    EXF_CHECK_ALIGNED("moe_expert_ffn", workspace);
    if (workspace_bytes < moe_expert_ffn_workspace_bytes(A, d, f, E_local, dt))
        return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "moe_expert_ffn: workspace %zu < %zu bytes", workspace_bytes,
                    moe_expert_ffn_workspace_bytes(A, d, f, E_local, dt));
    return EXF_OK;
}

extern "C" int moe_expert_ffn(const void* x_sorted, const int32_t* expert_offsets, const void* w1, const void* b1, const void* w2,
                              const void* b2, int64_t A, int d, int f, int E_local, int act, int dt, void* y_sorted,
                              void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace exf;
    if (int rc = check_ffn(x_sorted, expert_offsets, w1, w2, A, d, f, E_local, act, dt, y_sorted, workspace, workspace_bytes)) return rc;
    if (A == 0) return EXF_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int epi = act == EXF_ACT_GELU_ERF ? kEpiGeluErf : kEpiGeluTanh;
    int rc;
    if (stream_path_fits(A, d, f, E_local, dt)) {
        StreamGemm first{}, second{};
        first.act = x_sorted, first.weight = w1, first.bias = b1, first.out = workspace;
        first.K = d, first.N = f, first.epi = epi;
        second.act = workspace, second.weight = w2, second.bias = b2, second.out = y_sorted;
        second.K = f, second.N = d, second.epi = kEpiNone;
        first.offsets = second.offsets = expert_offsets;
        first.max_rows = second.max_rows = static_cast<int>(A);
        first.E_local = second.E_local = E_local;
        rc = launch_stream_pair(first, second, dt, s);
    } else {
        rc = launch_first_contraction(x_sorted, expert_offsets, w1, b1, A, d, f, E_local, epi, workspace, s, RowMap{});
        if (rc == EXF_OK) rc = launch_second_contraction(workspace, expert_offsets, w2, b2, A, f, d, E_local, y_sorted, s, RowMap{});
    }
    if (rc != EXF_OK) return rc;
    return check_launch("moe_expert_ffn");
}

extern "C" int moe_combine(const void* y_sorted, const int32_t* sorted_of_src, const float* topk_w, int64_t T, int d, int k,
                           int dt, void* out, void* stream);

extern "C" size_t moe_expert_ffn_fused_workspace_bytes(int64_t T, int k, int d, int f, int E_local, int dt)
{
    if (T < 0 || k < 1 || k > EXF_MAX_TOPK || d < 1 || f < 1 || (dt != EXF_BF16 && dt != EXF_F32)) return 0;
    const size_t elem = dt == EXF_BF16 ? 2 : 4;
    const size_t A = static_cast<size_t>(T > 0 ? T : 1) * static_cast<size_t>(k);
    size_t bytes = exf::hidden_bytes(static_cast<int64_t>(A), f, E_local, dt);  // hidden activations of A rows
    if (k > 1) bytes += exf::align_up(A * static_cast<size_t>(d) * elem, 256);   // sorted expert outputs [A,d]
    return bytes + (dt == EXF_BF16 ? exf::kReservedBytes : 0);
}

int exf::check_ffn_fused(const void* x, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                         const int32_t* expert_offsets, const void* w1, const void* w2, int64_t T, int k, int d, int f, int E_local, int act,
                         int dt, const void* out, const void* workspace, size_t workspace_bytes)
{
    if (dt != EXF_F32 && dt != EXF_BF16) return fail(EXF_ERR_BAD_DTYPE, "moe_expert_ffn_fused: dt = %d", dt);
    if (act != EXF_ACT_GELU_ERF && act != EXF_ACT_GELU_TANH) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: act = %d", act);
    if (k < 1 || k > EXF_MAX_TOPK) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: k = %d outside [1,%d]", k, EXF_MAX_TOPK);
    if (T < 0 || T * k >= (1ll << 31))
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: T = %lld, T*k outside [0,2^31)", static_cast<long long>(T));
    if (E_local < 1 || E_local > EXF_MAX_EXPERTS)
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: E_local = %d outside [1,%d]", E_local, EXF_MAX_EXPERTS);
    const int gran = dt == EXF_BF16 ? 64 : 4;
    if (d < gran || d % gran != 0 || f < gran || f % gran != 0)
        return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: d = %d and f = %d must be positive multiples of %d", d, f, gran);
    const int64_t A = T * k;
    if (dt == EXF_BF16) {  // the bf16 kernel addresses rows with 32-bit byte offsets
        const unsigned long long widest = static_cast<unsigned long long>(d > f ? d : f);
        const unsigned long long rows = static_cast<unsigned long long>(A) + static_cast<unsigned long long>(kReservedRowsPerExpert) * (E_local + 1);
        if (rows * widest * 2ull >= (1ull << 32) ||
            static_cast<unsigned long long>(d) * static_cast<unsigned long long>(f) * 2ull >= (1ull << 32))
            return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: (T*k + 32 (E_local + 1))*max(d,f) and d*f must stay below 2^31 elements");
    }
    if (T == 0) return EXF_OK;
    EXF_CHECK_PTR("moe_expert_ffn_fused", x);
    EXF_CHECK_PTR("moe_expert_ffn_fused", src_of_sorted);
    EXF_CHECK_PTR("moe_expert_ffn_fused", sorted_of_src);
    EXF_CHECK_PTR("moe_expert_ffn_fused", topk_w);
    EXF_CHECK_PTR("moe_expert_ffn_fused", expert_offsets);
    EXF_CHECK_PTR("moe_expert_ffn_fused", w1);
    EXF_CHECK_PTR("moe_expert_ffn_fused", w2);
    EXF_CHECK_PTR("moe_expert_ffn_fused", out);
    EXF_CHECK_PTR("moe_expert_ffn_fused", workspace);
    EXF_CHECK_ALIGNED("moe_expert_ffn_fused", x);
    EXF_CHECK_ALIGNED("moe_expert_ffn_fused", w1);
    EXF_CHECK_ALIGNED("moe_expert_ffn_fused", w2);
    EXF_CHECK_ALIGNED("moe_expert_ffn_fused", out);
    EXF_CHECK_ALIGNED("moe_expert_ffn_fused", workspace);
    if (x == out) return fail(EXF_ERR_BAD_SHAPE, "moe_expert_ffn_fused: out must not alias x");
    const size_t need = moe_expert_ffn_fused_workspace_bytes(T, k, d, f, E_local, dt);
    if (workspace_bytes < need) return fail(EXF_ERR_WORKSPACE_TOO_SMALL, "moe_expert_ffn_fused: workspace %zu < %zu bytes", workspace_bytes, need);
    return EXF_OK;
}

// Do the two rows of a token of a top-2 layer meet in the second contraction (meet() in ffn_stream.hip) instead of in a combine?  Where the first
// one sorts, so that the maps are this call's and the words have been cleared; of the separate calls, whose workspace has no room of its own for
// these, those in bf16 that get by with the reserve.  Past a gigabyte of weights of the second contraction the launch saved is
// less than a hundredth, and the wait for the exchange at the end of every block has cost more (8 tokens, 16 experts of 4096 x 16384 426 and 433 us).
constexpr int64_t kMeetingWeights = 1ll << 29;
static bool pairs_meet(int64_t T, int k, int d, int f, int E_local, int dt, bool fused)
{
    const int64_t A = T * k;
    return k == 2 && exf::routed_path_fits(A, d, f, E_local, dt) && (A < E_local ? A : E_local) * d * f <= kMeetingWeights &&
           (fused || (dt == EXF_BF16 && static_cast<size_t>(T) * d * 2 <= exf::kReservedBytes));
}

static int ffn_fused_run(const void* x, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                         const int32_t* expert_offsets, const void* w1, const void* b1, const void* w2, const void* b2, int64_t T, int k,
                         int d, int f, int E_local, int act, int dt, void* out, void* workspace, size_t workspace_bytes, void* stream,
                         unsigned long long* timeline, int timeline_cap, const exf::FfnRouting* routing = nullptr)
{
    using namespace exf;
    if (routing == nullptr) {  // (a layer's arguments have been checked)
        if (int rc = check_ffn_fused(x, src_of_sorted, sorted_of_src, topk_w, expert_offsets, w1, w2, T, k, d, f, E_local, act, dt, out, workspace,
                                     workspace_bytes))
            return rc;
    }
    if (T == 0) return EXF_OK;
    const int64_t A = T * k;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int epi = act == EXF_ACT_GELU_ERF ? kEpiGeluErf : kEpiGeluTanh;
    unsigned char* hidden = static_cast<unsigned char*>(workspace);
    RowMap gather{};
    gather.a_row = src_of_sorted;
    gather.a_div = k;
    gather.timeline = timeline;  // first contraction: records [0, cap), second: [cap, 2 cap)
    gather.timeline_cap = timeline_cap;
    RowMap scatter{};
    scatter.timeline = timeline != nullptr ? timeline + static_cast<size_t>(timeline_cap) * 8 : nullptr;
    scatter.timeline_cap = timeline_cap;
    const bool pairs = routing != nullptr && timeline == nullptr && pairs_meet(T, k, d, f, E_local, dt, routing->y_sorted == nullptr);
    if (k == 1 || pairs) {
        scatter.out_row = src_of_sorted;  // (k = 1: the flat assignment index is the token)
        scatter.out_scale = topk_w;
        scatter.unrouted = sorted_of_src;
        scatter.n_unrouted = static_cast<int>(T);
    }
    void* y_sorted = routing != nullptr && routing->y_sorted != nullptr ? routing->y_sorted : hidden + hidden_bytes(A, f, E_local, dt);
    void* second_out = k == 1 || pairs ? out : y_sorted;
    int rc;
    if (timeline == nullptr && stream_path_fits(A, d, f, E_local, dt)) {
        StreamGemm first{}, second{};
        first.act = x, first.weight = w1, first.bias = b1, first.out = hidden;
        first.a_row = src_of_sorted, first.a_div = k;
        if (routing != nullptr) {
            first.topk_idx = routing->topk_idx, first.expert_map = routing->expert_map, first.E = routing->E;
            first.src_of_sorted = routing->src_of_sorted, first.sorted_of_src = routing->sorted_of_src;
            first.expert_counts = routing->expert_counts, first.expert_offsets = routing->expert_offsets;
            first.w_gate = routing->w_gate, first.renormalize = routing->renormalize;
            first.k = second.k = k;
            first.gate_idx = routing->gate_idx, first.gate_w = routing->gate_w;
            first.sorted_act = routing->x_sorted;
            if (k == 1 || pairs) second.sorted_out = routing->y_sorted;
            if (pairs) first.exchange = second.exchange = reinterpret_cast<unsigned long long*>(hidden + hidden_bytes(A, f, E_local, dt));
            if (dt == EXF_BF16 && A <= kFewAssignments) {
                second.topk_idx = routing->topk_idx, second.expert_map = routing->expert_map, second.E = routing->E;
            }
        }
        first.K = d, first.N = f, first.epi = epi;
        second.act = hidden, second.weight = w2, second.bias = b2, second.out = second_out;
        second.out_row = scatter.out_row, second.out_scale = scatter.out_scale;
        second.unrouted = scatter.unrouted, second.n_unrouted = scatter.n_unrouted;
        second.K = f, second.N = d, second.epi = kEpiNone;
        first.offsets = second.offsets = expert_offsets;
        first.max_rows = second.max_rows = static_cast<int>(A);
        first.E_local = second.E_local = E_local;
        rc = launch_stream_pair(first, second, dt, s);
    } else {
        if (routing != nullptr) {
            const TileRouting route{routing->topk_idx,      routing->expert_map,     routing->src_of_sorted, routing->sorted_of_src,
                                    routing->expert_counts, routing->expert_offsets, static_cast<bf16_t*>(routing->x_sorted), routing->E, k};
            if (k == 1) scatter.sorted_out = static_cast<bf16_t*>(routing->y_sorted);
            rc = launch_routed_first(epi, x, w1, A, d, f, E_local, hidden, s, route);
        } else {
            rc = launch_first_contraction(x, expert_offsets, w1, b1, A, d, f, E_local, epi, hidden, s, gather);
        }
        if (rc == EXF_OK) rc = launch_second_contraction(hidden, expert_offsets, w2, b2, A, f, d, E_local, second_out, s, scatter);
    }
    if (rc != EXF_OK) return rc;
    if (k == 1 || pairs) return check_launch("moe_expert_ffn_fused");
    rc = check_launch("moe_expert_ffn_fused");
    if (rc != EXF_OK) return rc;
    return moe_combine(y_sorted, sorted_of_src, topk_w, T, d, k, dt, out, stream);
}

extern "C" int moe_expert_ffn_fused(const void* x, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                                    const int32_t* expert_offsets, const void* w1, const void* b1, const void* w2, const void* b2,
                                    int64_t T, int k, int d, int f, int E_local, int act, int dt, void* out, void* workspace,
                                    size_t workspace_bytes, void* stream)
{
    return ffn_fused_run(x, src_of_sorted, sorted_of_src, topk_w, expert_offsets, w1, b1, w2, b2, T, k, d, f, E_local, act, dt, out,
                         workspace, workspace_bytes, stream, nullptr, 0);
}

int exf::ffn_combined(const void* x_sorted, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                      const int32_t* expert_offsets, const void* w1, const void* w2, int64_t T, int d, int f, int E_local, int act, int dt,
                      void* y_sorted, void* out, void* workspace, void* stream)
{
    if (T == 0) return EXF_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int epi = act == EXF_ACT_GELU_ERF ? kEpiGeluErf : kEpiGeluTanh;
    int rc;
    if (stream_path_fits(T, d, f, E_local, dt)) {
        StreamGemm first{}, second{};
        first.act = x_sorted, first.weight = w1, first.out = workspace;
        first.K = d, first.N = f, first.epi = epi;
        second.act = workspace, second.weight = w2, second.out = out, second.sorted_out = y_sorted;
        second.out_row = src_of_sorted, second.out_scale = topk_w;
        second.unrouted = sorted_of_src, second.n_unrouted = static_cast<int>(T);
        second.K = f, second.N = d, second.epi = kEpiNone;
        first.offsets = second.offsets = expert_offsets;
        first.max_rows = second.max_rows = static_cast<int>(T);
        first.E_local = second.E_local = E_local;
        rc = launch_stream_pair(first, second, dt, s);
    } else {
        RowMap scatter{};
        scatter.out_row = src_of_sorted, scatter.out_scale = topk_w;
        scatter.unrouted = sorted_of_src, scatter.n_unrouted = static_cast<int>(T);
        scatter.sorted_out = static_cast<bf16_t*>(y_sorted);
        rc = launch_first_contraction(x_sorted, expert_offsets, w1, nullptr, T, d, f, E_local, epi, workspace, s, RowMap{});
        if (rc == EXF_OK) rc = launch_second_contraction(workspace, expert_offsets, w2, nullptr, T, f, d, E_local, out, s, scatter);
    }
    return rc == EXF_OK ? check_launch("moe_layer_forward") : rc;
}

int exf::ffn_fused_routed(const FfnRouting& r, const void* x, const float* topk_w, const void* w1, const void* w2, int64_t T, int k, int d, int f,
                          int E_local, int act, int dt, void* out, void* workspace, size_t workspace_bytes, void* stream)
{
    return ffn_fused_run(x, r.src_of_sorted, r.sorted_of_src, topk_w, r.expert_offsets, w1, nullptr, w2, nullptr, T, k, d, f,
                         E_local, act, dt, out, workspace, workspace_bytes, stream, nullptr, 0, &r);
}

// moe_expert_ffn_fused (bf16) with a per-workgroup timeline of both contractions (see RowMap::timeline).
extern "C" int exf_probe_ffn_timeline(const void* x, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                                      const int32_t* expert_offsets, const void* w1, const void* w2, int64_t T, int k, int d, int f,
                                      int E_local, void* out, void* workspace, size_t workspace_bytes, uint64_t* timeline,
                                      int capacity, void* stream)
{
    EXF_REQUIRE_PTR(timeline);
    if (capacity < 1) return exf::fail(EXF_ERR_BAD_SHAPE, "exf_probe_ffn_timeline: capacity = %d < 1", capacity);
    return ffn_fused_run(x, src_of_sorted, sorted_of_src, topk_w, expert_offsets, w1, nullptr, w2, nullptr, T, k, d, f,
                         E_local, EXF_ACT_GELU_ERF, EXF_BF16, out, workspace, workspace_bytes, stream,
                         reinterpret_cast<unsigned long long*>(timeline), capacity);
}
