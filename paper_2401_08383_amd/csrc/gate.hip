// moe_gate_topk / moe_topk_from_logits: gate GEMM + softmax + top-k routing.
//
// The gate contraction is skinny (N = E <= 64 outputs per token): bound by the HBM read of x for long batches and by the
// weights of all experts passing through every compute unit for short ones.  bf16 runs on the matrix cores (experts
// on the MFMA row axis, tokens on the column axis, so that a token's logits sit in 4 lanes); softmax and selection are
// fp32.  fp32 inputs (small layers) use one wavefront per token with wavefront reductions.
#include "gate_tile.hpp"

namespace exf {

// Wavefront routing: lane e holds logit e (lanes >= E hold -inf).  Every lane returns the result.
__device__ __forceinline__ void wave_argmax(float& v, int& i)
{
    best_of_pair<32>(v, i);
    best_of_pair<16>(v, i);
    best_of_pair<8>(v, i);
    best_of_pair<4>(v, i);
    best_of_pair<2>(v, i);
    best_of_pair<1>(v, i);
}

__device__ __forceinline__ Route route_wave(float my_logit, int E, int k, int renormalize)
{
    const int lane = lane_id();
    const bool live = lane < E;
    Route r;
    float v = live ? my_logit : -INFINITY;
    int i = live ? lane : kWave + lane;
    wave_argmax(v, i);
    const float l0 = v;
    r.i0 = i;
    float l1 = 0.0f;
    r.i1 = -1;
    if (k > 1) {
        v = (live && lane != r.i0) ? my_logit : -INFINITY;
        i = (live && lane != r.i0) ? lane : kWave + lane;
        wave_argmax(v, i);
        l1 = v;
        r.i1 = i;
    }
    const float s = wave_sum(live ? expf(my_logit - l0) : 0.0f);
    route_weights(r, l0, l1, s, k, renormalize);
    return r;
}

// ------------------------------------------------------------------------------------------
// Routing from stored logits: one wavefront per token, lane e reads logits[t][e].
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void topk_from_logits_kernel(const float* __restrict__ logits, int64_t T, int E, int k,
                                                                int renormalize, int32_t* __restrict__ topk_idx,
                                                                float* __restrict__ topk_w)
{
    const int lane = lane_id();
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x / kWave);
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave; t < T; t += waves) {
        const float l = lane < E ? logits[t * E + lane] : 0.0f;
        const Route r = route_wave(l, E, k, renormalize);
        if (lane == 0) store_route(r, t, k, topk_idx, topk_w);
    }
}

// ------------------------------------------------------------------------------------------
// fp32 gate: one wavefront per token; lanes split the reduction dimension.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gate_f32_kernel(const float* __restrict__ x, const float* __restrict__ wg, int64_t T,
                                                        int d, int E, int k, int renormalize,
                                                        float* __restrict__ logits_out, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_w)
{
    const int lane = lane_id();
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x / kWave);
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave; t < T; t += waves) {
        const float* xr = x + t * d;
        float mine = 0.0f;
        // eight experts at a time: their loads and their wavefront sums (six dependent steps each) overlap
        constexpr int EB = 8;
        for (int e0 = 0; e0 < E; e0 += EB) {
            float acc[EB];
#pragma unroll
            for (int j = 0; j < EB; ++j) acc[j] = 0.0f;
            for (int c = lane * 4; c < d; c += kWave * 4) {
                const float4 a = *reinterpret_cast<const float4*>(xr + c);
                float4 b[EB];
#pragma unroll
                for (int j = 0; j < EB; ++j) b[j] = *reinterpret_cast<const float4*>(wg + static_cast<int64_t>(min(e0 + j, E - 1)) * d + c);
#pragma unroll
                for (int j = 0; j < EB; ++j) {
                    acc[j] = fmaf(a.x, b[j].x, acc[j]);
                    acc[j] = fmaf(a.y, b[j].y, acc[j]);
                    acc[j] = fmaf(a.z, b[j].z, acc[j]);
                    acc[j] = fmaf(a.w, b[j].w, acc[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < EB; ++j) acc[j] = wave_sum(acc[j]);
#pragma unroll
            for (int j = 0; j < EB; ++j)
                if (lane == e0 + j) mine = acc[j];
        }
        if (logits_out != nullptr && lane < E) logits_out[t * E + lane] = mine;
        const Route r = route_wave(mine, E, k, renormalize);
        if (lane == 0) store_route(r, t, k, topk_idx, topk_w);
    }
}

// ------------------------------------------------------------------------------------------
// bf16 gate: a workgroup takes 16 MT tokens, its W wavefronts deal the 128-byte units of the reduction among themselves
// and stream weights and token rows through rings of their own in LDS (eight rows of 128 bytes per direct-to-LDS load,
// no barrier until the sums are added).  Loaded straight into registers in the lane layout of the matrix cores, each
// load touches 64 pieces of 16 bytes and the address unit is what the launch waits for: 64 experts x 4096 took 21.9 us
// for 256 tokens and 62 for 16384, 9.8 and 31 this way.
// ------------------------------------------------------------------------------------------
template <int NT, int MT, int W>
struct GateRing {
    static constexpr int kSlot = (NT + MT) * 2048;  // 16 NT expert rows, then 16 MT token rows, of 128 bytes
    static constexpr int kFit = 144 * 1024 / (W * kSlot);
    static constexpr int kSlots = kFit > 4 ? 4 : kFit;
    static constexpr size_t kBytes = static_cast<size_t>(W) * kSlots * kSlot;
};

template <int NT, int MT, int W>
__global__ __launch_bounds__(W * 64) void gate_stream_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg, int64_t T, int d,
                                                             int E, int k, int renormalize, float* __restrict__ logits_out,
                                                             int32_t* __restrict__ topk_idx, float* __restrict__ topk_w)
{
    typedef GateRing<NT, MT, W> Ring;
    constexpr int R = Ring::kSlots, SLOT = Ring::kSlot, LPU = 2 * (NT + MT);
    static_assert(MT <= W, "a wavefront per token tile routes");
    static_assert(R >= 2 && (R - 1) * LPU < 64, "ring depth against the 6-bit vmcnt");
    extern __shared__ __attribute__((aligned(1024))) unsigned char gate_smem[];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r8 = lane >> 3, c8 = lane & 7;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * (16 * MT);
    const uint32_t ring_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)gate_smem)) + wave * (R * SLOT);
    unsigned char* ring = gate_smem + wave * (R * SLOT);
    const uint32_t row_bytes = static_cast<uint32_t>(d) * 2u;
    const unsigned char* w_base = uniform_ptr(reinterpret_cast<const unsigned char*>(wg));
    const unsigned char* x_base = uniform_ptr(reinterpret_cast<const unsigned char*>(x) + static_cast<size_t>(t0) * row_bytes);
    // LDS row r of a slot holds 16-byte piece c at position c ^ ((r / 2) % 8); rows past the last expert or token repeat it
    uint32_t off[LPU];
#pragma unroll
    for (int i = 0; i < LPU; ++i) {
        const int r = i * 8 + r8;
        const int row = i < 2 * NT ? min(r, E - 1) : static_cast<int>(min(static_cast<int64_t>(r - 16 * NT), T - 1 - t0));
        off[i] = static_cast<uint32_t>(row) * row_bytes + ((c8 ^ ((r >> 1) & 7)) * 16);
    }
    const int units = (d + 63) / 64;
    const int cnt = wave < units ? (units - wave + W - 1) / W : 0;
    const int tail = d / 8 - (units - 1) * 8;  // 16-byte pieces of a row in the last unit (8 unless d is ragged)
    auto issue = [&](int u) {
        const size_t at = static_cast<size_t>(wave + u * W) * 128;
        const uint32_t slot = ring_addr + (u % R) * SLOT;
        if (tail == 8 || wave + u * W + 1 < units) {
#pragma unroll
            for (int i = 0; i < LPU; ++i) lds_dma_16B((i < 2 * NT ? w_base : x_base) + at, off[i], slot + i * 1024);
        } else {  // pieces past the row's end repeat the unit's first one; the tokens' are zeroed below
#pragma unroll
            for (int i = 0; i < LPU; ++i) {
                const int piece = c8 ^ (((i * 8 + r8) >> 1) & 7);
                lds_dma_16B((i < 2 * NT ? w_base : x_base) + at, off[i] - (piece >= tail ? piece * 16 : 0), slot + i * 1024);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u < cnt) issue(u);
    const int r16 = lane & 15, g = lane >> 4;
    int frag[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) frag[h] = r16 * 128 + (((4 * h + g) ^ (r16 >> 1)) * 16);
    f32x4_t acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int u = 0; u < cnt; ++u) {
        const int younger = min(R - 1, cnt - 1 - u);
        if (R >= 4 && younger >= 3) wait_vmcnt<(R >= 4 ? 3 : 0) * LPU>();
        else if (R >= 3 && younger >= 2) wait_vmcnt<(R >= 3 ? 2 : 0) * LPU>();
        else if (younger >= 1) wait_vmcnt<LPU>();
        else wait_vmcnt<0>();
        const unsigned char* s = ring + (u % R) * SLOT;
        bf16x8_t a[NT][2], b[MT][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) a[nt][h] = *reinterpret_cast<const bf16x8_t*>(s + nt * 2048 + frag[h]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) b[mt][h] = *reinterpret_cast<const bf16x8_t*>(s + (NT + mt) * 2048 + frag[h]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read: it may be filled again
        if (u + R < cnt) issue(u + R);
        if (tail < 8 && wave + u * W + 1 == units) {
            const bf16x8_t zero8 = {};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    if (4 * h + g >= tail) b[mt][h] = zero8;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[nt][h], b[mt][h], acc[mt][nt], 0, 0, 0);
    }
    // sums of the wavefronts, in order: wavefront mt adds and routes token tile mt
    static_assert(MT * NT * kWave * 16 <= R * SLOT, "the sums must fit the ring");
    f32x4_t* red = reinterpret_cast<f32x4_t*>(ring);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[(mt * NT + nt) * kWave + lane] = acc[mt][nt];
    __syncthreads();
    if (wave >= MT) return;
    f32x4_t sum[NT];
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const f32x4_t v = reinterpret_cast<const f32x4_t*>(gate_smem + w * (R * SLOT))[(wave * NT + nt) * kWave + lane];
            sum[nt] = w == 0 ? v : sum[nt] + v;
        }
    route_quads<NT>(sum, t0 + wave * 16 + r16, T, E, k, renormalize, logits_out, topk_idx, topk_w);
}

template <int NT, int MT, int W>
static int launch_gate_stream(const void* x, const void* wg, int64_t T, int d, int E, int k, int renormalize, float* logits_out,
                              int32_t* topk_idx, float* topk_w, hipStream_t stream)
{
    constexpr size_t lds = GateRing<NT, MT, W>::kBytes;
    auto kern = gate_stream_kernel<NT, MT, W>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_gate_topk")) return rc;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((T + 16 * MT - 1) / (16 * MT))), dim3(W * kWave), lds, stream, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(wg), T, d, E, k, renormalize, logits_out, topk_idx, topk_w);
    return EXF_OK;
}

// ------------------------------------------------------------------------------------------
// bf16 gate of a long batch: a workgroup takes 64 tokens, a wavefront 16 of them over the whole reduction, and the weights of a
// unit are fetched once for all four, into the slot of its token rows.  What bounds it is the read of x.  gate_stream_kernel reads
// the weights for every wavefront into rings of 128 KB and more, half of it weights: one workgroup per compute unit, so each
// round of workgroups waits for its first loads and for the addition of its sums.  Here 64 KB do, the next workgroup's
// loads run beside, and the sums need no LDS.  32768 tokens: 1024, 64 experts 20.7 us before and 15.6 now; 2048, 64
// experts 34.7 and 30.5; 1024, 8 experts 16.5 and 13.7; 2048, 8 experts 36.2 and 27.3 (2.5 to 4.9 TB/s of x).
// x loaded past the caches is up to 8 % faster here and 2 % slower in a layer, whose first contraction reads x next (32768
// tokens, 8 of 64 experts resident: 544 and 554 us with the gate at 15.5 and 15.9).
// ------------------------------------------------------------------------------------------
constexpr int kLongWaves = 4;
template <int NT>
struct GateLongRing {
    static constexpr int kSlot = (NT + kLongWaves) * 2048;  // 16 NT expert rows, then 16 token rows of every wavefront
    static constexpr int kSlots = 64 * 1024 / kSlot;        // (two or three workgroups a compute unit)
    static constexpr size_t kBytes = static_cast<size_t>(kSlots) * kSlot;
};

template <int NT, int SUMS>
__global__ __launch_bounds__(kLongWaves * 64) void gate_long_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg, int64_t T, int d,
                                                                    int E, int k, int renormalize, float* __restrict__ logits_out,
                                                                    int32_t* __restrict__ topk_idx, float* __restrict__ topk_w)
{
    typedef GateLongRing<NT> Ring;
    constexpr int R = Ring::kSlots, SLOT = Ring::kSlot;
    constexpr int LW = (2 * NT + kLongWaves - 1) / kLongWaves, LPU = LW + 2;  // eight-row loads of a wavefront and unit
    static_assert(R >= 4 && R <= 6 && (R - 2) * LPU < 64, "ring depth: the waits below, the 6-bit vmcnt");
    extern __shared__ __attribute__((aligned(1024))) unsigned char gate_smem[];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r8 = lane >> 3, c8 = lane & 7;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * (16 * kLongWaves) + wave * 16;
    const uint32_t ring_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)gate_smem));
    const uint32_t row_bytes = static_cast<uint32_t>(d) * 2u;
    const unsigned char* w_base = uniform_ptr(reinterpret_cast<const unsigned char*>(wg));
    const unsigned char* x_base = uniform_ptr(reinterpret_cast<const unsigned char*>(x) + static_cast<size_t>(min(t0, T - 1)) * row_bytes);
    const int last = static_cast<int>(min(max(T - 1 - t0, static_cast<int64_t>(0)), static_cast<int64_t>(15)));  // (a wavefront past the last token repeats it)
    // LDS row r of a group of 16 holds 16-byte piece c at position c ^ ((r / 2) % 8); rows past the last expert or token repeat it
    int group[LW];  // of eight experts; past the last one it is loaded once more
    uint32_t off_w[LW], off_x[2];
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        group[i] = min(i * kLongWaves + wave, 2 * NT - 1);
        const int r = group[i] * 8 + r8;
        off_w[i] = static_cast<uint32_t>(min(r, E - 1)) * row_bytes + ((c8 ^ ((r >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = i * 8 + r8;
        off_x[i] = static_cast<uint32_t>(min(r, last)) * row_bytes + ((c8 ^ ((r >> 1) & 7)) * 16);
    }
    const int units = (d + 63) / 64;
    const int tail = d / 8 - (units - 1) * 8;  // 16-byte pieces of a row in the last unit (8 unless d is ragged)
    auto issue = [&](int u) {
        const size_t at = static_cast<size_t>(u) * 128;
        const uint32_t slot = ring_addr + (u % R) * SLOT;
        const uint32_t slot_x = slot + (NT + wave) * 2048;
        if (tail == 8 || u + 1 < units) {
#pragma unroll
            for (int i = 0; i < LW; ++i) lds_dma_16B(w_base + at, off_w[i], slot + group[i] * 1024);
#pragma unroll
            for (int i = 0; i < 2; ++i) lds_dma_16B(x_base + at, off_x[i], slot_x + i * 1024);
        } else {  // pieces past the row's end repeat the unit's first one; the tokens' are zeroed below
            auto cut = [&](int r) {
                const int piece = c8 ^ ((r >> 1) & 7);
                return static_cast<uint32_t>(piece >= tail ? piece * 16 : 0);
            };
#pragma unroll
            for (int i = 0; i < LW; ++i) lds_dma_16B(w_base + at, off_w[i] - cut(group[i] * 8 + r8), slot + group[i] * 1024);
#pragma unroll
            for (int i = 0; i < 2; ++i) lds_dma_16B(x_base + at, off_x[i] - cut(i * 8 + r8), slot_x + i * 1024);
        }
    };
#pragma unroll
    for (int u = 0; u < R - 1; ++u)
        if (u < units) issue(u);
    const int r16 = lane & 15, g = lane >> 4;
    int frag[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) frag[h] = r16 * 128 + (((4 * h + g) ^ (r16 >> 1)) * 16);
    // sum j is that of the units j, j + SUMS, ..; added in order, they are the sums of gate_stream_kernel's wavefronts
    f32x4_t acc[SUMS][NT];
#pragma unroll
    for (int j = 0; j < SUMS; ++j)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[j][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int u0 = 0; u0 < units; u0 += SUMS) {
#pragma unroll
        for (int j = 0; j < SUMS; ++j) {
            const int u = u0 + j;
            if (u >= units) break;
            const int younger = min(R - 2, units - 1 - u);
            if (R >= 6 && younger >= 4) wait_vmcnt<(R >= 6 ? 4 : 0) * LPU>();
            else if (R >= 5 && younger >= 3) wait_vmcnt<(R >= 5 ? 3 : 0) * LPU>();
            else if (younger >= 2) wait_vmcnt<2 * LPU>();
            else if (younger >= 1) wait_vmcnt<LPU>();
            else wait_vmcnt<0>();
            // everyone's share of unit u has landed, and everyone has read unit u - 1: its slot may be filled again
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (u + R - 1 < units) issue(u + R - 1);
            const unsigned char* s = gate_smem + (u % R) * SLOT;
            bf16x8_t a[NT][2], b[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                b[h] = *reinterpret_cast<const bf16x8_t*>(s + (NT + wave) * 2048 + frag[h]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) a[nt][h] = *reinterpret_cast<const bf16x8_t*>(s + nt * 2048 + frag[h]);
            }
            if (tail < 8 && u + 1 == units) {
                const bf16x8_t zero8 = {};
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (4 * h + g >= tail) b[h] = zero8;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[nt][h], b[h], acc[j][nt], 0, 0, 0);
        }
    }
    f32x4_t sum[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        sum[nt] = acc[0][nt];
#pragma unroll
        for (int j = 1; j < SUMS; ++j) sum[nt] = sum[nt] + acc[j][nt];
    }
    route_quads<NT>(sum, t0 + r16, T, E, k, renormalize, logits_out, topk_idx, topk_w);
}

template <int NT, int SUMS>
static int launch_gate_long(const void* x, const void* wg, int64_t T, int d, int E, int k, int renormalize, float* logits_out,
                            int32_t* topk_idx, float* topk_w, hipStream_t stream)
{
    constexpr size_t lds = GateLongRing<NT>::kBytes;
    auto kern = gate_long_kernel<NT, SUMS>;
    static std::atomic<uint64_t> allowed{0};
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed, "moe_gate_topk")) return rc;
    constexpr int tokens = 16 * kLongWaves;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>((T + tokens - 1) / tokens)), dim3(kLongWaves * kWave), lds, stream,
                       static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(wg), T, d, E, k, renormalize, logits_out, topk_idx, topk_w);
    return EXF_OK;
}

// Tokens per workgroup of gate_stream_kernel: 16, or 64 where more than 16 experts' weights go through every compute unit and the
// batch still gives half of them a workgroup (12000 tokens x 1024, 64 experts: 14.6 us with 16, 9.8 with 64; 4096 x 1024, 64
// experts: 5.6 and 7.1).
// gate_long_kernel where that one would begin a second round of workgroups: more than 16 experts from 64 x 256 tokens on (there itself
// 10.9 us against 10.1 for 1024, 64 experts, but 29.6 against 31.0 for 4096, 48 experts; 17001 x 1024, 64 experts: 17.9 and 14.1).
// At most 16 experts: the other kernel deals 16 tokens at a time, so only where the rounds of 64-token workgroups are half full
// at least (8 experts x 1024: 20000 tokens 11.2 and 11.7, 24576 13.1 and 12.0, 65536 30.3 and 25.5) and the reduction is not so long
// that it keeps eight wavefronts busy (8 experts x 4096, 32768 tokens: 53.9 and 54.7; x 3072: 48.5 and 36.0).
constexpr int kLongRound = 256;  // one workgroup per compute unit
template <int NT>
static int dispatch_gate_bf16(const void* x, const void* wg, int64_t T, int d, int E, int k, int renormalize,
                              float* logits_out, int32_t* topk_idx, float* topk_w, hipStream_t stream)
{
    const int64_t workgroups = (T + 16 * kLongWaves - 1) / (16 * kLongWaves), last_round = workgroups % kLongRound;
    const bool full = workgroups >= kLongRound && (last_round == 0 || last_round >= kLongRound / 2 || workgroups > 2 * kLongRound);
    if (NT > 1 ? workgroups > kLongRound : (full && d <= 3072)) {
        if (NT == 1 && d >= 2048) return launch_gate_long<NT, NT == 1 ? 8 : 4>(x, wg, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, stream);
        return launch_gate_long<NT, 4>(x, wg, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, stream);
    }
    if (NT > 1 && T >= 64 * 128) return launch_gate_stream<NT, 4, 4>(x, wg, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, stream);
    if (gate_sums(NT, d) == 8) return launch_gate_stream<NT, 1, NT <= 2 ? 8 : 4>(x, wg, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, stream);
    return launch_gate_stream<NT, 1, 4>(x, wg, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, stream);
}

static int validate_topk_args(const char* fn, int64_t T, int E, int k)
{
    if (T < 0) return fail(EXF_ERR_BAD_SHAPE, "%s: T = %lld < 0", fn, static_cast<long long>(T));
    if (E < 1 || E > EXF_MAX_EXPERTS) return fail(EXF_ERR_BAD_SHAPE, "%s: E = %d outside [1,%d]", fn, E, EXF_MAX_EXPERTS);
    if (k < 1 || k > EXF_MAX_TOPK || k > E)
        return fail(EXF_ERR_BAD_SHAPE, "%s: k = %d outside [1,min(E,%d)]", fn, k, EXF_MAX_TOPK);
    if (T * k >= (1ll << 31)) return fail(EXF_ERR_BAD_SHAPE, "%s: T*k must be below 2^31", fn);
    return EXF_OK;
}

int check_gate(const void* x, const void* w_gate, int64_t T, int d, int E, int k, int dt, const int32_t* topk_idx, const float* topk_w)
{
    if (dt != EXF_F32 && dt != EXF_BF16) return fail(EXF_ERR_BAD_DTYPE, "moe_gate_topk: dt = %d", dt);
    if (int rc = validate_topk_args("moe_gate_topk", T, E, k)) return rc;
    const int gran = dt == EXF_BF16 ? 8 : 4;
    if (d < gran || d % gran != 0)
        return fail(EXF_ERR_BAD_SHAPE, "moe_gate_topk: d = %d must be a positive multiple of %d", d, gran);
    if (T == 0) return EXF_OK;
    EXF_CHECK_PTR("moe_gate_topk", x);
    EXF_CHECK_PTR("moe_gate_topk", w_gate);
    EXF_CHECK_PTR("moe_gate_topk", topk_idx);
    EXF_CHECK_PTR("moe_gate_topk", topk_w);
    EXF_CHECK_ALIGNED("moe_gate_topk", x);
    EXF_CHECK_ALIGNED("moe_gate_topk", w_gate);
    return EXF_OK;
}

}  // namespace exf

extern "C" int moe_gate_topk(const void* x, const void* w_gate, int64_t T, int d, int E, int k, int renormalize, int dt,
                             float* logits_out, int32_t* topk_idx, float* topk_w, void* stream)
{
    using namespace exf;
    if (int rc = check_gate(x, w_gate, T, d, E, k, dt, topk_idx, topk_w)) return rc;
    if (T == 0) return EXF_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dt == EXF_F32) {
        const int64_t blocks = (T + 3) / 4;
        hipLaunchKernelGGL(gate_f32_kernel, dim3(static_cast<unsigned>(blocks < 65536 ? blocks : 65536)), dim3(256), 0, s,
                           static_cast<const float*>(x), static_cast<const float*>(w_gate), T, d, E, k, renormalize,
                           logits_out, topk_idx, topk_w);
    } else {
        const int nt = (E + 15) / 16;
        int rc = EXF_OK;
        switch (nt) {
            case 1: rc = dispatch_gate_bf16<1>(x, w_gate, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, s); break;
            case 2: rc = dispatch_gate_bf16<2>(x, w_gate, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, s); break;
            case 3: rc = dispatch_gate_bf16<3>(x, w_gate, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, s); break;
            default: rc = dispatch_gate_bf16<4>(x, w_gate, T, d, E, k, renormalize, logits_out, topk_idx, topk_w, s); break;
        }
        if (rc != EXF_OK) return rc;
    }
    return check_launch("moe_gate_topk");
}

extern "C" int moe_topk_from_logits(const float* logits, int64_t T, int E, int k, int renormalize, int32_t* topk_idx,
                                    float* topk_w, void* stream)
{
    using namespace exf;
    if (int rc = validate_topk_args("moe_topk_from_logits", T, E, k)) return rc;
    if (T == 0) return EXF_OK;
    EXF_REQUIRE_PTR(logits);
    EXF_REQUIRE_PTR(topk_idx);
    EXF_REQUIRE_PTR(topk_w);
    const int64_t blocks = (T + 3) / 4;
    hipLaunchKernelGGL(topk_from_logits_kernel, dim3(static_cast<unsigned>(blocks < 65536 ? blocks : 65536)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), logits, T, E, k, renormalize, topk_idx, topk_w);
    return check_launch("moe_topk_from_logits");
}
