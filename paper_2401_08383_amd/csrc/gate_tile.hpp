// The gate's routing arithmetic and the gate of one token tile, shared by moe_gate_topk and by the expert layer of a handful of
// tokens (ffn_stream.hip).
#pragma once

#include <math.h>

#include "common.hpp"

namespace exf {

struct Route {
    int i0, i1;
    float w0, w1;
};

// Softmax weights of the selected experts from the two best logits and sum exp(l - l0).
__device__ __forceinline__ void route_weights(Route& r, float l0, float l1, float sum_exp, int k, int renormalize)
{
    if (k == 1) {
        r.w0 = 1.0f / sum_exp;
        r.w1 = 0.0f;
    } else {
        const float t = expf(l1 - l0);
        if (renormalize) {
            const float z = 1.0f + t;
            r.w0 = 1.0f / z;
            r.w1 = t / z;
        } else {
            r.w0 = 1.0f / sum_exp;
            r.w1 = t / sum_exp;
        }
    }
}

__device__ __forceinline__ void store_route(const Route& r, int64_t t, int k, int32_t* __restrict__ topk_idx,
                                            float* __restrict__ topk_w)
{
    topk_idx[t * k] = r.i0;
    topk_w[t * k] = r.w0;
    if (k > 1) {
        topk_idx[t * k + 1] = r.i1;
        topk_w[t * k + 1] = r.w1;
    }
}

constexpr int kNoExpert = 2 * kWave;
// A lane looks at its experts in ascending order: a tie keeps the earlier one, and anything beats kNoExpert.
__device__ __forceinline__ void pick_later(float& v, int& i, float ov, int oi, bool live)
{
    const bool better = live & ((ov > v) | ((ov == v) & (i == kNoExpert)));
    v = better ? ov : v;
    i = better ? oi : i;
}

template <int OFF>
__device__ __forceinline__ void best_of_pair(float& v, int& i)
{
    float v0, v1;
    uint32_t i0, i1;
    butterfly<OFF>(v, v0, v1);
    butterfly<OFF>(static_cast<uint32_t>(i), i0, i1);
    const bool second = v1 > v0 || (v1 == v0 && static_cast<int>(i1) < static_cast<int>(i0));
    v = second ? v1 : v0;
    i = static_cast<int>(second ? i1 : i0);
}
__device__ __forceinline__ void best_of_quads(float& v, int& i)
{
    best_of_pair<16>(v, i);
    best_of_pair<32>(v, i);
}

// Routing from the accumulator layout: lane (r16, g) holds the logits of token `tok` (its r16-th of the tile) for the experts
// nt*16 + 4g + v (ascending in (nt, v)), so the four lanes of a token need two shuffle steps.
template <int NT>
__device__ __forceinline__ Route route_of_quads(const f32x4_t (&acc)[NT], int E, int k, int renormalize)
{
    const int g = lane_id() >> 4;
    float l0 = -INFINITY;
    int i0 = kNoExpert;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int e = nt * 16 + 4 * g + v;
            pick_later(l0, i0, acc[nt][v], e, e < E);
        }
    best_of_quads(l0, i0);
    float l1 = -INFINITY;
    int i1 = kNoExpert;
    if (k > 1) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int e = nt * 16 + 4 * g + v;
                pick_later(l1, i1, acc[nt][v], e, e < E && e != i0);
            }
        best_of_quads(l1, i1);
    }
    float se = 0.0f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            se += nt * 16 + 4 * g + v < E ? expf(acc[nt][v] - l0) : 0.0f;
    se = butterfly_add<32>(butterfly_add<16>(se));
    Route r;
    r.i0 = i0;
    r.i1 = i1;
    route_weights(r, l0, l1, se, k, renormalize);
    return r;
}

template <int NT>
__device__ __forceinline__ void route_quads(const f32x4_t (&acc)[NT], int64_t tok, int64_t T, int E, int k, int renormalize,
                                            float* __restrict__ logits_out, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w)
{
    const int g = lane_id() >> 4;
    const Route r = route_of_quads<NT>(acc, E, k, renormalize);
    if (tok >= T) return;
    if (logits_out != nullptr) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int e = nt * 16 + 4 * g + v;
                if (e < E) logits_out[tok * E + e] = acc[nt][v];
            }
    }
    if (g == 0) store_route(r, tok, k, topk_idx, topk_w);
}

// Sums the reduction of d is dealt to (see gate_stream_kernel): a long one to eight while their rings fit.
__host__ __device__ constexpr int gate_sums(int NT, int d) { return d >= 2048 && NT <= 2 ? 8 : 4; }

// The gate of up to 16 tokens by a workgroup of W wavefronts that goes on to other work: x [T,d], wg [E,d], d % 64 == 0.  Every
// wavefront returns all routes, token lane%16 in lane.  P sums over the units of the reduction, added in order, as
// gate_stream_kernel<NT,1,P> adds them: the same bits.  `smem`: LDS bytes, free again on return.
constexpr int kGateFewTokens = 16;
template <int NT, int P, int W, int LDS>
__device__ __forceinline__ Route gate_few(const void* x, const void* wg, int T, int d, int E, int k, int renormalize, unsigned char* smem)
{
    constexpr int SLOT = (NT + 1) * 2048, LPU = 2 * (NT + 1);
    constexpr int FIT = LDS / ((P < W ? P : W) * SLOT), R = FIT > 4 ? 4 : FIT;  // (a wavefront without a sum has no ring)
    constexpr int OWN = P > W ? P / W : 1;  // sums of a wavefront
    constexpr int STEP = NT == 1 ? R : 2;    // units read at once: the launch waits for the LDS, unit by unit
    static_assert(R >= 2 && STEP <= R && (R - 1) * LPU < 64 && OWN * W >= P, "waits below; every sum has a wavefront");
    static_assert(OWN * NT * kWave * 16 <= R * SLOT, "the sums must fit the ring");
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r8 = lane >> 3, c8 = lane & 7;
    unsigned char* ring = smem + wave * (R * SLOT);
    const uint32_t ring_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem)) + wave * (R * SLOT);
    const uint32_t row_bytes = static_cast<uint32_t>(d) * 2u;
    const unsigned char* w_base = uniform_ptr(static_cast<const unsigned char*>(wg));
    const unsigned char* x_base = uniform_ptr(static_cast<const unsigned char*>(x));
    // LDS row r of a slot holds 16-byte piece c at position c ^ ((r / 2) % 8); rows past the last expert or token repeat it
    uint32_t off[LPU];
#pragma unroll
    for (int i = 0; i < LPU; ++i) {
        const int r = i * 8 + r8;
        const int row = i < 2 * NT ? min(r, E - 1) : min(r - 16 * NT, T - 1);
        off[i] = static_cast<uint32_t>(row) * row_bytes + ((c8 ^ ((r >> 1) & 7)) * 16);
    }
    const int units = d / 64;
    int cnt[OWN], total = 0;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
        const int sum = wave + o * W;
        cnt[o] = sum < P && sum < units ? (units - sum + P - 1) / P : 0;
        total += cnt[o];
    }
    auto issue = [&](int q) {  // the q-th unit of this wavefront: its sums one after the other
        const int unit = q < cnt[0] ? wave + q * P : wave + W + (q - cnt[0]) * P;
        const uint32_t slot = ring_addr + (q % R) * SLOT;
#pragma unroll
        for (int i = 0; i < LPU; ++i) lds_dma_16B((i < 2 * NT ? w_base : x_base) + static_cast<size_t>(unit) * 128, off[i], slot + i * 1024);
    };
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (q < total) issue(q);
    const int r16 = lane & 15, g = lane >> 4;
    int frag[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) frag[h] = r16 * 128 + (((4 * h + g) ^ (r16 >> 1)) * 16);
    f32x4_t acc[OWN][NT];
    int q = 0;
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[o][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int u = 0; u < cnt[o]; u += STEP) {
            const int n = min(STEP, cnt[o] - u), younger = min(R - n, total - n - q);  // units asked for behind these
            if (R >= 4 && younger >= 3) wait_vmcnt<(R >= 4 ? 3 : 0) * LPU>();
            else if (R >= 3 && younger >= 2) wait_vmcnt<(R >= 3 ? 2 : 0) * LPU>();
            else if (younger >= 1) wait_vmcnt<LPU>();
            else wait_vmcnt<0>();
            bf16x8_t a[STEP][NT][2], b[STEP][2];
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                if (i > 0 && i >= n) break;
                const unsigned char* s = ring + ((q + i) % R) * SLOT;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) a[i][nt][h] = *reinterpret_cast<const bf16x8_t*>(s + nt * 2048 + frag[h]);
                    b[i][h] = *reinterpret_cast<const bf16x8_t*>(s + NT * 2048 + frag[h]);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slots have been read: they may be filled again
#pragma unroll
            for (int i = 0; i < STEP; ++i)
                if (i < n && q + i + R < total) issue(q + i + R);
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                if (i > 0 && i >= n) break;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[o][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][nt][h], b[i][h], acc[o][nt], 0, 0, 0);
            }
            q += n;
        }
    }
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (wave + o * W < P) reinterpret_cast<f32x4_t*>(ring)[(o * NT + nt) * kWave + lane] = acc[o][nt];
    __syncthreads();
    f32x4_t sum[NT];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const f32x4_t v = reinterpret_cast<const f32x4_t*>(smem + p % W * (R * SLOT))[(p / W * NT + nt) * kWave + lane];
            sum[nt] = p == 0 ? v : sum[nt] + v;
        }
    const Route r = route_of_quads<NT>(sum, E, k, renormalize);
    __syncthreads();
    return r;
}

}  // namespace exf
