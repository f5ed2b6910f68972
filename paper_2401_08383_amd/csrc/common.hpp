// Shared host/device helpers of the gfx950 library: error reporting, bf16 conversion,
// wavefront primitives.  Nothing here is used by the CPU checker.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "exflow_moe.h"

namespace exf {

// ---- host side ---------------------------------------------------------------------------
// Records a formatted message for exf_last_error() on this thread and returns `code`.
int fail(int code, const char* fmt, ...);
// Maps the pending HIP launch error (if any) to EXF_ERR_HIP.
int check_launch(const char* what);

// Lets a kernel use more than 64 KiB of LDS; asks the runtime once per device (`allowed`: a bit per device).
inline int allow_lds(const void* kern, size_t lds, std::atomic<uint64_t>& allowed, const char* what)
{
    if (lds <= 64 * 1024) return EXF_OK;
    int dev = -1;
    const bool known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64;
    if (known && (allowed.load(std::memory_order_relaxed) >> dev & 1u) != 0) return EXF_OK;
    hipError_t err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (err != hipSuccess) return fail(EXF_ERR_HIP, "%s: LDS attribute: %s", what, hipGetErrorString(err));
    if (known) allowed.fetch_or(1ull << dev, std::memory_order_relaxed);
    return EXF_OK;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Refuse a null or misaligned pointer argument of the call `fn`.
#define EXF_CHECK_PTR(fn, p)                                                      \
    do {                                                                          \
        if ((p) == nullptr) return ::exf::fail(EXF_ERR_NULL_PTR, "%s: %s is NULL", fn, #p); \
    } while (0)
#define EXF_CHECK_ALIGNED(fn, p)                                                  \
    do {                                                                          \
        if (!::exf::aligned16(p))                                                 \
            return ::exf::fail(EXF_ERR_MISALIGNED, "%s: %s is not 16-byte aligned", fn, #p); \
    } while (0)
#define EXF_REQUIRE_PTR(p) EXF_CHECK_PTR(__func__, p)
#define EXF_REQUIRE_ALIGNED(p) EXF_CHECK_ALIGNED(__func__, p)

// What the calls of a layer refuse, without launching anything: moe_layer_forward asks all of them before its first launch.
int check_gate(const void* x, const void* w_gate, int64_t T, int d, int E, int k, int dt, const int32_t* topk_idx, const float* topk_w);
int check_dispatch(const void* x, const int32_t* topk_idx, int64_t T, int d, int k, int E, int E_local, int dt, const void* x_sorted,
                   const int32_t* src_of_sorted, const int32_t* sorted_of_src, const int32_t* expert_counts, const int32_t* expert_offsets,
                   const void* workspace, size_t workspace_bytes);
int check_ffn(const void* x_sorted, const int32_t* expert_offsets, const void* w1, const void* w2, int64_t A, int d, int f, int E_local,
              int act, int dt, const void* y_sorted, const void* workspace, size_t workspace_bytes);
int check_ffn_fused(const void* x, const int32_t* src_of_sorted, const int32_t* sorted_of_src, const float* topk_w,
                    const int32_t* expert_offsets, const void* w1, const void* w2, int64_t T, int k, int d, int f, int E_local, int act,
                    int dt, const void* out, const void* workspace, size_t workspace_bytes);
int check_combine(const void* y_sorted, const int32_t* sorted_of_src, const float* topk_w, int64_t T, int d, int k, int dt, const void* out);

constexpr int kWave = 64;  // CDNA wavefront width

// ---- device side -------------------------------------------------------------------------
typedef uint16_t bf16_t;  // storage only; arithmetic is fp32
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// Round-to-nearest-even; inputs are finite by contract (NaN is quieted).
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<bf16_t>((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<bf16_t>(u >> 16);
}

// Two floats -> two bf16 in one register (gfx950 has a packed round-to-nearest-even convert).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_v;
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_v;
    const f32x2_v f = {lo, hi};
    const bf16x2_v b = __builtin_convertvector(f, bf16x2_v);
    uint32_t u;
    __builtin_memcpy(&u, &b, sizeof(u));
    return u;
}

// 16-byte streaming accesses: data that is touched once should not displace reusable lines.
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_v;
__device__ __forceinline__ uint4 load_stream16(const uint4* p)
{
    const u32x4_v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_v*>(p));
    return uint4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void store_stream16(uint4* p, uint4 x)
{
    const u32x4_v v = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_v*>(p));
}
// Written through to memory by the L2 (a wide store's data registers may be overwritten two wait states after it at the earliest).
__device__ __forceinline__ void store_through16(uint4* p, uint4 x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const u32x4_v v = {x.x, x.y, x.z, x.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
#else
    (void)p;
    (void)x;
#endif
}

// Launch width of the pure streaming kernels: a grid-stride loop over about two workgroups per
// CU sustained the highest HBM rate when measured (many more workgroups were slower).
constexpr int kStreamWorkgroups = 512;

// Row batches of the gather / combine streams (see combine.hip): rows per wavefront batch, chosen
// so that about 2048 wavefronts have work (a short batch keeps a small problem parallel, a long
// one amortises the index fetch), and the row a flat chunk index falls in: c / vec_per_row
// through a float reciprocal with one correction step (c < 2^24).
inline int row_batch_for(int64_t rows)
{
    int b = 16;
    while (b > 1 && rows / b < 2048) b >>= 1;
    return b;
}
__device__ __forceinline__ int row_of_chunk(int c, int vec_per_row, float rcp)
{
    int q = static_cast<int>(static_cast<float>(c) * rcp);
    const int r = c - q * vec_per_row;
    if (r < 0) q -= 1;
    else if (r >= vec_per_row) q += 1;
    return q;
}

__device__ __forceinline__ int lane_id() { return static_cast<int>(threadIdx.x) & (kWave - 1); }

// A workgroup barrier behind which everybody's LDS accesses are done; loads from memory stay in flight across it.
__device__ __forceinline__ void barrier_for_lds()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#endif
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// The values of the two lanes that differ in bit OFF of their number, the same two in both of them (or the same pair of values: OFF 8,
// 4, 2, 1 expect that the lanes whose numbers differ in the higher bits below 16 already agree, as they do on the way
// through a butterfly).  Rows of 16 lanes trade places, lanes of a row rotate: no trip through the LDS pipeline.
template <int OFF>
__device__ __forceinline__ void butterfly(uint32_t v, uint32_t& a, uint32_t& b)
{
    if constexpr (OFF == 32) {
        const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = s[0], b = s[1];
    } else if constexpr (OFF == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = s[0], b = s[1];
    } else {
        a = v;
        b = __builtin_amdgcn_update_dpp(0, v, 0x120 + OFF, 0xf, 0xf, true);  // row_ror
    }
}
template <int OFF>
__device__ __forceinline__ void butterfly(float v, float& a, float& b)
{
    uint32_t x, y;
    butterfly<OFF>(__float_as_uint(v), x, y);
    a = __uint_as_float(x), b = __uint_as_float(y);
}
template <int OFF>
__device__ __forceinline__ float butterfly_add(float v)
{
    float a, b;
    butterfly<OFF>(v, a, b);
    return a + b;
}
// wave_sum of floats, added in the same order: the same bits.
__device__ __forceinline__ float wave_sum(float v)
{
    return butterfly_add<1>(butterfly_add<2>(butterfly_add<4>(butterfly_add<8>(butterfly_add<16>(butterfly_add<32>(v))))));
}

// Inclusive prefix sum across the 64 lanes of a wavefront, on the cross-lane data path of the vector
// ALU (a shuffle goes through the LDS pipeline and costs a round trip of its own per step; a tile
// lookup runs several scans in a row before a workgroup can request its first operand).  Steps 1-4 add
// the lanes 1, 2, 4 and 8 to the right inside every row of 16 lanes (zero shifted in at a row's
// start), step 5 adds lane 15 of rows 0 and 2 to rows 1 and 3, step 6 lane 31 to rows 2 and 3.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Asks for all 64-byte lines of a kernel's arguments (BYTES of them) at once.  They lie in host memory, and the first access to a
// line takes half a microsecond: left to the compiler, which loads an argument where it is used first, a kernel of a few
// microseconds pays that once per line.
template <int BYTES>
__device__ __forceinline__ void touch_arguments()
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto* a = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (BYTES + 63) / 64;
    uint32_t v[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) v[i] = a[i * 16];
#pragma unroll
    for (int i = 0; i < LINES; ++i) asm volatile("" ::"s"(v[i]));
#endif
}

// Value of `v` in lane `src`, where src is the same in every lane (read on the scalar path).
__device__ __forceinline__ int wave_read_lane(int v, int src)
{
    return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}

// Lanes of the wavefront that hold the same local expert as this lane (meaningful where e >= 0): the
// ids are compared bit by bit, log2(E_local) ballots instead of one ballot per expert.
__device__ __forceinline__ unsigned long long same_expert_lanes(int e, int E_local)
{
    unsigned long long m = __ballot(e >= 0);
    for (int bit = 1; bit < E_local; bit <<= 1) {
        const unsigned long long b = __ballot((e & bit) != 0);
        m &= (e & bit) != 0 ? b : ~b;
    }
    return m;
}

// ---------------------------------------------------------------------------- direct-to-LDS loads
// A pointer that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// One wavefront-wide direct-to-LDS load: lane i fetches 16 bytes at base + voff and they land at
// LDS byte address lds_addr + 16*i (M0 carries the wavefront-uniform LDS address).  Issued as
// inline assembly on purpose: the compiler then keeps exact lgkmcnt waits for the ds_read
// operand fetches, and the landing of these loads is awaited explicitly with wait_vmcnt.
__device__ __forceinline__ void lds_dma_16B(const unsigned char* base, uint32_t voff, uint32_t lds_addr)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory");
#else
    (void)base; (void)voff; (void)lds_addr;
#endif
}

// The same for data that is read once: streamed past the caches.
__device__ __forceinline__ void lds_dma_16B_stream(const unsigned char* base, uint32_t voff, uint32_t lds_addr)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory");
#else
    (void)base; (void)voff; (void)lds_addr;
#endif
}

// One wavefront-wide direct-to-LDS load of 4 bytes per lane: lane i fetches base + voff and the word
// lands at LDS byte address lds_addr + 4*i.
__device__ __forceinline__ void lds_dma_4B(const unsigned char* base, uint32_t voff, uint32_t lds_addr)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1\n" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory");
#else
    (void)base; (void)voff; (void)lds_addr;
#endif
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}


}  // namespace exf
