// Token vectors of a trace column and the calls of affinity_direct.hip, shared by the trace kernels.
#pragma once

#include "common.hpp"

namespace exf {

template <int VEC>
struct TokVec {
    int v[VEC];
};

// Loads the ids of tokens n .. n+VEC-1 of one trace column.  The load is UNCONDITIONAL: a lane past
// the end of its chunk re-reads the chunk's last vector (the caller masks such lanes through its own
// range test).  Keeping branches away from the loads matters: with a branch around each of them the
// compiler can no longer count the loads in flight and waits for all earlier ones before every new
// one, which leaves a single load in flight per wavefront.
// A column starts at any multiple of four bytes (its length is the number of tokens, any number): the
// 16-byte load of gfx950 needs no more, and it costs one more cache line per wavefront when it straddles.
// (Odd token counts used to take 4-byte loads: 46.5 us for the transfers of a 24 x 999983 trace, 24.9 now.)
// A lane whose vector is cut by the end of the chunk receives the LAST VEC ids; cut_vector() moves them.
// STREAM: the column is read once.
template <int VEC, bool STREAM = true>
__device__ __forceinline__ TokVec<VEC> load_tokens(const int32_t* __restrict__ col, int64_t n, int64_t end)
{
    TokVec<VEC> r;
    const int64_t n_safe = min(n, end - VEC);  // callers guarantee end >= VEC; earlier chunks may be touched
    if constexpr (VEC == 4) {
        typedef int i32x4_v __attribute__((vector_size(4 * sizeof(int)), aligned(4)));
        const i32x4_v* at = reinterpret_cast<const i32x4_v*>(col + n_safe);
        const i32x4_v q = STREAM ? __builtin_nontemporal_load(at) : *at;
        r.v[0] = q[0];
        r.v[1] = q[1];
        r.v[2] = q[2];
        r.v[3] = q[3];
    } else {
        r.v[0] = __builtin_nontemporal_load(col + n_safe);
    }
    return r;
}

// The ids of tokens n, n+1, .. in v[0], v[1], .. again, for a lane with n < end < n + VEC (other lanes
// are not changed; ids past the end are whatever is left, the caller's range test drops them).
template <int VEC>
__device__ __forceinline__ void cut_vector(TokVec<VEC>& t, int64_t n, int64_t end)
{
    if constexpr (VEC == 4) {
        const int64_t by = n - (end - VEC);
        const bool one = by == 1 || by == 3, two = by == 2 || by == 3;
        if (one) {
            t.v[0] = t.v[1];
            t.v[1] = t.v[2];
            t.v[2] = t.v[3];
        }
        if (two) {
            t.v[0] = t.v[2];
            t.v[1] = t.v[3];
        }
    }
}

// Short traces in one launch, see affinity_direct.hip.  Each says whether it takes the trace; launch errors are the caller's to check.
bool statistics_direct(const int32_t* trace, const int32_t* placement, int L, int64_t N, int E, int64_t* counts, int64_t* loads, float* cond_prob,
                       int64_t* n_invalid, int64_t* local_per_pair, hipStream_t stream);
bool multihop_direct(const int32_t* trace, int L, int64_t N, int E, int64_t* counts, float* cond_prob, hipStream_t stream);
bool locality_direct(const int32_t* trace, const int32_t* placement, const int32_t* home, int L, int64_t N, int E, int64_t* local_per_pair,
                     int64_t* away_per_layer, hipStream_t stream);

}  // namespace exf
