// The first contractions in tiles that sort the assignments themselves: an object of their own, as ffn_keep.hip and for its reason.
#include "ffn_tiles.hpp"

namespace exf {

int launch_routed_first(int epi, const void* act, const void* weight, int64_t A, int K, int N, int E_local, void* out, hipStream_t stream, const TileRouting& route)
{
    if (epi == kEpiGeluErf) return launch_routed_as<kEpiGeluErf>(act, weight, A, K, N, E_local, out, stream, route);
    return launch_routed_as<kEpiGeluTanh>(act, weight, A, K, N, E_local, out, stream, route);
}

}  // namespace exf
