// As ffn_routed.hip, with weights that one row tile reads streamed (ffn_once.hip).
#include "ffn_tiles.hpp"

namespace exf {

int launch_routed_once_first(int epi, const void* act, const void* weight, int64_t A, int K, int N, int E_local, void* out, hipStream_t stream, const TileRouting& route)
{
    if (epi == kEpiGeluErf) return launch_routed_as<kEpiGeluErf, true>(act, weight, A, K, N, E_local, out, stream, route);
    return launch_routed_as<kEpiGeluTanh, true>(act, weight, A, K, N, E_local, out, stream, route);
}

}  // namespace exf
