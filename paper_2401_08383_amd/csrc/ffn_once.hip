// The first contractions in tiles that stream the weights of experts of one row tile (GemmTile's ONCE): an object of their own, as ffn_keep.hip and for
// its reason.
#include "ffn_tiles.hpp"

namespace exf {

int launch_once_first(int epi, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N, int E_local,
                      void* out, hipStream_t stream, const RowMap& map)
{
    if (epi == kEpiGeluErf) return launch_bf16_as<256, 8, kEpiGeluErf, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    return launch_bf16_as<256, 8, kEpiGeluTanh, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
}

}  // namespace exf
