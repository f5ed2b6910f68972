// The second contractions that go with ffn_once.hip.
#include "ffn_tiles.hpp"

namespace exf {

int launch_once_second(bool wide, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N, int E_local,
                       void* out, hipStream_t stream, const RowMap& map)
{
    if (map.sorted_out == nullptr) {
        if (wide) return launch_bf16_as<256, 4, kEpiNone, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
        return launch_bf16_as<128, 4, kEpiNone, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    }
    if (wide) return launch_bf16_as<256, 4, kEpiKeepSorted, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    return launch_bf16_as<128, 4, kEpiKeepSorted, true>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
}

}  // namespace exf
