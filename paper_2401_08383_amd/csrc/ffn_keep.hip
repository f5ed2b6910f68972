// The second contractions in tiles that leave their sorted rows besides the output (RowMap::sorted_out), for the separate calls of a top-1 layer.  An
// object of their own: in one with the others they made its code half as large again (1.3 MB, 1.9 with them), and the launches of layers that do not
// use them took longer by as much as it takes to reach code further off, with the same instructions.  In one object, in two and before there were any, us:
// 1931 tokens top-2, 6 experts of 1024 x 4096 94.4, 93.5, 94.3; 6000 top-2, 8 of 512 x 2048 81.3, 80.8, 80.8; 656, 12 of 960 x 1984 34.3, 33.8, 33.9;
// 3000, 8 of 768 x 3072 53.8, 53.6, 54.0.  The layers that do use them pay some of it back (4000 tokens, separate calls, 8 of 1024 x 4096 90.7, 91.7; five
// launches 96.8).
#include "ffn_tiles.hpp"

namespace exf {

int launch_kept_contraction(bool wide, const void* act, const int32_t* offsets, const void* weight, const void* bias, int64_t A, int K, int N,
                            int E_local, void* out, hipStream_t stream, const RowMap& map)
{
    if (wide) return launch_bf16_as<256, 4, kEpiKeepSorted>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
    return launch_bf16_as<128, 4, kEpiKeepSorted>(act, offsets, weight, bias, A, K, N, E_local, out, stream, map);
}

}  // namespace exf
