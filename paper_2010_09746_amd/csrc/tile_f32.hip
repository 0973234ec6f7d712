// complex64 instantiations of the fused tile pass over whole 128-byte lines
// (non-temporal access); passes with lane gates, phase fans or a permuted
// store go to launch_tile_f32_ext, passes over partial lines to launch_tile_f32_plain
#include "kernels.h"
#include "tile_kernel.cuh"

namespace qsim {
void launch_tile_f32(const TileArgs &a, uint64_t n_tiles, int log_r, int log_nt, hipStream_t st)
{
    if (!(a.io & 8u))
        launch_tile_f32_plain(a, n_tiles, log_r, log_nt, st);
    else if (a.io & IO_EXT)
        launch_tile_f32_ext(a, n_tiles, log_r, log_nt, st);
    else
        launch_tile_t<float, 1>(a, n_tiles, log_r, log_nt, nullptr, st);
}
}  // namespace qsim
