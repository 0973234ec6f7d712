// complex128 instantiations of the fused tile pass over whole 128-byte lines
// with lane gates, phase fans and permuted stores
#include "kernels.h"
#include "tile_kernel.cuh"

namespace qsim {
void launch_tile_f64_ext(const TileArgs &a, uint64_t n_tiles, int log_r, int log_nt, hipStream_t st)
{
    launch_tile_t<double, 3>(a, n_tiles, log_r, log_nt, nullptr, st);
}
}  // namespace qsim
