// The float kernels of gemm_tile.hpp.
#include "gemm_tile.hpp"

namespace blstm {
namespace {

// 128x128 tiles, two workgroups per CU, or 64x64, up to five; two buffers (a third took 121 us where two take 116: 1344 x 4096,
// K = 1024, 64x64).
template <bool AT, bool BT, bool RS, int MODE>
hipError_t launch_direct_f32_rs(const Params& P, int tile, dim3 grid, hipStream_t stream) {
    if (tile == GEMM_TILE_64) return launch_kernel<float, float, AT, BT, 1, 1, 2, MODE, RS, 2>(P, grid, stream);
    return launch_kernel<float, float, AT, BT, 2, 2, 2, MODE, RS, 2>(P, grid, stream);
}
template <int MODE>
hipError_t launch_direct_f32(const GemmDesc& d, const Params& P, int tile, dim3 grid, hipStream_t stream) {
    if (d.atrans && d.btrans) return P.rowsum ? launch_direct_f32_rs<true, true, true, MODE>(P, tile, grid, stream) : launch_direct_f32_rs<true, true, false, MODE>(P, tile, grid, stream);
    if (P.rowsum) return hipErrorInvalidValue;
    if (!d.atrans && d.btrans) return launch_direct_f32_rs<false, true, false, MODE>(P, tile, grid, stream);
    if (!d.atrans && !d.btrans) return launch_direct_f32_rs<false, false, false, MODE>(P, tile, grid, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_f32(const GemmDesc& d, const Params& P, int mode, bool direct, int tile, dim3 grid, hipStream_t stream) {
    if (!direct) return launch_staged<float, float>(d, P, mode, grid, stream);
    return mode == WHOLE ? launch_direct_f32<WHOLE>(d, P, tile, grid, stream) : launch_direct_f32<EDGE>(d, P, tile, grid, stream);
}
hipError_t launch_group_f32_tiles(const GroupParams& G, int total, int mode, int tile, hipStream_t stream) {
    if (tile == GEMM_TILE_64) return mode == WHOLE ? launch_group_kernel<float, 1, 1, WHOLE, 2>(G, total, stream) : launch_group_kernel<float, 1, 1, EDGE, 2>(G, total, stream);
    return mode == WHOLE ? launch_group_kernel<float, 2, 2, WHOLE, 2>(G, total, stream) : launch_group_kernel<float, 2, 2, EDGE, 2>(G, total, stream);
}

}  // namespace blstm
