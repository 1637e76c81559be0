// Conversions between the row-major MXFP4 operand layout of the ABI and the tiled layout the
// fast GEMM reads (see duqpp_internal.h).  Pure byte permutations.
#include "duqpp_internal.h"
#include "layout_device.h"

namespace duqpp {

constexpr int kTileWaves = 4;

// Row-major -> tiled, a wave per unit; the units of a second operand (none if it has no rows) follow the first's.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void tile_kernel(LayoutParams a, LayoutParams b) {
    const int lane = threadIdx.x & 63;
    const int64_t unit = (int64_t)blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t of_a = tile_units(a);
    if (unit < of_a) tile_unit(a, unit, lane);
    else if (unit < of_a + tile_units(b)) tile_unit(b, unit - of_a, lane);
}

__global__ __launch_bounds__(256) void untile_kernel(LayoutParams p) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;   // over (row, group)
    const int64_t total = (int64_t)p.rows * p.G;
    if (idx >= total) return;
    const int j = (int)(idx % p.G);
    const int row = (int)(idx / p.G);
    const int rt = row / 32, r = row % 32;
    *(uint4*)(p.dst_codes + idx * 16) = *(const uint4*)(p.src_codes + (((int64_t)rt * p.GP + j) * 32 + r) * 16);
    p.dst_scales[idx] = p.src_scales[((((int64_t)rt * (p.GP / 8) + j / 8) * 2 + (j % 8) / 4) * 32 + r) * 4 + (j % 4)];
}

hipError_t launch_tile(const LayoutParams& a, const LayoutParams& b, hipStream_t stream) {
    const int64_t units = tile_units(a) + tile_units(b);
    if (units <= kTileWaves * kNumCU) return launch(tile_kernel<1>, dim3((unsigned)units), dim3(64), 0, stream, a, b);
    return launch(tile_kernel<kTileWaves>, dim3((unsigned)((units + kTileWaves - 1) / kTileWaves)), dim3(64 * kTileWaves), 0, stream, a, b);
}
hipError_t launch_tile(const LayoutParams& p, hipStream_t stream) {
    LayoutParams none = p;
    none.rows = 0;
    return launch_tile(p, none, stream);
}

hipError_t launch_untile(const LayoutParams& p, hipStream_t stream) {
    const int64_t total = (int64_t)p.rows * p.G;
    return launch(untile_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, p);
}

}  // namespace duqpp
