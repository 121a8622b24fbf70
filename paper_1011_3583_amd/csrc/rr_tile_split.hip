// rr_tile_split.hip -- tiles of short records split into planes (gfx950).
#include <hip/hip_runtime.h>

#include "rr_device.hpp"
#include "rr_kernels.hpp"

namespace rr {

// Crops of interleaved records to planes, and permutes of that form, whose tiles share
// 128-byte lines (tiles that do not, and de-interlaces to separate planes, stream their
// output and take k_tile).  Bound by LDS instructions before: every output byte was a
// read of its own.  Here an output vector is one 16-byte read and its share of a
// register split.  A kernel per record length, so the split is compile-time byte
// permutes.
// MI355X, RGB crops to planes, through write_ragged -> here: 224x224 of 256 u8
// images of 256x256 (77 MB, 12 us at the copy rate; short of that by the launch and
// one read-then-write round per workgroup) 26.2 -> 18.2 us; 30 MB 19.1 -> 14.9; 3.4 MB 11.0 -> 6.5; 727 MB of floats 143 -> 136
// (bound by memory); RGBA u8 6.7 MB 10.4 -> 6.5.
template <int U, int N>
__global__ __launch_bounds__(NT) void k_tile_split(const TileArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const TileCtx t = tile_decode(a, block_to_tile(a, blockIdx.x));
    read_segs<U, true>(a, t, smem, threadIdx.x);
    __syncthreads();
    write_split<U, N, false>(a, t, smem, threadIdx.x);
}

template <int U>
static hipError_t launch_u(const TileArgs& a, uint32_t grid, hipStream_t st) {
    const dim3 g(grid), b(NT);
    const uint32_t lds = a.lds_bytes;
    switch (a.TA) {
        case 2: hipLaunchKernelGGL((k_tile_split<U, 2>), g, b, lds, st, a); break;
        case 3: hipLaunchKernelGGL((k_tile_split<U, 3>), g, b, lds, st, a); break;
        case 4: hipLaunchKernelGGL((k_tile_split<U, 4>), g, b, lds, st, a); break;
        case 5: hipLaunchKernelGGL((k_tile_split<U, 5>), g, b, lds, st, a); break;
        case 6: hipLaunchKernelGGL((k_tile_split<U, 6>), g, b, lds, st, a); break;
        case 7: hipLaunchKernelGGL((k_tile_split<U, 7>), g, b, lds, st, a); break;
        case 8: hipLaunchKernelGGL((k_tile_split<U, 8>), g, b, lds, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_tile_split(const TileArgs& a, uint32_t grid, hipStream_t st) {
    switch (a.unit) {
        case 1: return launch_u<1>(a, grid, st);
        case 2: return launch_u<2>(a, grid, st);
        case 4: return launch_u<4>(a, grid, st);
        case 8: return launch_u<8>(a, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rr
