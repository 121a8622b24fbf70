// rr_batch_fused.hip -- one launch over all groups of a batch (gfx950).
#include <hip/hip_runtime.h>

#include "rr_device.hpp"
#include "rr_kernels.hpp"

namespace rr {

template <int U, int G>
__device__ __forceinline__ void fused_tile(const uint8_t* table, const FusedGroup& g, uint32_t b, uint8_t* smem) {
    const uint32_t j = find_job(reinterpret_cast<const uint32_t*>(table + g.prefix_off), g.njobs, b);
    const EntryRange r = reinterpret_cast<const EntryRange*>(table + g.range_off)[j];
    const TileArgs& a = reinterpret_cast<const TileArgs*>(table + g.args_off)[j];
    const TileCtx t = tile_decode(a, batch_block_to_tile(a.flags, r, b));
    read_dispatch<U, G>(a, t, smem, threadIdx.x);
    __syncthreads();
    write_phase<U, G>(a, t, smem, threadIdx.x);
}
template <int W>
__device__ __forceinline__ void fused_run(const uint8_t* table, const FusedGroup& g, uint32_t b) {
    batch_run_block<W>(reinterpret_cast<const RunArgs*>(table + g.args_off),
                       reinterpret_cast<const uint32_t*>(table + g.prefix_off),
                       reinterpret_cast<const EntryRange*>(table + g.range_off), g.njobs, b, threadIdx.x);
}
template <int W>
__device__ __forceinline__ void fused_copy(const uint8_t* table, const FusedGroup& g, uint32_t b) {
    batch_copy_block<W>(reinterpret_cast<const CopyArgs*>(table + g.args_off),
                        reinterpret_cast<const uint32_t*>(table + g.prefix_off),
                        reinterpret_cast<const EntryRange*>(table + g.range_off), g.njobs, b, threadIdx.x);
}

// A small batch is bound by its launches, not its bytes: up to 23 kernel families
// of a few dozen workgroups each, spread over four streams, took 90-100 us for
// 1 MB as for 77 MB.  Here every workgroup of every group is in one grid: it finds
// its group among the directory's starts (kernel arguments, scalar compares), then
// its job and tile as in k_batch_*, and branches uniformly to that body.  The
// bodies are those of the batch kernels, so the launch needs the registers of the
// widest one: 57 VGPRs (the table pointer is __restrict__, so job arguments are
// scalar loads; without it they took vector registers and spilled) and, past the
// scalar registers, 258 scalar values in vector-register lanes; asked for seven waves
// per SIMD it gets eight.  16 jobs / 1 MB: 93 -> 9 us; 256 jobs / 77 MB: 101 -> 40 us.
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(7, 8)))
void k_batch_fused(const FusedArgs f, const uint8_t* __restrict__ table) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const FusedGroup g = f.g[fused_group(f, blockIdx.x)];
    const uint32_t b = blockIdx.x - g.start;
    switch (g.code) {
        case 101: fused_tile<1, 1>(table, g, b, smem); break;
        case 104: fused_tile<1, 4>(table, g, b, smem); break;
        case 108: fused_tile<1, 8>(table, g, b, smem); break;
        case 204: fused_tile<2, 4>(table, g, b, smem); break;
        case 201: fused_tile<2, 1>(table, g, b, smem); break;
        case 401: fused_tile<4, 1>(table, g, b, smem); break;
        case 801: fused_tile<8, 1>(table, g, b, smem); break;
        case 1601: fused_tile<16, 1>(table, g, b, smem); break;
        case FUSED_RUN + 16: fused_run<16>(table, g, b); break;
        case FUSED_RUN + 8: fused_run<8>(table, g, b); break;
        case FUSED_RUN + 4: fused_run<4>(table, g, b); break;
        case FUSED_RUN + 2: fused_run<2>(table, g, b); break;
        case FUSED_RUN + 1: fused_run<1>(table, g, b); break;
        case 16: fused_copy<16>(table, g, b); break;
        case 8: fused_copy<8>(table, g, b); break;
        case 4: fused_copy<4>(table, g, b); break;
        case 2: fused_copy<2>(table, g, b); break;
        default: fused_copy<1>(table, g, b); break;
    }
}


hipError_t launch_batch_fused(const FusedArgs& f, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_fused, dim3(f.total), dim3(NT), f.lds_bytes, st, f, reinterpret_cast<const uint8_t*>(f.table));
    return hipGetLastError();
}

}  // namespace rr
