// One transfer from memory straight into LDS behind values that vector instructions wrote, for a look at the emitted code.
#include "flurka_fast.h"
#include "flurka_gemm_tile.h"

__global__ void one_transfer(const void* base, unsigned bytes, const int* offsets, float* out) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[2048];
    const flurka::u32x4 r = flurka::tile_rsrc(base, bytes);
    flurka::lds_dma16<1024>(r, (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)lds, 16 * threadIdx.x,
                            offsets[threadIdx.x], 0);
    flurka::wait_and_barrier<0>();
    out[threadIdx.x] = ((const float*)(lds + 1024))[threadIdx.x];
}
