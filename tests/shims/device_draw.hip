// A kernel that draws through the device-side API, for its register counts.
#include "mtgp_device.h"

extern "C" __global__ void __launch_bounds__(1024)
draw_kernel(const uint32_t *params, uint32_t *states, uint32_t stride, uint32_t draws,
            uint32_t *out, uint32_t lds_words) {
    extern __shared__ uint32_t lds[];
    mtgp_device_stream s;
    uint32_t *row = states + (uint64_t)blockIdx.x * stride;
    mtgp_device_begin(s, params, blockIdx.x, row, lds, lds_words);
    uint32_t *o = out + (uint64_t)blockIdx.x * draws * blockDim.x;
    for (uint32_t i = 0; i < draws; ++i)
        o[i * blockDim.x + threadIdx.x] = mtgp_device_draw_u32(s, blockDim.x);
    mtgp_device_end(s, row);
}
