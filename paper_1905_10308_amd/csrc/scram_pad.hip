// Copies between rows of the channel counts the kernels take and shorter rows.

#include "scram_device.h"

namespace scram {
namespace {

constexpr int kMaxPad = 4;

struct PadParams {
    PadTensor t[kMaxPad];
    int log_width;
};

// One block row (blockIdx.y) per tensor; a thread takes 4 consecutive elements
// of a wide row at a time, so that side is read or written in whole vectors.
// A small image is one short launch: 93 x 125 pixels of 3 channels, three
// tensors, 3.7 us where a fill and a strided copy per tensor took six launches.
template <typename E, bool UNPAD>
__global__ __launch_bounds__(kBlock) void pad_kernel(PadParams p)
{
    typedef E vec4 __attribute__((ext_vector_type(4)));
    const PadTensor t = p.t[blockIdx.y];
    const int lw = p.log_width;
    const int64_t quads = (t.rows << lw) >> 2;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < quads;
         i += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int64_t row = i >> (lw - 2);
        const int c = static_cast<int>(i << 2) & ((1 << lw) - 1);
        const int64_t at = row * t.width + c;  // in the short rows
        if constexpr (UNPAD) {
            const vec4 v = static_cast<const vec4*>(t.src)[i];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c + j < t.width) static_cast<E*>(t.dst)[at + j] = v[j];
        } else {
            vec4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = c + j < t.width ? static_cast<const E*>(t.src)[at + j] : E(0);
            static_cast<vec4*>(t.dst)[i] = v;
        }
    }
}

}  // namespace

hipError_t launch_pad(const PadTensor* t, int count, int width, int elem_bytes, bool unpad, hipStream_t stream)
{
    PadParams p{};
    int64_t most = 0;
    for (int i = 0; i < count; ++i) {
        p.t[i] = t[i];
        most = t[i].rows > most ? t[i].rows : most;
    }
    while ((1 << p.log_width) < width) ++p.log_width;
    const int64_t want = (most * width / 4 + kBlock - 1) / kBlock;
    const dim3 grid(static_cast<uint32_t>(want < 4096 ? want : 4096), count);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, stream, p);
        return hipGetLastError();
    };
    if (elem_bytes == 2) return unpad ? go(pad_kernel<uint16_t, true>) : go(pad_kernel<uint16_t, false>);
    return unpad ? go(pad_kernel<uint32_t, true>) : go(pad_kernel<uint32_t, false>);
}

}  // namespace scram
