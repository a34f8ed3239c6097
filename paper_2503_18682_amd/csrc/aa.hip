// Box downsampling for anti-aliasing evaluation: a view rendered at f times
// the resolution (f x f rays per output pixel on an ordered grid, centres at
// offsets (k + 1/2) / f) averaged back to the output grid.  With f = 2 this
// is the 4-ray multisampling baseline of Sec. 6.2; larger f gives
// supersampled references.
#include <algorithm>
#include <cstdint>

#include "internal.h"

namespace rgs {
namespace {

// One thread per output pixel and plane, summing row by row.  Bound by the reads;
// FACTOR (0: any, taken at run time) fixes the loops, so that a thread has
// its loads in flight together, four floats wide where rows allow it, and
// the index is split in 32 bits where it fits: 5120 x 3840 x 3 by 8 took 128 us with one
// float a load and 64-bit divisions and takes 37 us.
template <int FACTOR, class Index>
__global__ __launch_bounds__(256) void k_downsample_box(const float *__restrict__ src, int width, int height,
                                                        int factor, int planes, float *__restrict__ dst)
{
    const Index n = (Index)width * height * planes;
    const int f = FACTOR ? FACTOR : factor;
    const float inv = 1.0f / (float)(f * f);
    const int sw = width * f;
    for (Index i = (Index)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (Index)gridDim.x * blockDim.x) {
        const int x = (int)(i % (Index)width);
        const int64_t t = (int64_t)(i / (Index)width);  // output row of all planes
        const float *s = src + t * f * sw + (int64_t)x * f;
        float acc = 0.0f;
        if constexpr (FACTOR % 4 == 0 && FACTOR > 0) {
            float4 v[FACTOR][FACTOR / 4];
#pragma unroll
            for (int r = 0; r < FACTOR; ++r)
#pragma unroll
                for (int c = 0; c < FACTOR / 4; ++c) v[r][c] = reinterpret_cast<const float4 *>(s + (int64_t)r * sw)[c];
#pragma unroll
            for (int r = 0; r < FACTOR; ++r)
#pragma unroll
                for (int c = 0; c < FACTOR / 4; ++c) acc = (((acc + v[r][c].x) + v[r][c].y) + v[r][c].z) + v[r][c].w;
        } else if constexpr (FACTOR == 2) {
            const float2 a = *reinterpret_cast<const float2 *>(s), b = *reinterpret_cast<const float2 *>(s + sw);
            acc = (((acc + a.x) + a.y) + b.x) + b.y;
        } else {
            for (int r = 0; r < f; ++r)
                for (int c = 0; c < f; ++c) acc += s[(int64_t)r * sw + c];
        }
        dst[i] = acc * inv;
    }
}

template <int FACTOR>
void downsample(const float *src, int width, int height, int factor, int planes, float *dst, int64_t n,
                hipStream_t stream)
{
    const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
    if (n < (int64_t(1) << 31))  // (and the last stride past the end below 2^32)
        k_downsample_box<FACTOR, uint32_t><<<grid, 256, 0, stream>>>(src, width, height, factor, planes, dst);
    else
        k_downsample_box<FACTOR, int64_t><<<grid, 256, 0, stream>>>(src, width, height, factor, planes, dst);
}

}  // namespace

hipError_t launch_downsample_box(const float *src, int width, int height, int factor, int planes, float *dst,
                                 hipStream_t stream)
{
    const int64_t n = (int64_t)width * height * planes;
    if (n == 0) return hipSuccess;
    // rows of the source start at multiples of the factor, so the wide loads
    // are aligned if the image is
    const bool aligned = (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
    if (aligned && factor == 8)
        downsample<8>(src, width, height, factor, planes, dst, n, stream);
    else if (aligned && factor == 4)
        downsample<4>(src, width, height, factor, planes, dst, n, stream);
    else if (aligned && factor == 2)
        downsample<2>(src, width, height, factor, planes, dst, n, stream);
    else
        downsample<0>(src, width, height, factor, planes, dst, n, stream);
    return hipGetLastError();
}

}  // namespace rgs
