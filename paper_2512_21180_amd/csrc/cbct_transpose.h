// Volume copies for the forward sweeps: the tiles that sweep x planes
// stage their boxes from a copy of the volume with x and y swapped, so that
// a box row (fixed z, in-plane index y) is contiguous in memory.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>

#include "cbct_storage.h"

namespace cbct {
namespace {

// out[s][x][y] = in[s][y][x] for the n_slices (channel x z) slices of a
// volume: 32 x 32 tiles through LDS, both sides' accesses along rows.
template <class T>
__global__ void __launch_bounds__(256)
transpose_xy(const T *__restrict__ in, T *__restrict__ out, int nx, int ny, int n_slices)
{
    __shared__ T tile[32][33];
    const int tx = (nx + 31) >> 5;
    const int x0 = (blockIdx.x % tx) * 32, y0 = (blockIdx.x / tx) * 32;
    const int lx = threadIdx.x & 31, ly = threadIdx.x >> 5;   // 32 x 8
    const size_t plane = (size_t)nx * ny;
    for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
        const T *src = in + sl * plane;
        T *dst = out + sl * plane;
        __syncthreads();   // the previous slice's readers of the tile are done
#pragma unroll
        for (int j = ly; j < 32; j += 8) {
            const int x = x0 + lx, y = y0 + j;
            if (x < nx && y < ny)
                tile[j][lx] = src[(size_t)y * nx + x];
        }
        __syncthreads();
#pragma unroll
        for (int j = ly; j < 32; j += 8) {
            const int y = y0 + lx, x = x0 + j;
            if (x < nx && y < ny)
                dst[(size_t)x * ny + y] = tile[lx][j];
        }
    }
}

// The two FP32 copies the forward sweeps stage from: the volume as it is
// ([z][y][pitch]) and with x and y swapped ([z][x][pitch]), rows between zero
// pads (sweep_pitch), so that the sweeps load quads of voxels without a test
// of their single voxels, whatever the storage.  A copy that no tile reads (a
// single projection's rays mostly run along one axis) is null and not made.
template <class VS>
__global__ void __launch_bounds__(256)
sweep_copies(const typename VS::T *__restrict__ in, float *__restrict__ wide,
             float *__restrict__ out, int nx, int ny, int n_slices)
{
    __shared__ float tile[32][33];
    const int px = sweep_pitch(nx), py = sweep_pitch(ny);
    // tiles cover the padded rows of both copies
    const int tx = (px + 31) >> 5;
    const int x0 = (blockIdx.x % tx) * 32 - kSweepPad, y0 = (blockIdx.x / tx) * 32 - kSweepPad;
    const int lx = threadIdx.x & 31, ly = threadIdx.x >> 5;   // 32 x 8
    for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
        __syncthreads();   // the previous slice's readers of the tile are done
#pragma unroll
        for (int j = ly; j < 32; j += 8) {
            const int x = x0 + lx, y = y0 + j;
            float v = 0.0f;
            if ((unsigned)x < (unsigned)nx && (unsigned)y < (unsigned)ny)
                v = VS::wide(VS::raw(in, ((size_t)sl * ny + y) * nx + x));
            if (wide && (unsigned)y < (unsigned)ny && x + kSweepPad < px)
                wide[((size_t)sl * ny + y) * px + x + kSweepPad] = v;
            tile[j][lx] = v;
        }
        if (!out)
            continue;
        __syncthreads();
#pragma unroll
        for (int j = ly; j < 32; j += 8) {
            const int y = y0 + lx, x = x0 + j;
            if ((unsigned)x < (unsigned)nx && y + kSweepPad < py)
                out[((size_t)sl * nx + x) * py + y + kSweepPad] = tile[lx][j];
        }
    }
}

// Launch transpose_xy over n_slices slices of nx x ny elements.
template <class T>
inline void launch_transpose_xy(const T *in, T *out, int nx, int ny, int n_slices, hipStream_t s)
{
    const dim3 grid(((nx + 31) / 32) * ((ny + 31) / 32), std::min(n_slices, 65535));
    hipLaunchKernelGGL((transpose_xy<T>), grid, dim3(256), 0, s, in, out, nx, ny, n_slices);
}

// FP32 words of the copies of n_slices slices that a plan's tiles read (axes:
// 1 x planes, the swapped copy; 2 y planes), and the copies made in `buf`.
inline size_t sweep_words(int nx, int ny, size_t n_slices, int axes)
{
    return n_slices * ((axes & 2 ? (size_t)ny * sweep_pitch(nx) : 0) +
                       (axes & 1 ? (size_t)nx * sweep_pitch(ny) : 0));
}

struct SweepVolumes {
    const float *vol, *volt;
};

inline SweepVolumes make_sweep_volumes(const void *vol, cbct_dtype t, float *buf, int nx, int ny,
                                       int n_slices, int axes, hipStream_t s)
{
    if (!axes)
        return {buf, buf};   // no tile meets the volume
    float *wide = axes & 2 ? buf : nullptr;
    float *out = axes & 1 ? buf + sweep_words(nx, ny, n_slices, axes & 2) : nullptr;
    const dim3 grid(((sweep_pitch(nx) + 31) / 32) * ((sweep_pitch(ny) + 31) / 32),
                    std::min(n_slices, 65535));
    if (t == CBCT_F32)
        hipLaunchKernelGGL(sweep_copies<F32>, grid, dim3(256), 0, s, (const F32::T *)vol, wide, out,
                           nx, ny, n_slices);
    else if (t == CBCT_BF16)
        hipLaunchKernelGGL(sweep_copies<BF16>, grid, dim3(256), 0, s, (const BF16::T *)vol, wide,
                           out, nx, ny, n_slices);
    else
        hipLaunchKernelGGL(sweep_copies<F16>, grid, dim3(256), 0, s, (const F16::T *)vol, wide, out,
                           nx, ny, n_slices);
    return {wide, out};
}

}  // namespace
}  // namespace cbct
