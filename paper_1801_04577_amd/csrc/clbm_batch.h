// clbm_batch.h -- what the kernels of the batched form share (gfx950).
#pragma once

#include "clbm_device.h"

namespace clbm {

struct BatchInst {
    LatticeConst c;
    unsigned long long buf[2];  // device addresses of the two population buffers
    unsigned long long snap;    // device address of the (u_x, u_y, T) snapshot
    int tiles_x[2];             // tiles in a row: of the list, of kBlock columns
    int tile_off, tile_count;
};

__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Tile k of this workgroup among n active tiles (n when there is none). With at least 8
// workgroups, the workgroups of XCD x (blockIdx % 8 == x) sweep the x-th of eight
// contiguous bands of the list (instance by instance, row by row), so the ring nodes that
// neighbouring tiles of an instance share stay in that XCD's L2.
__device__ __forceinline__ int banded_tile(int k, int n)
{
    const int b = blockIdx.x, G = gridDim.x;
    if (G < 8) {
        const int t = b + k * G;
        return t < n ? t : n;
    }
    const int x = b & 7, i = b >> 3, per = (G - x + 7) >> 3, band = (n + 7) >> 3;
    const int j = i + k * per, t = x * band + j;
    return j < band && t < n ? t : n;
}

}  // namespace clbm
