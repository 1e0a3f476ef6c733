// clbm_multi.hip -- the kernels of clbm_multi.h: a single lattice and the batched form.
#include <hip/hip_runtime.h>

#include "clbm_batch.h"
#include "clbm_host.h"
#include "clbm_multi.h"

namespace clbm {

// A workgroup owns one tile; workgroups are dealt to the XCDs in contiguous bands of tiles,
// so the ring nodes that neighbouring tiles share stay in that XCD's L2 (512^2 FP32,
// 32 x 16 tiles: 4.1 against 4.5 us per step).
template <typename S, int SRC, int TX, int TY, int NS>
__global__ void __launch_bounds__((MultiTile<TX, TY, NS>::NT))
k_multi(const S* __restrict__ src, S* __restrict__ dst, const LatticeConst c, int tiles_x, int tiles_total,
        int steps, unsigned inv)
{
    __shared__ S lds[MultiTile<TX, TY, NS>::elems];
    const int t = tile_of_block(tiles_total, 1);
    if (t >= tiles_total) return;
    multi_tile<S, SRC, TX, TY, NS>(src, dst, c, lds, (t % tiles_x) * TX, (t / tiles_x) * TY, (int)threadIdx.x,
                                   steps, inv);
}

// Waves per SIMD that k_batch_multi is held to: in FP32 with every combination of source
// terms compiled in, those that the LDS tiles of as many workgroups as fit need, at most six (80
// registers). Left to itself that variant takes 87 to 95, and of the two workgroups of 32 x 16 tiles on a
// CU one stays: 16 lattices of 512^2 with none, viscous heating and a field in turn took 84.5 us per step
// (k_batch_step2: 62.1), now 57.1. The others fit by themselves, and were 7 % slower when held.
template <typename S, int MODE, int TX, int TY, int NS>
constexpr int multi_waves_per_eu()
{
    typedef MultiTile<TX, TY, NS> T;
    constexpr int w = (160 * 1024 / (int)(T::elems * sizeof(S)) * (T::NT / 64) + 3) / 4;
    return MODE != 2 || sizeof(S) == 2 ? 1 : w < 6 ? w : 6;
}

// The same over the active tile list of a batch; MODE and bands as in k_batch_step2.
template <typename S, int MODE, int TX, int TY, int NS>
__global__ void __launch_bounds__((MultiTile<TX, TY, NS>::NT))
__attribute__((amdgpu_waves_per_eu(multi_waves_per_eu<S, MODE, TX, TY, NS>())))
k_batch_multi(const BatchInst* __restrict__ insts, const int2* __restrict__ list, const int* __restrict__ count,
              int parity, int bands, int steps, unsigned inv)
{
    __shared__ S lds[MultiTile<TX, TY, NS>::elems];
    const int n = uniform_int(*count);
    const int tid = (int)threadIdx.x;
    for (int k = 0;; ++k) {
        int t = (int)blockIdx.x + k * (int)gridDim.x;
        if (bands) t = banded_tile(k, n);
        if (t >= n) break;
        const int2 e = list[t];
        const int inst = uniform_int(e.x), id = uniform_int(e.y);
        const BatchInst& I = insts[inst];
        const LatticeConst c = I.c;
        const int tiles_x = uniform_int(I.tiles_x[0]);
        const int X0 = (id % tiles_x) * TX, Y0 = (id / tiles_x) * TY;
        const S* src = reinterpret_cast<const S*>(I.buf[parity]);
        S* dst = reinterpret_cast<S*>(I.buf[parity ^ 1]);
        const int terms = MODE == 0 ? 0 : MODE == 1 ? kSrcVisc : uniform_int(runtime_src(c));
        if (MODE != 0 && terms == kSrcVisc)
            multi_tile<S, kSrcVisc, TX, TY, NS>(src, dst, c, lds, X0, Y0, tid, steps, inv);
        else if (MODE == 2 && terms == kSrcField)
            multi_tile<S, kSrcField, TX, TY, NS>(src, dst, c, lds, X0, Y0, tid, steps, inv);
        else if (MODE == 2 && terms == (kSrcVisc | kSrcField))
            multi_tile<S, kSrcVisc | kSrcField, TX, TY, NS>(src, dst, c, lds, X0, Y0, tid, steps, inv);
        else if (MODE != 1)
            multi_tile<S, 0, TX, TY, NS>(src, dst, c, lds, X0, Y0, tid, steps, inv);
        __syncthreads();  // the next tile overwrites the LDS tiles
    }
}

template <typename S, int TX, int TY, int NS>
static const void* single_of(int src)
{
    switch (src) {
        case kSrcVisc: return reinterpret_cast<const void*>(&k_multi<S, kSrcVisc, TX, TY, NS>);
        case kSrcField: return reinterpret_cast<const void*>(&k_multi<S, kSrcField, TX, TY, NS>);
        case kSrcVisc | kSrcField:
            return reinterpret_cast<const void*>(&k_multi<S, kSrcVisc | kSrcField, TX, TY, NS>);
        default: return reinterpret_cast<const void*>(&k_multi<S, 0, TX, TY, NS>);
    }
}

template <typename S, int TX, int TY, int NS>
static const void* batch_of(int mode)
{
    return mode == 0   ? reinterpret_cast<const void*>(&k_batch_multi<S, 0, TX, TY, NS>)
           : mode == 1 ? reinterpret_cast<const void*>(&k_batch_multi<S, 1, TX, TY, NS>)
                       : reinterpret_cast<const void*>(&k_batch_multi<S, 2, TX, TY, NS>);
}

template <int TX, int TY, int NS>
struct Entry {
    static const void* single(int precision, int src)
    {
        return precision == CLBM_FP16_SHIFTED ? single_of<__half, TX, TY, NS>(src) : single_of<float, TX, TY, NS>(src);
    }
    static const void* batch(int precision, int mode)
    {
        return precision == CLBM_FP16_SHIFTED ? batch_of<__half, TX, TY, NS>(mode) : batch_of<float, TX, TY, NS>(mode);
    }
    static MultiShape shape() { return {TX, TY, NS, MultiTile<TX, TY, NS>::NT, &single, &batch}; }
};

const MultiShape* multi_shapes()
{
    static const MultiShape shapes[kMultiShapes] = {Entry<16, 4, 6>::shape(), Entry<32, 8, 6>::shape(),
                                                    Entry<32, 12, 4>::shape(), Entry<32, 16, 3>::shape()};
    return shapes;
}

}  // namespace clbm
