// clbm_multi.h -- several time steps per launch on small tiles (gfx950).
//
// A lattice of up to a few million nodes leaves most of the GPU idle or waiting: a launch
// of the two-step kernel takes 7.5 us on 64 x 32 nodes and 9 us on 256 x 256, nearly all
// of it the chain launch - load - collide (up to five nodes in sequence per wave) - store.
// Here a workgroup owns a smaller tile, gives every node of it and of its ring a thread of
// its own, and takes up to NS steps before it stores, so the chain of one launch is paid
// once for all of them. The price is the ring, which is collided again by each tile that
// touches it: the more tiles there are per CU, the fewer steps pay (multi_shape).
#pragma once

#include "../../include/clbm.h"
#include "clbm_kernels.h"

namespace clbm {

// Phase with ring r (r = steps - 1 first, 0 last) advances the tile and r nodes around it
// by one step: the first pulls from the stored buffer, the later ones from the LDS tile
// the phase before has written (they alternate between two), the last one stores. Each
// phase runs the per-node code of k_step on values rounded as stored, so a launch equals
// that many launches of k_step bit for bit.
template <int TX, int TY, int NS>
struct MultiTile {
    static constexpr int R = NS - 1;                          // ring of the first of NS phases
    static constexpr int XE = TX + 2 * R, YE = TY + 2 * R;    // LDS tile with the ring
    static constexpr unsigned P = XE * YE;                    // LDS population stride
    static_assert(NS > 1, "one step per launch is k_step");
    static constexpr unsigned elems = 2 * 14 * P;             // two tiles: ring r writes tile r % 2
    static constexpr int NT = (XE * YE + 63) / 64 * 64;       // a thread per node of the first phase
};

// Lattice coordinate of g in a periodic direction of n nodes, which may be fewer than the
// ring is wide.
__device__ __forceinline__ int wrap_ring(int g, int n)
{
    if (g >= 0 && g < n) return g;
    g %= n;
    return g < 0 ? g + n : g;
}

// Pull gather of node (x, y), at element o of an LDS tile [14][YE][XE] that holds the node's
// neighbours: the populations of gather_mem. The loads take no wall into account (what
// they fetch across a wall is never used); the wave's wall nodes are completed afterwards,
// so a wave without one pays nothing for them. Coordinates do not wrap in a periodic
// direction (the ring holds the wrapped nodes).
template <int SRC, typename S, typename T>
__device__ __forceinline__ void gather_tile(const S* from, const LatticeConst& c, unsigned o, int x, int y,
                                            float a[9], float b[5])
{
    constexpr unsigned P = T::P;
#pragma unroll
    for (int i = 0; i < 9; ++i) a[i] = ld(from + (o - ey(i) * T::XE - ex(i)) + i * P);
#pragma unroll
    for (int i = 0; i < 5; ++i) b[i] = ld(from + (o - ey(i) * T::XE - ex(i)) + (9 + i) * P);
    const bool oxm = !c.periodic_x && x == 0, oxp = !c.periodic_x && x == c.nx - 1;
    const bool oym = !c.periodic_y && y == 0, oyp = !c.periodic_y && y == c.ny - 1;
    if (!(oxm | oxp | oym | oyp)) return;
    auto own = [&](int i) { return ld(from + o + i * P); };
    auto theta = [&](unsigned off, int qx, int qy) {
        return theta_at<SRC, S, P>(from, c, off, node_q<SRC>(c, wrap_ring(qx, c.nx), wrap_ring(qy, c.ny)));
    };
    const float th1 = theta(o, x, y);
    if (oxm | oxp) {
        const int d = oxm ? 1 : -1, s = oxm ? 0 : 1;
        const float t2 = theta(o + d, x + d, y);
        const float tw = c.a1[s] * th1 + c.a2[s] * t2 + c.a3[s];
        if (oxm) {
            a[1] = own(3);
            b[1] = -own(12) + CT2 * tw;
        } else {
            a[3] = own(1);
            b[3] = -own(10) + CT2 * tw;
        }
    }
    if (oym | oyp) {
        const int d = oym ? 1 : -1, s = oym ? 2 : 3;
        const float t2 = theta(o + d * T::XE, x, y + d);
        const float tw = c.a1[s] * th1 + c.a2[s] * t2 + c.a3[s];
        if (oym) {
            a[2] = own(4);
            b[2] = -own(13) + CT2 * tw;
        } else {
            a[4] = own(2);
            b[4] = -own(11) + CT2 * tw;
        }
    }
    if (oxm | oym) a[5] = own(7);
    if (oxp | oym) a[6] = own(8);
    if (oxp | oyp) a[7] = own(5);
    if (oxm | oyp) a[8] = own(6);
    if (c.moving) add_wall_motion(c, from + o, P, oxm, oxp, oym, oyp, a);
}

// Result of node (gx, gy) of the tile: rounded, then into the LDS tile `to` at element o,
// or in the last phase into the other buffer.
template <typename S, unsigned P>
__device__ __forceinline__ void multi_finish(S* __restrict__ dst, const LatticeConst& c, S* to, unsigned o,
                                             bool last, const typename Wide<S>::type fa[9],
                                             const typename Wide<S>::type tb[5], int gx, int gy)
{
    S v[14];
    round_node<S>(fa, tb, v, gx, gy);
    if (last) {
        S* out = dst + (unsigned)node_off(c, gx, gy);
#pragma unroll
        for (int i = 0; i < 14; ++i) st_nt(out + i * kBlock, v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 14; ++i) to[i * P + o] = v[i];
    }
}

// Whether a phase with ring r has work at node (gx, gy), in coordinates that do not wrap:
// a node beyond a wall does not exist, and one further than r beyond a periodic end is
// read by nothing.
__device__ __forceinline__ bool multi_skip(const LatticeConst& c, int gx, int gy, int r)
{
    if (gx >= c.nx + (c.periodic_x ? r : 0) || gy >= c.ny + (c.periodic_y ? r : 0)) return true;
    return (gx < 0 && !c.periodic_x) || (gy < 0 && !c.periodic_y);
}

// The first phase, from the stored buffer. The ring is known at run time only: w = TX + 2 r
// nodes per row, and id / w is taken as (id * inv) >> 16 with inv = 65536 / w rounded up,
// exact while id * w <= 65536.
template <typename S, int SRC, int TX, int TY, int NS>
__device__ __forceinline__ void multi_first(const S* __restrict__ src, S* __restrict__ dst,
                                            const LatticeConst& c, S* lds, int X0, int Y0, int tid, int r,
                                            unsigned inv, bool interior)
{
    typedef typename Wide<S>::type W;
    typedef MultiTile<TX, TY, NS> T;
    const int w = TX + 2 * r, row = (int)(((unsigned)tid * inv) >> 16);
    if (row >= TY + 2 * r) return;
    const int tx = tid - row * w - r, ty = row - r;
    const unsigned o = (unsigned)(ty + T::R) * T::XE + (unsigned)(tx + T::R);
    S* to = lds + (r & 1) * 14 * T::P;
    int gx = X0 + tx, gy = Y0 + ty;
    W fa[9], tb[5];
    NodeMacro m;
    if (interior) {
        typename LoadT<S>::type a[9], b[5];
        const char* rc = stored_row(src, c.rowlen, gy);
        const size_t rb = (size_t)c.rowlen * sizeof(S);
        gather_interior<S, kBlock>(rc - rb, rc, rc + rb, stored_cols<S>(gx), a, b);
        collide<float, SRC, W>(c, a, b, fa, tb, m, node_q<SRC>(c, gx, gy));
    } else {
        if (multi_skip(c, gx, gy, r)) return;
        gx = wrap_ring(gx, c.nx);
        gy = wrap_ring(gy, c.ny);
        float a[9], b[5];
        gather_node<S, SRC, unsigned>(src, c, gx, gy, a, b);
        collide<float, SRC, W>(c, a, b, fa, tb, m, node_q<SRC>(c, gx, gy));
    }
    multi_finish<S, T::P>(dst, c, to, o, r == 0, fa, tb, gx, gy);
}

// A later phase with ring r, from the LDS tile of ring r + 1.
template <typename S, int SRC, int TX, int TY, int NS, int r>
__device__ __forceinline__ void multi_next(S* __restrict__ dst, const LatticeConst& c, S* lds, int X0, int Y0,
                                           int tid, bool interior)
{
    typedef typename Wide<S>::type W;
    typedef MultiTile<TX, TY, NS> T;
    constexpr int w = TX + 2 * r;
    if (tid >= w * (TY + 2 * r)) return;
    const S* from = lds + ((r + 1) & 1) * 14 * T::P;
    S* to = lds + (r & 1) * 14 * T::P;
    const int tx = tid % w - r, ty = tid / w - r;
    const unsigned o = (unsigned)(ty + T::R) * T::XE + (unsigned)(tx + T::R);
    int gx = X0 + tx, gy = Y0 + ty;
    W fa[9], tb[5];
    NodeMacro m;
    if (interior) {
        typename LoadT<S>::type a[9], b[5];
        constexpr unsigned e = (unsigned)sizeof(S), rb = T::XE * e;
        const char* rc = reinterpret_cast<const char*>(from + o);
        gather_interior<S, T::P>(rc - rb - e, rc - e, rc + rb - e, ColBytes{0, e, 2 * e}, a, b);
        collide<float, SRC, W>(c, a, b, fa, tb, m, node_q<SRC>(c, gx, gy));
    } else {
        if (multi_skip(c, gx, gy, r)) return;
        float a[9], b[5];
        gather_tile<SRC, S, T>(from, c, o, gx, gy, a, b);
        gx = wrap_ring(gx, c.nx);
        gy = wrap_ring(gy, c.ny);
        collide<float, SRC, W>(c, a, b, fa, tb, m, node_q<SRC>(c, gx, gy));
    }
    multi_finish<S, T::P>(dst, c, to, o, r == 0, fa, tb, gx, gy);
}

template <typename S, int SRC, int TX, int TY, int NS, int r>
__device__ __forceinline__ void multi_rest(S* __restrict__ dst, const LatticeConst& c, S* lds, int X0, int Y0,
                                           int tid, int steps, bool interior)
{
    if (r < steps - 1) {   // the same for the whole workgroup
        __syncthreads();
        multi_next<S, SRC, TX, TY, NS, r>(dst, c, lds, X0, Y0, tid, interior);
    }
    if constexpr (r > 0) multi_rest<S, SRC, TX, TY, NS, r - 1>(dst, c, lds, X0, Y0, tid, steps, interior);
}

// `steps` (1 to NS) steps of the tile at (X0, Y0); lds holds MultiTile::elems elements.
template <typename S, int SRC, int TX, int TY, int NS>
__device__ __forceinline__ void multi_tile(const S* __restrict__ src, S* __restrict__ dst,
                                           const LatticeConst& c, S* lds, int X0, int Y0, int tid, int steps,
                                           unsigned inv)
{
    // no node that a phase advances lies at a wall, and nothing wraps
    const bool interior = X0 >= steps && X0 + TX - 1 + steps < c.nx && Y0 >= steps && Y0 + TY - 1 + steps < c.ny;
    multi_first<S, SRC, TX, TY, NS>(src, dst, c, lds, X0, Y0, tid, steps - 1, inv, interior);
    multi_rest<S, SRC, TX, TY, NS, NS - 2>(dst, c, lds, X0, Y0, tid, steps, interior);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// A tile shape: tx x ty nodes, at most `steps` steps per launch, `threads` per workgroup.
struct MultiShape {
    int tx, ty, steps, threads;
    const void* (*single)(int precision, int src);         // k_multi for the source terms
    const void* (*batch)(int precision, int mode);         // k_batch_multi (MODE of k_batch_step2)
};

constexpr int kMultiShapes = 4;
const MultiShape* multi_shapes();

// The shape for a lattice (or the lattices of a batch), or nullptr for the two-step kernel.
// tiles(tx, ty) is the number of tiles of that size, or 0 if they cannot be listed.
// While every tile has a CU of its own the time is the chain of one workgroup, so the
// smallest tile and the most steps win; with more tiles than CUs the ring is paid for, and
// the shapes with less of it win. Microseconds per step on square lattices in FP32
// (two-step kernel first):
//   128^2: 4.7, 16x4 1.68, 32x8 2.07     192^2: 4.4, 16x4 2.23, 32x8 2.08
//   256^2: 4.5, 32x8 2.13, 32x12 2.38    384^2: 4.8, 32x8 4.8, 32x12 3.26, 32x16 3.8
//   512^2: 6.6, 32x12 4.5, 32x16 4.1    1500^2: 29.4, 32x12 27.9, 32x16 25.8
//  2048^2: 49.2, 32x16 45.5            4096^2: 179, 32x16 175
// 2^23 nodes is how far the shapes are taken, not where they stop to pay: 32x16 is the faster one beyond it
// too (3200^2 110.7 and 106.8, 4096^2 177.5 and 173.6, 6000^2 381 and 373; 256 cavities of 64 to 512 a
// side, 28.8 million nodes, 389 and 331). In FP16 the two-step kernel's taller tile wins from about 1.6 million nodes:
//   512^2: 6.0, 32x16 4.0   1200^2: 15.8, 32x16 14.2   1400^2: 18.8, 32x16 19.0   2048^2: 34.6, 32x16 38.3
template <typename Tiles>
const MultiShape* multi_shape(Tiles tiles, size_t nodes, int precision)
{
    constexpr size_t kCUs = 256;
    constexpr size_t most[kMultiShapes] = {kCUs, kCUs, 2 * kCUs, ~(size_t)0};
    if (nodes > (precision == CLBM_FP16_SHIFTED ? (size_t)3 << 19 : (size_t)1 << 23)) return nullptr;
    for (int k = 0; k < kMultiShapes; ++k) {
        const MultiShape& m = multi_shapes()[k];
        const size_t n = tiles(m.tx, m.ty);
        if (n > 0 && n <= most[k]) return &m;
    }
    return nullptr;
}

// Whether two steps that are left of a call are a launch of m too, not one of the two-step
// kernel. On large lattices it pays the ring and hides less: FP32, two-step kernel first, 1000 x 777
// 25 and 26 us, 1400^2 50 and 54, 2800^2 171 and 193, but 800 x 600 20 and 17; FP16 1200^2 32 and 34,
// 1000 x 777 20 and 24 the other way round. A batch gives its tile counts too (else 0): of 32 x 16 nodes,
// which collide 1124 for two steps, and of 64 x 14 for the two-step kernel, 1952, each node 3 % faster
// in FP32 and 10 % in FP16. Calls of two steps, two-step kernel first, FP32: 6 lattices of 700^2 (deeper
// tiles 1.3 % more nodes) 88 and 91 us, 16 of 512^2 (0.4 % fewer) 124 and 126, 64 from 64^2 to 505^2 (4 %
// fewer) 207 and 191; FP16: 8 of 330^2 (8 % fewer) 32 and 36, 24 from 64 x 60 to 156 x 129 (12 % fewer)
// 25 and 20.
inline bool multi_pairs(const MultiShape& m, size_t nodes, int precision, size_t tiles = 0, size_t two_step_tiles = 0)
{
    const bool half = precision == CLBM_FP16_SHIFTED;
    if (m.steps != 3) return true;
    if (tiles > 0 && (half || nodes > (size_t)5 << 17))
        return (half ? 1.1 : 1.03) * 1124 * (double)tiles < 1952.0 * (double)two_step_tiles;
    return nodes <= (half ? (size_t)1 << 20 : (size_t)5 << 17);
}

// Whether a lone step of a batch goes over the tiles of m, not over those of the two-step kernel
// (`nodes2` places in them): less of small tiles lies outside the lattices, but their short rows cost in
// FP16 and where there is little to hide them. The two-step kernel's tiles first: FP32 24 lattices
// of 96^2 (27 % fewer places) 18 and 16 us, 8 of 330^2 35 and 33, 64 from 64^2 to 505^2 159 and 150, but
// 4 of 300^2 (1 % fewer) 20 and 21; FP16 the first 16 and 14, the last 16 and 18.
inline bool multi_lone(const MultiShape& m, size_t nodes, int precision, size_t tiles, size_t nodes2)
{
    if (precision != CLBM_FP16_SHIFTED && nodes > (size_t)5 << 17) return true;
    return 1.15 * (double)(tiles * m.tx * m.ty) < (double)nodes2;
}

// How many of n steps are taken in launches of m; the others take the one- and two-step
// kernels (all of them give the same bits). A lone step is always theirs: 1000 x 777 in FP32
// 17.5 against 20.3 us, 1200^2 26 against 32. Without pairs only whole launches of three are
// left, and four steps are two pairs.
inline int multi_part(const MultiShape& m, bool pairs, int n)
{
    if (n < 2) return 0;
    return pairs ? n : n - (n % 3 == 1 ? 4 : n % 3);
}

// n steps as launches of at most `most` steps, as even as they come; parity 0 or 1: an even or odd
// number of launches (of n > 1 steps).
struct StepSplit {
    int launches, base, extra;   // the first `extra` launches take base + 1 steps
    StepSplit(int n, int most, int parity = -1)
    {
        launches = (n + most - 1) / most;
        if (parity >= 0 && launches % 2 != parity) ++launches;
        base = launches ? n / launches : 0;
        extra = launches ? n % launches : 0;
    }
    int steps(int k) const { return base + (k < extra ? 1 : 0); }
};

// Launches of n steps by the two-step kernel.
inline int two_step_launches(int n) { return n / 2 + n % 2; }

// Whether steps issued now are recorded into a caller's stream capture. The recorded launches
// start from one of two buffers and can be repeated only if they end in it too. With the two-step
// kernel that held for every multiple of four steps, and launches of the deeper tiles are
// recorded in a number of the same parity; where steps run at once it does not matter.
inline bool is_captured(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    // (the null stream cannot be captured)
    return stream && hipStreamIsCapturing(stream, &status) == hipSuccess && status == hipStreamCaptureStatusActive;
}

// The divisor of multi_first for launches of `steps` steps.
inline unsigned multi_inv(const MultiShape& m, int steps)
{
    const unsigned w = (unsigned)(m.tx + 2 * (steps - 1));
    return (65536u + w - 1) / w;
}

}  // namespace clbm
