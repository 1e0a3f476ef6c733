// clbm_wgrad.h -- weight and bias gradients of a 3x3 convolution (gfx950).
//
// dW[co][tap][ci] = sum over pixels p of dz[p][co] x[p shifted by the tap][ci]: a GEMM whose
// K is the pixel, the slow index of NHWC. Both operands are staged as they lie in memory
// and read with LDS transpose reads (ds_read_b64_tr_b16: four pixels x 16 channels per 16
// lanes), so a tap is a constant LDS offset and nothing is staged more than once.
#pragma once

#include <type_traits>

#include "clbm_conv.h"

namespace clbm {

// Four consecutive pixels (LDS rows of 64 bytes) of 16 channels, transposed: lane l of each 16
// gives the address of pixel l / 4, channels 4 (l % 4), and receives channel l % 16.
__device__ __forceinline__ bf16x8 tr_pair(const bf16* p0, const bf16* p1)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_p;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p0));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p1));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

struct WgradArgs {
    const bf16* dz;
    int zC;
    const bf16* x;
    int xC, xoff;
    int zocts, xocts;           // octets of channels that are stored (the others are zero)
    int H, W, P;
    int co_blocks, ci_blocks;   // blocks of 16 NA x 32 channels
    int pixels, splits;         // pixels per split (a multiple of 32) and their number
    float *part, *bpart;        // [split][block][9 x 16 NA x 32], [split][co_blocks x 16 NA]
};

// The split of a layer, which fixes the order its gradient is summed in: about 512 blocks
// of 64 x 64 channels (32 or 16 where the channels do not divide), at most 256 splits, at
// least 256 pixels each.
inline int wgrad_pixels_per_split(size_t P, int cout, int cin_pad)
{
    auto block = [](int n16) { return n16 % 4 == 0 ? 4 : (n16 % 2 == 0 ? 2 : 1); };
    const int co16 = (cout + 15) / 16, ci16 = cin_pad / 16;
    const size_t blocks = (size_t)(co16 / block(co16)) * (ci16 / block(ci16));
    size_t splits = 512 / blocks;
    splits = splits > 256 ? 256 : splits < 1 ? 1 : splits;
    const size_t most = P / 256 > 1 ? P / 256 : 1;
    splits = splits < most ? splits : most;
    const size_t pixels = (P + splits - 1) / splits;
    return (int)((pixels + 31) / 32 * 32);
}

constexpr int kWgStep = 96;   // pixels staged per step: three chunks of K = 32

// A workgroup owns 16 NA x 32 channels and the consecutive pixels of one split. Wave dy
// takes the three taps of kernel row dy, so a chunk costs it NA + 6 fragment reads for 6 NA
// MFMAs. A wave's chain of reads and multiplies bounds it, covered by the other workgroup of
// the CU: reading a chunk ahead takes the registers of that one (64 -> 64 at 64^2: 34 us
// against 21), and waves of 16 input channels, which read more per MFMA, were slower although
// twice as many. The input lies in LDS as a ring over consecutive pixels of
// the batch that spans the rows above and below the current pixels: a pixel is staged once
// and a tap is a constant distance in the ring (rows too long for that have a ring per
// kernel row, and are staged three times). A lane whose pixel has no such neighbour reads
// zeros instead. Input and gradient of the next two steps are in registers or on their way
// while one is multiplied. Each split leaves one partial; the bias gradient is the product
// with ones, taken by the first input block. Workgroups of the same pixels follow each other
// on one XCD.
// ALIGNED: rows are a multiple of 32 pixels, so a chunk lies in one row and its places in the
// ring are a uniform base plus constants of the lane (the general form spends more time on
// addresses than on MFMAs).
// LDS: 32 channels (64 bytes) per pixel, whose halves swap with bit 3 of its place, so the
// eight pixels that a half-wave reads cover all banks.
// 32 -> 32 channels at batch 32 on 128^2 (67 MB of operands): 33 us; 64 -> 64 at 64^2:
// 21 us; three waves staging nine shifted, transposed copies took 144 and 74 us.
template <int NA, int RING, bool WIDE, bool ALIGNED>
__global__ void __launch_bounds__(192) k_wgrad(const WgradArgs a)
{
    constexpr int D = 2;        // steps in flight between memory and LDS
    constexpr int kPass = 48;   // pixels staged by one pass of the workgroup, two per step
    constexpr int kRings = WIDE ? 3 : 1;
    constexpr int kPlane = kWgStep * 32, kPlanes = NA / 2, kZ = kPlanes * kPlane;
    __shared__ __attribute__((aligned(64))) bf16 lds[kRings * RING * 32 + 2 * kZ + 32];
    bf16* const zbuf = lds + kRings * RING * 32;
    constexpr unsigned kZero = kRings * RING * 32 + 2 * kZ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int dy = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = a.co_blocks * a.ci_blocks;
    const int local = blockIdx.x >> 3, split = (blockIdx.x & 7) + 8 * (local / blocks), blk = local % blocks;
    if (split >= a.splits) return;
    const int cob = blk % a.co_blocks, cib = blk / a.co_blocks;
    const int pbeg = split * a.pixels, pend = min(a.P, pbeg + a.pixels), chunks = (pend - pbeg) / 32;
    const int W = a.W;
    const int oct = tid & 3, px = tid >> 2;   // staged octet and pixel (the first of two)
    const bf16* xb = a.x + a.xoff + cib * 32 + 8 * oct;
    const bf16* zb = a.dz + cob * 16 * NA + 8 * oct;
    const bool xin = cib * 4 + oct < a.xocts;
    const bf16x8 zero = {};
    if (tid < 4) *reinterpret_cast<bf16x8*>(lds + kZero + 8 * tid) = zero;
    // Ring d holds the input at a distance of (d - 1) rows (WIDE), or the one ring all of it;
    // pixel q of a ring has `halo` neighbours on either side of the pixels being multiplied.
    // A pixel outside the batch is read by no lane.
    const int halo = WIDE ? 1 : W + 1;
    auto xload = [&](int d, int q) {
        if (WIDE) q += (d - 1) * W;
        return xin && q >= 0 && q < a.P ? *reinterpret_cast<const bf16x8*>(xb + (size_t)q * a.xC) : zero;
    };
    auto xput = [&](int d, int q, const bf16x8 v) {
        const unsigned slot = (unsigned)q & (RING - 1);
        *reinterpret_cast<bf16x8*>(lds + (d * RING + slot) * 32 + ((oct * 8) ^ ((slot & 8) << 1))) = v;
    };
    bf16x8 rx[D][2][kRings], rz[D][2][kPlanes];
    // gradient of the step's 96 pixels and input of the 96 pixels that the step adds
    auto fetch = [&](int s, int st, bool input) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int p = pbeg + st * kWgStep + px + u * kPass;
#pragma unroll
            for (int k = 0; k < kPlanes; ++k)
                rz[s][u][k] = p < pend && cob * 2 * NA + 4 * k + oct < a.zocts ? *reinterpret_cast<const bf16x8*>(zb + (size_t)p * a.zC + 32 * k) : zero;
#pragma unroll
            for (int d = 0; d < kRings; ++d)
                if (input) rx[s][u][d] = xload(d, p + halo);
        }
    };
    auto put = [&](int s, int st, bool input) {
        bf16* z = zbuf + (st & 1) * kZ;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int l = px + u * kPass;
#pragma unroll
            for (int k = 0; k < kPlanes; ++k)
                *reinterpret_cast<bf16x8*>(z + k * kPlane + l * 32 + ((oct * 8) ^ ((l & 8) << 1))) = rz[s][u][k];
#pragma unroll
            for (int d = 0; d < kRings; ++d)
                if (input) xput(d, pbeg + st * kWgStep + l + halo, rx[s][u][d]);
        }
    };
    f32x4 acc[3][NA][2], bacc[NA];
    const f32x4 fz = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        bacc[i] = fz;
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[0][i][j] = acc[1][i][j] = acc[2][i][j] = fz;
    }
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (bf16)1.f;
    const bool bias = cib == 0 && dy == 1;
    fetch(0, 0, false);
#pragma unroll
    for (int d = 0; d < kRings; ++d)
        for (int q = pbeg - halo + px; q < pbeg + kWgStep + halo; q += kPass) xput(d, q, xload(d, q));
    put(0, 0, false);
    // The two pixels of a chunk whose address this lane gives, as places of the image
    // (ALIGNED: of the chunk's first pixel, the same for every lane), and the elements of
    // their fragments: input relative to the chunk's place in the ring, gradient.
    const int c4 = (lane & 3) * 4, l0 = 8 * (lane >> 4) + ((lane >> 2) & 3);
    int y[2], x[2], tc[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int rem = (pbeg + (ALIGNED ? 0 : l0 + 4 * h)) % (a.H * W);
        y[h] = rem / W;
        x[h] = rem - y[h] * W;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const int t = l0 + 4 * h + dx - 1;
            tc[dx][h] = t * 32 + (c4 ^ ((t & 8) << 1));
        }
    }
    unsigned za[NA][2];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int l = l0 + 4 * h;
            za[i][h] = (unsigned)((i >> 1) * kPlane + l * 32 + ((c4 + 16 * (i & 1)) ^ ((l & 8) << 1)));
        }
    const unsigned mine = (unsigned)c4;
    // chunk c, the k-th of the step at z
    auto chunk = [&](int c, const bf16* z, int k) {
        unsigned xa[3][2];
        const int p = pbeg + c * 32 + (WIDE ? 0 : (dy - 1) * W);
        if constexpr (ALIGNED) {
            const int base = (int)((unsigned)p & (RING - 1)), ring = WIDE ? dy * RING : 0;
            const bool vy = (unsigned)(y[0] + dy - 1) < (unsigned)a.H;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int h = 0; h < 2; ++h) xa[dx][h] = vy ? (unsigned)((ring + base) * 32 + tc[dx][h]) : kZero + mine;
            // the neighbours before the chunk's first pixel and after its last: across the
            // ring's end, or outside the row
            if (l0 == 0) xa[0][0] = !vy || x[0] == 0 ? kZero + mine : xa[0][0] + (base == 0 ? RING * 32 : 0);
            if (l0 == 27) xa[2][1] = !vy || x[0] + 32 == W ? kZero + mine : xa[2][1] - (base == RING - 32 ? RING * 32 : 0);
            x[0] += 32;
            if (x[0] == W) {
                x[0] = 0;
                if (++y[0] == a.H) y[0] = 0;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool vy = (unsigned)(y[h] + dy - 1) < (unsigned)a.H;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    const bool v = vy && (dx != 0 || x[h] > 0) && (dx != 2 || x[h] < W - 1);
                    const unsigned slot = (unsigned)(p + l0 + 4 * h + dx - 1) & (RING - 1);
                    xa[dx][h] = (v ? ((WIDE ? dy * RING : 0) + slot) * 32 + ((slot & 8) << 1) : kZero) ^ mine;
                }
                x[h] += 32;
                while (x[h] >= W) {
                    x[h] -= W;
                    if (++y[h] == a.H) y[h] = 0;
                }
            }
        }
        bf16x8 az[NA], bx[3][2];
#pragma unroll
        for (int i = 0; i < NA; ++i) az[i] = tr_pair(z + za[i][0] + k * 32 * 32, z + za[i][1] + k * 32 * 32);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                bx[dx][j] = tr_pair(lds + (xa[dx][0] ^ (16u * j)), lds + (xa[dx][1] ^ (16u * j)));
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[dx][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(az[i], bx[dx][j], acc[dx][i][j], 0, 0, 0);
        if (bias)
#pragma unroll
            for (int i = 0; i < NA; ++i)
                bacc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(az[i], ones, bacc[i], 0, 0, 0);
    };
    const int steps = (chunks + 2) / 3;
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s + 1 < steps) fetch(s, s + 1, true);
    __syncthreads();
    for (int st0 = 0; st0 < steps; st0 += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const int st = st0 + s, c = 3 * st;
            if (st >= steps) break;
            const bf16* z = zbuf + (st & 1) * kZ;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (c + k < chunks) chunk(c + k, z, k);
            if (st + 1 < steps) put(s, st + 1, true);
            if (st + 1 + D < steps) fetch(s, st + 1 + D, true);
            __syncthreads();
        }
    }
    f32x4* out = reinterpret_cast<f32x4*>(a.part) + ((size_t)split * blocks + blk) * (9 * NA * 2 * 64) + lane;
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) out[(((dy * 3 + dx) * NA + i) * 2 + j) * 64] = acc[dx][i][j];
    // every column of the product with ones holds the sum; rows 4 (lane / 16) .. + 3
    if (bias && (lane & 15) == 0)
#pragma unroll
        for (int i = 0; i < NA; ++i)
            reinterpret_cast<f32x4*>(a.bpart)[((size_t)split * a.co_blocks + cob) * (4 * NA) + 4 * i + (lane >> 4)] = bacc[i];
}

// Geometry of k_wgrad_octets: pixels staged per step, and LDS bytes of one channel's pixels,
// the last 16 of them zeros. Channels start a multiple of 128 bytes and 16 apart, octets
// of channels 32 more: the eight channels that a group of lanes reads cover all banks, and so do the
// four octets x two pixel groups that it writes.
template <int NA>
struct OctetGeom {
    static constexpr int S = NA == 4 ? 128 : 192;   // (NA/2 + 1 planes) x S/8 x 4 octets: 192 items
    static constexpr int HALO = 8;   // pixels kept on either side
    static constexpr int ZS = 2 * S + 16;
    static constexpr int Z = 16 * NA * ZS + 64 * NA;
    __host__ __device__ static int ring(int W) { return 2 * W + 2 * HALO + 2 * S; }
    __host__ __device__ static int xs(int W) { return (2 * ring(W) + 127) / 128 * 128 + 16; }
    __host__ __device__ static int x_bytes(int W) { return 32 * xs(W) + 128; }
    static size_t lds(int W) { return (size_t)x_bytes(W) + 2 * Z; }
};

// Rows of whole octets of pixels. A workgroup owns 16 NA x 32 channels and the consecutive pixels
// of one split; wave (dy, j) takes the three taps of kernel row dy and half j of the input
// channels. Operands are transposed on their way to LDS: an item is eight pixels x
// eight channels, 16-byte loads of a pixel's channels and 16-byte stores of a channel's
// pixels, so a fragment (one channel, eight consecutive pixels per lane) is one plain 16-byte
// read. The taps to the left and right are the same fragment shifted by one pixel with
// the neighbouring pair from LDS. The input is a ring over consecutive pixels of the batch that
// holds the rows above and below, staged once; an octet lies in one row, so a pixel outside
// the image is a whole fragment or a neighbouring pair, read from the zeros behind the lane's
// channel instead. Two steps are in registers or on their way (the halves of the
// workgroup stage alternate ones), one barrier per step; the fragments of the next chunk are
// read while one is multiplied. It reads more of LDS per MFMA than k_wgrad and is the faster one
// where a CU has a single workgroup: 32 -> 32 channels at batch 32 on 128^2, 256 workgroups:
// 25 against 33 us; with 512 of 64 x 32 channels 26 against 21 us.
template <int NA>
__global__ void __launch_bounds__(384) __attribute__((amdgpu_waves_per_eu(2))) k_wgrad_octets(const WgradArgs a)
{
    using G = OctetGeom<NA>;
    constexpr int S = G::S, ZS = G::ZS, HALO = G::HALO, kZPlanes = NA / 2;
    extern __shared__ __attribute__((aligned(128))) char oct_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), dy = wave % 3, jb = wave / 3;
    const int blocks = a.co_blocks * a.ci_blocks;
    const int local = blockIdx.x >> 3, split = (blockIdx.x & 7) + 8 * (local / blocks), blk = local % blocks;
    if (split >= a.splits) return;
    const int cob = blk % a.co_blocks, cib = blk / a.co_blocks;
    const int pbeg = split * a.pixels, pend = min(a.P, pbeg + a.pixels), chunks = (pend - pbeg) / 32;
    const int W = a.W, H = a.H, ring = G::ring(W), XS = G::xs(W), last = a.P - 8;
    char* const zlds = oct_lds + G::x_bytes(W);
    const bf16x8 zero = {};
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    // eight pixels x eight channels in, a channel's eight pixels out
    auto store = [](char* to, int stride, const bf16x8 (&v)[8]) {
        u32x4 in[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] = __builtin_bit_cast(u32x4, v[j]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            u32x4 out;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[i] = __builtin_amdgcn_perm(in[2 * i + 1][k / 2], in[2 * i][k / 2], k % 2 ? 0x07060302u : 0x05040100u);
            *reinterpret_cast<u32x4*>(to + k * stride) = out;
        }
    };
    // this thread's item of a step: octet o of the channels of a plane, pixel group
    const int item = tid - 192 * jb, o = item & 3, pg = (item >> 2) % (S / 8), plane = item / (S / 2);
    const bool isx = plane == kZPlanes;
    const bool have = isx ? cib * 4 + o < a.xocts : cob * 2 * NA + 4 * plane + o < a.zocts;
    const int istride = isx ? a.xC : a.zC;
    const bf16* const isrc = isx ? a.x + a.xoff + cib * 32 + 8 * o : a.dz + cob * 16 * NA + plane * 32 + 8 * o;
    const int ipix = pbeg + 8 * pg + (isx ? W + HALO : 0);   // its first pixel in step 0
    // Pixels after the split's (gradient) or the batch's last (input) are multiplied by no lane:
    // any pixel's channels do.
    bf16x8 v[8];
    auto load = [&](const bf16* src, int p, int stride) {
        src += (size_t)max(0, min(p, last)) * stride;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const bf16x8*>(src + (size_t)j * stride);
    };
    auto fetch = [&](int st) {
        if (have) load(isrc, ipix + st * S, istride);
    };
    char* const zrow = zlds + (plane * 4 + o) * (8 * ZS + 32) + 16 * pg;
    char* const xrow = oct_lds + o * (8 * XS + 32);
    int slot = 2 * W + 2 * HALO + 8 * pg + (jb == 0 ? 2 * S : S);   // ring place of its next put
    slot = slot >= ring ? slot - ring : slot;
    auto put = [&](int st) {
        if (have) {
            if (isx) store(xrow + 2 * slot, XS, v);
            else store(zrow + (st & 1) * G::Z, ZS, v);
        }
        slot += 2 * S;
        slot = slot >= ring ? slot - ring : slot;
    };
    const int steps = (chunks * 32 + S - 1) / S;
    // channels that are not stored, and the pixels outside the image, read as zeros
    if (cib * 4 + 4 > a.xocts || cob * 2 * NA + 2 * NA > a.zocts) {
        for (int t = tid; t < (G::x_bytes(W) + 2 * G::Z) / 16; t += 384) reinterpret_cast<bf16x8*>(oct_lds)[t] = zero;
        __syncthreads();
    }
    if (tid < 32) *reinterpret_cast<bf16x8*>(oct_lds + tid * XS + (tid >> 3) * 32 + XS - 16) = zero;
    // input of the first step with the rows around it: ring places 0 .. 2 W + 2 HALO + S
    for (int t = tid; t < (2 * W + 2 * HALO + S) / 2; t += 384) {
        const int oc = t & 3;
        if (cib * 4 + oc < a.xocts) {
            load(a.x + a.xoff + cib * 32 + 8 * oc, pbeg - W - HALO + 2 * (t & ~3), a.xC);
            store(oct_lds + oc * (8 * XS + 32) + 4 * (t & ~3), XS, v);
        }
    }
    if (jb == 0 && !isx && have) {
        fetch(0);
        store(zrow, ZS, v);
    }
    if (2 - jb < steps) fetch(2 - jb);
    f32x4 acc[3][NA], bacc[NA];
    const f32x4 fz = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[0][i] = acc[1][i] = acc[2][i] = bacc[i] = fz;
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (bf16)1.f;
    const bool bias = cib == 0 && dy == 1 && jb == 0;
    // the next chunk's octet of pixels of this lane: row and column of the image and byte in a
    // channel's ring
    const int r16 = lane & 15, g = lane >> 4;
    const int rem = (pbeg + 8 * g) % (H * W);
    int y = rem / W, x = rem - y * W;
    unsigned at = 2 * (dy * W + HALO + 8 * g);
    const unsigned end = 2 * ring, none = XS - 16;
    const int down = 32 / W % H, right = 32 % W;
    const char* const xl = oct_lds + (16 * jb + r16) * XS + (2 * jb + (r16 >> 3)) * 32;
    const unsigned zl = r16 * ZS + (r16 >> 3) * 32 + 16 * g;
    struct Frags {
        bf16x8 z[NA];
        u32x4 x;
        unsigned left, right;
    } f[2];
    auto read = [&](Frags& f, const char* z, int k) {
        const bool vy = (unsigned)(y + dy - 1) < (unsigned)H;
        const unsigned mid = vy ? at : none;
        const unsigned lef = vy && x > 0 ? (at ? at : end) - 4 : none;
        const unsigned rig = vy && x + 8 < W ? (at + 16 == end ? 0 : at + 16) : none;
        x += right;
        const bool next = x >= W;
        x = next ? x - W : x;
        y += down + next;
        y = y >= H ? y - H : y;
        at += 64;
        at = at >= end ? at - end : at;
        f.x = *reinterpret_cast<const u32x4*>(xl + mid);
        f.left = *reinterpret_cast<const unsigned*>(xl + lef);
        f.right = *reinterpret_cast<const unsigned*>(xl + rig);
#pragma unroll
        for (int i = 0; i < NA; ++i)
            f.z[i] = *reinterpret_cast<const bf16x8*>(z + zl + k * 64 + i * (16 * ZS + 64));
    };
    auto multiply = [&](const Frags& f, auto with_bias) {
        const u32x4 c = f.x;
        const unsigned m1 = __builtin_amdgcn_alignbit(c[1], c[0], 16), m2 = __builtin_amdgcn_alignbit(c[2], c[1], 16);
        const unsigned m3 = __builtin_amdgcn_alignbit(c[3], c[2], 16);
        const bf16x8 bx[3] = {
            __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_alignbit(c[0], f.left, 16), m1, m2, m3}),
            __builtin_bit_cast(bf16x8, c),
            __builtin_bit_cast(bf16x8, u32x4{m1, m2, m3, __builtin_amdgcn_alignbit(f.right, c[3], 16)})};
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int i = 0; i < NA; ++i)
                acc[dx][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.z[i], bx[dx], acc[dx][i], 0, 0, 0);
        if constexpr (with_bias.value)
#pragma unroll
            for (int i = 0; i < NA; ++i)
                bacc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.z[i], ones, bacc[i], 0, 0, 0);
    };
    // the chunks of a step: fragments of the next are read while one is multiplied (left to
    // the compiler, each chunk waited for its own)
    auto step = [&](const char* z, int n, auto with_bias) {
        read(f[0], z, 0);
        if (n == S / 32) {
#pragma unroll
            for (int k = 0; k < S / 32; ++k) {
                if (k + 1 < S / 32) read(f[(k + 1) & 1], z, k + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(f[k & 1], with_bias);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            for (int k = 0; k < n; ++k) {
                multiply(f[0], with_bias);
                if (k + 1 < n) read(f[0], z, k + 1);
            }
        }
    };
    __syncthreads();
    for (int st = 0; st < steps; ++st) {
        const int n = min(S / 32, chunks - st * (S / 32));
        const char* z = zlds + (st & 1) * G::Z;
        if (bias) step(z, n, std::true_type{});
        else step(z, n, std::false_type{});
        if (jb != (st & 1)) {
            if (st + 1 < steps) put(st + 1);
            if (st + 3 < steps) fetch(st + 3);
        }
        __syncthreads();
    }
    f32x4* out = reinterpret_cast<f32x4*>(a.part) + ((size_t)split * blocks + blk) * (9 * NA * 2 * 64) + lane;
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int i = 0; i < NA; ++i) out[(((dy * 3 + dx) * NA + i) * 2 + jb) * 64] = acc[dx][i];
    // every column of the product with ones holds the sum; rows 4 (lane / 16) .. + 3
    if (bias && r16 == 0)
#pragma unroll
        for (int i = 0; i < NA; ++i)
            reinterpret_cast<f32x4*>(a.bpart)[((size_t)split * a.co_blocks + cob) * (4 * NA) + 4 * i + g] = bacc[i];
}

// Sums of the split partials in split order, written to the canonical gradient
// grad[co][ci][tap] (co < Cout, ci < Cin); the workgroups after the weights' sum the biases.
// One float per thread, 32 splits' loads in flight (8 took three times as long where a
// layer has few weights and many splits).
template <int NA>
__global__ void __launch_bounds__(64) k_wgrad_reduce(const float* __restrict__ part, const float* __restrict__ bpart,
                                                     int splits, int co_blocks, int ci_blocks, int Cout, int Cin,
                                                     float* __restrict__ grad, float* __restrict__ bgrad)
{
    constexpr int kBlock = 9 * NA * 2 * 256;
    const int blocks = co_blocks * ci_blocks, wgs = blocks * (kBlock / 64);
    const bool bias = (int)blockIdx.x >= wgs;
    const size_t stride = bias ? (size_t)co_blocks * 16 * NA : (size_t)blocks * kBlock;
    const size_t at = (size_t)(bias ? blockIdx.x - wgs : blockIdx.x) * 64 + threadIdx.x;
    if (at >= stride) return;
    const float* p = (bias ? bpart : part) + at;
    float s = 0.f;
    int k = 0;
    for (; k + 32 <= splits; k += 32) {
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = p[(size_t)(k + u) * stride];
#pragma unroll
        for (int u = 0; u < 32; ++u) s += v[u];
    }
#pragma unroll 4
    for (; k < splits; ++k) s += p[(size_t)k * stride];
    if (bias) {
        if ((int)at < Cout) bgrad[at] = s;
        return;
    }
    const int blk = (int)(at / kBlock), e = (int)(at % kBlock);
    const int v = e & 3, l = (e >> 2) & 63, j = (e >> 8) & 1, i = (e >> 9) % NA, tap = (e >> 9) / NA;
    const int co = (blk % co_blocks) * 16 * NA + 16 * i + 4 * (l >> 4) + v, ci = (blk / co_blocks) * 32 + 16 * j + (l & 15);
    if (ci < Cin && co < Cout) grad[((size_t)co * Cin + ci) * 9 + tap] = s;
}

}  // namespace clbm
