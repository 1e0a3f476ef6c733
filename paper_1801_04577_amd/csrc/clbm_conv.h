// clbm_conv.h -- 3x3 convolutions of the warm-start network as implicit GEMMs (gfx950).
//
// M = output channels, N = pixels, K = 9 taps x input channels, on
// v_mfma_f32_16x16x32_bf16: lane l holds row (l % 16) of the first operand (a channel) and
// column (l % 16) of the second (a pixel), elements k = 8 (l/16) .. 8 (l/16) + 7; the
// result holds column (l % 16), rows 4 (l/16) .. 4 (l/16) + 3. Channels are taken as rows,
// so a lane ends with consecutive channels of one pixel, and two row blocks are dealt so
// that it has eight of them: one 16-byte store where NHWC is written.
//
// Every output is accumulated in FP32 in one of two orders, which fix its rounding: with
// the chunk of 32 input channels outermost and the taps inside (k_conv_rows), or with the
// taps outermost (k_conv_tile, k_conv_taps).
#pragma once

#include <hip/hip_runtime.h>

namespace clbm {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kKChunk = 32;          // K per MFMA (one tap, 32 input channels)
constexpr int kFrag = 512;           // elements of one operand fragment (64 lanes x 8)
constexpr int kChunkW = 18 * kFrag;  // weights of 32 channels over a chunk: 9 taps x 2 row blocks

__device__ __forceinline__ float bf2f(bf16 v) { return (float)v; }
__device__ __forceinline__ bf16 f2bf(float v) { return (bf16)v; }

// What an epilogue does besides (kPostPool) or instead of writing its output: everything that the
// network does between two convolutions, on values still in registers and rounded to bf16
// as they would have been stored. Pool and Sum need 2 x 2 pixels in one wave: rows are in its
// registers, columns in neighbouring lanes. As kernels of their own these passes took 150 us of
// a training step at batch 32 on 128^2; in the epilogues they add about 65.
enum ConvPost : int {
    kPostNone,
    kPostPool,     // also the 2 x 2 average, to e (half resolution)
    kPostUp,       // four copies, to e (double resolution)
    kPostSum,      // channels below eN: 2 x 2 sums to e (half resolution), zero where mask is not positive at
                   // the first pixel of the four (the upsampled activations); the others as they are
    kPostUnpool    // four times a quarter plus e2, zero where mask is not positive, to e (all double resolution)
};

// The weights w of one direction of a layer lie as its convolution reads them: per group of 32
// output channels, chunk of 32 input channels and tap (in the order they are accumulated) and
// row block h one fragment of 1 KB, lane after lane. Row i of block h is channel
// 8 (i/4) + 4 h + i % 4 of the group.
struct ConvArgs {
    const bf16* x;       // input, NHWC
    int xC, xoff, Cin;   // channel stride and offset; input channels, a multiple of 32
    int octs;            // octets of channels that are stored, when fewer than Cin (one chunk; the others are zero)
    const bf16* w;
    const float* bias;
    int N, H, W, P;      // output channels, image, pixels in all
    int mode;            // 0: relu(acc + bias) as bf16; 1: acc as bf16 (input gradients); 2: acc + bias, FP32 NCHW
    const bf16* mask;    // mode 1: nullptr, or activations at the output's pixels: zero where not positive (ReLU)
    int maskC;
    bf16* y;
    int yC, yoff;
    float *yf, *yf2;     // mode 2: the output, and a second place for it or nullptr
    int post;            // ConvPost; its views of the operands' channels
    bf16* e;
    int eC, eN;
    const bf16* e2;
    int e2C;
};

// Epilogue of one pixel: lane group g = lane / 16 holds channels n0 + 8 g .. + 7.
template <int NH>
__device__ __forceinline__ void conv_bias(const ConvArgs& a, int n, float (&bias)[4 * NH])
{
#pragma unroll
    for (int k = 0; k < 4 * NH; ++k) bias[k] = a.mode != 1 && n + k < a.N ? a.bias[n + k] : 0.f;
}

// The pixel's eight channels as they are stored.
__device__ __forceinline__ bf16x8 conv_value(const ConvArgs& a, const f32x4 (&acc)[2], const float (&bias)[8])
{
    bf16x8 o;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float r = acc[h][v];
            if (a.mode == 0) r = fmaxf(r + bias[4 * h + v], 0.f);
            o[4 * h + v] = f2bf(r);
        }
    return o;
}

// Where the pixel (x, y) of image img and the rows below it go and find their masks, as pointers and
// their steps per row: one 64-bit product each instead of one per pixel and operand.
template <bool POST>
struct ConvPlace {
    bf16 *y, *e;
    const bf16 *mask, *e2;
    size_t yS, eS, maskS, e2S;
    __device__ __forceinline__ ConvPlace(const ConvArgs& a, int n, int img, int py, int px)
    {
        const size_t HW = (size_t)a.H * a.W, p = img * HW + (unsigned)(py * a.W + px);
        const bool twice = POST && (a.post == kPostUp || a.post == kPostUnpool);
        // double resolution: two rows per row; half: a row per two (eS is per pair)
        const size_t q = twice ? 4 * img * HW + (size_t)(4 * py) * a.W + 2 * px : p;
        y = a.y + p * a.yC + a.yoff + n;
        yS = (size_t)a.W * a.yC;
        mask = a.mask + q * a.maskC + n;
        maskS = (size_t)(twice ? 4 * a.W : a.W) * a.maskC;
        if constexpr (POST) {
            e = a.e + (twice ? q : img * (HW / 4) + (unsigned)((py / 2) * (a.W / 2) + px / 2)) * a.eC + n;
            eS = (size_t)(twice ? 4 * a.W : a.W / 2) * a.eC;
            e2 = a.e2 + q * a.e2C + n;
            e2S = (size_t)(4 * a.W) * a.e2C;
        }
    }
};

// Row r of a place (its channels n .. n + 7): output and what follows it pixel by pixel.
template <bool POST>
__device__ __forceinline__ void conv_pixel(const ConvArgs& a, const ConvPlace<POST>& t, int r, int n, bf16x8 o)
{
    if (POST && a.post == kPostSum && n < a.eN) return;
    if (POST && (a.post == kPostUp || a.post == kPostUnpool)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const size_t at = (size_t)((k >> 1) * 2 * a.W + (k & 1));
            bf16x8 v = o;
            if (a.post == kPostUnpool) {
                const bf16x8 skip = *reinterpret_cast<const bf16x8*>(t.e2 + r * t.e2S + at * a.e2C);
                const bf16x8 m = *reinterpret_cast<const bf16x8*>(t.mask + r * t.maskS + at * a.maskC);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v[i] = bf2f(m[i]) > 0.f ? f2bf(bf2f(skip[i]) + 0.25f * bf2f(o[i])) : (bf16)0.f;
            }
            *reinterpret_cast<bf16x8*>(t.e + r * t.eS + at * a.eC) = v;
        }
        return;
    }
    if (a.mask && !(POST && a.post == kPostSum)) {
        const bf16x8 m = *reinterpret_cast<const bf16x8*>(t.mask + r * t.maskS);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (!(bf2f(m[k]) > 0.f)) o[k] = (bf16)0.f;
    }
    *reinterpret_cast<bf16x8*>(t.y + r * t.yS) = o;
}

// The output layer: pixel (x, y) of image img.
template <int NH>
__device__ __forceinline__ void conv_planes(const ConvArgs& a, const f32x4 (&acc)[NH], const float (&bias)[4 * NH],
                                            int n, int img, int y, int x)
{
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = n + 4 * h + v;
            if (c >= a.N) continue;
            const float r = acc[h][v] + bias[4 * h + v];
            const size_t at = ((size_t)img * a.N + c) * ((size_t)a.H * a.W) + y * a.W + x;
            a.yf[at] = r;
            if (a.yf2) a.yf2[at] = r;
        }
}

// 2 x 2 pixels: this lane's column (odd or even) of rows r (r0) and r + 1 (r1), r even, and the
// neighbouring lane's. The lane of the even column finishes the first four channels, the other the
// last four.
__device__ __forceinline__ void conv_pair(const ConvArgs& a, const ConvPlace<true>& t, int r, bool odd, bf16x8 r0,
                                          bf16x8 r1)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const int half = 4 * odd;
    float sum[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const u32x4 w = __builtin_bit_cast(u32x4, i ? r1 : r0);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const unsigned own = odd ? w[2 + d] : w[d], give = odd ? w[d] : w[2 + d];
            const unsigned got = __builtin_amdgcn_update_dpp(0u, give, 0xB1, 0xF, 0xF, true);   // lanes 1 0 3 2
            const unsigned left = odd ? got : own, right = odd ? own : got;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float l = __builtin_bit_cast(float, k ? left & 0xffff0000u : left << 16);
                const float m = __builtin_bit_cast(float, k ? right & 0xffff0000u : right << 16);
                float& s = sum[2 * d + k];
                s = i ? s + l + m : l + m;
            }
        }
    }
    bf16x4 o;
    if (a.post == kPostPool) {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = f2bf(0.25f * sum[k]);
    } else {
        const bf16x4 m = *reinterpret_cast<const bf16x4*>(t.mask + r * t.maskS - (odd ? a.maskC : 0) + half);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = bf2f(m[k]) > 0.f ? f2bf(sum[k]) : (bf16)0.f;
    }
    *reinterpret_cast<bf16x4*>(t.e + (r / 2) * t.eS + half) = o;
}

// R rows of a wave's column x from row y, an even one where 2 x 2 pixels are asked for. POST:
// a.post is set.
template <int R, int NH, bool POST>
__device__ __forceinline__ void conv_rows_store(const ConvArgs& a, const f32x4 (&acc)[R][NH],
                                                const float (&bias)[4 * NH], int n, int img, int y, int x)
{
    if (x >= a.W) return;
    if (a.mode == 2) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (y + r < a.H) conv_planes<NH>(a, acc[r], bias, n, img, y + r, x);
        return;
    }
    if constexpr (NH == 2) {
        const ConvPlace<POST> t(a, n, img, y, x);
        const bool pairs = POST && (a.post == kPostPool || (a.post == kPostSum && n < a.eN));
#pragma unroll
        for (int r = 0; r < R; r += 2) {
            if (y + r >= a.H) break;
            const bf16x8 v0 = conv_value(a, acc[r], bias), v1 = conv_value(a, acc[r + 1], bias);
            conv_pixel<POST>(a, t, r, n, v0);
            if (y + r + 1 < a.H) conv_pixel<POST>(a, t, r + 1, n, v1);
            if constexpr (POST)
                if (pairs) conv_pair(a, t, r, x & 1, v0, v1);
        }
    }
}

// Chunk-outermost order. A workgroup owns a block of 16 PX x R PY pixels of one image and
// 32 CW channels (CW x PX x PY waves); a wave owns 16 columns x R rows and 32 channels (or,
// NH = 1, the first four of 32: the output layer). Per chunk the pixel block with its
// one-pixel halo is staged in LDS, and each wave holds the nine taps' weights in registers,
// loaded in fragment order straight from memory. It then goes down the R + 2 input rows:
// the three fragments of a row (one per dx) serve the up to three output rows that the row
// is a neighbour of, so a pixel is read from LDS 3 (R + 2)/R times per wave instead of
// nine, and the weights never pass through LDS (with both staged and read per tap, LDS
// reads took as long as the MFMAs). The next chunk's pixels are loaded into registers and
// its weights replaced tap row by tap row while the current chunk is multiplied.
// LDS: [pixel][32 channels], the four 16-byte octets of a pixel rotated by its column so
// that 16 neighbouring pixels cover all banks.
template <int R, int CW, int PX, int PY, int NH, bool ONE, bool POST>
__global__ void __launch_bounds__(64 * CW * PX * PY) k_conv_rows(const ConvArgs a)
{
    constexpr int NT = 64 * CW * PX * PY, HX = 16 * PX + 2, HY = R * PY + 2, NPIX = HX * HY;
    constexpr int NA = (NPIX * 4 + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) bf16 sa[ONE ? 1 : 2][NPIX * kKChunk];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % CW, wx = (wave / CW) % PX, wy = wave / (CW * PX);
    const int nbx = (a.W + 16 * PX - 1) / (16 * PX), nby = (a.H + R * PY - 1) / (R * PY);
    const int bx = blockIdx.x % nbx, by = (blockIdx.x / nbx) % nby, img = blockIdx.x / (nbx * nby);
    const int x0 = bx * 16 * PX, y0 = by * R * PY;
    const int r16 = lane & 15, g = lane >> 4;
    const int nch = ONE ? 1 : a.Cin / kKChunk;
    // the pixels this thread stages (octet tid % 4 of each; -1: outside the image, zero)
    const bf16* xi = a.x + (size_t)img * a.H * a.W * a.xC + a.xoff + 8 * (tid & 3);
    int so[NA];
    unsigned dst[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int t = tid + NT * i, px = t >> 2, oct = t & 3;
        const int hy = px / HX, hx = px - hy * HX, sy = y0 + hy - 1, sx = x0 + hx - 1;
        so[i] = t < NPIX * 4 && oct < a.octs && sy >= 0 && sy < a.H && sx >= 0 && sx < a.W ? sy * a.W + sx : -1;
        dst[i] = t < NPIX * 4 ? (unsigned)(px * kKChunk + ((oct ^ ((hx >> 2) & 3)) << 3)) : ~0u;
    }
    const bf16x8 zero = {};
    bf16x8 ra[NA];
    auto fetch = [&](int c) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            ra[i] = so[i] >= 0 ? *reinterpret_cast<const bf16x8*>(xi + (size_t)so[i] * a.xC + c * kKChunk) : zero;
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if (dst[i] != ~0u) *reinterpret_cast<bf16x8*>(&sa[buf][dst[i]]) = ra[i];
    };
    const bf16* wp = a.w + (size_t)(blockIdx.y * CW + cw) * nch * kChunkW + lane * 8;
    bf16x8 w[3][3][NH];
    auto weights = [&](int c, int dy) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int h = 0; h < NH; ++h)
                w[dy][dx][h] =
                    *reinterpret_cast<const bf16x8*>(wp + (size_t)c * kChunkW + ((dy * 3 + dx) * 2 + h) * kFrag);
    };
    // LDS element of this lane's pixel in the wave's first input row, per dx
    unsigned base[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int hx = wx * 16 + r16 + dx;
        base[dx] = (unsigned)((wy * R * HX + hx) * kKChunk + ((g ^ ((hx >> 2) & 3)) << 3));
    }
    f32x4 acc[R][NH];
#pragma unroll
    for (int o = 0; o < R; ++o)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[o][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) weights(0, dy);
    const int n0 = (blockIdx.y * CW + cw) * 32 + 8 * g;
    float bias[4 * NH];
    if (ONE) conv_bias<NH>(a, n0, bias);   // with more chunks the registers are worth more than the wait
    put(0);
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const bool more = !ONE && c + 1 < nch;
        const bf16* s = sa[ONE ? 0 : c & 1];
        if (more) fetch(c + 1);
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            bf16x8 v[3];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) v[dx] = *reinterpret_cast<const bf16x8*>(&s[base[dx] + r * HX * kKChunk]);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int o = r - dy;
                    if (o < 0 || o >= R) continue;
#pragma unroll
                    for (int h = 0; h < NH; ++h)
                        acc[o][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[dy][dx][h], v[dx], acc[o][h], 0, 0, 0);
                }
            // tap row dy has served its last input row r = R - 1 + dy
            if (more && r >= R - 1) weights(c + 1, r - (R - 1));
        }
        if (more) {
            put((c + 1) & 1);
            __syncthreads();
        }
    }
    const int xx = x0 + wx * 16 + r16;
    if (!ONE) conv_bias<NH>(a, n0, bias);
    conv_rows_store<R, NH, POST>(a, acc, bias, n0, img, y0 + wy * R, xx);
}

// Tap-outermost order on a staged tile. The pixel block of a workgroup (16 columns x R PY rows
// of one image, with its halo) is staged in LDS with all its input channels, so each tap
// reads it there at an offset instead of fetching it again; a wave owns 16 columns x R
// rows and 32 channels. A step is one tap of one chunk; the weights lie in the order of the
// steps and come from memory 2 U steps ahead, the pixels of the next step are read while
// one is multiplied. U divides the chunks, so U steps share a tap and everything that depends
// on the tap is decided between groups of U: with a decision per step its branches and the
// exposed LDS read took three times the MFMAs' time. 16 images of 24 x 20, 384 -> 128
// channels: 27 us, 42 with every tap's pixels from memory.
// LDS: [chunk][pixel][32 channels], octets rotated as in k_conv_rows.
template <int R, int CW, int PY, int NH, int U, bool POST>
__global__ void __launch_bounds__(64 * CW * PY) k_conv_tile(const ConvArgs a)
{
    constexpr int NT = 64 * CW * PY, HX = 18, HY = R * PY + 2, NPIX = HX * HY;
    extern __shared__ __attribute__((aligned(16))) bf16 st[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), cw = wave % CW, wy = wave / CW;
    const int nbx = (a.W + 15) / 16, nby = (a.H + R * PY - 1) / (R * PY);
    const int bx = blockIdx.x % nbx, by = (blockIdx.x / nbx) % nby, img = blockIdx.x / (nbx * nby);
    const int x0 = bx * 16, y0 = by * R * PY;
    const int r16 = lane & 15, g = lane >> 4;
    const int nch = a.Cin / kKChunk, steps = 9 * nch;
    const bf16* wp = a.w + (size_t)(blockIdx.y * CW + cw) * nch * kChunkW + lane * 8;
    bf16x8 w[2 * U][NH];
    auto weights = [&](int d, int s) {   // past the last step: the last again
#pragma unroll
        for (int h = 0; h < NH; ++h)
            w[d][h] = *reinterpret_cast<const bf16x8*>(wp + (size_t)min(s, steps - 1) * (2 * kFrag) + h * kFrag);
    };
#pragma unroll
    for (int d = 0; d < 2 * U; ++d) weights(d, d);
    // stage: octets of a pixel are neighbouring threads; whole chunks of a pixel one after the other
    const bf16* xi = a.x + (size_t)img * a.H * a.W * a.xC + a.xoff;
    const int octs = a.octs, per = 4 * nch;
    const bf16x8 zero = {};
    for (int t = tid; t < NPIX * per; t += NT) {
        const int px = t / per, o = t - px * per, c = o >> 2, oct = o & 3;
        const int hy = px / HX, hx = px - hy * HX, sy = y0 + hy - 1, sx = x0 + hx - 1;
        const bool in = o < octs && sy >= 0 && sy < a.H && sx >= 0 && sx < a.W;
        *reinterpret_cast<bf16x8*>(&st[(c * NPIX + px) * kKChunk + ((oct ^ ((hx >> 2) & 3)) << 3)]) =
            in ? *reinterpret_cast<const bf16x8*>(xi + (size_t)(sy * a.W + sx) * a.xC + 8 * o) : zero;
    }
    unsigned base[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int hx = r16 + dx;
        base[dx] = (unsigned)((wy * R * HX + hx) * kKChunk + ((g ^ ((hx >> 2) & 3)) << 3));
    }
    // first pixel of the group that starts with chunk c of tap (dy, dx)
    int dy = 0, dx = 0, c = 0;
    auto group = [&]() {
        return st + (c * NPIX + dy * HX) * kKChunk + (dx == 0 ? base[0] : dx == 1 ? base[1] : base[2]);
    };
    auto turn = [&]() {
        c += U;
        if (c == nch) {
            c = 0;
            if (++dx == 3) {
                dx = 0;
                if (++dy == 3) dy = 0;   // past the last step: the first again
            }
        }
    };
    bf16x8 v[2][R];
    auto pixels = [&](int d, const bf16* p) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[d][r] = *reinterpret_cast<const bf16x8*>(p + r * HX * kKChunk);
    };
    f32x4 acc[R][NH];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[r][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int n0 = (blockIdx.y * CW + cw) * 32 + 8 * g;
    float bias[4 * NH];
    conv_bias<NH>(a, n0, bias);
    __syncthreads();
    const bf16* p = group();
    pixels(0, p);
    for (int s = 0; s < steps; s += 2 * U) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half == 1 && s + U >= steps) break;
            turn();
            const bf16* next = group();
#pragma unroll
            for (int d = half * U; d < (half + 1) * U; ++d) {
                const int k = d - half * U + 1;
                pixels((d + 1) & 1, k < U ? p + k * NPIX * kKChunk : next);
                __builtin_amdgcn_sched_barrier(0);   // the reads stay ahead of the multiply
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int h = 0; h < NH; ++h)
                        acc[r][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[d][h], v[d & 1][r], acc[r][h], 0, 0, 0);
                weights(d, s + d + 2 * U);
                __builtin_amdgcn_sched_barrier(0);
            }
            p = next;
        }
    }
    const int xx = x0 + r16;
    conv_rows_store<R, NH, POST>(a, acc, bias, n0, img, y0 + wy * R, xx);
}

// Tap-outermost order where there is too little work for tiles, or a tile with all its
// channels does not fit in LDS. A wave owns MP blocks of 16 consecutive pixels (of the whole
// batch) and 32 channels, and its operands come from memory, D steps ahead: bound by the
// latency of those loads (four 32 x 32 images, the six layers at 8 x 8 and 4 x 4: 7 to 21 us
// each; loaded in the step that multiplies them, 62 us on average).
template <int MP, int NH>
__global__ void __launch_bounds__(256) k_conv_taps(const ConvArgs a)
{
    constexpr int D = MP == 1 ? 9 : 3;   // divides the number of steps
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int HW = a.H * a.W, nch = a.Cin / kKChunk, steps = 9 * nch;
    const int groups = (a.N + 31) / 32;
    // waves of a workgroup: neighbouring channel groups first (they share the pixels)
    const int id = blockIdx.x * 4 + wave, ng = id % groups;
    const int p0 = id / groups * 16 * MP;
    if (p0 >= a.P) return;
    int py[MP], px[MP];
    const bf16* xb[MP];
#pragma unroll
    for (int j = 0; j < MP; ++j) {
        const int p = min(p0 + 16 * j + r16, a.P - 1);
        const int img = p / HW, rem = p - img * HW;
        py[j] = rem / a.W;
        px[j] = rem - py[j] * a.W;
        xb[j] = a.x + (size_t)p * a.xC + a.xoff + (g < a.octs ? 8 * g : 0);
    }
    const bf16x8 zero = {};
    const bf16* wp = a.w + (size_t)ng * nch * kChunkW + lane * 8;
    bf16x8 va[D][MP], vw[D][NH];
    bool in[D][MP];
    int ls = 0, ly = 0, lx = 0, lc = 0;   // next step to load: its tap (row, column) and chunk
    auto load = [&](int d) {
        const int dy = ly - 1, dx = lx - 1;
#pragma unroll
        for (int j = 0; j < MP; ++j) {
            in[d][j] = g < a.octs && (unsigned)(py[j] + dy) < (unsigned)a.H && (unsigned)(px[j] + dx) < (unsigned)a.W;
            // a source outside the image is replaced by the pixel itself and not used
            const int off = in[d][j] ? (dy * a.W + dx) * a.xC : 0;
            va[d][j] = *reinterpret_cast<const bf16x8*>(xb[j] + off + lc * kKChunk);
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
            vw[d][h] = *reinterpret_cast<const bf16x8*>(wp + (size_t)min(ls, steps - 1) * (2 * kFrag) + h * kFrag);
        ++ls;
        const bool turn = ++lc == nch;   // past the last step the first again
        lc = turn ? 0 : lc;
        lx += turn;
        const bool down = lx == 3;
        lx = down ? 0 : lx;
        ly += down;
        ly = ly == 3 ? 0 : ly;
    };
    f32x4 acc[MP][NH];
#pragma unroll
    for (int j = 0; j < MP; ++j)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[j][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d) load(d);
    float bias[4 * NH];
    conv_bias<NH>(a, ng * 32 + 8 * g, bias);
    for (int s = 0; s < steps; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
#pragma unroll
            for (int j = 0; j < MP; ++j) {
                const bf16x8 v = in[d][j] ? va[d][j] : zero;
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    acc[j][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vw[d][h], v, acc[j][h], 0, 0, 0);
            }
            load(d);
        }
    }
#pragma unroll
    for (int j = 0; j < MP; ++j) {
        const int p = p0 + 16 * j + r16;
        if (p >= a.P) continue;
        const int img = p / HW, rem = p - img * HW, y = rem / a.W;
        const int n = ng * 32 + 8 * g, x = rem - y * a.W;
        if (a.mode == 2) {
            conv_planes<NH>(a, acc[j], bias, n, img, y, x);
        } else if constexpr (NH == 2) {
            const ConvPlace<MP == 1> t(a, n, img, y, x);
            conv_pixel<MP == 1>(a, t, 0, n, conv_value(a, acc[j], bias));
        }
    }
}

// All layers' weights from the canonical FP32 vector into the fragments of both directions
// in one launch. A workgroup takes 32 x 32 channels with their taps: rows of 288 consecutive
// floats, read once and written from LDS as lanes' eight elements of either direction (read
// element by element where they are needed, a cache line each, 1.9 million weights took
// 22 us). Elements outside a layer's real sizes are zero. The input gradient's weights are the
// transposed, flipped kernel: output channel = input channel of the layer, tap 8 - tap.
struct PrepLayer {
    size_t woff;
    bf16 *wf, *wb;
    int cin, cout, chunks_f, chunks_b;
    int taps;     // the tap is the outer index, not the chunk
    int first;    // index of the layer's first block
};
constexpr int kPrepMax = 16;
struct PrepTable {
    PrepLayer l[kPrepMax];
    int layers, total;
};

static __global__ void __launch_bounds__(256) k_weight_prep(const float* __restrict__ params, const PrepTable t)
{
    constexpr int kRow = 288 + 1;
    __shared__ float w[32 * kRow];
    int li = 0;
    while (li + 1 < t.layers && (int)blockIdx.x >= t.l[li + 1].first) ++li;
    const PrepLayer& L = t.l[li];
    const int blk = blockIdx.x - L.first, cb = blk / L.chunks_f, c = blk - cb * L.chunks_f, tid = threadIdx.x;
    const float* W = params + L.woff;
    const int cout = L.cout, len = L.cin * 9;
    float v[36];
#pragma unroll
    for (int u = 0; u < 36; ++u) {   // all in flight: one after the other they are the kernel's time
        const int k = tid + 256 * u, row = k / 288, co = cb * 32 + row, at = c * 288 + k - row * 288;
        v[u] = co < cout && at < len ? W[(size_t)co * len + at] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 36; ++u) {
        const int k = tid + 256 * u, row = k / 288;
        w[row * kRow + k - row * 288] = v[u];
    }
    __syncthreads();
    for (int k = tid; k < 2 * 9 * 128; k += 256) {
        const bool back = k >= 9 * 128;
        if (back && !L.wb) break;
        const int lane = k & 63, h = (k >> 6) & 1, tap = (k >> 7) % 9;
        const int i = lane & 15, n = 8 * (i >> 2) + 4 * h + (i & 3), k0 = 8 * (lane >> 4);
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            o[j] = f2bf(back ? w[(k0 + j) * kRow + n * 9 + 8 - tap] : w[n * kRow + (k0 + j) * 9 + tap]);
        const int chunks = back ? L.chunks_b : L.chunks_f, chunk = back ? cb : c, grp = back ? c : cb;
        const int step = L.taps ? tap * chunks + chunk : chunk * 9 + tap;
        *reinterpret_cast<bf16x8*>((back ? L.wb : L.wf)
                                   + ((((size_t)grp * 9 * chunks + step) * 2 + h) * 64 + lane) * 8) = o;
    }
}

}  // namespace clbm
