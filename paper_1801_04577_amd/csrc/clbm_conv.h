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
// taps outermost (k_conv_taps).
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

// Weights of one direction of a layer as its convolution reads them: per group of 32 output
// channels, chunk of 32 input channels, tap and row block h one fragment of 1 KB, lane
// after lane. Row i of block h is channel 8 (i/4) + 4 h + i % 4 of the group.
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
    float* yf;
};

// Epilogue of one pixel: lane group g = lane / 16 holds channels n0 + 8 g .. + 7.
template <int NH>
__device__ __forceinline__ void conv_bias(const ConvArgs& a, int n, float (&bias)[4 * NH])
{
#pragma unroll
    for (int k = 0; k < 4 * NH; ++k) bias[k] = a.mode != 1 && n + k < a.N ? a.bias[n + k] : 0.f;
}

template <int NH>
__device__ __forceinline__ void conv_store(const ConvArgs& a, const f32x4 (&acc)[NH], const float (&bias)[4 * NH],
                                           int n, size_t p, int img, int rem)
{
    if (a.mode == 2) {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = n + 4 * h + v;
                if (c < a.N) a.yf[((size_t)img * a.N + c) * ((size_t)a.H * a.W) + rem] = acc[h][v] + bias[4 * h + v];
            }
        return;
    }
    if constexpr (NH == 2) {
        bf16x8 o;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float r = acc[h][v];
                if (a.mode == 0) r = fmaxf(r + bias[4 * h + v], 0.f);
                o[4 * h + v] = f2bf(r);
            }
        if (a.mask) {
            const bf16x8 m = *reinterpret_cast<const bf16x8*>(a.mask + p * a.maskC + n);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (!(bf2f(m[k]) > 0.f)) o[k] = (bf16)0.f;
        }
        *reinterpret_cast<bf16x8*>(a.y + p * a.yC + a.yoff + n) = o;
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
template <int R, int CW, int PX, int PY, int NH, bool ONE>
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
    if (xx >= a.W) return;
    if (!ONE) conv_bias<NH>(a, n0, bias);
#pragma unroll
    for (int o = 0; o < R; ++o) {
        const int yy = y0 + wy * R + o, rem = yy * a.W + xx;
        if (yy < a.H)
            conv_store<NH>(a, acc[o], bias, n0, (size_t)img * a.H * a.W + rem, img, rem);
    }
}

// Tap-outermost order, for images that k_conv_rows does not tile in its own order. A wave
// owns MP blocks of 16 consecutive pixels (of the whole batch) and NG groups of 32
// channels, its operands come from memory, and the fragments of the next D steps (a step
// is one tap of one chunk) are in flight while one is multiplied: with few waves per CU
// the time is otherwise the latency of every step's loads.
template <int MP, int NG, int NH>
__global__ void __launch_bounds__(256) k_conv_taps(const ConvArgs a)
{
    constexpr int D = 4;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int HW = a.H * a.W, nch = a.Cin / kKChunk, steps = 9 * nch;
    const int groups = (a.N + 32 * NG - 1) / (32 * NG);
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
    const bf16* wp = a.w + (size_t)ng * NG * nch * kChunkW + lane * 8;
    bf16x8 va[D][MP], vw[D][NG][NH];
    bool in[D][MP];
    int lt = 0, lc = 0;   // tap and chunk of the next step to load
    auto load = [&](int d) {
        const int dy = lt / 3 - 1, dx = lt % 3 - 1;
#pragma unroll
        for (int j = 0; j < MP; ++j) {
            in[d][j] = g < a.octs && (unsigned)(py[j] + dy) < (unsigned)a.H && (unsigned)(px[j] + dx) < (unsigned)a.W;
            // a source outside the image is replaced by the pixel itself and not used
            const int off = in[d][j] ? (dy * a.W + dx) * a.xC : 0;
            va[d][j] = *reinterpret_cast<const bf16x8*>(xb[j] + off + lc * kKChunk);
        }
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int h = 0; h < NH; ++h)
                vw[d][n][h] = *reinterpret_cast<const bf16x8*>(wp + (size_t)(n * nch + lc) * kChunkW
                                                               + (lt * 2 + h) * kFrag);
        if (++lc == nch) {
            lc = 0;
            ++lt;
        }
    };
    f32x4 acc[MP][NG][NH];
#pragma unroll
    for (int j = 0; j < MP; ++j)
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int h = 0; h < NH; ++h) acc[j][n][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < steps) load(d);
    float bias[NG][4 * NH];
#pragma unroll
    for (int n = 0; n < NG; ++n) conv_bias<NH>(a, (ng * NG + n) * 32 + 8 * g, bias[n]);
    for (int s = 0; s < steps; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (s + d >= steps) break;
#pragma unroll
            for (int j = 0; j < MP; ++j) {
                const bf16x8 v = in[d][j] ? va[d][j] : zero;
#pragma unroll
                for (int n = 0; n < NG; ++n)
#pragma unroll
                    for (int h = 0; h < NH; ++h)
                        acc[j][n][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vw[d][n][h], v, acc[j][n][h], 0, 0, 0);
            }
            if (s + d + D < steps) load(d);
        }
    }
#pragma unroll
    for (int j = 0; j < MP; ++j) {
        const int p = p0 + 16 * j + r16;
        if (p >= a.P) continue;
        const int img = p / HW;
#pragma unroll
        for (int n = 0; n < NG; ++n)
            if ((ng * NG + n) * 32 < a.N)
                conv_store<NH>(a, acc[j][n], bias[n], (ng * NG + n) * 32 + 8 * g, (size_t)p, img, p - img * HW);
    }
}

// All layers' weights from the canonical FP32 vector into the fragments of both directions
// in one launch; each thread writes one lane's eight elements. Elements outside a layer's
// real sizes are zero. The input gradient's weights are the transposed, flipped kernel:
// output channel = input channel of the layer, tap 8 - tap.
struct PrepLayer {
    size_t woff;
    bf16 *wf, *wb;
    int cin, cout, chunks_f, chunks_b;
    int first;    // index of the layer's first lane fragment
    int lanes_f;  // lane fragments of the forward direction
};
constexpr int kPrepMax = 16;
struct PrepTable {
    PrepLayer l[kPrepMax];
    int layers, total;
};

static __global__ void __launch_bounds__(256) k_weight_prep(const float* __restrict__ params, const PrepTable t)
{
    int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= t.total) return;
    int li = 0;
    while (li + 1 < t.layers && k >= t.l[li + 1].first) ++li;
    const PrepLayer& L = t.l[li];
    k -= L.first;
    const bool back = k >= L.lanes_f;
    if (back) k -= L.lanes_f;
    const int lane = k & 63, h = (k >> 6) & 1, rest = k >> 7;
    const int tap = rest % 9, chunks = back ? L.chunks_b : L.chunks_f;
    const int c = rest / 9 % chunks, grp = rest / 9 / chunks;
    const int i = lane & 15, n = grp * 32 + 8 * (i >> 2) + 4 * h + (i & 3), k0 = c * kKChunk + 8 * (lane >> 4);
    const float* W = params + L.woff;
    bf16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int co = back ? k0 + j : n, ci = back ? n : k0 + j, tp = back ? 8 - tap : tap;
        o[j] = f2bf(co < L.cout && ci < L.cin ? W[((size_t)co * L.cin + ci) * 9 + tp] : 0.f);
    }
    *reinterpret_cast<bf16x8*>((back ? L.wb : L.wf) + (size_t)k * 8) = o;
}

}  // namespace clbm
