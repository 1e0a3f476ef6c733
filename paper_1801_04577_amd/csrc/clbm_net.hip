// clbm_net.hip -- the warm-start network on gfx950: a four-level convolutional
// encoder-decoder with skip connections, trained and run by the library's own
// kernels. 3x3 convolutions are implicit GEMMs on BF16 MFMA
// (v_mfma_f32_16x16x32_bf16) with FP32 accumulation; activations and activation
// gradients are BF16 in NHWC layout, master weights, weight gradients and the Adam
// state are FP32.
//
// Layer order (15 convolutions, widths w1..w4, input planes cin, output fields cout):
//   0: cin->w1   1: w1->w1 (= s1)                       at H x W
//   2: w1->w2    3: w2->w2 (= s2)      after avg-pool   at H/2
//   4: w2->w3    5: w3->w3 (= s3)      after avg-pool   at H/4
//   6: w3->w4    7: w4->w4             after avg-pool   at H/8
//   8: (w4+w3)->w3  9: w3->w3   on concat[up(h), s3]    at H/4
//  10: (w3+w2)->w2 11: w2->w2   on concat[up(h), s2]    at H/2
//  12: (w2+w1)->w1 13: w1->w1   on concat[up(h), s1]    at H
//  14: w1->cout (no activation)
// Every convolution but the last is followed by ReLU. The concatenations are free:
// the skip tensor is written straight into the upper channel range of the buffer the
// decoder reads. The canonical parameter vector stores, per layer in this order,
// W[cout][cin][3][3] then b[cout] (FP32).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <new>
#include <vector>

#include "clbm_conv.h"
#include "clbm_host.h"
#include "clbm_wgrad.h"

namespace clbm {

constexpr int kLayers = 15;

// fp32 NCHW input planes -> bf16 NHWC, channels padded to whole octets with zeros. A thread
// writes one octet of one pixel; neighbouring threads read neighbouring pixels of a plane.
__global__ void __launch_bounds__(256) k_pack_input(const float* __restrict__ xin, int Cin, int HW, int P,
                                                    bf16* __restrict__ x, int xC)
{
    const int p = blockIdx.x * 256 + threadIdx.x, c0 = blockIdx.y * 8;
    if (p >= P) return;
    const int b = p / HW, r = p - b * HW;
    bf16x8 o;
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = f2bf(c0 + c < Cin ? xin[((size_t)b * Cin + c0 + c) * HW + r] : 0.f);
    *reinterpret_cast<bf16x8*>(x + (size_t)p * xC + c0) = o;
}

// 2x2 average pooling of a channel view, for the layers whose epilogue cannot (ConvPost).
// A thread handles eight channels of one pixel.
__global__ void __launch_bounds__(256) k_avgpool(const bf16* __restrict__ x, int xC, int C, int H, int W, int B,
                                                 bf16* __restrict__ y, int yC)
{
    const int Ho = H / 2, Wo = W / 2, CV = C / 8;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= B * Ho * Wo * CV) return;
    const int c = (k % CV) * 8, p = k / CV;
    const int b = p / (Ho * Wo), r = p - b * Ho * Wo, oy = r / Wo, ox = r - oy * Wo;
    const bf16* src = x + ((size_t)b * H * W + (2 * oy) * W + 2 * ox) * xC + c;
    bf16x8 v[4], o;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const bf16x8*>(src + (size_t)((i >> 1) * W + (i & 1)) * xC);
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = f2bf(0.25f * (bf2f(v[0][i]) + bf2f(v[1][i]) + bf2f(v[2][i]) + bf2f(v[3][i])));
    *reinterpret_cast<bf16x8*>(y + (size_t)p * yC + c) = o;
}

// Gradient through the nearest upsampling and the ReLU before it, likewise: 2x2 sums of dy
// (2H x 2W), zero where the upsampled activation a (2H x 2W) is not positive.
__global__ void __launch_bounds__(256) k_upsample_bwd(const bf16* __restrict__ dy, int dyC, int C, int H, int W, int B,
                                                      const bf16* __restrict__ a, int aC, bf16* __restrict__ dz, int zC)
{
    const int Wi = 2 * W, CV = C / 8;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= B * H * W * CV) return;
    const int c = (k % CV) * 8, p = k / CV;
    const int b = p / (H * W), r = p - b * H * W, oy = r / W, ox = r - oy * W;
    const size_t at = (size_t)b * 4 * H * W + (2 * oy) * Wi + 2 * ox;
    const bf16x8 m = *reinterpret_cast<const bf16x8*>(a + at * aC + c);
    bf16x8 v[4], o;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const bf16x8*>(dy + (at + (i >> 1) * Wi + (i & 1)) * dyC + c);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        o[i] = bf2f(m[i]) > 0.f ? f2bf(bf2f(v[0][i]) + bf2f(v[1][i]) + bf2f(v[2][i]) + bf2f(v[3][i])) : (bf16)0.f;
    *reinterpret_cast<bf16x8*>(dz + (size_t)p * zC + c) = o;
}

// Mean squared error: dy = 2 (y - t)/n into a bf16 NHWC buffer (channels padded to whole
// octets with zeros), per-block sums of (y - t)^2 in FP64. A thread takes whole pixels, so
// the planes are read along their rows and an octet is one store; at most kMseBlocks partial
// sums are left, in a fixed order (one block per 256 elements left 65 536 for one workgroup
// to add: 56 + 65 us at batch 32 on 128^2, now 8.5 + 4.7).
constexpr int kMseBlocks = 1024;

__device__ __forceinline__ double block_sum_256(double s, double* lds)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

__global__ void __launch_bounds__(256) k_mse(const float* __restrict__ yv, const float* __restrict__ t,
                                             int Cout, int HW, int P, int zC, double inv_n,
                                             bf16* __restrict__ dz, double* __restrict__ part)
{
    __shared__ double lds[4];
    double s = 0.0;
    for (int p = blockIdx.x * 256 + threadIdx.x; p < P; p += gridDim.x * 256) {
        const int b = p / HW, r = p - b * HW;
        for (int c0 = 0; c0 < zC; c0 += 8) {
            bf16x8 o;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float g = 0.f;
                if (c0 + c < Cout) {
                    const size_t i = ((size_t)b * Cout + c0 + c) * HW + r;
                    const double d = (double)yv[i] - (double)t[i];
                    s += d * d;
                    g = (float)(2.0 * d * inv_n);
                }
                o[c] = f2bf(g);
            }
            *reinterpret_cast<bf16x8*>(dz + (size_t)p * zC + c0) = o;
        }
    }
    s = block_sum_256(s, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_sum_d(const double* __restrict__ part, int n, double* __restrict__ out)
{
    __shared__ double lds[4];
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += 256) s += part[k];
    s = block_sum_256(s, lds);
    if (threadIdx.x == 0) *out = s;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.f - b1) * gk;
    const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// Bilinear resampling of nf fields [nf][sh][sw] onto [nf][dh][dw] (cell-centred grids,
// edge values held), dst = scale[f] * value + shift[f].
struct FieldAffine {
    float scale[16], shift[16];
};

// A thread takes V neighbouring cells of one field: one row for all of them, one store. Bound
// by its launch and one chain of loads: 32 lattices of three fields 128^2 onto 512^2 take 127 us,
// 160 with a cell per thread.
template <int V>
__global__ void __launch_bounds__(256) k_resample(const float* __restrict__ src, int sh, int sw, float* __restrict__ dst,
                                                  int dh, int dw, FieldAffine af)
{
    const int per = dw / V, k = blockIdx.x * 256 + threadIdx.x, f = blockIdx.y;
    if (k >= dh * per) return;
    const int y = k / per, x = (k - y * per) * V;
    const float fy = fminf(fmaxf((y + 0.5f) * sh / dh - 0.5f, 0.f), (float)(sh - 1));
    const int y0 = (int)fy, y1 = min(y0 + 1, sh - 1);
    const float ty = fy - y0;
    int x0[V], x1[V];
    float tx[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const float fx = fminf(fmaxf((x + i + 0.5f) * sw / dw - 0.5f, 0.f), (float)(sw - 1));
        x0[i] = (int)fx;
        x1[i] = min(x0[i] + 1, sw - 1);
        tx[i] = fx - x0[i];
    }
    const float* s = src + (size_t)f * sh * sw;
    float o[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const float v = (1.f - ty) * ((1.f - tx[i]) * s[y0 * sw + x0[i]] + tx[i] * s[y0 * sw + x1[i]]) +
                        ty * ((1.f - tx[i]) * s[y1 * sw + x0[i]] + tx[i] * s[y1 * sw + x1[i]]);
        o[i] = af.scale[f] * v + af.shift[f];
    }
    float* to = dst + ((size_t)f * dh + y) * dw + x;
    if constexpr (V == 4) *reinterpret_cast<f32x4*>(to) = f32x4{o[0], o[1], o[2], o[3]};
    else to[0] = o[0];
}

// Input planes of the warm-start network for one problem per sample (see
// clbm_net_features in include/clbm.h for the channel list).
__global__ void k_features(const clbm_problem_code* __restrict__ codes, int B, int H, int W,
                           float* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= B * H * W) return;
    const int b = k / (H * W), r = k - b * H * W, y = r / W, x = r - y * W;
    const clbm_problem_code c = codes[b];
    // boundary cells of the network grid, side order x-, x+, y-, y+
    const bool at[4] = {x == 0, x == W - 1, y == 0, y == H - 1};
    float tw = 0.f, dir = 0.f, neu = 0.f;
    for (int s = 0; s < 4; ++s) {
        if (!at[s]) continue;
        if (c.kind[s] == 1) { dir = 1.f; tw = c.theta_wall[s]; }
        if (c.kind[s] == 2) neu = 1.f;
    }
    float* o = out + (size_t)b * 8 * H * W + r;
    const size_t pl = (size_t)H * W;
    o[0] = (c.log10_ra - 4.5f) / 1.5f;
    o[pl] = (c.pr - 3.85f) / 3.15f;
    o[2 * pl] = c.q_star / 4.f;
    o[3 * pl] = tw;
    o[4 * pl] = dir;
    o[5 * pl] = neu;
    o[6 * pl] = 2.f * (x + 0.5f) / W - 1.f;
    o[7 * pl] = c.log2_aspect;
}

}  // namespace clbm

using namespace clbm;

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

namespace {

struct TView {
    bf16* p;
    int C;    // channel stride
    int off;  // channel offset
};

struct Layer {
    int cin, cout;       // real sizes
    int cin_pad;         // K channels (multiple of 32)
    int cout_kpad;       // K channels of the input-gradient convolution (multiple of 32)
    int H, W;            // resolution it runs at
    size_t woff, boff;   // offsets of W and b in the canonical vector
    bf16* wf;
    bf16* wb;
    TView in, out;       // forward input and output views
    TView dz;            // gradient w.r.t. the pre-activation (and output) of the layer
    TView din;           // gradient w.r.t. the input (nullptr p for layer 0)
};

int round_up(int v, int a) { return (v + a - 1) / a * a; }

}  // namespace

struct clbm_net {
    clbm_net_desc d;
    hipStream_t stream;
    Layer L[kLayers];
    size_t nparams;
    float *params, *grads, *adam_m, *adam_v;
    float* wpart;      // weight-gradient split partials
    size_t wpart_floats;
    float* bpart;      // bias-gradient partials
    double* lpart;     // loss partials
    double* loss;
    bf16* xin;         // packed input (cin padded to whole octets)
    float* yout;       // network output fp32 NCHW
    bf16* dyout;       // loss gradient (cout padded to whole octets)
    // activations
    bf16 *a1, *cat1, *p1, *a2, *cat2, *p2, *a3, *cat3, *p3, *a4, *d3a, *d2a, *d1a, *d1b;
    // activation gradients
    bf16 *g_d1b, *g_d1a, *g_cat1, *g_d2b, *g_d2a, *g_cat2, *g_d3b, *g_d3a, *g_cat3, *g_m4, *g_a4,
        *g_a3, *g_a2, *g_a1, *g_z;  // g_z: scratch for dz of the current layer
    size_t zscratch;
    int weights_stale;
};

namespace {

struct Alloc {
    char* base;
    size_t off;
    bool dry;
    template <typename T>
    T* take(size_t count)
    {
        const size_t o = off;
        off = align_up(off + count * sizeof(T), kAlign);
        return dry ? nullptr : reinterpret_cast<T*>(base + o);
    }
};

clbm_status check_desc(const clbm_net_desc* d)
{
    if (!d) return CLBM_ERR_INVALID_ARG;
    if (d->batch < 1 || d->cin < 1 || d->cin > 32 || d->cout < 1 || d->cout > 16)
        return CLBM_ERR_INVALID_ARG;
    if (d->height < 16 || d->width < 16 || d->height % 8 || d->width % 8) return CLBM_ERR_INVALID_ARG;
    // the coarsest level must hold whole 64-pixel tiles
    if (((long)d->batch * (d->height / 8) * (d->width / 8)) % 64 != 0) return CLBM_ERR_INVALID_ARG;
    for (int k = 0; k < 4; ++k)
        if (d->widths[k] < 32 || d->widths[k] % 32) return CLBM_ERR_INVALID_ARG;
    return CLBM_OK;
}

// Lays out every buffer; with a.dry only counts bytes.
void layout_net(clbm_net* n, Alloc& a)
{
    const clbm_net_desc& d = n->d;
    const int B = d.batch, H = d.height, W = d.width;
    const int w1 = d.widths[0], w2 = d.widths[1], w3 = d.widths[2], w4 = d.widths[3];
    const size_t P1 = (size_t)B * H * W, P2 = P1 / 4, P3 = P1 / 16, P4 = P1 / 64;
    const int cinp = round_up(d.cin, 8), coutp = round_up(d.cout, 8);
    // activations (input and output gradient hold whole octets of channels)
    n->xin = a.take<bf16>(P1 * cinp);
    n->a1 = a.take<bf16>(P1 * w1);
    n->cat1 = a.take<bf16>(P1 * (w2 + w1));
    n->p1 = a.take<bf16>(P2 * w1);
    n->a2 = a.take<bf16>(P2 * w2);
    n->cat2 = a.take<bf16>(P2 * (w3 + w2));
    n->p2 = a.take<bf16>(P3 * w2);
    n->a3 = a.take<bf16>(P3 * w3);
    n->cat3 = a.take<bf16>(P3 * (w4 + w3));
    n->p3 = a.take<bf16>(P4 * w3);
    n->a4 = a.take<bf16>(P4 * w4);
    n->d3a = a.take<bf16>(P3 * w3);
    n->d2a = a.take<bf16>(P2 * w2);
    n->d1a = a.take<bf16>(P1 * w1);
    n->d1b = a.take<bf16>(P1 * w1);
    n->yout = a.take<float>(P1 * d.cout);
    n->dyout = a.take<bf16>(P1 * coutp);
    // gradients
    n->g_d1b = a.take<bf16>(P1 * w1);
    n->g_d1a = a.take<bf16>(P1 * w1);
    n->g_cat1 = a.take<bf16>(P1 * (w2 + w1));
    n->g_d2b = a.take<bf16>(P2 * w2);
    n->g_d2a = a.take<bf16>(P2 * w2);
    n->g_cat2 = a.take<bf16>(P2 * (w3 + w2));
    n->g_d3b = a.take<bf16>(P3 * w3);
    n->g_d3a = a.take<bf16>(P3 * w3);
    n->g_cat3 = a.take<bf16>(P3 * (w4 + w3));
    n->g_m4 = a.take<bf16>(P4 * w4);
    n->g_a4 = a.take<bf16>(P4 * w4);
    n->g_a3 = a.take<bf16>(P3 * w3);
    n->g_a2 = a.take<bf16>(P2 * w2);
    n->g_a1 = a.take<bf16>(P1 * w1);
    const size_t zmax = std::max({P1 * (size_t)w1, P2 * (size_t)w2, P3 * (size_t)w3, P4 * (size_t)w4});
    n->zscratch = zmax;
    n->g_z = a.take<bf16>(zmax);

    // layers
    const int cin_[kLayers] = {d.cin, w1, w1, w2, w2, w3, w3, w4, w4 + w3, w3, w3 + w2, w2, w2 + w1, w1, w1};
    const int cout_[kLayers] = {w1, w1, w2, w2, w3, w3, w4, w4, w3, w3, w2, w2, w1, w1, d.cout};
    const int res_[kLayers] = {1, 1, 2, 2, 4, 4, 8, 8, 4, 4, 2, 2, 1, 1, 1};
    size_t off = 0;
    for (int k = 0; k < kLayers; ++k) {
        Layer& l = n->L[k];
        l.cin = cin_[k];
        l.cout = cout_[k];
        l.cin_pad = round_up(l.cin, 32);
        l.cout_kpad = round_up(l.cout, 32);
        l.H = H / res_[k];
        l.W = W / res_[k];
        l.woff = off;
        off += (size_t)l.cout * l.cin * 9;
        l.boff = off;
        off += l.cout;
        l.wf = a.take<bf16>((size_t)l.cout_kpad * 9 * l.cin_pad);
        l.wb = k == 0 ? nullptr : a.take<bf16>((size_t)l.cin_pad * 9 * l.cout_kpad);
    }
    n->nparams = off;
    n->params = a.take<float>(off);
    n->grads = a.take<float>(off);
    n->adam_m = a.take<float>(off);
    n->adam_v = a.take<float>(off);
    // split-K partials of the weight and bias gradients
    size_t wp = 0, bp = 0;
    for (int k = 0; k < kLayers; ++k) {
        const Layer& l = n->L[k];
        const size_t P = (size_t)B * l.H * l.W, pixels = wgrad_pixels_per_split(P, l.cout, l.cin_pad);
        const size_t splits = (P + pixels - 1) / pixels;
        wp = std::max(wp, splits * l.cout_kpad * 9 * l.cin_pad);
        bp = std::max(bp, splits * l.cout_kpad);
    }
    n->wpart_floats = wp;
    n->wpart = a.take<float>(wp);
    n->bpart = a.take<float>(bp);
    n->lpart = a.take<double>(kMseBlocks);
    n->loss = a.take<double>(1);

    // views: forward input/output of each layer
    auto V = [](bf16* p, int C, int off) { return TView{p, C, off}; };
    Layer* L = n->L;
    L[0].in = V(n->xin, cinp, 0);      L[0].out = V(n->a1, w1, 0);
    L[1].in = V(n->a1, w1, 0);         L[1].out = V(n->cat1, w2 + w1, w2);   // s1
    L[2].in = V(n->p1, w1, 0);         L[2].out = V(n->a2, w2, 0);
    L[3].in = V(n->a2, w2, 0);         L[3].out = V(n->cat2, w3 + w2, w3);   // s2
    L[4].in = V(n->p2, w2, 0);         L[4].out = V(n->a3, w3, 0);
    L[5].in = V(n->a3, w3, 0);         L[5].out = V(n->cat3, w4 + w3, w4);   // s3
    L[6].in = V(n->p3, w3, 0);         L[6].out = V(n->a4, w4, 0);
    L[7].in = V(n->a4, w4, 0);
    L[8].in = V(n->cat3, w4 + w3, 0);  L[8].out = V(n->d3a, w3, 0);
    L[9].in = V(n->d3a, w3, 0);
    L[10].in = V(n->cat2, w3 + w2, 0); L[10].out = V(n->d2a, w2, 0);
    L[11].in = V(n->d2a, w2, 0);
    L[12].in = V(n->cat1, w2 + w1, 0); L[12].out = V(n->d1a, w1, 0);
    L[13].in = V(n->d1a, w1, 0);       L[13].out = V(n->d1b, w1, 0);
    L[14].in = V(n->d1b, w1, 0);       L[14].out = V(nullptr, 0, 0);
    // gradient w.r.t. each layer's input
    L[0].din = V(nullptr, 0, 0);
    L[1].din = V(n->g_a1, w1, 0);
    L[3].din = V(n->g_a2, w2, 0);
    L[5].din = V(n->g_a3, w3, 0);
    L[7].din = V(n->g_a4, w4, 0);
    L[8].din = V(n->g_cat3, w4 + w3, 0);
    L[9].din = V(n->g_d3a, w3, 0);
    L[10].din = V(n->g_cat2, w3 + w2, 0);
    L[11].din = V(n->g_d2a, w2, 0);
    L[12].din = V(n->g_cat1, w2 + w1, 0);
    L[13].din = V(n->g_d1a, w1, 0);
    L[14].din = V(n->g_d1b, w1, 0);
}

dim3 grid1(size_t n, int block = 256) { return dim3((unsigned)((n + block - 1) / block)); }

clbm_status pool(clbm_net* n, TView x, int C, int H, int W, TView y)
{
    const int B = n->d.batch;
    hipLaunchKernelGGL(k_avgpool, grid1((size_t)B * (H / 2) * (W / 2) * (C / 8)), dim3(256), 0, n->stream,
                       x.p + x.off, x.C, C, H, W, B, y.p + y.off, y.C);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

// dy and the activations act are 2H x 2W, dz is H x W.
clbm_status upsample_bwd(clbm_net* n, TView dy, int C, int H, int W, TView act, TView dz)
{
    const int B = n->d.batch;
    hipLaunchKernelGGL(k_upsample_bwd, grid1((size_t)B * H * W * (C / 8)), dim3(256), 0, n->stream, dy.p + dy.off,
                       dy.C, C, H, W, B, act.p + act.off, act.C, dz.p + dz.off, dz.C);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

template <int R, int CW, int PX, int PY, int NH, bool POST = false>
clbm_status launch_rows(clbm_net* n, const ConvArgs& a)
{
    if constexpr (NH == 2 && !POST)
        if (a.post) return launch_rows<R, CW, PX, PY, NH, true>(n, a);
    const int B = a.P / (a.H * a.W);
    const size_t blocks = (size_t)((a.W + 16 * PX - 1) / (16 * PX)) * ((a.H + R * PY - 1) / (R * PY)) * B;
    const dim3 grid((unsigned)blocks, (a.N + 32 * CW - 1) / (32 * CW)), block(64 * CW * PX * PY);
    if (a.Cin == kKChunk) hipLaunchKernelGGL((k_conv_rows<R, CW, PX, PY, NH, true, POST>), grid, block, 0, n->stream, a);
    else hipLaunchKernelGGL((k_conv_rows<R, CW, PX, PY, NH, false, POST>), grid, block, 0, n->stream, a);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

template <int MP, int NH>
clbm_status launch_taps(clbm_net* n, const ConvArgs& a)
{
    const int waves = (a.P + 16 * MP - 1) / (16 * MP) * ((a.N + 31) / 32);
    hipLaunchKernelGGL((k_conv_taps<MP, NH>), dim3((waves + 3) / 4), dim3(256), 0, n->stream, a);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

template <int R, int CW, int PY, int NH, bool POST = false>
clbm_status launch_tile(clbm_net* n, const ConvArgs& a)
{
    if constexpr (NH == 2 && !POST)
        if (a.post) return launch_tile<R, CW, PY, NH, true>(n, a);
    const int B = a.P / (a.H * a.W);
    const size_t blocks = (size_t)((a.W + 15) / 16) * ((a.H + R * PY - 1) / (R * PY)) * B;
    const dim3 grid((unsigned)blocks, (a.N + 32 * CW - 1) / (32 * CW)), block(64 * CW * PY);
    const size_t lds = (size_t)18 * (R * PY + 2) * a.Cin * sizeof(bf16);
    const int nch = a.Cin / kKChunk;
    if (nch % 4 == 0) hipLaunchKernelGGL((k_conv_tile<R, CW, PY, NH, 4, POST>), grid, block, lds, n->stream, a);
    else if (nch % 3 == 0) hipLaunchKernelGGL((k_conv_tile<R, CW, PY, NH, 3, POST>), grid, block, lds, n->stream, a);
    else if (nch % 2 == 0) hipLaunchKernelGGL((k_conv_tile<R, CW, PY, NH, 2, POST>), grid, block, lds, n->stream, a);
    else hipLaunchKernelGGL((k_conv_tile<R, CW, PY, NH, 1, POST>), grid, block, lds, n->stream, a);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

// Whether a layer accumulates with the chunk outermost: images that 256-pixel blocks of 64,
// 32 or 16 columns tile. The order fixes the rounding of every output, so it depends on
// the image alone. One chunk gives both orders the same.
bool chunk_order(int H, int W)
{
    const int bw = W >= 64 ? 64 : W;
    return (bw == 64 || bw == 32 || bw == 16) && W % bw == 0 && H % (256 / bw) == 0;
}

struct Post {
    int kind;        // ConvPost
    TView e, e2;
    int n;
};
constexpr TView kNoView{nullptr, 0, 0};
constexpr Post kNoPost{kPostNone, kNoView, kNoView, 0};

clbm_status conv_launch(clbm_net* n, const Layer& l, TView in, int cin_pad, const bf16* w, const float* bias, int N,
                        int mode, TView out, float* yf, float* yf2, TView mask, const Post& post)
{
    ConvArgs a;
    a.x = in.p;
    a.xC = in.C;
    a.xoff = in.off;
    a.Cin = cin_pad;
    a.octs = in.C < cin_pad ? in.C / 8 : cin_pad / 8;
    a.w = w;
    a.bias = bias;
    a.N = N;
    a.H = l.H;
    a.W = l.W;
    a.P = n->d.batch * l.H * l.W;
    a.mode = mode;
    a.y = out.p;
    a.yC = out.C;
    a.yoff = out.off;
    a.yf = yf;
    a.mask = mask.p ? mask.p + mask.off : nullptr;
    a.maskC = mask.C;
    a.yf2 = yf2;
    a.post = post.kind;
    a.e = post.e.p ? post.e.p + post.e.off : nullptr;
    a.eC = post.e.C;
    a.eN = post.n;
    a.e2 = post.e2.p ? post.e2.p + post.e2.off : nullptr;
    a.e2C = post.e2.C;
    // 16-pixel waves hold no 2 x 2 pixels
    auto taps = [&](bool big) {
        const int kind = a.post;
        if (kind == kPostPool || kind == kPostSum) a.post = kPostNone;
        if (kind == kPostSum) a.mask = nullptr;
        const clbm_status st = big && !a.post ? launch_taps<4, 2>(n, a) : launch_taps<1, 2>(n, a);
        if (st == CLBM_OK && kind == kPostPool) return pool(n, out, N, l.H, l.W, post.e);
        if (st == CLBM_OK && kind == kPostSum) return upsample_bwd(n, out, post.n, l.H / 2, l.W / 2, mask, post.e);
        return st;
    };
    const bool one = cin_pad == kKChunk;
    if (mode == 2) {
        // the output layer: at most 16 channels, in one group; the first four need one row block
        if (one && a.W >= 16) return N <= 4 ? launch_rows<4, 1, 2, 2, 1>(n, a) : launch_rows<4, 1, 2, 2, 2>(n, a);
        if (18 * 10 * a.Cin * 2 <= 160 * 1024) return N <= 4 ? launch_tile<4, 1, 2, 1>(n, a) : launch_tile<4, 1, 2, 2>(n, a);
        return N <= 4 ? launch_taps<4, 1>(n, a) : launch_taps<4, 2>(n, a);
    }
    const int groups = N / 32;
    if ((one && a.W >= 16) || chunk_order(a.H, a.W)) {
        const bool narrow = a.W <= 16;
        // eight rows per wave where that still gives every SIMD two waves
        const size_t waves8 = (size_t)a.P / 128 * groups;
        const bool tall = waves8 >= 2048;
        if (groups % 4 == 0) return tall ? launch_rows<8, 4, 1, 1, 2>(n, a) : launch_rows<4, 4, 1, 1, 2>(n, a);
        if (groups % 2 == 0) {
            if (narrow) return tall ? launch_rows<8, 2, 1, 2, 2>(n, a) : launch_rows<4, 2, 1, 2, 2>(n, a);
            return tall ? launch_rows<8, 2, 2, 1, 2>(n, a) : launch_rows<4, 2, 2, 1, 2>(n, a);
        }
        return narrow ? launch_rows<4, 1, 1, 4, 2>(n, a) : launch_rows<4, 1, 2, 2, 2>(n, a);
    }
    // Under 512 waves of tiles (half of the SIMDs) 16-pixel waves spread the layer further: four
    // 32 x 32 images, all six layers at 8 x 8 and 4 x 4: 73 us against 78 us; 16 images of
    // 24 x 20 (768 waves) already take 17.5 against 13.7 us.
    const size_t tile_waves = (size_t)((a.W + 15) / 16) * ((a.H + 3) / 4) * (a.P / (a.H * a.W)) * groups;
    if (tile_waves < 512) return taps(false);
    // tiles of four rows per wave, 18 x 6 (one wave down) or 18 x 10 (two) pixels with the halo,
    // within the 160 KB of LDS
    if (groups % 4 == 0 && 18 * 6 * a.Cin * 2 <= 160 * 1024) return launch_tile<4, 4, 1, 2>(n, a);
    if (groups % 2 == 0 && 18 * 10 * a.Cin * 2 <= 160 * 1024) return launch_tile<4, 2, 2, 2>(n, a);
    if (18 * 10 * a.Cin * 2 <= 160 * 1024) return launch_tile<4, 1, 2, 2>(n, a);
    return taps((size_t)a.P / 64 * groups >= 2048);
}

clbm_status prep_weights(clbm_net* n)
{
    PrepTable t;
    std::memset(&t, 0, sizeof t);
    t.layers = kLayers;
    for (int k = 0; k < kLayers; ++k) {
        const Layer& l = n->L[k];
        PrepLayer& p = t.l[k];
        p.woff = l.woff;
        p.wf = l.wf;
        p.wb = l.wb;
        p.cin = l.cin;
        p.cout = l.cout;
        // (the output layer sums taps outermost always; its input gradient has one chunk)
        p.taps = k == kLayers - 1 || !chunk_order(l.H, l.W);
        p.chunks_f = l.cin_pad / kKChunk;
        p.chunks_b = l.cout_kpad / kKChunk;
        p.first = t.total;
        t.total += l.cout_kpad / 32 * p.chunks_f;
    }
    hipLaunchKernelGGL(k_weight_prep, dim3(t.total), dim3(256), 0, n->stream, n->params, t);
    CLBM_HIP(hipGetLastError());
    n->weights_stale = 0;
    return CLBM_OK;
}

template <int NA, int RING, bool WIDE>
clbm_status wgrad_ring(clbm_net* n, const WgradArgs& g)
{
    const dim3 grid((g.splits + 7) / 8 * 8 * g.co_blocks * g.ci_blocks), block(192);
    if (g.W % 32 == 0)
        hipLaunchKernelGGL((k_wgrad<NA, RING, WIDE, true>), grid, block, 0, n->stream, g);
    else
        hipLaunchKernelGGL((k_wgrad<NA, RING, WIDE, false>), grid, block, 0, n->stream, g);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

template <int NA>
clbm_status wgrad_octets(clbm_net* n, const WgradArgs& g)
{
    const dim3 grid((g.splits + 7) / 8 * 8 * g.co_blocks * g.ci_blocks), block(384);
    hipLaunchKernelGGL((k_wgrad_octets<NA>), grid, block, OctetGeom<NA>::lds(g.W), n->stream, g);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

// Weight and bias gradients of a layer.
template <int NA>
clbm_status wgrad_launch(clbm_net* n, const Layer& l, TView dz)
{
    WgradArgs g;
    g.dz = dz.p;
    g.zC = dz.C;
    g.x = l.in.p;
    g.xC = l.in.C;
    g.xoff = l.in.off;
    g.zocts = dz.C < l.cout_kpad ? dz.C / 8 : l.cout_kpad / 8;
    g.xocts = l.in.C < l.cin_pad ? l.in.C / 8 : l.cin_pad / 8;
    g.H = l.H;
    g.W = l.W;
    g.P = n->d.batch * l.H * l.W;
    g.co_blocks = l.cout_kpad / (16 * NA);
    g.ci_blocks = l.cin_pad / 32;
    g.pixels = wgrad_pixels_per_split((size_t)g.P, l.cout, l.cin_pad);
    g.splits = (g.P + g.pixels - 1) / g.pixels;
    g.part = n->wpart;
    g.bpart = n->bpart;
    // the ring holds two rows and two steps: rows of up to 159 pixels in 512
    const int need = 2 * l.W + 2 + 2 * kWgStep;
    // one workgroup per CU at most: the latency of each counts, not the chip's LDS traffic
    const bool few = g.splits * g.co_blocks * g.ci_blocks <= 256;
    const clbm_status st = few && l.W % 8 == 0 && OctetGeom<NA>::lds(l.W) <= 160 * 1024 ? wgrad_octets<NA>(n, g)
                           : need <= 256                                            ? wgrad_ring<NA, 256, false>(n, g)
                           : need <= 512                                            ? wgrad_ring<NA, 512, false>(n, g)
                                                                                    : wgrad_ring<NA, 256, true>(n, g);
    if (st != CLBM_OK) return st;
    const size_t weights = (size_t)l.cout_kpad * 9 * l.cin_pad;
    hipLaunchKernelGGL(k_wgrad_reduce<NA>, dim3((unsigned)(weights / 64 + (l.cout_kpad + 63) / 64)), dim3(64), 0,
                       n->stream, n->wpart, n->bpart, g.splits, g.co_blocks, g.ci_blocks, l.cout, l.cin,
                       n->grads + l.woff, n->grads + l.boff);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

// Backward through one convolution: dz (gradient w.r.t. its output pre-activation,
// ReLU already applied) -> weight and bias gradients, and the input gradient when the
// layer has one, taken through the ReLU of the activations `mask` where that is given.
clbm_status conv_backward(clbm_net* n, int k, TView dz, TView mask = kNoView, const Post& post = kNoPost)
{
    const Layer& l = n->L[k];
    const clbm_status st = l.cout_kpad % 64 == 0 ? wgrad_launch<4>(n, l, dz) : wgrad_launch<2>(n, l, dz);
    if (st != CLBM_OK) return st;
    // input gradient: convolution of dz with the flipped, transposed kernel
    if (k == 0) return CLBM_OK;
    return conv_launch(n, l, dz, l.cout_kpad, l.wb, nullptr, l.cin, 1, l.din, nullptr, nullptr, mask, post);
}

}  // namespace

extern "C" {

clbm_status clbm_net_param_count(const clbm_net_desc* d, size_t* count)
{
    if (!count) return CLBM_ERR_INVALID_ARG;
    clbm_status st = check_desc(d);
    if (st != CLBM_OK) return st;
    clbm_net tmp;
    std::memset(&tmp, 0, sizeof tmp);
    tmp.d = *d;
    Alloc a{nullptr, 0, true};
    layout_net(&tmp, a);
    *count = tmp.nparams;
    return CLBM_OK;
}

clbm_status clbm_net_workspace_bytes(const clbm_net_desc* d, size_t* bytes)
{
    if (!bytes) return CLBM_ERR_INVALID_ARG;
    clbm_status st = check_desc(d);
    if (st != CLBM_OK) return st;
    clbm_net tmp;
    std::memset(&tmp, 0, sizeof tmp);
    tmp.d = *d;
    Alloc a{nullptr, 0, true};
    layout_net(&tmp, a);
    *bytes = a.off;
    return CLBM_OK;
}

clbm_status clbm_net_create(const clbm_net_desc* d, void* d_workspace, size_t bytes, void* hip_stream,
                            clbm_net** out)
{
    if (!out) return CLBM_ERR_INVALID_ARG;
    *out = nullptr;
    clbm_status st = check_desc(d);
    if (st != CLBM_OK) return st;
    size_t need = 0;
    clbm_net_workspace_bytes(d, &need);
    if (!d_workspace || ((uintptr_t)d_workspace) % kAlign) return CLBM_ERR_INVALID_ARG;
    if (bytes < need) return CLBM_ERR_BUFFER_TOO_SMALL;
    clbm_net* n = new (std::nothrow) clbm_net;
    if (!n) return CLBM_ERR_INVALID_ARG;
    std::memset(n, 0, sizeof *n);
    n->d = *d;
    n->stream = (hipStream_t)hip_stream;
    Alloc a{(char*)d_workspace, 0, false};
    layout_net(n, a);
    // zero everything once (padding channels must read as zeros), Adam moments included
    hipError_t e = hipMemsetAsync(d_workspace, 0, need, n->stream);
    if (e != hipSuccess) {
        delete n;
        set_last_hip_error(e, "hipMemsetAsync", __FILE__, __LINE__);
        return CLBM_ERR_HIP;
    }
    n->weights_stale = 1;
    *out = n;
    return CLBM_OK;
}

void clbm_net_destroy(clbm_net* n) { delete n; }

clbm_status clbm_net_set_params(clbm_net* n, const float* d_params)
{
    if (!n || !d_params) return CLBM_ERR_INVALID_ARG;
    CLBM_HIP(hipMemcpyAsync(n->params, d_params, n->nparams * sizeof(float), hipMemcpyDeviceToDevice,
                            n->stream));
    n->weights_stale = 1;
    return CLBM_OK;
}

clbm_status clbm_net_get_params(clbm_net* n, float* d_params)
{
    if (!n || !d_params) return CLBM_ERR_INVALID_ARG;
    CLBM_HIP(hipMemcpyAsync(d_params, n->params, n->nparams * sizeof(float), hipMemcpyDeviceToDevice,
                            n->stream));
    return CLBM_OK;
}

clbm_status clbm_net_get_grads(clbm_net* n, float* d_grads)
{
    if (!n || !d_grads) return CLBM_ERR_INVALID_ARG;
    CLBM_HIP(hipMemcpyAsync(d_grads, n->grads, n->nparams * sizeof(float), hipMemcpyDeviceToDevice,
                            n->stream));
    return CLBM_OK;
}

clbm_status clbm_net_forward(clbm_net* n, const float* d_x, float* d_y)
{
    if (!n || !d_x) return CLBM_ERR_INVALID_ARG;
    const clbm_net_desc& d = n->d;
    const int B = d.batch, H = d.height, W = d.width;
    const int w1 = d.widths[0], w2 = d.widths[1], w3 = d.widths[2], w4 = d.widths[3];
    clbm_status st = CLBM_OK;
    if (n->weights_stale && (st = prep_weights(n)) != CLBM_OK) return st;
    const int cinp = round_up(d.cin, 8);
    hipLaunchKernelGGL(k_pack_input, dim3((B * H * W + 255) / 256, cinp / 8), dim3(256), 0, n->stream, d_x, d.cin,
                       H * W, B * H * W, n->xin, cinp);
    CLBM_HIP(hipGetLastError());
    Layer* L = n->L;
    auto fwd = [&](int k, const Post& post = kNoPost) {
        const Layer& l = L[k];
        return conv_launch(n, l, l.in, l.cin_pad, l.wf, n->params + l.boff, l.cout, k == 14 ? 2 : 0, l.out,
                           k == 14 ? n->yout : nullptr, k == 14 ? d_y : nullptr, kNoView, post);
    };
    auto pooled = [&](bf16* p, int C) { return Post{kPostPool, TView{p, C, 0}, kNoView, 0}; };
    auto up = [&](bf16* p, int C) { return Post{kPostUp, TView{p, C, 0}, kNoView, 0}; };
    if ((st = fwd(0)) || (st = fwd(1, pooled(n->p1, w1)))) return st;
    if ((st = fwd(2)) || (st = fwd(3, pooled(n->p2, w2)))) return st;
    if ((st = fwd(4)) || (st = fwd(5, pooled(n->p3, w3)))) return st;
    if ((st = fwd(6)) || (st = fwd(7, up(n->cat3, w4 + w3)))) return st;
    if ((st = fwd(8)) || (st = fwd(9, up(n->cat2, w3 + w2)))) return st;
    if ((st = fwd(10)) || (st = fwd(11, up(n->cat1, w2 + w1)))) return st;
    if ((st = fwd(12)) || (st = fwd(13)) || (st = fwd(14))) return st;
    return CLBM_OK;
}

clbm_status clbm_net_backward(clbm_net* n, const float* d_target, double* loss)
{
    if (!n || !d_target) return CLBM_ERR_INVALID_ARG;
    const clbm_net_desc& d = n->d;
    const int B = d.batch, H = d.height, W = d.width;
    const int w1 = d.widths[0], w2 = d.widths[1], w3 = d.widths[2], w4 = d.widths[3];
    const int P1 = B * H * W;
    auto V = [](bf16* p, int C, int off) { return TView{p, C, off}; };
    clbm_status st = CLBM_OK;
    // loss and its gradient
    const int nblk = std::min((P1 + 255) / 256, kMseBlocks), coutp = round_up(d.cout, 8);
    hipLaunchKernelGGL(k_mse, dim3(nblk), dim3(256), 0, n->stream, n->yout, d_target, d.cout, H * W, P1, coutp,
                       1.0 / ((double)P1 * d.cout), n->dyout, n->lpart);
    CLBM_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_sum_d, dim3(1), dim3(256), 0, n->stream, n->lpart, nblk, n->loss);
    CLBM_HIP(hipGetLastError());
    auto zv = [&](int C) { return TView{n->g_z, C, 0}; };
    // output layer (no activation); each input gradient leaves its convolution as the gradient
    // before the ReLU of the layer below
    if ((st = conv_backward(n, 14, V(n->dyout, coutp, 0), V(n->d1b, w1, 0)))) return st;
    // decoder; the gradient of [up | skip] leaves the upsampled part as the gradient of the level
    // below, the skip's for the encoder
    auto sum = [&](bf16* dz, int C) { return Post{kPostSum, V(dz, C, 0), kNoView, C}; };
    auto cat = [&](bf16* p, int up, int skip) { return V(p, up + skip, 0); };
    if ((st = conv_backward(n, 13, V(n->g_d1b, w1, 0), V(n->d1a, w1, 0)))) return st;
    if ((st = conv_backward(n, 12, V(n->g_d1a, w1, 0), cat(n->cat1, w2, w1), sum(n->g_d2b, w2)))) return st;
    if ((st = conv_backward(n, 11, V(n->g_d2b, w2, 0), V(n->d2a, w2, 0)))) return st;
    if ((st = conv_backward(n, 10, V(n->g_d2a, w2, 0), cat(n->cat2, w3, w2), sum(n->g_d3b, w3)))) return st;
    if ((st = conv_backward(n, 9, V(n->g_d3b, w3, 0), V(n->d3a, w3, 0)))) return st;
    if ((st = conv_backward(n, 8, V(n->g_d3a, w3, 0), cat(n->cat3, w4, w3), sum(n->g_m4, w4)))) return st;
    // bottom level
    if ((st = conv_backward(n, 7, V(n->g_m4, w4, 0), V(n->a4, w4, 0)))) return st;
    // encoder: the pooled activations' gradient, with the skip's and through the ReLU to g_z
    auto unpool = [&](bf16* skip, int up, int C) { return Post{kPostUnpool, zv(C), V(skip, up + C, up), 0}; };
    if ((st = conv_backward(n, 6, V(n->g_a4, w4, 0), V(n->cat3, w4 + w3, w4), unpool(n->g_cat3, w4, w3)))) return st;
    if ((st = conv_backward(n, 5, zv(w3), V(n->a3, w3, 0)))) return st;
    if ((st = conv_backward(n, 4, V(n->g_a3, w3, 0), V(n->cat2, w3 + w2, w3), unpool(n->g_cat2, w3, w2)))) return st;
    if ((st = conv_backward(n, 3, zv(w2), V(n->a2, w2, 0)))) return st;
    if ((st = conv_backward(n, 2, V(n->g_a2, w2, 0), V(n->cat1, w2 + w1, w2), unpool(n->g_cat1, w2, w1)))) return st;
    if ((st = conv_backward(n, 1, zv(w1), V(n->a1, w1, 0)))) return st;
    if ((st = conv_backward(n, 0, V(n->g_a1, w1, 0)))) return st;
    if (loss) {
        double sum = 0.0;
        CLBM_HIP(hipMemcpyAsync(&sum, n->loss, sizeof(double), hipMemcpyDeviceToHost, n->stream));
        CLBM_HIP(hipStreamSynchronize(n->stream));
        *loss = sum / ((double)P1 * d.cout);
    }
    return CLBM_OK;
}

clbm_status clbm_net_adam(clbm_net* n, float lr, float beta1, float beta2, float eps, int t)
{
    if (!n || t < 1) return CLBM_ERR_INVALID_ARG;
    const float c1 = 1.f - std::pow(beta1, (float)t), c2 = 1.f - std::pow(beta2, (float)t);
    hipLaunchKernelGGL(k_adam, grid1(n->nparams), dim3(256), 0, n->stream, n->params, n->grads, n->adam_m,
                       n->adam_v, n->nparams, lr, beta1, beta2, eps, c1, c2);
    CLBM_HIP(hipGetLastError());
    n->weights_stale = 1;
    return CLBM_OK;
}

clbm_status clbm_resample_bilinear(const float* d_src, int sh, int sw, float* d_dst, int dh, int dw,
                                   int nfields, const float* scale, const float* shift,
                                   void* hip_stream)
{
    if (!d_src || !d_dst || sh < 1 || sw < 1 || dh < 1 || dw < 1 || nfields < 1 || nfields > 16)
        return CLBM_ERR_INVALID_ARG;
    FieldAffine af;
    for (int f = 0; f < 16; ++f) {
        af.scale[f] = (scale && f < nfields) ? scale[f] : 1.f;
        af.shift[f] = (shift && f < nfields) ? shift[f] : 0.f;
    }
    if (dw % 4 == 0 && (uintptr_t)d_dst % 16 == 0)
        hipLaunchKernelGGL(k_resample<4>, dim3(grid1((size_t)dh * (dw / 4)).x, nfields), dim3(256), 0, (hipStream_t)hip_stream,
                           d_src, sh, sw, d_dst, dh, dw, af);
    else
        hipLaunchKernelGGL(k_resample<1>, dim3(grid1((size_t)dh * dw).x, nfields), dim3(256), 0, (hipStream_t)hip_stream,
                           d_src, sh, sw, d_dst, dh, dw, af);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

clbm_status clbm_net_features(const clbm_problem_code* d_codes, int batch, int height, int width,
                              float* d_out, void* hip_stream)
{
    if (!d_codes || !d_out || batch < 1 || height < 1 || width < 1) return CLBM_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_features, grid1((size_t)batch * height * width), dim3(256), 0,
                       (hipStream_t)hip_stream, d_codes, batch, height, width, d_out);
    CLBM_HIP(hipGetLastError());
    return CLBM_OK;
}

clbm_status clbm_problem_encode(const clbm_params* p, clbm_problem_code* out)
{
    if (!p || !out) return CLBM_ERR_INVALID_ARG;
    Rates r;
    clbm_status st = derive_rates(p, &r);
    if (st != CLBM_OK) return st;
    // Sec. 3.3: the cavity height H = ny, dT = T(x-) - T(x+) of the Dirichlet side walls
    // (1 when they are not both Dirichlet); Ra = g beta dT H^3/(nu alpha), Pr = nu/alpha.
    const double H = p->ny;
    double dT = 1.0;
    if (p->side[0].kind == CLBM_WALL && p->side[1].kind == CLBM_WALL && p->side[0].b1 == 0.0 &&
        p->side[1].b1 == 0.0 && p->side[0].b2 != 0.0 && p->side[1].b2 != 0.0) {
        const double d = p->side[0].b3 / p->side[0].b2 - p->side[1].b3 / p->side[1].b2;
        if (d != 0.0) dT = std::fabs(d);
    }
    const double Ra = std::max(p->g_beta * dT * H * H * H / (p->nu * p->alpha), 1.0);
    std::memset(out, 0, sizeof *out);
    out->log10_ra = (float)std::log10(Ra);
    out->pr = (float)(p->nu / p->alpha);
    out->q_star = (float)(p->Q * H * H / (p->alpha * dT));
    out->log2_aspect = (float)std::log2((double)p->nx / p->ny);
    for (int s = 0; s < 4; ++s) {
        const clbm_side& sd = p->side[s];
        if (sd.kind != CLBM_WALL) {
            out->kind[s] = 0;
        } else if (sd.b1 == 0.0) {
            out->kind[s] = 1;
            out->theta_wall[s] = (float)((sd.b3 / sd.b2 - p->T0) / dT);
        } else {
            out->kind[s] = (sd.b2 == 0.0 && sd.b3 == 0.0) ? 2 : 3;
        }
    }
    out->u_scale = (float)std::sqrt(p->g_beta * dT * H);
    out->t_scale = (float)dT;
    return CLBM_OK;
}

}  // extern "C"
