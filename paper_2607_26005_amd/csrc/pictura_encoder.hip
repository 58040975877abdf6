// The policy's image encoder on rendered views (inference): five 3x3
// convolutions, one cross-attention block of 16 learned queries per camera, mean
// over the queries, projection.
//
// Activations are channel-last.  The convolutions after the first are implicit
// GEMMs on the bf16 matrix cores at fp32 accuracy: an fp32 value is cut into
// three bf16 parts of 8 significant bits each, which add up to it exactly, and
// a product of two such values is the sum of the six largest part products.
// With weights cut by truncation (second and third part below 2^-7 and 2^-15 of
// the value's power of two) and activations to the nearest (2^-8 and 2^-17, of
// either sign), the three left out are below 2^-22 of the product and mostly
// cancel in a sum.  Six bf16 products run 2.6 times as fast as one on the fp32
// matrix cores (2.5 PFLOP/s / 6 against 157 TFLOP/s).  Values are cut once,
// where they are produced, and stored as [pixel][channels / 32][3][32].
//
// Measured on 8,192 views of 96x54 of a town: 5.0 ms a call, 15.6 ms through
// PyTorch's layers (MIOpen's Winograd convolutions 8.1 ms, the planes, ReLUs and
// layout changes around them 6 ms, the attention 2 ms).  The error against the
// same encoder in fp64 is 2.7e-8, 3.1e-8 through the layers, and of the
// convolutions alone with positive weights 1.1e-7, 1.4e-7 through the layers.
// Kernels: first convolution 0.71 ms (2.0 GB written), then 0.98, 1.12, 0.68 and
// 1.00 ms (0.62, 1.09, 0.90 and 1.22 PFLOP/s of bf16 products; a large bf16 matrix
// product reaches 1.15 on this card), attention 0.39 ms, the rest 0.08 ms.
#include <cmath>

#include "pictura.h"
#include "pictura_internal.h"

#pragma clang fp contract(off)

namespace pictura {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kEmb = PICTURA_ENCODER_WIDTH;       // tokens, queries and the embedding of a camera
constexpr int kHeads = PICTURA_ENCODER_HEADS, kHeadDim = kEmb / kHeads;
constexpr int kQueries = PICTURA_ENCODER_QUERIES;
constexpr int kC1 = 32, kC2 = 64, kC3 = 64, kC4 = 128, kC5 = kEmb;
constexpr int kTaps = 9;
constexpr int kKC = 32;                           // input channels of one staged chunk

// n / d for n < 2^31 (see Div31)
__device__ __forceinline__ uint32_t div31(uint32_t n, Div31 d) { return d.m ? (__umulhi(n, d.m) >> d.s) : n; }

// A weight: x = hi + mid + lo exactly (each the leading 8 significant bits of what
// is left, by truncation, so no part overflows and all have x's sign); an
// infinity or NaN stays whole in hi.
__device__ __forceinline__ void split3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo)
{
    const uint32_t u = __float_as_uint(x);
    hi = u & 0xFFFF0000u;
    const bool fin = (u & 0x7F800000u) != 0x7F800000u;
    const float r = fin ? x - __uint_as_float(hi) : 0.0f;
    if (!fin && (u & 0x007FFFFFu)) hi |= 0x00400000u;   // a NaN whose payload sat in the cut bits
    mid = __float_as_uint(r) & 0xFFFF0000u;
    lo = __float_as_uint(r - __uint_as_float(mid)) & 0xFFFF0000u;
}

// Activations (0 or more, or NaN) are cut to the nearest instead: x0 and x1, packed
// in this order.  The second and third part then have either sign, so that what
// the products leave out does not add up.  The first part is held below
// infinity: of an infinity (or NaN) the second is one, and the third, the
// difference of the two, is held to a number that no finite value's reaches
// and that adds to the same side.  Without branches: with one per pair for
// such values the first convolution took 969 us instead of 711.
__device__ __forceinline__ void split3_pair(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    auto nearest = [](float a, float b) {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
    };
    auto first = [](uint32_t p) { return __uint_as_float(p << 16); };
    auto second = [](uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); };
    constexpr float kMost = 0x1.FEp127f;
    hi = nearest(fminf(x0, kMost), fminf(x1, kMost));
    const float r0 = x0 - first(hi), r1 = x1 - second(hi);
    mid = nearest(r0, r1);
    lo = nearest(fminf(r0 - first(mid), 0x1p112f), fminf(r1 - second(mid), 0x1p112f));
}

// ---------------------------------------------------------------------------
// weights in the kernels' layouts (every call: the caller may have changed them)
// ---------------------------------------------------------------------------

struct EncWeights {
    // caller's tensors
    const float* cw[5];
    const float* cb[5];
    const float* queries;
    const float* in_w; const float* in_b;
    const float* out_w; const float* out_b;
    const float* proj_w; const float* proj_b;
    int32_t cams, classes;
    // prepared
    float* table;          // [tap][classes + 1][32]: first convolution, the last plane that of the inverse depth
    uint16_t* wk[4];       // [tap][Cin / 32][3][Cout][32]: convolutions 2..5
    float* qk;             // [cams][heads][queries][kEmb]: query . key as a product with the token
    float* vt; float* ot; float* pt;   // value, output and final projections, transposed [in][out]
};

__device__ void prep_conv(const float* w, uint16_t* o, int cin, int cout, int64_t i)
{
    const int k = (int)(i % kKC);
    const int n = (int)(i / kKC % cout);
    const int ch = (int)(i / kKC / cout % (cin / kKC));
    const int tap = (int)(i / kKC / cout / (cin / kKC));
    uint32_t h, m, l;
    const float x = w[((int64_t)n * cin + ch * kKC + k) * kTaps + tap];
    split3(x, h, m, l);
    // An infinite pixel's second part is the infinite one; times a weight's second
    // part of zero it would be a NaN beside the infinite products.  Such a part takes
    // the least normal number, of the weight's sign (2^-126, below 2^-26 of any
    // weight it is added to).
    if (fabsf(x) >= 0x1p-100f && fabsf(x) < INFINITY && !(m << 1)) m = (h & 0x80000000u) | 0x00800000u;
    uint16_t* b = o + ((int64_t)(tap * (cin / kKC) + ch) * 3 * cout + n) * kKC + k;
    b[0] = (uint16_t)(h >> 16);
    b[(int64_t)cout * kKC] = (uint16_t)(m >> 16);
    b[(int64_t)2 * cout * kKC] = (uint16_t)(l >> 16);
}

__global__ __launch_bounds__(256) void enc_prep_kernel(const EncWeights W)
{
    constexpr int kCin[4] = {kC1, kC2, kC3, kC4}, kCout[4] = {kC2, kC3, kC4, kC5};
    __shared__ float qv[kQueries][kHeadDim];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < W.cams * kHeads) {
        // q = queries Wq^T + bq; its product with a key, scaled, is a product with
        // the token: (q_h / sqrt(d)) . (Wk_h t) = (Wk_h^T q_h / sqrt(d)) . t.  The
        // keys' bias adds the same to every token's score, which the softmax drops.
        const int cam = blockIdx.x / kHeads, h = blockIdx.x % kHeads;
        for (int i = tid; i < kQueries * kHeadDim; i += 256) {
            const int q = i / kHeadDim, c = h * kHeadDim + i % kHeadDim;
            const float* x = W.queries + ((int64_t)cam * kQueries + q) * kEmb;
            const float* y = W.in_w + (int64_t)c * kEmb;
            float s = 0.0f;
#pragma unroll 32
            for (int k = 0; k < kEmb; ++k) s = fmaf(x[k], y[k], s);
            qv[q][i % kHeadDim] = s + W.in_b[c];
        }
        __syncthreads();
        const float scale = 1.0f / sqrtf((float)kHeadDim);
        for (int i = tid; i < kQueries * kEmb; i += 256) {
            const int k = i % kEmb, q = i / kEmb;
            float s = 0.0f;
#pragma unroll
            for (int j = 0; j < kHeadDim; ++j) s = fmaf(qv[q][j], W.in_w[(int64_t)(kEmb + h * kHeadDim + j) * kEmb + k], s);
            W.qk[((int64_t)(cam * kHeads + h) * kQueries + q) * kEmb + k] = s * scale;
        }
        return;
    }
    const int64_t n0 = (int64_t)kTaps * (W.classes + 1) * kC1;
    const int64_t step = (int64_t)(gridDim.x - W.cams * kHeads) * 256;
    const int64_t first = (int64_t)(blockIdx.x - W.cams * kHeads) * 256 + tid;
    for (int64_t i = first; i < n0; i += step) {
        const int c = (int)(i % kC1), p = (int)(i / kC1 % (W.classes + 1)), tap = (int)(i / kC1 / (W.classes + 1));
        W.table[i] = W.cw[0][((int64_t)c * (W.classes + 1) + p) * kTaps + tap];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        for (int64_t i = first; i < (int64_t)kTaps * kCin[q] * kCout[q]; i += step)
            prep_conv(W.cw[q + 1], W.wk[q], kCin[q], kCout[q], i);
    for (int64_t i = first; i < (int64_t)kEmb * kEmb; i += step) {
        const int o = (int)(i % kEmb), k = (int)(i / kEmb);
        W.vt[i] = W.in_w[(int64_t)(2 * kEmb + o) * kEmb + k];
        W.ot[i] = W.out_w[(int64_t)o * kEmb + k];
        W.pt[i] = W.proj_w[(int64_t)o * kEmb + k];
    }
}

// ---------------------------------------------------------------------------
// first convolution, from the rendered images
// ---------------------------------------------------------------------------

// Its input planes (one per class, then 1 / depth) are never built: a tap adds
// the weights of its pixel's class and 1 / depth times the last plane's.  Four
// threads per output pixel, eight channels each; they share the set-up of the
// nine taps (three each, handed round the quad), since that and not the sums
// was most of the instructions.  Bound by the vector ALU and the stores of the
// output (six bytes a value).
template <int kLane>
__device__ __forceinline__ uint32_t quad_get(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kLane * 0x55, 0xf, 0xf, true);
}

__global__ __launch_bounds__(256) void enc_conv1_kernel(const uint8_t* __restrict__ cls, const float* __restrict__ depth,
                                                        const float* __restrict__ table, const float* __restrict__ bias,
                                                        int classes, int H, int W, int h, int w, Div31 by_hw,
                                                        Div31 by_w, int pixels, uint16_t* __restrict__ out)
{
    extern __shared__ float tb[];   // [tap][classes + 1][32]: the classes, then zeros (a class beyond the planes)
    const int rows = classes + 1;
    for (int i = threadIdx.x; i < kTaps * rows * kC1; i += 256)
        tb[i] = i / kC1 % rows < classes ? table[i] : 0.0f;
    __syncthreads();
    const int part = threadIdx.x & 3;
    float b[8], td[kTaps][8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        b[c] = bias[part * 8 + c];
#pragma unroll
        for (int t = 0; t < kTaps; ++t) td[t][c] = table[(t * rows + classes) * kC1 + part * 8 + c];
    }
    // (whole waves stay in the loop: one past the last pixel computes it again)
    __shared__ u32x4 sout[4][16 * 12];
    u32x4* const wave_out = sout[threadIdx.x >> 6];
    for (int px = blockIdx.x * 64 + (threadIdx.x >> 2); px - (int)(threadIdx.x >> 2 & 15) < pixels; px += gridDim.x * 64) {
        const int pc = min(px, pixels - 1), v = (int)div31((uint32_t)pc, by_hw);
        const int r = pc - v * (h * w), y = (int)div31((uint32_t)r, by_w), x = r - y * w;
        // taps part, part + 4 and 8: the class's row of the table and 1 / depth (outside the image: zeros and 0)
        uint32_t row[3], inv[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int t = s == 2 ? 8 : 4 * s + part;
            const int dy = (t * 11) >> 5, iy = 2 * y + dy - 1, ix = 2 * x + (t - 3 * dy) - 1;
            int k = classes;
            float n = 0.0f;
            if ((unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W) {
                const int64_t i = ((int64_t)v * H + iy) * W + ix;
                k = min((int)cls[i], classes);
                // correctly rounded, as the division: one Newton step with fused
                // residual where the hardware reciprocal's error allows it
                const float d = depth[i];
                n = __builtin_amdgcn_rcpf(d);
                if (d >= 0.000244140625f && d < 1048576.0f) n = fmaf(fmaf(-d, n, 1.0f), n, n);
                else if (d != INFINITY) n = 1.0f / d;
            }
            row[s] = (uint32_t)((t * rows + k) * kC1);
            inv[s] = __float_as_uint(n);
        }
        float acc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = b[c];
        auto tap = [&](int t, uint32_t ro, uint32_t in) {
            const float n = __uint_as_float(in);
            const f32x4* tc = (const f32x4*)&tb[ro + part * 8];
            const f32x4 c0 = tc[0], c1 = tc[1];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                acc[c] = fmaf(n, td[t][c], acc[c] + c0[c]);
                acc[4 + c] = fmaf(n, td[t][4 + c], acc[4 + c] + c1[c]);
            }
        };
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            tap(4 * s, quad_get<0>(row[s]), quad_get<0>(inv[s]));
            tap(4 * s + 1, quad_get<1>(row[s]), quad_get<1>(inv[s]));
            tap(4 * s + 2, quad_get<2>(row[s]), quad_get<2>(inv[s]));
            tap(4 * s + 3, quad_get<3>(row[s]), quad_get<3>(inv[s]));
        }
        tap(8, row[2], inv[2]);
        uint32_t parts[3][4];
#pragma unroll
        for (int c = 0; c < 8; c += 2)
            split3_pair(acc[c] < 0.0f ? 0.0f : acc[c], acc[c + 1] < 0.0f ? 0.0f : acc[c + 1], parts[0][c / 2],
                        parts[1][c / 2], parts[2][c / 2]);
        // through LDS, so that the wave's 16 pixels of 192 bytes leave as whole kilobytes
        u32x4* const row16 = wave_out + (threadIdx.x >> 2 & 15) * 12 + part;
#pragma unroll
        for (int q = 0; q < 3; ++q) row16[4 * q] = u32x4{parts[q][0], parts[q][1], parts[q][2], parts[q][3]};
        __builtin_amdgcn_wave_barrier();
        const int lane = threadIdx.x & 63, px0 = px - (lane >> 2);   // the wave's first pixel
        u32x4* const o = (u32x4*)out + (int64_t)px0 * 12;
#pragma unroll
        for (int s = 0; s < 3; ++s)
            if (px0 + (s * 64 + lane) / 12 < pixels) o[s * 64 + lane] = wave_out[s * 64 + lane];
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// 3x3 convolutions as implicit GEMMs
// ---------------------------------------------------------------------------

// A workgroup of four waves makes MT output pixels times all kCout channels, a
// wave 64 x 64 of them in 2 x 2 tiles of 32x32 (rows channels, columns pixels:
// a lane then holds four consecutive channels of a pixel).  K runs over the
// nine taps and kKC = 32 channels of one at a time; a chunk's pixels and
// weights (three parts each) are staged through LDS, the next chunk's loads
// in flight in registers meanwhile.  LDS rows are 64 bytes at a pitch of 80, so
// 16-byte reads of consecutive rows fall on distinct banks.  Two workgroups
// fit a CU (LDS, 256 registers a lane): one's staging hides behind the other's
// products.  Bound by the matrix cores and the LDS reads that feed them (12 of
// 16 bytes a lane for 24 products of 32 cycles).
constexpr int kRowBytes = 80;

// The products of a staged chunk: weight rows of this lane (parts kCout rows
// apart), and its two pixel rows (parts kARows rows apart).
template <int kCout, int kARows>
__device__ __forceinline__ void enc_products(const uint8_t* wrow, const uint8_t* prow0, const uint8_t* prow1, int lane,
                                             f32x16 (&acc)[2][2])
{
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int ko = ks * 32 + (lane >> 5) * 16;
        bf16x8 wf[2][3], pf[2][3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            wf[0][q] = *(const bf16x8*)(wrow + q * kCout * kRowBytes + ko);
            wf[1][q] = *(const bf16x8*)(wrow + (q * kCout + 32) * kRowBytes + ko);
            pf[0][q] = *(const bf16x8*)(prow0 + q * kARows * kRowBytes + ko);
            pf[1][q] = *(const bf16x8*)(prow1 + q * kARows * kRowBytes + ko);
        }
        // the smallest products first
        constexpr int kW[6] = {2, 0, 1, 1, 0, 0}, kP[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][kW[t]], pf[j][kP[t]], acc[i][j], 0, 0, 0);
    }
}

template <int kCout, int MT, bool kLast>
__device__ __forceinline__ void enc_store(f32x16 (&acc)[2][2], uint8_t* sA, const float* __restrict__ bias, int64_t p0,
                                          int64_t pixels, int wm, int wn, void* __restrict__ out)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // bias, ReLU (a NaN stays one); lane: pixel column lane & 31, channels 8 g + 4 (lane >> 5) .. + 3 of group g.
    // The parts of 32 channels go through the wave's share of LDS, so that the stores are whole rows of 192 bytes.
    constexpr int kOutPitch = 208;
    if constexpr (!kLast) __syncthreads();
    uint8_t* const so = sA + wid * 64 * kOutPitch;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = g * 8 + (lane >> 5) * 4, n = wn * 64 + i * 32 + c;
                const f32x4 b = *(const f32x4*)(bias + n);
                f32x4 x;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float s = acc[i][j][g * 4 + r] + b[r];
                    x[r] = s < 0.0f ? 0.0f : s;
                }
                if constexpr (kLast) {
                    const int64_t px = p0 + wm * 64 + j * 32 + (lane & 31);
                    if (px < pixels) *(f32x4*)((float*)out + px * kCout + n) = x;
                } else {
                    uint32_t w[6];
                    split3_pair(x[0], x[1], w[0], w[1], w[2]);
                    split3_pair(x[2], x[3], w[3], w[4], w[5]);
                    uint8_t* o = so + (j * 32 + (lane & 31)) * kOutPitch + c * 2;
                    *(u32x2*)o = u32x2{w[0], w[3]};
                    *(u32x2*)(o + 64) = u32x2{w[1], w[4]};
                    *(u32x2*)(o + 128) = u32x2{w[2], w[5]};
                }
            }
        if constexpr (!kLast) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = 0; s < 12; ++s) {
                const int q = s * 64 + lane, row = q / 12, at = q - row * 12;
                const int64_t px = p0 + wm * 64 + row;
                const u32x4 d = *(const u32x4*)(so + row * kOutPitch + at * 16);
                if (px < pixels) *((u32x4*)out + (px * (kCout / 32) + wn * 2 + i) * 12 + at) = d;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

template <int kCin, int kCout, int kStride, int MT, bool kLast>
__global__ __launch_bounds__(256, 2) void enc_conv_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ wk,
                                                          const float* __restrict__ bias, int hi, int wi, int h, int w,
                                                          int64_t pixels, void* __restrict__ out)
{
    constexpr int kWavesN = kCout / 64, kWavesM = 4 / kWavesN;
    static_assert(MT == 64 * kWavesM, "four waves of 64 x 64");
    constexpr int kSteps = kCin / kKC, kChunks = kTaps * kSteps;
    constexpr int kRows = MT / 64;                      // pixel rows a thread stages a 16-byte piece of, per part
    constexpr int kBLoads = kCout * 3 * 4 / 256;        // 16-byte weight pieces per thread
    constexpr int kABytes = 3 * MT * kRowBytes;
    constexpr int kLdsBytes = kABytes + 3 * kCout * kRowBytes;
    __shared__ __align__(16) uint8_t sA[kLdsBytes];
    uint8_t* const sB = sA + kABytes;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid % kWavesM, wn = wid / kWavesM;
    const int64_t p0 = (int64_t)blockIdx.x * MT;

    // the thread's pixel rows of a staged chunk: four lanes to a row's 64 bytes of a part
    const int piece = tid & 3;
    int iy0[kRows], ix0[kRows], pix0[kRows];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int64_t px = p0 + i * 64 + (tid >> 2);
        iy0[i] = ix0[i] = -4;   // (no tap of a row past the last pixel is inside)
        pix0[i] = 0;
        if (px < pixels) {
            const int v = (int)(px / (h * w)), r = (int)(px - (int64_t)v * (h * w)), y = r / w;
            iy0[i] = y * kStride - 1;
            ix0[i] = (r - y * w) * kStride - 1;
            pix0[i] = (v * hi + iy0[i]) * wi + ix0[i];
        }
    }
    u32x4 ra[3 * kRows], rb[kBLoads];
    auto fetch = [&](int ch) {
        const int tap = ch / kSteps, dy = tap / 3, dx = tap - 3 * dy;
        const u32x4* a = (const u32x4*)in + (ch - tap * kSteps) * 12 + piece;   // a pixel's chunk: 12 pieces
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int iy = iy0[i] + dy, ix = ix0[i] + dx;
            const bool ok = (unsigned)iy < (unsigned)hi && (unsigned)ix < (unsigned)wi;
            const u32x4* p = a + (int64_t)(pix0[i] + dy * wi + dx) * (12 * kSteps);
#pragma unroll
            for (int q = 0; q < 3; ++q) ra[i * 3 + q] = ok ? p[4 * q] : u32x4{0u, 0u, 0u, 0u};
        }
        const u32x4* b = (const u32x4*)(wk + (int64_t)ch * 3 * kCout * kKC);
#pragma unroll
        for (int s = 0; s < kBLoads; ++s) rb[s] = b[tid + 256 * s];
    };
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    fetch(0);
#pragma unroll 1
    for (int ch = 0; ch < kChunks; ++ch) {
        __syncthreads();   // the last chunk's reads are done
#pragma unroll
        for (int i = 0; i < kRows; ++i)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *(u32x4*)&sA[(q * MT + i * 64 + (tid >> 2)) * kRowBytes + piece * 16] = ra[i * 3 + q];
#pragma unroll
        for (int s = 0; s < kBLoads; ++s) {
            const int p = tid + 256 * s;
            *(u32x4*)&sB[(p >> 2) * kRowBytes + (p & 3) * 16] = rb[s];
        }
        __syncthreads();
        if (ch + 1 < kChunks) fetch(ch + 1);
        enc_products<kCout, MT>(sB + (wn * 64 + (lane & 31)) * kRowBytes, sA + (wm * 64 + (lane & 31)) * kRowBytes,
                                sA + (wm * 64 + 32 + (lane & 31)) * kRowBytes, lane, acc);
    }
    enc_store<kCout, MT, kLast>(acc, sA, bias, p0, pixels, wm, wn, out);
}

// The same with stride 1, where the three taps of a kernel row read the same
// pixels one apart: a row of MT + 2 consecutive pixels is staged once for the
// three (their weights one tap at a time), and a lane whose pixel has no
// neighbour there reads a row of zeros.  Staging is what holds the general
// kernel back: with 0.47 and 0.67 of its bytes the 64- and 128-channel
// convolutions of 8,192 views take 1.12 instead of 1.47 ms and 1.00 instead of
// 1.16.
template <int kCin, int kCout, int MT, bool kLast>
__global__ __launch_bounds__(256, 2) void enc_conv_s1_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ wk,
                                                             const float* __restrict__ bias, int h, int w, int64_t pixels,
                                                             void* __restrict__ out)
{
    constexpr int kWavesN = kCout / 64, kWavesM = 4 / kWavesN;
    static_assert(MT == 64 * kWavesM, "four waves of 64 x 64");
    constexpr int kSteps = kCin / kKC;
    constexpr int kRows = MT / 64, kARows = MT + 3;   // the last row is zero
    constexpr int kBLoads = kCout * 3 * 4 / 256;
    constexpr int kABytes = 3 * kARows * kRowBytes, kLdsBytes = kABytes + 3 * kCout * kRowBytes;
    __shared__ __align__(16) uint8_t sA[kLdsBytes];
    static_assert(kLast || 4 * 64 * 208 <= kLdsBytes, "output rows of four waves");
    uint8_t* const sB = sA + kABytes;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid % kWavesM, wn = wid / kWavesM;
    const int64_t p0 = (int64_t)blockIdx.x * MT;
    const int piece = tid & 3, hw = h * w;
    if (tid < 3 * kRowBytes / 16)
        *(u32x4*)&sA[((tid / 5) * kARows + kARows - 1) * kRowBytes + (tid % 5) * 16] = u32x4{0u, 0u, 0u, 0u};
    // this lane's two pixels: the taps that have a neighbour, a bit each
    uint32_t taps[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t px = p0 + wm * 64 + j * 32 + (lane & 31);
        taps[j] = 0;
        if (px < pixels) {
            const int r = (int)(px % hw), y = r / w, x = r - y * w;
#pragma unroll
            for (int t = 0; t < kTaps; ++t)
                if (y + t / 3 - 1 >= 0 && y + t / 3 - 1 < h && x + t % 3 - 1 >= 0 && x + t % 3 - 1 < w) taps[j] |= 1u << t;
        }
    }
    u32x4 ra[3 * kRows], rx[3], rb[kBLoads];
    // pixel rows of kernel row dy and chunk c; row r is pixel p0 - 1 + r + (dy - 1) w
    // (one outside the buffer is loaded from its end: no lane reads it)
    auto fetch_a = [&](int dy, int c) {
        const u32x4* a = (const u32x4*)in + c * 12 + piece;
        const int64_t q0 = p0 - 1 + (int64_t)(dy - 1) * w + (tid >> 2);
        auto at = [&](int64_t q) { return a + (q < 0 ? 0 : q < pixels ? q : pixels - 1) * (12 * kSteps); };
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const u32x4* p = at(q0 + i * 64);
#pragma unroll
            for (int q = 0; q < 3; ++q) ra[i * 3 + q] = p[4 * q];
        }
        if (tid < 8) {
            const u32x4* p = at(q0 + MT);
#pragma unroll
            for (int q = 0; q < 3; ++q) rx[q] = p[4 * q];
        }
    };
    auto fetch_b = [&](int tap, int c) {
        const u32x4* b = (const u32x4*)(wk + (int64_t)(tap * kSteps + c) * 3 * kCout * kKC);
#pragma unroll
        for (int s = 0; s < kBLoads; ++s) rb[s] = b[tid + 256 * s];
    };
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    fetch_a(0, 0);
    fetch_b(0, 0);
#pragma unroll 1
    for (int g = 0; g < 3 * kSteps; ++g) {   // kernel row and chunk
        const int dy = g / kSteps, c = g - dy * kSteps;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            __syncthreads();   // the last tap's reads are done
            if (dx == 0) {
#pragma unroll
                for (int i = 0; i < kRows; ++i)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        *(u32x4*)&sA[(q * kARows + i * 64 + (tid >> 2)) * kRowBytes + piece * 16] = ra[i * 3 + q];
                if (tid < 8) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        *(u32x4*)&sA[(q * kARows + MT + (tid >> 2)) * kRowBytes + piece * 16] = rx[q];
                }
            }
#pragma unroll
            for (int s = 0; s < kBLoads; ++s) {
                const int p = tid + 256 * s;
                *(u32x4*)&sB[(p >> 2) * kRowBytes + (p & 3) * 16] = rb[s];
            }
            __syncthreads();
            if (dx < 2) fetch_b(dy * 3 + dx + 1, c);
            else if (g + 1 < 3 * kSteps) fetch_b((g + 1) / kSteps * 3, (g + 1) % kSteps);
            if (dx == 0 && g + 1 < 3 * kSteps) fetch_a((g + 1) / kSteps, (g + 1) % kSteps);
            const int t = dy * 3 + dx, r0 = wm * 64 + (lane & 31) + dx;
            const int a0 = (taps[0] >> t) & 1u ? r0 : kARows - 1, a1 = (taps[1] >> t) & 1u ? r0 + 32 : kARows - 1;
            enc_products<kCout, kARows>(sB + (wn * 64 + (lane & 31)) * kRowBytes, sA + a0 * kRowBytes, sA + a1 * kRowBytes,
                                        lane, acc);
        }
    }
    enc_store<kCout, MT, kLast>(acc, sA, bias, p0, pixels, wm, wn, out);
}

// ---------------------------------------------------------------------------
// cross-attention, averaged over the queries
// ---------------------------------------------------------------------------

// One workgroup per view, a wave per head.  Only the mean over the queries of
// the attended values is used, and values are linear in the tokens, so a head's
// result is Wv_h applied to one weighted token average: keys, values and the
// per-query results are never formed.  Scores of 16 queries x 16 tokens come
// from the fp32 matrix cores (lane: column token lane & 15, and of each 16
// channels the four from 4 (lane >> 4) on).  The first pass over the tokens finds
// each query's maximum, the second its sum of exponentials, the third the
// tokens' mean weights and the average.  kStore: the scores wait in LDS between
// the passes (each lane its own, 16 bytes a lane and 16 tokens); without, for
// maps whose scores would take more than 64 KB (over 256 tokens), they are
// computed again (8,192 views of 84 tokens: 505 us that way).
template <bool kStore>
__global__ __launch_bounds__(256) void enc_attn_kernel(const float* __restrict__ tok, const float* __restrict__ qk,
                                                       int cams, int64_t v0, int n, float* __restrict__ pooled)
{
    const int lane = threadIdx.x & 63, head = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
    const int64_t v = blockIdx.x;
    const float* t0 = tok + v * n * kEmb;
    const float* q0 = qk + (((v0 + v) % cams * kHeads + head) * kQueries + c) * kEmb + g * 4;
    float qf[32];
#pragma unroll
    for (int k = 0; k < 32; k += 4) *(f32x4*)&qf[k] = *(const f32x4*)(q0 + 4 * k);
    float tf[32];
    auto load = [&](int b) {
        const float* t = t0 + (int64_t)min(b + c, n - 1) * kEmb + g * 4;
#pragma unroll
        for (int k = 0; k < 32; k += 4) *(f32x4*)&tf[k] = *(const f32x4*)(t + 4 * k);
    };
    auto scores = [&](int b) -> f32x4 {
        load(b);
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 32; ++k) s = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[k], tf[k], s, 0, 0, 0);
        return s;   // queries 4 g + r, token b + c
    };
    extern __shared__ f32x4 store[];   // [tile][thread]
    float mx[4], sum[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        mx[r] = -INFINITY;
        sum[r] = 0.0f;
    }
    for (int b = 0; b < n; b += 16) {
        const f32x4 s = scores(b);
        if constexpr (kStore) store[b * 16 + threadIdx.x] = s;
        // (a clamped lane repeats the last token: the same maximum)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[r] = fmaxf(mx[r], s[r]);
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[r] = fmaxf(mx[r], __shfl_xor(mx[r], d));
    for (int b = 0; b < n; b += 16) {
        f32x4 s;
        if constexpr (kStore) s = store[b * 16 + threadIdx.x];
        else s = scores(b);
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = expf(s[r] - mx[r]);
        if constexpr (kStore) store[b * 16 + threadIdx.x] = s;
        if (b + c < n) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += s[r];
        }
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] += __shfl_xor(sum[r], d);
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] = 1.0f / sum[r];
    float acc[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) acc[k] = 0.0f;
    for (int b = 0; b < n; b += 16) {
        f32x4 s;
        if constexpr (kStore) {
            s = store[b * 16 + threadIdx.x];
            load(b);
        } else {
            s = scores(b);
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = expf(s[r] - mx[r]);
        }
        float p = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) p = fmaf(s[r], sum[r], p);
        p += __shfl_xor(p, 16);
        p += __shfl_xor(p, 32);
        p = b + c < n ? p * (1.0f / kQueries) : 0.0f;
#pragma unroll
        for (int k = 0; k < 32; ++k) acc[k] = fmaf(p, tf[k], acc[k]);
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1)
#pragma unroll
        for (int k = 0; k < 32; ++k) acc[k] += __shfl_xor(acc[k], d);
    float* o = pooled + (v * kHeads + head) * kEmb + g * 4;
#pragma unroll
    for (int k = 0; k < 32; ++k)
        if ((k & 15) == c) o[(k >> 2) * 16 + (k & 3)] = acc[k];
}

// Values, output projection and final projection of 16 views per workgroup.  The
// sums are in fp64 (no time: 0.4 G products of a call of 8,192 views): their
// roundings would be most of the embedding's error.
constexpr int kTailViews = 16;
__global__ __launch_bounds__(256) void enc_tail_kernel(const EncWeights W, const float* __restrict__ pooled, int64_t views,
                                                       float* __restrict__ emb)
{
    __shared__ float sp[kTailViews][kHeads * kEmb];
    __shared__ float sx[2][kTailViews][kEmb];
    const int64_t v0 = (int64_t)blockIdx.x * kTailViews;
    const int nv = (int)min((int64_t)kTailViews, views - v0);
    for (int i = threadIdx.x; i < kTailViews * kHeads * kEmb; i += 256)
        sp[0][i] = i < nv * kHeads * kEmb ? pooled[v0 * kHeads * kEmb + i] : 0.0f;
    __syncthreads();
    const int c = threadIdx.x % kEmb, half = threadIdx.x / kEmb;   // channel, and views 8 half .. + 7
    const float* wt[3] = {W.vt, W.ot, W.pt};
    const float bias[3] = {W.in_b[2 * kEmb + c], W.out_b[c], W.proj_b[c]};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        double acc[8] = {};
#pragma unroll 4
        for (int k = 0; k < kEmb; ++k) {
            const double wv = (double)wt[l][k * kEmb + c];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int v = half * 8 + j;
                const float x = l == 0 ? sp[v][c / kHeadDim * kEmb + k] : sx[l - 1][v][k];
                acc[j] = fma(wv, (double)x, acc[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int v = half * 8 + j;
            const float y = (float)(acc[j] + (double)bias[l]);
            if (l < 2) sx[l][v][c] = y;
            else if (v < nv) emb[(v0 + v) * kEmb + c] = y;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------

namespace {

// Views encoded at a time: their activations (six bytes a value) stay near
// kActBytes, so a call's workspace is bounded whatever the number of views.
constexpr int64_t kActBytes = 3ll << 30;

struct EncPlan {
    int h[5], w[5];
    int64_t chunk;           // views at a time
    size_t off_table, off_wk[4], off_qk, off_vt, off_ot, off_pt, off_a, off_b, off_pool, total;
};

EncPlan enc_plan(const pictura_encoder& e, int64_t views, int H, int W)
{
    EncPlan p{};
    constexpr int st[5] = {2, 2, 1, 2, 1}, ch[6] = {0, kC1, kC2, kC3, kC4, kC5};
    for (int i = 0; i < 5; ++i) {
        p.h[i] = ((i ? p.h[i - 1] : H) - 1) / st[i] + 1;
        p.w[i] = ((i ? p.w[i - 1] : W) - 1) / st[i] + 1;
    }
    // x1, x3 and the tokens share one buffer, x2 and x4 the other
    int64_t a = 0, b = 0;
    for (int i = 0; i < 5; ++i) {
        const int64_t n = (int64_t)p.h[i] * p.w[i] * ch[i + 1] * (i == 4 ? 4 : 6);
        if (i & 1) b = n > b ? n : b;
        else a = n > a ? n : a;
    }
    int64_t chunk = kActBytes / (a + b);
    chunk = chunk < 1 ? 1 : chunk > views ? views : chunk;
    // equal chunks
    const int64_t nc = (views + chunk - 1) / chunk;
    p.chunk = nc > 0 ? (views + nc - 1) / nc : 0;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += (bytes + 255) & ~(size_t)255;
        return at;
    };
    p.off_table = take(sizeof(float) * kTaps * (e.num_classes + 1) * kC1);
    for (int i = 0; i < 4; ++i) p.off_wk[i] = take(sizeof(uint16_t) * 3 * kTaps * ch[i + 1] * ch[i + 2]);
    p.off_qk = take(sizeof(float) * (size_t)e.cams * kHeads * kQueries * kEmb);
    p.off_vt = take(sizeof(float) * kEmb * kEmb);
    p.off_ot = take(sizeof(float) * kEmb * kEmb);
    p.off_pt = take(sizeof(float) * kEmb * kEmb);
    p.off_a = take((size_t)(a * p.chunk));
    p.off_b = take((size_t)(b * p.chunk));
    p.off_pool = take(sizeof(float) * (size_t)p.chunk * kHeads * kEmb);
    p.total = o;
    return p;
}

pictura_status enc_check(const pictura_encoder* e, int64_t views, int32_t height, int32_t width)
{
    if (!e) return PICTURA_EINVAL;
    if (e->cams < 1 || e->cams > 4096 || e->num_classes < 1 || e->num_classes > PICTURA_ENCODER_MAX_CLASSES)
        return PICTURA_EINVAL;
    if (views < 0 || views > 0x7FFFFFFFll || height < 1 || width < 1 || height > 4096 || width > 4096) return PICTURA_EINVAL;
    return PICTURA_OK;
}

}  // namespace
}  // namespace pictura

using namespace pictura;

extern "C" {

pictura_status pictura_encoder_workspace(const pictura_encoder* e, int64_t views, int32_t height, int32_t width,
                                         uint64_t* bytes)
{
    const pictura_status st = enc_check(e, views, height, width);
    if (st != PICTURA_OK) return st;
    if (!bytes) return PICTURA_EINVAL;
    *bytes = (uint64_t)enc_plan(*e, views, height, width).total;
    return PICTURA_OK;
}

pictura_status pictura_encode_views(const pictura_encoder* e, const uint8_t* cls, const float* depth, int64_t views,
                                    int32_t height, int32_t width, void* workspace, uint64_t workspace_bytes,
                                    float* out, void* stream)
{
    pictura_status st = enc_check(e, views, height, width);
    if (st != PICTURA_OK) return st;
    if (views == 0) return PICTURA_OK;
    if (!cls || !depth || !workspace || !out) return PICTURA_EINVAL;
    for (int i = 0; i < 5; ++i)
        if (!e->conv_w[i] || !e->conv_b[i]) return PICTURA_EINVAL;
    if (!e->queries || !e->in_proj_w || !e->in_proj_b || !e->out_proj_w || !e->out_proj_b || !e->proj_w || !e->proj_b)
        return PICTURA_EINVAL;
    // 16-byte loads of the biases and of the workspace
    for (int i = 1; i < 5; ++i)
        if (reinterpret_cast<uintptr_t>(e->conv_b[i]) & 15u) return PICTURA_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return PICTURA_EINVAL;
    const EncPlan p = enc_plan(*e, views, height, width);
    if (workspace_bytes < p.total) return PICTURA_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    uint8_t* ws = (uint8_t*)workspace;
    EncWeights W{};
    for (int i = 0; i < 5; ++i) {
        W.cw[i] = e->conv_w[i];
        W.cb[i] = e->conv_b[i];
    }
    W.queries = e->queries;
    W.in_w = e->in_proj_w; W.in_b = e->in_proj_b;
    W.out_w = e->out_proj_w; W.out_b = e->out_proj_b;
    W.proj_w = e->proj_w; W.proj_b = e->proj_b;
    W.cams = e->cams;
    W.classes = e->num_classes;
    W.table = (float*)(ws + p.off_table);
    for (int i = 0; i < 4; ++i) W.wk[i] = (uint16_t*)(ws + p.off_wk[i]);
    W.qk = (float*)(ws + p.off_qk);
    W.vt = (float*)(ws + p.off_vt);
    W.ot = (float*)(ws + p.off_ot);
    W.pt = (float*)(ws + p.off_pt);
    float* pooled = (float*)(ws + p.off_pool);
    uint16_t* A = (uint16_t*)(ws + p.off_a);
    uint16_t* B = (uint16_t*)(ws + p.off_b);
    hipLaunchKernelGGL(enc_prep_kernel, dim3((unsigned)W.cams * kHeads + 512u), dim3(256), 0, s, W);
    auto blocks = [](int64_t n, int64_t per) { return dim3((unsigned)((n + per - 1) / per)); };
    const size_t lds1 = sizeof(float) * kTaps * (W.classes + 1) * kC1;
    for (int64_t v0 = 0; v0 < views; v0 += p.chunk) {
        const int64_t nv = views - v0 < p.chunk ? views - v0 : p.chunk;
        int64_t px[5];
        for (int i = 0; i < 5; ++i) px[i] = nv * p.h[i] * p.w[i];
        const int64_t at = v0 * height * width;
        const int64_t b1 = (px[0] + 63) / 64;
        hipLaunchKernelGGL(enc_conv1_kernel, dim3((unsigned)(b1 < 4096 ? b1 : 4096)), dim3(256), lds1, s, cls + at,
                           depth + at, W.table, W.cb[0], W.classes, height, width, p.h[0], p.w[0],
                           make_div31((uint32_t)(p.h[0] * p.w[0])), make_div31((uint32_t)p.w[0]), (int)px[0], A);
        hipLaunchKernelGGL((enc_conv_kernel<kC1, kC2, 2, 256, false>), blocks(px[1], 256), dim3(256), 0, s, A, W.wk[0],
                           W.cb[1], p.h[0], p.w[0], p.h[1], p.w[1], px[1], (void*)B);
        hipLaunchKernelGGL((enc_conv_s1_kernel<kC2, kC3, 256, false>), blocks(px[2], 256), dim3(256), 0, s, B, W.wk[1],
                           W.cb[2], p.h[2], p.w[2], px[2], (void*)A);
        hipLaunchKernelGGL((enc_conv_kernel<kC3, kC4, 2, 128, false>), blocks(px[3], 128), dim3(256), 0, s, A, W.wk[2],
                           W.cb[3], p.h[2], p.w[2], p.h[3], p.w[3], px[3], (void*)B);
        hipLaunchKernelGGL((enc_conv_s1_kernel<kC4, kC5, 128, true>), blocks(px[4], 128), dim3(256), 0, s, B, W.wk[3],
                           W.cb[4], p.h[4], p.w[4], px[4], (void*)A);
        const int tokens = p.h[4] * p.w[4];
        if (tokens <= 256)
            hipLaunchKernelGGL(enc_attn_kernel<true>, dim3((unsigned)nv), dim3(256),
                               (size_t)((tokens + 15) / 16) * 256 * sizeof(f32x4), s, (const float*)A, W.qk, W.cams, v0,
                               tokens, pooled);
        else
            hipLaunchKernelGGL(enc_attn_kernel<false>, dim3((unsigned)nv), dim3(256), 0, s, (const float*)A, W.qk, W.cams,
                               v0, tokens, pooled);
        hipLaunchKernelGGL(enc_tail_kernel, blocks(nv, kTailViews), dim3(256), 0, s, W, pooled, nv,
                           out + v0 * kEmb);
    }
    return hipGetLastError() == hipSuccess ? PICTURA_OK : PICTURA_EDEVICE;
}

}  // extern "C"
