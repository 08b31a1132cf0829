// Residual CNN of the learned preconditioner: forward, backward and Adam on
// the device (see cnn.h).
//
// Convolutions are implicit GEMMs on the BF16 matrix cores (FP32
// accumulation): gfx950's v_mfma_f32_16x16x32_bf16 for K-steps of 32, the
// 16x16x16 form where a layer has only 16 (padded) input channels.  A
// workgroup owns a 16 x 16 pixel tile of one image and all output channels;
// its input tile with a one-pixel halo and the layer's 3x3 x C_out x C_in
// weights sit in LDS.  Each of the 4 waves computes 4 rows of 16 pixels; per
// tap (dy, dx) and K-step of input channels, operand A is the tap's weights, 16
// output channels x K, and operand B 16 pixels' K channels read from the halo
// tile at the shifted position.  Operand layouts (wave64; checked on the device
// against a host product): with K = 32, A: lane l holds A[l % 16][8 (l / 16) + e],
// B: lane l holds B[8 (l / 16) + e][l % 16] (e < 8); with K = 16 the same
// with 4 (l / 16) + e (e < 4); D: lane l item v holds D[4 (l / 16) + v][l % 16].
//
// The backward pass reuses the same kernel: the input gradient of a
// convolution is a convolution of the output gradient with the weights
// transposed in the channels and flipped in space.  Weight gradients are
// per-tile MFMA products (pixels as the K dimension) reduced over tiles in a
// fixed order.
#include <algorithm>
#include <cmath>
#include <vector>

#include "cnn.h"

namespace hinv {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef short s8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

// D += A B with K = 32 (operands as BF16 bit patterns)
__device__ inline f4_t mfma_k32(s8_t a, s8_t b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b), c, 0,
                                                   0, 0);
}

constexpr int kT = 16;       // output tile side (pixels)
constexpr int kH = kT + 2;   // tile side with halo
constexpr int kWgStride = 9 * 32 * 32 + 32;  // floats per workgroup in the weight-gradient partials

enum { EPI_RELU = 0, EPI_RELU_RES = 1, EPI_LINEAR = 2, EPI_BWD = 3 };

__device__ inline short bf16_bits(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest, ties to even
    return (short)(u >> 16);
}

__device__ inline float bf16_value(short s) { return __uint_as_float(((unsigned)(unsigned short)s) << 16); }

struct LayerDesc {
    int co, ci;    // real channel counts
    int COp, CIp;  // padded
    int woff, boff;  // offsets of W and b in the packed parameters
};

const LayerDesc* layers() {
    static LayerDesc L[Cnn::kLayers];
    static bool init = false;
    if (!init) {
        const int co[6] = {32, 32, 32, 32, 32, 1}, ci[6] = {3, 32, 32, 32, 32, 32};
        int off = 0;
        for (int l = 0; l < 6; ++l) {
            L[l].co = co[l];
            L[l].ci = ci[l];
            L[l].COp = co[l] == 1 ? Cnn::kPadIn : co[l];
            L[l].CIp = ci[l] == 3 ? Cnn::kPadIn : ci[l];
            L[l].woff = off;
            off += co[l] * ci[l] * 9;
            L[l].boff = off;
            off += co[l];
        }
        init = true;
    }
    return L;
}

// Padded BF16 weights: forward wf[t][co][ci] = W[co][ci][t], backward
// wb[t][ci][co] = W[co][ci][8 - t] (channels transposed, taps flipped).
__global__ void k_weights_prep(const float* __restrict__ W, int co_r, int ci_r, int COp, int CIp,
                               short* __restrict__ wf, short* __restrict__ wb) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= 9 * COp * CIp) return;
    const int t = id / (COp * CIp), rem = id % (COp * CIp), co = rem / CIp, ci = rem % CIp;
    const bool real = co < co_r && ci < ci_r;
    wf[id] = real ? bf16_bits(W[(co * ci_r + ci) * 9 + t]) : (short)0;
    wb[(t * CIp + ci) * COp + co] = real ? bf16_bits(W[(co * ci_r + ci) * 9 + (8 - t)]) : (short)0;
}

// Planar FP32 [B][3][S][S] -> pixel-major BF16 with 16 channels (3 used).
__global__ void k_pack_input(int B, int S, const float* __restrict__ in, short* __restrict__ out) {
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long np = (long long)S * S;
    if (id >= np * B) return;
    const long long b = id / np, p = id % np;
    short* o = out + id * Cnn::kPadIn;
    for (int c = 0; c < Cnn::kPadIn; ++c)
        o[c] = c < Cnn::kInCh ? bf16_bits(in[(b * Cnn::kInCh + c) * np + p]) : (short)0;
}

// Convolution with fused epilogue.  Grid: (tiles x, tiles y, images).
//   EPI_RELU:     z = conv + b; h = relu(z)
//   EPI_RELU_RES: z = conv + b; h = res + relu(z)
//   EPI_LINEAR:   z = conv + b, channel 0 only (the one real channel), planar
//   EPI_BWD:      g = conv + res (res optional); out16 = bf16(g * [z > 0])
// The weights are operand A and the pixels operand B, so a lane's results are
// four consecutive channels of one pixel: the epilogue moves 16 bytes a lane.
// [z > 0] is all the backward pass needs of z: a lane's 32 results give one
// word, which the backward kernel's lane of the same place reads (mask).
// Bound by the traffic of h, its BF16 copy and the residual (about 50 MB a layer at
// 32 images of 64 x 64: ~10 us); the residual is requested before the products,
// and the LDS pixel stride of 80 bytes keeps 16-byte reads of 16 neighbouring
// pixels off each other's banks.  Keeping z itself in FP32, with 4-byte
// accesses, took 25.5 us a layer forward and 29.5 backward there, this 11.7
// and 11.3.
template <int CI, int CO, int EPI>
__global__ __launch_bounds__(256) void k_conv(int S, const short* __restrict__ in, const short* __restrict__ w,
                                              const float* __restrict__ bias, const float* __restrict__ res,
                                              unsigned* __restrict__ mask, float* __restrict__ out32,
                                              short* __restrict__ out16) {
    constexpr int PS = CI == 32 ? 40 : CI;  // LDS stride of a pixel / weight row
    constexpr int CQ = CI / 8;              // 16-byte pieces of it
    constexpr int NI = kH * kH * CQ, NW = 9 * CO * CQ;
    __shared__ __attribute__((aligned(16))) short sin[kH * kH * PS];
    __shared__ __attribute__((aligned(16))) short sw[9 * CO * PS];
    const int tx0 = blockIdx.x * kT, ty0 = blockIdx.y * kT, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int pi = lane & 15, kq = (lane >> 4) * 4;
    constexpr int NT = CO / 16;
    {
        s8_t vi[(NI + 255) / 256], vw[(NW + 255) / 256];
#pragma unroll
        for (int u = 0; u < (NI + 255) / 256; ++u) {
            const int e = threadIdx.x + 256 * u, pix = e / CQ, q = e % CQ;
            const int gy = ty0 + pix / kH - 1, gx = tx0 + pix % kH - 1;
            vi[u] = s8_t{0, 0, 0, 0, 0, 0, 0, 0};
            if (e < NI && gy >= 0 && gy < S && gx >= 0 && gx < S)
                vi[u] = reinterpret_cast<const s8_t*>(in + (((size_t)b * S + gy) * S + gx) * CI)[q];
        }
#pragma unroll
        for (int u = 0; u < (NW + 255) / 256; ++u)
            vw[u] = reinterpret_cast<const s8_t*>(w)[min((int)threadIdx.x + 256 * u, NW - 1)];
#pragma unroll
        for (int u = 0; u < (NI + 255) / 256; ++u) {
            const int e = threadIdx.x + 256 * u;
            if (e < NI) *reinterpret_cast<s8_t*>(sin + e / CQ * PS + e % CQ * 8) = vi[u];
        }
#pragma unroll
        for (int u = 0; u < (NW + 255) / 256; ++u) {
            const int e = threadIdx.x + 256 * u;
            if (e < NW) *reinterpret_cast<s8_t*>(sw + e / CQ * PS + e % CQ * 8) = vw[u];
        }
    }
    // this lane's results: pixel (gx, gy0 + r), channels nt * 16 + kq + v
    const int gx = tx0 + pi, gy0 = ty0 + wave * 4;
    auto at = [&](int r, int nt) { return (((size_t)b * S + gy0 + r) * S + gx) * CO + nt * 16 + kq; };
    f4_t rs[4][NT];
    if constexpr (EPI == EPI_RELU_RES || EPI == EPI_BWD) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                rs[r][nt] = f4_t{0.f, 0.f, 0.f, 0.f};
                if (res && gx < S && gy0 + r < S) rs[r][nt] = *reinterpret_cast<const f4_t*>(res + at(r, nt));
            }
    }
    const size_t mo = (((size_t)b * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
    unsigned mk = EPI == EPI_BWD ? mask[mo] : 0u;
    __syncthreads();
    f4_t acc[4][NT];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[r][nt] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int dy = t / 3, dx = t % 3;
        if constexpr (CI == 32) {
            const int k8 = (lane >> 4) * 8;
            s8_t aw[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                aw[nt] = *reinterpret_cast<const s8_t*>(sw + (t * CO + nt * 16 + pi) * PS + k8);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const s8_t px = *reinterpret_cast<const s8_t*>(sin + ((wave * 4 + r + dy) * kH + pi + dx) * PS + k8);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[r][nt] = mfma_k32(aw[nt], px, acc[r][nt]);
            }
        } else {
            static_assert(CI == 16, "16 or 32 input channels");
            s4_t aw[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                aw[nt] = *reinterpret_cast<const s4_t*>(sw + (t * CO + nt * 16 + pi) * PS + kq);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const s4_t px = *reinterpret_cast<const s4_t*>(sin + ((wave * 4 + r + dy) * kH + pi + dx) * PS + kq);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[r][nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aw[nt], px, acc[r][nt], 0, 0, 0);
            }
        }
    }
    if constexpr (EPI == EPI_LINEAR) {
        const float b0 = bias[0];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (kq == 0 && gx < S && gy0 + r < S) out32[((size_t)b * S + gy0 + r) * S + gx] = acc[r][0][0] + b0;
        return;
    }
    float bc[NT][4];
    if constexpr (EPI == EPI_RELU || EPI == EPI_RELU_RES) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) bc[nt][v] = bias[nt * 16 + kq + v];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            f4_t o32;
            s4_t o16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const unsigned bit = 1u << ((r * NT + nt) * 4 + v);
                const float val = acc[r][nt][v];
                if constexpr (EPI == EPI_BWD) {
                    const float g = val + rs[r][nt][v];
                    o32[v] = g;
                    o16[v] = bf16_bits(mk & bit ? g : 0.f);
                } else {
                    const float z = val + bc[nt][v];
                    if (z > 0.f) mk |= bit;
                    float h = fmaxf(z, 0.f);
                    if constexpr (EPI == EPI_RELU_RES) h += rs[r][nt][v];
                    o32[v] = h;
                    o16[v] = bf16_bits(h);
                }
            }
            if (gx < S && gy0 + r < S) {
                *reinterpret_cast<f4_t*>(out32 + at(r, nt)) = o32;
                *reinterpret_cast<s4_t*>(out16 + at(r, nt)) = o16;
            }
        }
    }
    if constexpr (EPI != EPI_BWD) mask[mo] = mk;
}

// Four BF16 values of a channel for a lane: a transposing LDS read.  Lane j of
// each 16 gives the address of pixel j / 4 and channels 4 (j % 4) .. + 3, and
// receives channel j of the four pixels.
__device__ inline s4_t read_tr(const short* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4_t*)p);
}

// Layers of one shape whose gradients one launch takes.
struct DwArgs {
    const short* in[4];
    const short* dz[4];
};

// Weight and bias gradients per tile: part[layer][wg][t][co][ci] = sum over
// the tile's pixels p of dz[p][co] in[p + tap t][ci]; then
// part[layer][wg][9 CO CI + co] = sum_p dz[p][co].  Grid: (tiles x, tiles y,
// images x layers).  The products run over pixels, which LDS holds as rows of
// channels, so the operands come through transposing reads (16 LDS reads of
// two bytes an operand without them); a wave keeps its taps' tiles in
// registers and shares dz between them, and the bias is a product with ones.
// Bound by LDS reads (~70 wave reads of 512 bytes a wave) and the partials'
// 37 KB a tile.  The LDS pixel stride of 96 bytes spreads 8 pixels' 32-byte
// pieces over all banks.  32 images of 64 x 64, 32 channels: 23.2 us a layer
// with two-byte reads and a layer a launch, this 35.5 for four.
template <int CI, int CO>
__global__ __launch_bounds__(256) void k_conv_dw(int S, int B, DwArgs args, float* __restrict__ part) {
    constexpr int PI = CI == 32 ? 48 : CI, PO = CO == 32 ? 48 : CO;  // LDS strides of a pixel
    constexpr int QI = CI / 8, QO = CO / 8;
    constexpr int NI = kH * kH * QI, NO = kT * kT * QO;
    __shared__ __attribute__((aligned(16))) short sin[kH * kH * PI];
    __shared__ __attribute__((aligned(16))) short sdz[kT * kT * PO];
    const int layer = blockIdx.z / B, b = blockIdx.z - layer * B;
    const int tx0 = blockIdx.x * kT, ty0 = blockIdx.y * kT;
    const size_t wg = ((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const short *in = args.in[layer], *dz = args.dz[layer];
    {
        s8_t vi[(NI + 255) / 256], vo[NO / 256];
#pragma unroll
        for (int u = 0; u < (NI + 255) / 256; ++u) {
            const int e = threadIdx.x + 256 * u, pix = e / QI, q = e % QI;
            const int gy = ty0 + pix / kH - 1, gx = tx0 + pix % kH - 1;
            vi[u] = s8_t{0, 0, 0, 0, 0, 0, 0, 0};
            if (e < NI && gy >= 0 && gy < S && gx >= 0 && gx < S)
                vi[u] = reinterpret_cast<const s8_t*>(in + (((size_t)b * S + gy) * S + gx) * CI)[q];
        }
#pragma unroll
        for (int u = 0; u < NO / 256; ++u) {
            const int e = threadIdx.x + 256 * u, pix = e / QO, q = e % QO;
            const int gy = ty0 + pix / kT, gx = tx0 + pix % kT;
            vo[u] = s8_t{0, 0, 0, 0, 0, 0, 0, 0};
            if (gy < S && gx < S) vo[u] = reinterpret_cast<const s8_t*>(dz + (((size_t)b * S + gy) * S + gx) * CO)[q];
        }
#pragma unroll
        for (int u = 0; u < (NI + 255) / 256; ++u) {
            const int e = threadIdx.x + 256 * u;
            if (e < NI) *reinterpret_cast<s8_t*>(sin + e / QI * PI + e % QI * 8) = vi[u];
        }
#pragma unroll
        for (int u = 0; u < NO / 256; ++u) {
            const int e = threadIdx.x + 256 * u;
            *reinterpret_cast<s8_t*>(sdz + e / QO * PO + e % QO * 8) = vo[u];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pi = lane & 15, kq = (lane >> 4) * 4;
    // wave w: 16 input channels cit, taps t0 .. t0 + ntap - 1, all output
    // channels; the waves with fewer taps take the bias of 16 output channels
    constexpr int NCO = CO / 16, NCI = CI / 16, MT = NCI == 2 ? 5 : 3;
    const int cit = NCI == 2 ? wave & 1 : 0;
    const int t0 = NCI == 2 ? (wave >> 1) * 5 : (wave ? 2 * wave + 1 : 0);
    const int ntap = NCI == 2 ? 5 - (wave >> 1) : (wave ? 2 : 3);
    const int bt = NCI == 2 ? wave - 2 : wave - 1;  // its bias tile
    const bool bias = bt >= 0 && bt < NCO;
    f4_t acc[MT][NCO], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < MT; ++q)
#pragma unroll
        for (int c = 0; c < NCO; ++c) acc[q][c] = f4_t{0.f, 0.f, 0.f, 0.f};
    constexpr short kOne = 0x3f80;
    const s8_t ones = {kOne, kOne, kOne, kOne, kOne, kOne, kOne, kOne};
    // K = the tile's pixels, 32 (two rows) per step: pixel 32 st + 8 (l / 16) + e;
    // this lane addresses pixels + pi / 4 (e < 4) and + 4 + pi / 4
    const int p8 = (lane >> 4) * 8 + (pi >> 2), ch = (pi & 3) * 4;
    const short* dzp = sdz + p8 * PO + ch;
    const short* inp = sin + (p8 / kT * kH + p8 % kT) * PI + cit * 16 + ch;
    auto join = [](s4_t lo, s4_t hi) { return s8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}; };
#pragma unroll 2
    for (int st = 0; st < kT * kT / 32; ++st) {
        s8_t a[NCO];
#pragma unroll
        for (int c = 0; c < NCO; ++c)
            a[c] = join(read_tr(dzp + 32 * st * PO + c * 16), read_tr(dzp + (32 * st + 4) * PO + c * 16));
#pragma unroll
        for (int q = 0; q < MT; ++q) {
            if (q >= ntap) break;
            const int t = t0 + q, dy = t / 3, dx = t - 3 * dy;
            const short* ip = inp + ((2 * st + dy) * kH + dx) * PI;
            const s8_t x = join(read_tr(ip), read_tr(ip + 4 * PI));
#pragma unroll
            for (int c = 0; c < NCO; ++c) acc[q][c] = mfma_k32(a[c], x, acc[q][c]);
        }
        if (bias) accb = mfma_k32(NCO == 1 || bt == 0 ? a[0] : a[NCO - 1], ones, accb);
    }
    float* pw = part + wg * kWgStride;
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        if (q >= ntap) break;
#pragma unroll
        for (int c = 0; c < NCO; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                pw[((t0 + q) * CO + c * 16 + kq + v) * CI + cit * 16 + pi] = acc[q][c][v];
    }
    if (bias && pi == 0)
#pragma unroll
        for (int v = 0; v < 4; ++v) pw[9 * CO * CI + bt * 16 + kq + v] = accb[v];
}

// Weight and bias gradients from the per-tile partials, in two fixed-order
// stages that read the partials coalesced (index j runs over one tile's
// partial layout [t][co][ci] then the biases):
//   tmp[layer][sp][j] = sum over the tiles of split sp of part[layer][tile][j],
//   then the kDwSplit sums in order, scattered into the packed gradient.
// Every layer in one launch (grid.z; l0: the first one, its partials at part).
constexpr int kDwSplit = 16;
struct DwLayers {
    int J[Cnn::kLayers];
    int co[Cnn::kLayers], ci[Cnn::kLayers], COp[Cnn::kLayers], CIp[Cnn::kLayers], woff[Cnn::kLayers],
        boff[Cnn::kLayers];
};
__global__ void k_dw_partial(int nwg, int l0, DwLayers L, const float* __restrict__ part, double* __restrict__ tmp) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int sp = blockIdx.y, l = l0 + blockIdx.z;
    if (j >= L.J[l]) return;
    const int g0 = (int)((long long)sp * nwg / kDwSplit), g1 = (int)((long long)(sp + 1) * nwg / kDwSplit);
    const float* p = part + (size_t)blockIdx.z * nwg * kWgStride + j;
    double s = 0.0;
#pragma unroll 8
    for (int g = g0; g < g1; ++g) s += p[(size_t)g * kWgStride];
    tmp[((size_t)l * kDwSplit + sp) * kWgStride + j] = s;
}

__global__ void k_dw_reduce(DwLayers L, const double* __restrict__ tmp, float* __restrict__ grad) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x, l = blockIdx.y;
    if (j >= L.J[l]) return;
    double s = 0.0;
#pragma unroll
    for (int sp = 0; sp < kDwSplit; ++sp) s += tmp[((size_t)l * kDwSplit + sp) * kWgStride + j];
    const int COp = L.COp[l], CIp = L.CIp[l], nw = 9 * COp * CIp;
    if (j < nw) {
        const int t = j / (COp * CIp), r = j - t * COp * CIp, co = r / CIp, ci = r - co * CIp;
        if (co < L.co[l] && ci < L.ci[l]) grad[L.woff[l] + (co * L.ci[l] + ci) * 9 + t] = (float)s;
    } else if (j - nw < L.co[l]) {
        grad[L.boff[l] + j - nw] = (float)s;
    }
}

// Per-sample partial sums of |y - t|^2 and |t|^2 (grid: chunks x images).
__global__ void k_loss_part(long long np, const float* __restrict__ y, const float* __restrict__ tg,
                            double* __restrict__ part) {
    const int b = blockIdx.y;
    double num = 0.0, den = 0.0;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (long long)gridDim.x * blockDim.x) {
        const double yv = y[(size_t)b * np + p], tv = tg[(size_t)b * np + p];
        num += (yv - tv) * (yv - tv);
        den += tv * tv;
    }
    __shared__ double sn[256], sd[256];
    sn[threadIdx.x] = num;
    sd[threadIdx.x] = den;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, c = 0.0;
        for (int i = 0; i < (int)blockDim.x; ++i) {
            a += sn[i];
            c += sd[i];
        }
        part[((size_t)b * gridDim.x + blockIdx.x) * 2] = a;
        part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = c;
    }
}

// dL/dy = 2 (y - t) / (|t|^2 B) in channel 0 of a 16-channel BF16 image; the
// first workgroup of each image records |y - t|^2 / |t|^2.
__global__ void k_loss_grad(int B, long long np, int nchunk, const float* __restrict__ y,
                            const float* __restrict__ tg, const double* __restrict__ part,
                            short* __restrict__ gy, double* __restrict__ ratio) {
    const int b = blockIdx.y;
    double num = 0.0, den = 0.0;
    for (int c = 0; c < nchunk; ++c) {
        num += part[((size_t)b * nchunk + c) * 2];
        den += part[((size_t)b * nchunk + c) * 2 + 1];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ratio[b] = den > 0 ? num / den : 0.0;
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const double yv = y[(size_t)b * np + p], tv = tg[(size_t)b * np + p];
    const float g = den > 0 ? (float)(2.0 * (yv - tv) / (den * B)) : 0.f;
    short* o = gy + ((size_t)b * np + p) * Cnn::kPadIn;
    o[0] = bf16_bits(g);
    for (int c = 1; c < Cnn::kPadIn; ++c) o[c] = 0;
}

// Relative energy norm: per pixel d = (y - t) m, (A d) from the 5-point
// stencil (wE, wN, diag) of the target channels 1..3, neighbours outside the
// image zero; A t likewise.  Partials of d^T A d and t^T A t per chunk.
struct EnergyPix {
    double dAd, tAt, Ad;
};

__device__ inline EnergyPix energy_at(int S, long long b, int row, int col, const float* __restrict__ y,
                                      const float* __restrict__ tg, const float* __restrict__ in) {
    const long long np = (long long)S * S;
    const float* t = tg + b * 4 * np;
    const float* wE = t + np;
    const float* wN = t + 2 * np;
    const float* dg = t + 3 * np;
    const float* mk = in + (b * Cnn::kInCh + 2) * np;
    auto dv = [&](int r, int c) -> double {
        const long long p = (long long)r * S + c;
        return ((double)y[b * np + p] - (double)t[p]) * (double)mk[p];
    };
    auto tv = [&](int r, int c) -> double {
        const long long p = (long long)r * S + c;
        return (double)t[p] * (double)mk[p];
    };
    const long long p = (long long)row * S + col;
    const double d0 = dv(row, col), t0 = tv(row, col);
    double Ad = (double)dg[p] * d0, At = (double)dg[p] * t0;
    if (col + 1 < S) {
        Ad -= (double)wE[p] * dv(row, col + 1);
        At -= (double)wE[p] * tv(row, col + 1);
    }
    if (col > 0) {
        Ad -= (double)wE[p - 1] * dv(row, col - 1);
        At -= (double)wE[p - 1] * tv(row, col - 1);
    }
    if (row + 1 < S) {
        Ad -= (double)wN[p] * dv(row + 1, col);
        At -= (double)wN[p] * tv(row + 1, col);
    }
    if (row > 0) {
        Ad -= (double)wN[p - S] * dv(row - 1, col);
        At -= (double)wN[p - S] * tv(row - 1, col);
    }
    const double m = (double)mk[p];
    return EnergyPix{d0 * Ad * m, t0 * At * m, Ad * m};
}

__global__ void k_energy_part(int S, const float* __restrict__ y, const float* __restrict__ tg,
                              const float* __restrict__ in, double* __restrict__ part) {
    const int b = blockIdx.y;
    const long long np = (long long)S * S;
    double num = 0.0, den = 0.0;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (long long)gridDim.x * blockDim.x) {
        const EnergyPix e = energy_at(S, b, (int)(p / S), (int)(p % S), y, tg, in);
        num += e.dAd;
        den += e.tAt;
    }
    __shared__ double sn[256], sd[256];
    sn[threadIdx.x] = num;
    sd[threadIdx.x] = den;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, c = 0.0;
        for (int i = 0; i < (int)blockDim.x; ++i) {
            a += sn[i];
            c += sd[i];
        }
        part[((size_t)b * gridDim.x + blockIdx.x) * 2] = a;
        part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = c;
    }
}

// dL/dy = 2 m (A d) / (t^T A t B) in channel 0 of the BF16 gradient image.
__global__ void k_energy_grad(int B, int S, int nchunk, const float* __restrict__ y, const float* __restrict__ tg,
                              const float* __restrict__ in, const double* __restrict__ part,
                              short* __restrict__ gy, double* __restrict__ ratio) {
    const int b = blockIdx.y;
    const long long np = (long long)S * S;
    double num = 0.0, den = 0.0;
    for (int c = 0; c < nchunk; ++c) {
        num += part[((size_t)b * nchunk + c) * 2];
        den += part[((size_t)b * nchunk + c) * 2 + 1];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ratio[b] = den > 0 ? num / den : 0.0;
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const EnergyPix e = energy_at(S, b, (int)(p / S), (int)(p % S), y, tg, in);
    const float g = den > 0 ? (float)(2.0 * e.Ad / (den * B)) : 0.f;
    short* o = gy + ((size_t)b * np + p) * Cnn::kPadIn;
    o[0] = bf16_bits(g);
    for (int c = 1; c < Cnn::kPadIn; ++c) o[c] = 0;
}

__global__ void k_adam(int n, float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mi = b1 * m[i] + (1.f - b1) * g[i];
    const float vi = b2 * v[i] + (1.f - b2) * g[i] * g[i];
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

__global__ void k_fill_f(int n, float v, float* __restrict__ a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

}  // namespace

Cnn::Cnn(Ctx* ctx) : ctx_(ctx) {
    const int n = nparams();
    theta_.ensure(n);
    grad_.ensure(n);
    m_.ensure(n);
    v_.ensure(n);
    const LayerDesc* L = layers();
    for (int l = 0; l < kLayers; ++l) {
        wf_[l].ensure((size_t)9 * L[l].COp * L[l].CIp);
        wb_[l].ensure((size_t)9 * L[l].COp * L[l].CIp);
    }
    loss_.ensure(1);
    hipStream_t s = ctx_->stream;
    for (DBuf<float>* b : {&theta_, &grad_, &m_, &v_}) {
        k_fill_f<<<ceil_div(n, 256), 256, 0, s>>>(n, 0.f, b->get());
        HINV_LAUNCH_CHECK();
    }
}

int Cnn::nparams() {
    const LayerDesc* L = layers();
    return L[kLayers - 1].boff + L[kLayers - 1].co;
}

void Cnn::set_params(const float* host) {
    const int n = nparams();
    hipStream_t s = ctx_->stream;
    HINV_HIP(hipMemcpyAsync(theta_.get(), host, sizeof(float) * n, hipMemcpyHostToDevice, s));
    k_fill_f<<<ceil_div(n, 256), 256, 0, s>>>(n, 0.f, m_.get());
    k_fill_f<<<ceil_div(n, 256), 256, 0, s>>>(n, 0.f, v_.get());
    HINV_LAUNCH_CHECK();
    HINV_HIP(hipStreamSynchronize(s));
    step_ = 0;
    weights_fresh_ = false;
}

void Cnn::get_params(float* host) const {
    HINV_HIP(hipMemcpyAsync(host, theta_.get(), sizeof(float) * nparams(), hipMemcpyDeviceToHost, ctx_->stream));
    HINV_HIP(hipStreamSynchronize(ctx_->stream));
}

void Cnn::refresh_weights() {
    if (weights_fresh_) return;
    const LayerDesc* L = layers();
    for (int l = 0; l < kLayers; ++l) {
        const int tot = 9 * L[l].COp * L[l].CIp;
        k_weights_prep<<<ceil_div(tot, 256), 256, 0, ctx_->stream>>>(theta_.get() + L[l].woff, L[l].co, L[l].ci,
                                                                     L[l].COp, L[l].CIp, wf_[l].get(),
                                                                     wb_[l].get());
        HINV_LAUNCH_CHECK();
    }
    weights_fresh_ = true;
}

// Whether the partials of every layer's gradient are kept until one launch
// sums them: while they take at most 512 MB (2400 tiles), where a launch a
// layer would be mostly latency; beyond, layer after layer reuses the space.
static bool dw_together(int nwg) { return (size_t)nwg * kWgStride * sizeof(float) * Cnn::kLayers <= (512u << 20); }

void Cnn::ensure(int B, int S) {
    if (B <= 0 || S <= 0) fail(HINV_EINVAL, "empty image batch");
    if (S > 8193) fail(HINV_EINVAL, "image side above 8193");
    const size_t np = (size_t)B * S * S;
    const int tiles = ceil_div(S, kT);
    const int nwg = tiles * tiles * B;
    if (np > (size_t)B_ * S_ * S_ || nwg > nwg_) {
        B_ = S_ = nwg_ = 0;  // until every buffer is there
        in0_.ensure(np * kPadIn);
        for (int l = 0; l < kLayers - 1; ++l) {
            a_[l].ensure(np * kCh);
            h_[l].ensure(np * kCh);
        }
        y_.ensure(np);
        for (auto& d : dz_) d.ensure(np * kCh);
        for (auto& d : gh_) d.ensure(np * kCh);
        gy_.ensure(np * kPadIn);
        for (auto& m : mask_) m.ensure((size_t)nwg * 256);
        B_ = B;
        S_ = S;
        nwg_ = nwg;
    }
}

void Cnn::run_forward(int B, int S, float* y) {
    refresh_weights();
    const LayerDesc* L = layers();
    hipStream_t s = ctx_->stream;
    const int tiles = ceil_div(S, kT), top = kLayers - 1;
    const dim3 g(tiles, tiles, B);
    const float* th = theta_.get();
    k_conv<16, 32, EPI_RELU><<<g, 256, 0, s>>>(S, in0_.get(), wf_[0].get(), th + L[0].boff, nullptr, mask_[0].get(),
                                                h_[0].get(), a_[0].get());
    HINV_LAUNCH_CHECK();
    for (int l = 1; l < top; ++l) {
        k_conv<32, 32, EPI_RELU_RES><<<g, 256, 0, s>>>(S, a_[l - 1].get(), wf_[l].get(), th + L[l].boff,
                                                        h_[l - 1].get(), mask_[l].get(), h_[l].get(), a_[l].get());
        HINV_LAUNCH_CHECK();
    }
    k_conv<32, 16, EPI_LINEAR><<<g, 256, 0, s>>>(S, a_[top - 1].get(), wf_[top].get(), th + L[top].boff, nullptr,
                                                  nullptr, y, nullptr);
    HINV_LAUNCH_CHECK();
}

void Cnn::forward(int B, int S, const float* in, float* out) {
    ensure(B, S);
    const long long np = (long long)B * S * S;
    k_pack_input<<<(unsigned)ceil_div((int)std::min<long long>(np, 1LL << 30), 256), 256, 0, ctx_->stream>>>(
        B, S, in, in0_.get());
    HINV_LAUNCH_CHECK();
    run_forward(B, S, out);
}

short* Cnn::packed_input(int S) {
    ensure(1, S);
    return in0_.get();
}

void Cnn::forward_packed(int B, int S) {
    ensure(B, S);
    run_forward(B, S, y_.get());
}

double Cnn::gradient(int B, int S, const float* in, const float* target, int tchan, float* grad_host) {
    ensure(B, S);
    hipStream_t s = ctx_->stream;
    const long long np = (long long)S * S;
    k_pack_input<<<(unsigned)ceil_div((int)(np * B), 256), 256, 0, s>>>(B, S, in, in0_.get());
    HINV_LAUNCH_CHECK();
    run_forward(B, S, y_.get());
    // loss and dL/dy
    const int nchunk = std::min(64, ceil_div((int)np, 256));
    lpart_.ensure((size_t)2 * B * nchunk);
    ratio_.ensure(B);
    if (tchan == 1) {
        k_loss_part<<<dim3(nchunk, B), 256, 0, s>>>(np, y_.get(), target, lpart_.get());
        HINV_LAUNCH_CHECK();
        k_loss_grad<<<dim3(ceil_div((int)np, 256), B), 256, 0, s>>>(B, np, nchunk, y_.get(), target,
                                                                     lpart_.get(), gy_.get(), ratio_.get());
    } else {
        k_energy_part<<<dim3(nchunk, B), 256, 0, s>>>(S, y_.get(), target, in, lpart_.get());
        HINV_LAUNCH_CHECK();
        k_energy_grad<<<dim3(ceil_div((int)np, 256), B), 256, 0, s>>>(B, S, nchunk, y_.get(), target,
                                                                       in, lpart_.get(), gy_.get(), ratio_.get());
    }
    HINV_LAUNCH_CHECK();
    // backward
    const LayerDesc* L = layers();
    const int tiles = ceil_div(S, kT);
    const dim3 g(tiles, tiles, B);
    const int nwg = tiles * tiles * B;
    float* gr = grad_.get();
    part_.ensure((size_t)nwg * kWgStride * (dw_together(nwg) ? kLayers : 1));
    dwtmp_.ensure((size_t)kLayers * kDwSplit * kWgStride);
    const int top = kLayers - 1;
    // dL/dh_{top-1} and dZ_{top-1} = dL/dh * [z > 0]; then dL/dh_{l-1} =
    // conv^T(dZ_l) + dL/dh_l (identity path) and dZ_{l-1}
    k_conv<16, 32, EPI_BWD><<<g, 256, 0, s>>>(S, gy_.get(), wb_[top].get(), nullptr, nullptr, mask_[top - 1].get(),
                                               gh_[0].get(), dz_[top - 1].get());
    HINV_LAUNCH_CHECK();
    int cur = 0;
    for (int l = top - 1; l >= 1; --l) {
        k_conv<32, 32, EPI_BWD><<<g, 256, 0, s>>>(S, dz_[l].get(), wb_[l].get(), nullptr, gh_[cur].get(),
                                                   mask_[l - 1].get(), gh_[1 - cur].get(), dz_[l - 1].get());
        HINV_LAUNCH_CHECK();
        cur = 1 - cur;
    }
    DwLayers D{};
    int Jmax = 0;
    for (int l = 0; l < kLayers; ++l) {
        D.J[l] = 9 * L[l].COp * L[l].CIp + L[l].COp;
        D.co[l] = L[l].co;
        D.ci[l] = L[l].ci;
        D.COp[l] = L[l].COp;
        D.CIp[l] = L[l].CIp;
        D.woff[l] = L[l].woff;
        D.boff[l] = L[l].boff;
        Jmax = std::max(Jmax, D.J[l]);
    }
    // weight gradients of layers l0 .. l0 + n - 1, n > 1 for the middle ones only
    auto dw = [&](int l0, int n, float* part) {
        DwArgs a{};
        for (int i = 0; i < n; ++i) {
            a.in[i] = l0 + i ? a_[l0 + i - 1].get() : in0_.get();
            a.dz[i] = l0 + i == top ? gy_.get() : dz_[l0 + i].get();
        }
        const dim3 gd(tiles, tiles, B * n);
        if (l0 == top)
            k_conv_dw<32, 16><<<gd, 256, 0, s>>>(S, B, a, part);
        else if (l0 > 0)
            k_conv_dw<32, 32><<<gd, 256, 0, s>>>(S, B, a, part);
        else
            k_conv_dw<16, 32><<<gd, 256, 0, s>>>(S, B, a, part);
        HINV_LAUNCH_CHECK();
    };
    auto partials = [&](int l0, int n) {
        k_dw_partial<<<dim3(ceil_div(Jmax, 256), kDwSplit, n), 256, 0, s>>>(nwg, l0, D, part_.get(), dwtmp_.get());
        HINV_LAUNCH_CHECK();
    };
    if (dw_together(nwg)) {
        const size_t ps = (size_t)nwg * kWgStride;
        dw(0, 1, part_.get());
        dw(1, top - 1, part_.get() + ps);
        dw(top, 1, part_.get() + top * ps);
        partials(0, kLayers);
    } else {
        for (int l = 0; l < kLayers; ++l) {
            dw(l, 1, part_.get());
            partials(l, 1);
        }
    }
    k_dw_reduce<<<dim3(ceil_div(Jmax, 256), kLayers), 256, 0, s>>>(D, dwtmp_.get(), gr);
    HINV_LAUNCH_CHECK();
    std::vector<double> r(B);
    HINV_HIP(hipMemcpyAsync(r.data(), ratio_.get(), sizeof(double) * B, hipMemcpyDeviceToHost, s));
    if (grad_host)
        HINV_HIP(hipMemcpyAsync(grad_host, gr, sizeof(float) * nparams(), hipMemcpyDeviceToHost, s));
    HINV_HIP(hipStreamSynchronize(s));
    double Lsum = 0.0;
    for (double v : r) Lsum += v;
    return Lsum / B;
}

double Cnn::train_step(int B, int S, const float* in, const float* target, int tchan, float lr) {
    const double L = gradient(B, S, in, target, tchan, nullptr);
    ++step_;
    const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, step_)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, step_)));
    const int n = nparams();
    k_adam<<<ceil_div(n, 256), 256, 0, ctx_->stream>>>(n, theta_.get(), grad_.get(), m_.get(), v_.get(), lr, c1, c2);
    HINV_LAUNCH_CHECK();
    weights_fresh_ = false;
    return L;
}

}  // namespace hinv
