// Dense kernels: matrix-core tall-skinny products and s x s factorizations
// (s = k + oversampling <= 512), blocked over the compute units; the
// eigenproblems of small s in one workgroup's LDS.
//
// Matrix-core operand layouts (wave64), checked on the device:
//   f64 16x16x4:   A (16 x 4): lane l holds A[l % 16][l / 16]
//                  B (4 x 16): lane l holds B[l / 16][l % 16]
//                  D (16 x 16): lane l, item v holds D[4 v + l / 16][l % 16]
//   bf16 16x16x32 (gfx950): A: lane l holds A[l % 16][8 (l / 16) + e], e = 0..7
//                  B: lane l holds B[8 (l / 16) + e][l % 16]
//                  D: lane l, item v holds D[4 (l / 16) + v][l % 16]
#include <algorithm>
#include <vector>

#include "dense.h"
#include "grid.h"

namespace hinv {

namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef short s8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

__device__ inline short to_bf16(double x) {
    // round-to-nearest-even of the float value
    const float f = (float)x;
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

// Block products: a workgroup of kBlkWaves waves owns a 128 x 128 block of the
// output; wave w computes its rows [16 w, 16 w + 16) against all 128 columns
// (kBlkTiles matrix-core tiles sharing one operand), so each column of X and
// Y is read by ceil(s / 128) workgroups instead of ceil(s / 16).
constexpr int kBlkWaves = 8, kBlkTiles = 8, kBlk = 128;

// Split-K Gram C = X^T Y: grid.x = output block, grid.y = K chunk (a multiple
// of kGramKC rows).  The block's 128 columns of Y are staged in LDS kGramKC
// rows at a time (double-buffered: the next stage is loaded into registers
// while the matrix cores work on the current one), so the eight waves share
// one read of Y; each wave loads its 16 columns of X for the stage's eight K
// steps at once.  Products are accumulated in K order.
constexpr int kGramKC = 32;   // K rows per LDS stage

// XCD-aware order of the workgroups of a (per x chunks) grid: the hardware
// hands consecutive workgroups to the eight XCDs in turn, so with the plain
// order the `per` output blocks of one K chunk (which read the same rows of
// X and Y) land on different XCDs and each XCD's L2 fetches those rows again.
// Workgroup h is mapped to block b and chunk c such that the blocks of chunk
// c run on one XCD one after another (h = 8 j + x: XCD x, its j-th
// workgroup); the chunks beyond the last multiple of 8 keep the plain order.
// A bijection of [0, per * chunks) onto the (block, chunk) pairs, whatever
// the grid's shape (h is the dispatch order, x fastest).
__device__ inline void xcd_block_chunk(int per, int chunks, int& b, int& c) {
    const int h = blockIdx.x + gridDim.x * blockIdx.y;
    const int full = chunks & ~7;
    if (h < full * per) {
        const int x = h & 7, j = h >> 3;
        b = j % per;
        c = (j / per) * 8 + x;
    } else {
        const int t = h - full * per;
        b = t % per;
        c = full + t / per;
    }
}
constexpr int kGramLd = 144;  // LDS row stride (doubles): rows k and k + 1 fall in different bank halves
__global__ __launch_bounds__(512) void k_gram_f64(int n, int s1, int s2, int chunk,
                                                  const double* __restrict__ X, int ldx,
                                                  const double* __restrict__ Y, int ldy,
                                                  double* __restrict__ part) {
    __shared__ double ys[2][kGramKC * kGramLd];
    const int blocks_i = (s1 + kBlk - 1) / kBlk;
    int blk, split;
    xcd_block_chunk(gridDim.x, gridDim.y, blk, split);
    const int bi = blk % blocks_i, bj = blk / blocks_i;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = bi * kBlk + wave * 16 + (lane & 15);
    const bool rows_on = bi * kBlk + wave * 16 < s1;  // this wave has output rows (all waves stage Y)
    const int kr = lane >> 4;
    const int k_begin = split * chunk;
    const int k_end = min(n, k_begin + chunk);
    const double* xc = X + (size_t)(i < s1 ? i : 0) * ldx;
    // staging: thread t loads rows 8 (t mod 4) .. + 8 of block column t / 4
    const int jj = threadIdx.x >> 2, r8 = (threadIdx.x & 3) * 8;
    const bool jok = bj * kBlk + jj < s2;
    const double* ycol = Y + (size_t)(jok ? bj * kBlk + jj : 0) * ldy;
    double stg[8];
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + r8 + e;
            stg[e] = (jok && k < k_end) ? ycol[k] : 0.0;
        }
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < 8; ++e) ys[buf][(r8 + e) * kGramLd + jj] = stg[e];
    };
    d4_t acc[kBlkTiles];
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
    load_stage(k_begin);
    store_stage(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += kGramKC) {
        const bool more = k0 + kGramKC < k_end;
        if (more) load_stage(k0 + kGramKC);
        if (rows_on) {
            double a[kGramKC / 4];
#pragma unroll
            for (int u = 0; u < kGramKC / 4; ++u) {
                const int k = k0 + 4 * u + kr;
                a[u] = (i < s1 && k < k_end) ? xc[k] : 0.0;
            }
            const double* yb = ys[buf] + kr * kGramLd + (lane & 15);
#pragma unroll
            for (int u = 0; u < kGramKC / 4; ++u)
#pragma unroll
                for (int t = 0; t < kBlkTiles; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], yb[4 * u * kGramLd + t * 16], acc[t], 0, 0, 0);
        }
        // the other buffer was last read before the previous barrier
        if (more) store_stage(1 - buf);
        __syncthreads();
        buf = 1 - buf;
    }
    if (!rows_on) return;
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t)
        for (int v = 0; v < 4; ++v) {
            const int gi = bi * kBlk + wave * 16 + 4 * v + (lane >> 4);
            const int gj = bj * kBlk + t * 16 + (lane & 15);
            if (gi < s1 && gj < s2) part[((size_t)split * s2 + gj) * s1 + gi] = acc[t][v];
        }
}

__global__ __launch_bounds__(512) void k_gram_bf16(int n, int s1, int s2, int chunk,
                                                   const double* __restrict__ X, int ldx,
                                                   const double* __restrict__ Y, int ldy,
                                                   double* __restrict__ part) {
    const int blocks_i = (s1 + kBlk - 1) / kBlk;
    int blk, split;
    xcd_block_chunk(gridDim.x, gridDim.y, blk, split);
    const int bi = blk % blocks_i, bj = blk / blocks_i;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = bi * kBlk + wave * 16 + (lane & 15);
    if (bi * kBlk + wave * 16 >= s1) return;  // no rows for this wave (no barrier below)
    const int kq = (lane >> 4) * 8;  // gfx950 16x16x32 BF16: 8 consecutive K per lane
    const int k_begin = split * chunk;
    const int k_end = min(n, k_begin + chunk);
    const double* xc = X + (size_t)(i < s1 ? i : 0) * ldx;
    const double* yc[kBlkTiles];
    bool jv[kBlkTiles];
    f4_t acc[kBlkTiles];
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t) {
        const int j = bj * kBlk + t * 16 + (lane & 15);
        jv[t] = j < s2;
        yc[t] = Y + (size_t)(jv[t] ? j : 0) * ldy;
        acc[t] = f4_t{0.f, 0.f, 0.f, 0.f};
    }
    for (int k0 = k_begin; k0 < k_end; k0 += 32) {
        s8_t a;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + kq + e;
            a[e] = to_bf16((i < s1 && k < k_end) ? xc[k] : 0.0);
        }
#pragma unroll
        for (int t = 0; t < kBlkTiles; ++t) {
            s8_t b;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + kq + e;
                b[e] = to_bf16((jv[t] && k < k_end) ? yc[t][k] : 0.0);
            }
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b),
                                                             acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < kBlkTiles; ++t)
        for (int v = 0; v < 4; ++v) {
            const int gi = bi * kBlk + wave * 16 + 4 * (lane >> 4) + v;
            const int gj = bj * kBlk + t * 16 + (lane & 15);
            if (gi < s1 && gj < s2) part[((size_t)split * s2 + gj) * s1 + gi] = (double)acc[t][v];
        }
}

// Wide Gram for s2 <= 16 kWideMaxCT: grid.x = row blocks of rt row tiles,
// grid.y = K chunk.  A workgroup of eight waves stages the K step's rows of
// Y for all CT column tiles in LDS (double-buffered), so a K chunk of Y is
// read once per row block, and waves 0 .. rt-1 each compute one 16-row tile
// of the output against the CT column tiles (CT matrix-core accumulators).
// The output is covered by 16 x 16 tiles instead of 128 x 128 blocks (s =
// 220: 224^2 instead of 256^2 products).  For X = Y (self) a wave's A
// operand comes from the same staged rows, so X is not read at all.
constexpr int kWideKC = 32, kWideMaxCT = 16;
__host__ __device__ constexpr int wide_ld(int ct) { return 16 * ct + 16; }  // rows k, k + 1 in different bank halves

template <int CT>
__global__ __launch_bounds__(512) void k_gram_wide(int n, int s1, int s2, int chunk, int rt, int self,
                                                   const double* __restrict__ X, int ldx,
                                                   const double* __restrict__ Y, int ldy,
                                                   double* __restrict__ part) {
    extern __shared__ double wsh[];  // [2][kWideKC][LD]
    constexpr int LD = wide_ld(CT), SEG = 16 * CT * (kWideKC / 8), SPT = (SEG + 511) / 512;
    int blk, split;
    xcd_block_chunk(gridDim.x, gridDim.y, blk, split);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rtile = blk * rt + wave;
    const bool rows_on = wave < rt && rtile * 16 < s1;  // this wave has output rows (all waves stage Y)
    const int i = rtile * 16 + (lane & 15);
    const int kr = lane >> 4;
    const int k_begin = split * chunk;
    const int k_end = min(n, k_begin + chunk);
    const double* xc = X + (size_t)(i < s1 ? i : 0) * ldx;
    // staging: segment g = 8 consecutive rows (g mod 4) of column g / 4
    double stg[SPT][8];
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int sp = 0; sp < SPT; ++sp) {
            const int g = threadIdx.x + 512 * sp;
            const int j = g >> 2, r8 = (g & 3) * 8;
            const bool jok = g < SEG && j < s2;
            const double* yc = Y + (size_t)(jok ? j : 0) * ldy;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + r8 + e;
                stg[sp][e] = (jok && k < k_end) ? yc[k] : 0.0;
            }
        }
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int sp = 0; sp < SPT; ++sp) {
            const int g = threadIdx.x + 512 * sp;
            if (g < SEG) {
                const int j = g >> 2, r8 = (g & 3) * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e) wsh[(buf * kWideKC + r8 + e) * LD + j] = stg[sp][e];
            }
        }
    };
    // X != Y: a wave's A operand of the next K step is loaded with the staging
    // loads, a step ahead of its use
    double xa[kWideKC / 4];
    auto load_x = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kWideKC / 4; ++u) {
            const int k = k0 + 4 * u + kr;
            xa[u] = (!self && rows_on && i < s1 && k < k_end) ? xc[k] : 0.0;
        }
    };
    d4_t acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
    load_stage(k_begin);
    load_x(k_begin);
    store_stage(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += kWideKC) {
        const bool more = k0 + kWideKC < k_end;
        double a[kWideKC / 4];
#pragma unroll
        for (int u = 0; u < kWideKC / 4; ++u) a[u] = xa[u];
        if (more) {
            load_stage(k0 + kWideKC);
            load_x(k0 + kWideKC);
        }
        if (rows_on) {
            // A[l % 16][l / 16] = X[k0 + 4 u + l / 16][i], B[l / 16][l % 16] = Y[k0 + 4 u + l / 16][16 t + l % 16]
            const double* yb = wsh + (buf * kWideKC + kr) * LD + (lane & 15);
            if (self) {
#pragma unroll
                for (int u = 0; u < kWideKC / 4; ++u) a[u] = yb[4 * u * LD + 16 * rtile];
            }
#pragma unroll
            for (int u = 0; u < kWideKC / 4; ++u)
#pragma unroll
                for (int t = 0; t < CT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], yb[4 * u * LD + t * 16], acc[t], 0, 0, 0);
        }
        // the other buffer was last read before the previous barrier
        if (more) store_stage(1 - buf);
        __syncthreads();
        buf = 1 - buf;
    }
    if (!rows_on) return;
#pragma unroll
    for (int t = 0; t < CT; ++t)
        for (int v = 0; v < 4; ++v) {
            const int gi = rtile * 16 + 4 * v + (lane >> 4);
            const int gj = t * 16 + (lane & 15);
            if (gi < s1 && gj < s2) part[((size_t)split * s2 + gj) * s1 + gi] = acc[t][v];
        }
}

template <int CT>
void launch_gram_wide(Ctx* ctx, double flops, dim3 g, size_t shm, int n, int s1, int s2, int chunk, int rt, int self,
                      const double* X, int ldx, const double* Y, int ldy, double* part) {
    timed_launch_shm(ctx, kKGram, flops, k_gram_wide<CT>, g, dim3(512), shm, ctx->stream, n, s1, s2, chunk, rt, self,
                     X, ldx, Y, ldy, part);
}

// C = sum of the nsplit partial products.  A workgroup of 64 x kRedLanes
// threads owns 64 consecutive entries: lane y sums chunks y, y + kRedLanes, ...
// and the kRedLanes sums are added in lane order (a fixed order).
constexpr int kRedLanes = 16;
__global__ __launch_bounds__(64 * kRedLanes) void k_gram_reduce(int s1, int s2, int nsplit,
                                                                const double* __restrict__ part,
                                                                double* __restrict__ C, int ldc) {
    __shared__ double acc[kRedLanes][64];
    const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
    const int id = blockIdx.x * 64 + x;
    const size_t tot = (size_t)s1 * s2;
    double s = 0.0;
    if (id < s1 * s2)
        for (int p = y; p < nsplit; p += kRedLanes) s += part[(size_t)p * tot + id];
    acc[y][x] = s;
    __syncthreads();
    if (y == 0 && id < s1 * s2) {
        double t = 0.0;
        for (int l = 0; l < kRedLanes; ++l) t += acc[l][x];
        C[id % s1 + (size_t)(id / s1) * ldc] = t;
    }
}

// C = alpha X B + beta C (X: n x s, B: s x t).  grid.x: strips of 16
// kBlkWaves rows (one 16-row strip per wave), grid.y: 128-column blocks; a
// wave computes its 16 rows against the block's kBlkTiles column tiles, so
// X is read once per column block.  The block's columns of B are staged in
// LDS kGramKC rows at a time and shared by the eight waves, as in the Gram.
__global__ __launch_bounds__(512) void k_gemm_tall(int n, int s, int t, double alpha,
                                                   const double* __restrict__ X, int ldx,
                                                   const double* __restrict__ B, int ldb,
                                                   double beta, double* __restrict__ C, int ldc) {
    __shared__ double bsh[2][kGramKC * kGramLd];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the column blocks of one row strip read the same rows of X: they run on
    // one XCD one after another (grid: row strips x column blocks)
    int cb, strip;
    xcd_block_chunk(gridDim.y, gridDim.x, cb, strip);
    const int r0 = (strip * kBlkWaves + wave) * 16;
    const bool rows_on = r0 < n;  // this wave has output rows (all waves stage B)
    const int c0 = cb * kBlk;
    const int row = r0 + (lane & 15), kr = lane >> 4;
    const int jj = threadIdx.x >> 2, r8 = (threadIdx.x & 3) * 8;
    const bool jok = c0 + jj < t;
    const double* bcol = B + (size_t)(jok ? c0 + jj : 0) * ldb;
    double stg[8];
    auto load_stage = [&](int k0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + r8 + e;
            stg[e] = (jok && k < s) ? bcol[k] : 0.0;
        }
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bsh[buf][(r8 + e) * kGramLd + jj] = stg[e];
    };
    d4_t acc[kBlkTiles];
#pragma unroll
    for (int tt = 0; tt < kBlkTiles; ++tt) acc[tt] = d4_t{0.0, 0.0, 0.0, 0.0};
    load_stage(0);
    store_stage(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < s; k0 += kGramKC) {
        const bool more = k0 + kGramKC < s;
        if (more) load_stage(k0 + kGramKC);
        if (rows_on) {
            double a[kGramKC / 4];
#pragma unroll
            for (int u = 0; u < kGramKC / 4; ++u) {
                const int k = k0 + 4 * u + kr;
                a[u] = (row < n && k < s) ? X[(size_t)k * ldx + row] : 0.0;
            }
            const double* bb = bsh[buf] + kr * kGramLd + (lane & 15);
#pragma unroll
            for (int u = 0; u < kGramKC / 4; ++u)
#pragma unroll
                for (int tt = 0; tt < kBlkTiles; ++tt)
                    acc[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], bb[4 * u * kGramLd + tt * 16], acc[tt], 0,
                                                                   0, 0);
        }
        // the other buffer was last read before the previous barrier
        if (more) store_stage(1 - buf);
        __syncthreads();
        buf = 1 - buf;
    }
    if (!rows_on) return;
#pragma unroll
    for (int tt = 0; tt < kBlkTiles; ++tt) {
        const int cc = c0 + tt * 16 + (lane & 15);
        if (cc >= t) continue;
        for (int v = 0; v < 4; ++v) {
            const int rr = r0 + 4 * v + (lane >> 4);
            if (rr < n) {
                double* dst = C + (size_t)cc * ldc + rr;
                *dst = alpha * acc[tt][v] + (beta != 0.0 ? beta * *dst : 0.0);
            }
        }
    }
}

// The factorizations below treat nb matrices of a launch at once: matrix b's
// at base + b * stride (strides in elements); A(a, c) = A[a + c lda].

// 1 / sqrt(x) for normal x > 0, to about one ulp: the hardware's estimate, a
// third-order and a second-order step.
__device__ __forceinline__ double rsqrt_full(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double e = __builtin_fma(-x * y, y, 1.0);
    y = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
    e = __builtin_fma(-x * y, y, 1.0);
    return __builtin_fma(y * e, 0.5, y);
}

__device__ __forceinline__ double lane_value(double v, int lane) {  // lane: uniform
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

constexpr int kFacB = 32;           // block of the Cholesky factor and its inverse
constexpr int kFacLd = kFacB + 1;   // LDS column stride: a lane a column, no bank conflicts

// Block row j of the upper Cholesky factor R, left-looking: workgroup x forms
// tile (j, j + x) of A - R(0..j-1, j)^T R(0..j-1, j + x) and, again in each
// workgroup, the diagonal tile, on the matrix cores (one quadrant of both a
// wave); then wave 0 eliminates with a column of [diagonal | tile] in the
// registers of each lane, pivot row entries broadcast by lane reads: the
// diagonal's factor and the tile's triangular solve in one pass without LDS
// or barriers.  shift: per-matrix diagonal shifts (device) or null.
// All workgroups of a launch read the diagonal tile of A, so its factor goes
// to dbuf (two slots by the parity of j) and is copied into A by the next
// launch, whose workgroups do not read it; the last one's goes to A itself.
// Bound by that chain, ~10-16 us a block row; one workgroup updating the whole
// trailing matrix for each of the s pivots took 0.09 / 0.30 / 3.9 / 19 ms at
// s = 64 / 139 / 300 / 512 (whole factor with the flag's read-back), this
// 0.04 / 0.08 / 0.20 / 0.50 ms.
__global__ __launch_bounds__(256) void k_cholesky_row(int s, int j, double* __restrict__ A, int lda, size_t sa,
                                                      const double* __restrict__ shift, double* __restrict__ dbuf,
                                                      int* __restrict__ flag) {
    __shared__ double sm[2 * kFacB * kFacLd];
    A += blockIdx.y * sa;
    dbuf += (size_t)blockIdx.y * 2 * kFacB * kFacB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
    const int m0 = (wave & 1) * 16, n0 = (wave >> 1) * 16;
    const int oj = j * kFacB, ok = (j + blockIdx.x) * kFacB;
    const bool tile = blockIdx.x > 0, last = oj + kFacB >= s;
    const double sh = shift ? shift[blockIdx.y] : 0.0;
    if (j > 0 && !tile) {  // the previous diagonal factor, lower part zero
        const double* d = dbuf + ((j - 1) & 1) * kFacB * kFacB;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = threadIdx.x + 256 * u, r = id & 31, c = id >> 5;
            A[oj - kFacB + r + (size_t)(oj - kFacB + c) * lda] = d[id];
        }
    }
    auto col = [&](int c) { return A + (size_t)min(c, s - 1) * lda; };  // columns past the end are not stored
    const double *ca = col(oj + m0 + lm), *cd = col(oj + n0 + lm), *ct = col(ok + n0 + lm);
    double av[2][8], dv[2][8], tv[2][8];
    auto load = [&](int k0, int b) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + 4 * u + lk;
            av[b][u] = ca[k];
            dv[b][u] = cd[k];
            tv[b][u] = ct[k];  // workgroup 0 does its tile twice
        }
    };
    d4_t ad = {0.0, 0.0, 0.0, 0.0}, at = ad, od, ot;
    if (j > 0) load(0, 0);
    // this lane's entries of A itself
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = min(oj + m0 + 4 * v + lk, s - 1);
        od[v] = cd[r];
        ot[v] = ct[r];
    }
    for (int k0 = 0; k0 < oj; k0 += 2 * kFacB) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int k = k0 + b * kFacB;
            if (k >= oj) break;
            if (k + kFacB < oj) load(k + kFacB, 1 - b);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                ad = __builtin_amdgcn_mfma_f64_16x16x4f64(av[b][u], dv[b][u], ad, 0, 0, 0);
                at = __builtin_amdgcn_mfma_f64_16x16x4f64(av[b][u], tv[b][u], at, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = m0 + 4 * v + lk, c = n0 + lm;
        const bool in = oj + r < s && oj + c < s;  // beyond: the identity
        const double dd = od[v] + (r == c ? sh : 0.0) - ad[v];
        sm[r + c * kFacLd] = in ? dd : (r == c ? 1.0 : 0.0);
        sm[r + (kFacB + c) * kFacLd] = tile ? ot[v] - at[v] : 0.0;
    }
    __syncthreads();
    if (wave == 0) {
        double x[kFacB];
#pragma unroll
        for (int r = 0; r < kFacB; ++r) x[r] = sm[r + lane * kFacLd];
        bool bad = false;
#pragma unroll
        for (int i = 0; i < kFacB; ++i) {
            const double piv = lane_value(x[i], i);
            bad |= !(piv > 0.0);
            x[i] *= rsqrt_full(piv);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = i + 1; r < kFacB; ++r) {
                x[r] = __builtin_fma(-lane_value(x[i], r), x[i], x[r]);
                if ((r & 7) == 7) __builtin_amdgcn_sched_barrier(0);  // few broadcast entries live at once
            }
        }
#pragma unroll
        for (int r = 0; r < kFacB; ++r) sm[r + lane * kFacLd] = lane >= kFacB || r <= lane ? x[r] : 0.0;
        if (!tile && lane == 0) flag[blockIdx.y] = (j > 0 ? flag[blockIdx.y] : 0) | (bad ? 1 : 0);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int id = threadIdx.x + 256 * u, r = id & 31, c = id >> 5;
        if (!tile) {
            if (!last)
                dbuf[(j & 1) * kFacB * kFacB + id] = sm[r + c * kFacLd];
            else if (oj + r < s && oj + c < s)
                A[oj + r + (size_t)(oj + c) * lda] = sm[r + c * kFacLd];
        } else if (ok + c < s) {
            A[oj + r + (size_t)(ok + c) * lda] = sm[r + (kFacB + c) * kFacLd];
        }
        if (tile && ok + r < s) A[ok + r + (size_t)(oj + c) * lda] = 0.0;  // the tile below the diagonal
    }
}

// Diagonal blocks of Ri = R^-1: one wave a block, a column of R and one of the
// inverse in the registers of each lane, back substitution with lane reads.
__global__ __launch_bounds__(64) void k_tri_inverse_diag(int s, const double* __restrict__ R, int ldr, size_t sr,
                                                         double* __restrict__ Ri, int ldi, size_t si) {
    __shared__ double sm[kFacB * kFacLd];
    R += blockIdx.y * sr;
    Ri += blockIdx.y * si;
    const int lane = threadIdx.x, o = blockIdx.x * kFacB;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int id = lane + 64 * u, r = id & 31, c = id >> 5;
        double v = r == c ? 1.0 : 0.0;  // beyond the matrix: the identity
        if (o + c < s && r <= c) v = R[o + r + (size_t)(o + c) * ldr];
        sm[r + c * kFacLd] = v;
    }
    __syncthreads();
    const int c = lane & 31;
    double x[kFacB], y[kFacB];
#pragma unroll
    for (int r = 0; r < kFacB; ++r) {
        x[r] = sm[r + c * kFacLd];
        y[r] = r == c ? 1.0 : 0.0;
    }
    const double inv = 1.0 / sm[c + c * kFacLd];
#pragma unroll
    for (int i = kFacB - 1; i >= 0; --i) {
        y[i] *= lane_value(inv, i);
#pragma unroll
        for (int r = 0; r < i; ++r) y[r] = __builtin_fma(-lane_value(x[r], i), y[i], y[r]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFacB; ++r) sm[r + c * kFacLd] = y[r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int id = lane + 64 * u, r = id & 31, cc = id >> 5;
        if (o + r < s && o + cc < s) Ri[o + r + (size_t)(o + cc) * ldi] = sm[r + cc * kFacLd];
    }
}

// Block column J of Ri off the diagonal, given its diagonal blocks: upwards,
// Ri(I, J) = -Ri(I, I) sum_{K = I+1..J} R(I, K) Ri(K, J), the column kept in
// dynamic LDS (ld: its rows, padded), one quadrant of the tile a wave.  The
// columns are independent, so one launch does them all: 0.056 / 0.10 ms with
// the diagonal blocks at s = 300 / 512; block products a launch each over
// 128 x 128 blocks took 0.44 / 0.88 ms.
__global__ __launch_bounds__(256) void k_tri_inverse_cols(int s, const double* __restrict__ R, int ldr, size_t sr,
                                                          double* __restrict__ Ri, int ldi, size_t si, int ld) {
    extern __shared__ double col[];
    __shared__ double ws[kFacB * kFacLd];
    R += blockIdx.y * sr;
    Ri += blockIdx.y * si;
    const int J = gridDim.x - 1 - blockIdx.x, oj = J * kFacB;  // longest first
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
    const int m0 = (wave & 1) * 16, n0 = (wave >> 1) * 16;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int id = threadIdx.x + 256 * u, r = id & 31, c = id >> 5;
        col[oj + r + c * ld] = oj + r < s && oj + c < s ? Ri[oj + r + (size_t)(oj + c) * ldi] : 0.0;
    }
    for (int I = J - 1; I >= 0; --I) {
        const int oi = I * kFacB, n = oj + kFacB;
        const double* ra = R + oi + m0 + lm;
        double av[2][8], dv[8];
        auto load = [&](int k0, int b) {
#pragma unroll
            for (int u = 0; u < 8; ++u) av[b][u] = ra[(size_t)min(k0 + 4 * u + lk, s - 1) * ldr];  // beyond: times 0
        };
        load(oi + kFacB, 0);
#pragma unroll
        for (int u = 0; u < 8; ++u) dv[u] = Ri[oi + m0 + lm + (size_t)(oi + 4 * u + lk) * ldi];
        d4_t acc = {0.0, 0.0, 0.0, 0.0};
        __syncthreads();  // the column's rows from block I + 1 on are there, ws is free
        for (int k0 = oi + kFacB; k0 < n; k0 += 2 * kFacB) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int k = k0 + b * kFacB;
                if (k >= n) break;
                if (k + kFacB < n) load(k + kFacB, 1 - b);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[b][u], col[k + 4 * u + lk + (n0 + lm) * ld], acc, 0,
                                                               0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ws[m0 + 4 * v + lk + (n0 + lm) * kFacLd] = acc[v];
        __syncthreads();
        acc = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 8; ++u)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(dv[u], ws[4 * u + lk + (n0 + lm) * kFacLd], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) col[oi + m0 + 4 * v + lk + (n0 + lm) * ld] = -acc[v];
    }
    __syncthreads();
    for (int id = threadIdx.x; id < s * kFacB; id += 256) {
        const int c = id / s, r = id - c * s;
        if (oj + c < s && (r < oj || r >= oj + kFacB)) Ri[r + (size_t)(oj + c) * ldi] = r < oj ? col[r + c * ld] : 0.0;
    }
}

// Pair k of step `step` of the round-robin ordering of an even number m of
// indices (every pair meets once in m - 1 steps), ordered so that p < q.
__device__ __forceinline__ void rr_pair(int step, int k, int m, int& p, int& q) {
    if (k == 0) {
        p = step;
        q = m - 1;
    } else {
        p = (step + k) % (m - 1);
        q = (step - k + (m - 1)) % (m - 1);
    }
    if (p > q) {
        const int tmp = p;
        p = q;
        q = tmp;
    }
}

// Plane rotation (c, sv) that zeroes the off-diagonal entry of the symmetric
// 2 x 2 block [app apq; apq aqq] (the smaller of the two rotation angles):
// with h = aqq - app and g = 2 apq, t = sign(h) g / (|h| + sqrt(h^2 + g^2)).
// h and g are scaled by the larger one's exponent, so the squares neither
// overflow nor vanish.  No branch and no IEEE division or root sequence: the
// rotations are the serial chain of a step (in a launch of its own 16.7 -> 12.1 us a step).
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double& c, double& sv) {
    double h = aqq - app, g = 2.0 * apq;
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(h), fabs(g)));
    h = ldexp(h, ex);
    g = ldexp(g, ex);
    const double r2 = __builtin_fma(h, h, g * g);
    const double den = fabs(h) + r2 * rsqrt_full(r2);  // in [1/2, 4)
    double rc = __builtin_amdgcn_rcp(den);
    double e = __builtin_fma(-den, rc, 1.0);
    rc = __builtin_fma(rc * e, 1.0 + e, rc);
    const double gs = h >= 0.0 ? g : -g;
    double t = gs * rc;
    t = __builtin_fma(__builtin_fma(-den, t, gs), rc, t);
    const double cc = rsqrt_full(__builtin_fma(t, t, 1.0));
    const bool on = apq != 0.0;
    c = on ? cc : 1.0;
    sv = on ? t * cc : 0.0;
}

// Squared off-diagonal and total Frobenius norms of the s x s matrix T (ld),
// summed in a fixed order; every thread returns both.
__device__ __forceinline__ void jacobi_norms(int s, const double* T, int ld, double& offn, double& totn) {
    __shared__ double wsum[32];
    double o = 0.0, t = 0.0;
    for (int id = threadIdx.x; id < s * s; id += blockDim.x) {
        const int a = id % s, c = id / s;
        const double v = T[a + (size_t)c * ld];
        t += v * v;
        if (a != c) o += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) {
        o += __shfl_xor(o, off, 64);
        t += __shfl_xor(t, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        wsum[threadIdx.x >> 6] = o;
        wsum[16 + (threadIdx.x >> 6)] = t;
    }
    __syncthreads();
    double so = 0.0, st = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
        so += wsum[w];
        st += wsum[16 + w];
    }
    offn = so;
    totn = st;
    __syncthreads();  // wsum is reused by the next call
}

// Stopping test of the Jacobi sweeps: the off-diagonal Frobenius norm is below
// 1e-12 of the total, or, once it is below 1e-8, a sweep no longer halves it
// (rounding in the rotations keeps it near s eps |T|, so a fixed tighter
// bound may never be met).  prev: squared off-diagonal norm of the previous
// sweep (negative before the first).
__device__ __forceinline__ bool jacobi_done(double offn, double totn, double prev) {
    if (offn <= 1e-24 * totn || totn == 0.0) return true;
    return prev >= 0.0 && offn <= 1e-16 * totn && offn > 0.25 * prev;
}

// One step of the parallel Jacobi sweep: the np rotations (pp, qq, cs, sn)
// applied to both sides of T and to the columns of S.  The thread of pair
// block (k, l) forms rows p_k, q_k of J^T T on columns p_l, q_l and rotates
// those columns: the same products in the same order as a row pass followed
// by a column pass, with every entry of T read and written once.  A pair
// with q >= s (odd s) has the identity rotation and no row or column q.  Each
// thread advances its item indices by the workgroup size without dividing.
__device__ __forceinline__ void jacobi_apply(int s, int np, double* T, int ldt, double* S, int lds,
                                             const int* pp, const int* qq, const double* cs, const double* sn) {
    const int bd = blockDim.x;
    {
        const int nb = np * np, dk = bd % np, dl = bd / np;
        int k = threadIdx.x % np, l = threadIdx.x / np;
        for (int id = threadIdx.x; id < nb; id += bd) {
            const int pk = pp[k], qk = qq[k], pl = pp[l], ql = qq[l];
            const double va = T[pk + (size_t)pl * ldt];
            const double vb = ql < s ? T[pk + (size_t)ql * ldt] : 0.0;
            const double vc = qk < s ? T[qk + (size_t)pl * ldt] : 0.0;
            const double vd = qk < s && ql < s ? T[qk + (size_t)ql * ldt] : 0.0;
            const double ck = cs[k], sk = sn[k], cl = cs[l], sl = sn[l];
            const double r0x = ck * va - sk * vc, r0y = ck * vb - sk * vd;
            const double r1x = sk * va + ck * vc, r1y = sk * vb + ck * vd;
            T[pk + (size_t)pl * ldt] = cl * r0x - sl * r0y;
            if (ql < s) T[pk + (size_t)ql * ldt] = sl * r0x + cl * r0y;
            if (qk < s) T[qk + (size_t)pl * ldt] = cl * r1x - sl * r1y;
            if (qk < s && ql < s) T[qk + (size_t)ql * ldt] = sl * r1x + cl * r1y;
            k += dk;
            l += dl;
            if (k >= np) {
                k -= np;
                ++l;
            }
        }
    }
    const int ns = np * s, dr = bd % s, dq = bd / s;
    int r = threadIdx.x % s, k = threadIdx.x / s;
    for (int id = threadIdx.x; id < ns; id += bd) {
        if (qq[k] < s) {
            const double vp = S[r + (size_t)pp[k] * lds], vq = S[r + (size_t)qq[k] * lds];
            S[r + (size_t)pp[k] * lds] = cs[k] * vp - sn[k] * vq;
            S[r + (size_t)qq[k] * lds] = sn[k] * vp + cs[k] * vq;
        }
        r += dr;
        k += dq;
        if (r >= s) {
            r -= s;
            ++k;
        }
    }
}

// The one-workgroup sweeps (two copies of the matrix in LDS) take nb matrices of
// a launch at the price of one, ~2 us a step; a block step of 16 indices
// beyond takes ~16 us and np + 2 np^2 workgroups a matrix.  So the former serve
// s <= 56 and, where the blocks come in threes (64 < s <= 96), large batches:
// one matrix, LDS / blocked, s = 48 / 64 / 70 / 80 / 96 590 / 1088 / 1486 / 1809 / 3080
// against 762 / 838 / 1180 / 1287 / 1182 us; 32 matrices, s = 65 / 72 / 80 1350 /
// 1603 / 1989 against 1632 / 1647 / 1760; 52 (more than 1024 workgroups a step),
// s = 65 / 72 / 76 1332 / 1607 / 1820 against 2144 / 2187 / 2204.
constexpr int kJacLdsMax = 80;
inline bool jacobi_one_group(int nb, int s) {
    return s <= 56 || (s > 64 && s <= kJacLdsMax && nb >= (s <= 72 ? 32 : 49));
}

// Parallel cyclic Jacobi (round-robin pairing), one workgroup, on T and S
// (ld ldt, lds): per step, the np disjoint rotations, then jacobi_apply.
__device__ __forceinline__ void jacobi_sweeps(int s, double* T, int ldt, double* S, int lds, int max_sweeps) {
    const int m = s + (s & 1);
    const int np = m / 2;
    __shared__ double cs[kJacLdsMax / 2], sn[kJacLdsMax / 2];
    __shared__ int pp[kJacLdsMax / 2], qq[kJacLdsMax / 2];
    double prev = -1.0;  // off-diagonal norm^2 of the previous sweep
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        double offn, totn;
        jacobi_norms(s, T, ldt, offn, totn);
        if (jacobi_done(offn, totn, prev)) break;
        prev = offn;
        for (int step = 0; step < m - 1; ++step) {
            for (int k = threadIdx.x; k < np; k += blockDim.x) {
                int p, q;
                rr_pair(step, k, m, p, q);
                double c = 1.0, sv = 0.0;
                if (q < s)
                    jacobi_rotation(T[p + (size_t)p * ldt], T[q + (size_t)q * ldt], T[p + (size_t)q * ldt], c, sv);
                pp[k] = p;
                qq[k] = q;
                cs[k] = c;
                sn[k] = sv;
            }
            __syncthreads();
            jacobi_apply(s, np, T, ldt, S, lds, pp, qq, cs, sn);
            __syncthreads();
        }
    }
}

// Blocked Jacobi for matrices beyond the LDS of one compute unit, over all
// compute units.  The matrix is padded with zero rows and columns to sp (a
// multiple of 32) and cut into blocks of kJacB indices; step t of a sweep
// pairs the blocks by rr_pair.  For each block pair k_jacobi_step runs the
// rotations of every index pair between the two blocks once (in the first step of a sweep also those within the blocks), so
// a sweep meets each index pair once, as a cyclic sweep does, and leaves the
// product of its rotations in Q (32 x 32), which is applied on the matrix cores:
// T <- Q^T T Q and S <- S Q, one 32 x 32 tile a workgroup.
// Padding stays exactly zero (a zero off-diagonal has the identity rotation).
// One workgroup rotating T in global memory moved 2 s^2 doubles through one
// compute unit s - 1 times a sweep.  Whole eigenproblem, s = 99 / 300 / 512:
// 4.4 / 96 / 486 ms there, 1.8 / 4.8 / 9.3 ms here (as many sweeps).
constexpr int kJacB = 16, kJacT = 2 * kJacB;
constexpr int kJacLd = 48;  // LDS column stride: two columns' 16-row runs cover all banks

__global__ __launch_bounds__(256) void k_jacobi_init(int s, int sp, const double* __restrict__ A, int lda, size_t sa,
                                                     double* __restrict__ T, double* __restrict__ S,
                                                     int* __restrict__ done, double* __restrict__ prev) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.y;
    if (id == 0) {
        done[b] = 0;
        prev[b] = -1.0;
    }
    if (id >= sp * sp) return;
    const int r = id % sp, c = id / sp;
    A += b * sa;
    const size_t o = (size_t)b * sp * sp + id;
    double v = 0.0;
    if (r < s && c < s)
        v = r == c ? A[r + (size_t)r * lda] : 0.5 * (A[r + (size_t)c * lda] + A[c + (size_t)r * lda]);
    T[o] = v;
    S[o] = r == c ? 1.0 : 0.0;
}

// Pair index of block A in step `step` of rr_pair's order of m blocks.
__device__ __forceinline__ int rr_index(int step, int A, int m) {
    if (A == step || A == m - 1) return 0;
    const int e = A > step ? A - step : A - step + m - 1;
    return e <= (m - 2) / 2 ? e : m - 1 - e;
}

// One step in one launch (grid: pairs of the next step, then tiles; matrix).
// The first np workgroups find the rotations of step `next`: a block pair's
// 32 x 32 entries after this step, Q_k^T T Q_l of the four blocks (a wave each),
// then the rotations in LDS, a chain of LDS reads, two rotations (every thread
// computes those of its row and column pair itself, which saves a barrier) and
// LDS writes into the other buffer; their product goes to Qn.  The others
// apply this step's rotations Q: Tn = Q^T T Q, S <- S Q, one 32 x 32 tile a
// workgroup, one quadrant a wave.  norms (last step of a sweep): the tile's
// squared off-diagonal and total sums to part.  step < 0: the rotations of
// step `next` from T itself, nothing applied.
// Bound by the chain of rotations; with the rotations and the tiles in launches
// of their own a step took 12.1 + 6.3 us (s = 300), 15.9 in one.
__global__ __launch_bounds__(256) void k_jacobi_step(int sp, int step, int next, const double* __restrict__ T,
                                                     double* __restrict__ Tn, double* __restrict__ S,
                                                     const double* __restrict__ Q, double* __restrict__ Qn,
                                                     double* __restrict__ part, int norms,
                                                     const int* __restrict__ done) {
    if (done[blockIdx.y]) return;
    constexpr int kQ = kJacT * kJacT, kA = kJacT * kJacLd, kPs = kJacT * (kJacB + 1), kLd = kJacT + 2;
    __shared__ double sm[3 * kA];
    static_assert(4 * kPs <= 2 * kA && kJacT * kLd <= 3 * kA, "scratch within the LDS");
    const int np = sp / kJacT, nblk = sp / kJacB;
    const size_t mo = (size_t)blockIdx.y * sp * sp, qo = (size_t)blockIdx.y * np * kQ;
    T += mo;
    Q += qo;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
    if ((int)blockIdx.x < np) {
        double *t0 = sm, *t1 = sm + kA, *qq = sm + 2 * kA;
        int I, J;
        rr_pair(next, blockIdx.x, nblk, I, J);
        if (step < 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int id = threadIdx.x + 256 * u, r = id & 31, c = id >> 5;
                auto at = [&](int x) { return (x < kJacB ? I : J - 1) * kJacB + x; };
                t0[r + c * kJacLd] = T[at(r) + (size_t)at(c) * sp];
            }
        } else {
            // wave (a, b): block (a ? J : I, b ? J : I) of Q^T T Q
            const int a = wave & 1, b = wave >> 1, A = a ? J : I, B = b ? J : I;
            const int ka = rr_index(step, A, nblk), kb = rr_index(step, B, nblk);
            int Ia, Ja, Ib, Jb;
            rr_pair(step, ka, nblk, Ia, Ja);
            rr_pair(step, kb, nblk, Ib, Jb);
            const double* qa = Q + (size_t)ka * kQ + (A == Ja ? kJacB : 0) * kJacT;  // its 16 columns
            const double* qb = Q + (size_t)kb * kQ + (B == Jb ? kJacB : 0) * kJacT;
            double tv[2][8], bv[8], av[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = 4 * u + lk, col = (k < kJacB ? Ib : Jb - 1) * kJacB + k;
                tv[0][u] = T[Ia * kJacB + lm + (size_t)col * sp];
                tv[1][u] = T[Ja * kJacB + lm + (size_t)col * sp];
                bv[u] = qb[k + lm * kJacT];
                av[u] = qa[k + lm * kJacT];
            }
            double* ps = t1 + wave * kPs;  // this wave's 32 x 16 product T Q_l
            d4_t acc[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                acc[h] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[h][u], bv[u], acc[h], 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) ps[(h * kJacB + 4 * v + lk) * (kJacB + 1) + lm] = acc[h][v];
            }
            __syncthreads();
            d4_t n = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 8; ++u)
                n = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], ps[(4 * u + lk) * (kJacB + 1) + lm], n, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) t0[a * kJacB + 4 * v + lk + (b * kJacB + lm) * kJacLd] = n[v];
            __syncthreads();  // ps has been read
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = threadIdx.x + 256 * u, r = id & 31, c = id >> 5;
            qq[r + c * kJacLd] = r == c ? 1.0 : 0.0;
        }
        __syncthreads();
        const int k = threadIdx.x & 15, l = threadIdx.x >> 4;
        const bool all = next == 0;  // the first step of a sweep: also the pairs within the blocks
        const int nst = all ? kJacT - 1 : kJacB;
        for (int t = 0; t < nst; ++t) {
            int pk = k, qk = kJacB + ((k + t) & 15), pl = l, ql = kJacB + ((l + t) & 15);
            if (all) {
                rr_pair(t, k, kJacT, pk, qk);
                rr_pair(t, l, kJacT, pl, ql);
            }
            const double* a = t & 1 ? t1 : t0;
            double* b = t & 1 ? t0 : t1;
            const double va = a[pk + pl * kJacLd], vb = a[pk + ql * kJacLd], vc = a[qk + pl * kJacLd],
                         vd = a[qk + ql * kJacLd];
            const double q0p = qq[k + pl * kJacLd], q0q = qq[k + ql * kJacLd];
            const double q1p = qq[k + 16 + pl * kJacLd], q1q = qq[k + 16 + ql * kJacLd];
            double ck, sk, cl, sl;
            jacobi_rotation(a[pk + pk * kJacLd], a[qk + qk * kJacLd], a[pk + qk * kJacLd], ck, sk);
            jacobi_rotation(a[pl + pl * kJacLd], a[ql + ql * kJacLd], a[pl + ql * kJacLd], cl, sl);
            const double r0x = ck * va - sk * vc, r0y = ck * vb - sk * vd;
            const double r1x = sk * va + ck * vc, r1y = sk * vb + ck * vd;
            b[pk + pl * kJacLd] = cl * r0x - sl * r0y;
            b[pk + ql * kJacLd] = sl * r0x + cl * r0y;
            b[qk + pl * kJacLd] = cl * r1x - sl * r1y;
            b[qk + ql * kJacLd] = sl * r1x + cl * r1y;
            // columns pl, ql of Q are this thread row's alone during the step
            qq[k + pl * kJacLd] = cl * q0p - sl * q0q;
            qq[k + ql * kJacLd] = sl * q0p + cl * q0q;
            qq[k + 16 + pl * kJacLd] = cl * q1p - sl * q1q;
            qq[k + 16 + ql * kJacLd] = sl * q1p + cl * q1q;
            __syncthreads();
        }
        Qn += qo + (size_t)blockIdx.x * kQ;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = threadIdx.x + 256 * u;
            Qn[id] = qq[(id & 31) + (id >> 5) * kJacLd];
        }
        return;
    }
    double* ps = sm;
    const int tile = blockIdx.x - np, ky = tile / np, l = tile - ky * np;
    const bool is_t = ky < np;
    const int k = is_t ? ky : ky - np;
    const int m0 = (wave & 1) * 16, n0 = (wave >> 1) * 16;
    const double* M = is_t ? T : S + mo;
    double* Mn = is_t ? Tn + mo : S + mo;
    int Ik = 2 * k, Jk = 2 * k + 1, Il, Jl;
    rr_pair(step, l, nblk, Il, Jl);
    if (is_t) rr_pair(step, k, nblk, Ik, Jk);
    auto row = [&](int r) { return (r < kJacB ? Ik : Jk - 1) * kJacB + r; };
    auto col = [&](int c) { return (size_t)((c < kJacB ? Il : Jl - 1) * kJacB + c) * sp; };
    double bq[8], p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) bq[u] = Q[(size_t)l * kQ + 4 * u + lk + (n0 + lm) * kJacT];
    if (is_t) {
        double aq[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            aq[u] = Q[(size_t)k * kQ + 4 * u + lk + (m0 + lm) * kJacT];
            p[u] = M[row(4 * u + lk) + col(n0 + lm)];
        }
        d4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(aq[u], p[u], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) ps[m0 + 4 * v + lk + (n0 + lm) * kLd] = acc[v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = ps[m0 + lm + (4 * u + lk) * kLd];
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = M[row(m0 + lm) + col(4 * u + lk)];
        __syncthreads();  // both waves of these rows have read them
    }
    d4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(p[u], bq[u], acc, 0, 0, 0);
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = m0 + 4 * v + lk, c = n0 + lm;
        Mn[row(r) + col(c)] = acc[v];
        tot += acc[v] * acc[v];
        if (k != l || r != c) off += acc[v] * acc[v];
    }
    if (!norms || !is_t) return;
    off = wave_sum(off);
    tot = wave_sum(tot);
    __syncthreads();  // ps has been read
    if (lane == 0) {
        ps[wave] = off;
        ps[4 + wave] = tot;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double* o = part + (((size_t)blockIdx.y * np + k) * np + l) * 2;
        o[0] = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        o[1] = (ps[4] + ps[5]) + (ps[6] + ps[7]);
    }
}

// Stopping test of a sweep, one workgroup a matrix.
__global__ __launch_bounds__(256) void k_jacobi_check(int np, const double* __restrict__ part,
                                                      double* __restrict__ prev, int* __restrict__ done) {
    const int b = blockIdx.x;
    if (done[b]) return;
    __shared__ double w[8];
    part += (size_t)b * np * np * 2;
    double off = 0.0, tot = 0.0;
    for (int i = threadIdx.x; i < np * np; i += 256) {
        off += part[2 * i];
        tot += part[2 * i + 1];
    }
    off = wave_sum(off);
    tot = wave_sum(tot);
    if ((threadIdx.x & 63) == 0) {
        w[threadIdx.x >> 6] = off;
        w[4 + (threadIdx.x >> 6)] = tot;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        off = (w[0] + w[1]) + (w[2] + w[3]);
        tot = (w[4] + w[5]) + (w[6] + w[7]);
        done[b] = jacobi_done(off, tot, prev[b]);
        prev[b] = off;
    }
}

// The cyclic sweeps on copies of T and S in LDS (ld s), written back at the end.
__global__ __launch_bounds__(1024) void k_jacobi_lds(int s, double* __restrict__ T, int ldt, size_t st,
                                                     double* __restrict__ S, int lds, size_t ss, int max_sweeps) {
    extern __shared__ double sm[];
    T += blockIdx.x * st;
    S += blockIdx.x * ss;
    double* tl = sm;
    double* sl = sm + (size_t)s * s;
    for (int id = threadIdx.x; id < s * s; id += blockDim.x) {
        const int a = id % s, c = id / s;
        tl[id] = a == c ? T[a + (size_t)a * ldt] : 0.5 * (T[a + (size_t)c * ldt] + T[c + (size_t)a * ldt]);
        sl[id] = a == c ? 1.0 : 0.0;
    }
    __syncthreads();
    jacobi_sweeps(s, tl, s, sl, s, max_sweeps);
    for (int id = threadIdx.x; id < s * s; id += blockDim.x) {
        const int a = id % s, c = id / s;
        T[a + (size_t)c * ldt] = tl[id];
        S[a + (size_t)c * lds] = sl[id];
    }
}

// Sorts the eigenpairs by decreasing eigenvalue: column c of S goes to column
// rank(c) of Sout, and lam[rank(c)] = lam_unsorted[c] (ties keep index order).
// grid.y: matrix of the batch (S, Sout, lam_unsorted and lam at their strides).
__global__ void k_eig_permute(int s, const double* __restrict__ lam_unsorted, size_t slu,
                              const double* __restrict__ S, int lds, size_t ss, double* __restrict__ Sout, int ldo,
                              size_t so, double* __restrict__ lam, size_t sl) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= s * s) return;
    lam_unsorted += blockIdx.y * slu;
    S += blockIdx.y * ss;
    Sout += blockIdx.y * so;
    lam += blockIdx.y * sl;
    const int r = id % s, c = id / s;
    const double lc = lam_unsorted[c];
    int rank = 0;
    for (int j = 0; j < s; ++j) {
        const double lj = lam_unsorted[j];
        rank += (lj > lc) || (lj == lc && j < c);
    }
    Sout[r + (size_t)rank * ldo] = S[r + (size_t)c * lds];
    if (r == 0) lam[rank] = lc;
}

// lam[c] = v_c^T p_c / v_c^T v_c, one workgroup a column (grid.y: matrix): the
// Rayleigh quotients of the columns of V with P = T V.
__global__ __launch_bounds__(64) void k_rayleigh(int s, const double* __restrict__ V, const double* __restrict__ P,
                                                 int ld, size_t st, double* __restrict__ lam, size_t sl) {
    const double* v = V + blockIdx.y * st + (size_t)blockIdx.x * ld;
    const double* p = P + blockIdx.y * st + (size_t)blockIdx.x * ld;
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < s; i += 64) {
        a += v[i] * p[i];
        b += v[i] * v[i];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if (threadIdx.x == 0) lam[blockIdx.y * sl + blockIdx.x] = a / b;
}

__global__ void k_diag_copy(int s, const double* __restrict__ T, int ldt, size_t st, double* __restrict__ d,
                            size_t sd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < s) d[blockIdx.y * sd + i] = T[blockIdx.y * st + i + (size_t)i * ldt];
}

// out[b] = factor * trace(A_b), one workgroup per matrix.
__global__ void k_scaled_trace(int s, const double* __restrict__ A, int lda, size_t sa, double factor,
                               double* __restrict__ out) {
    __shared__ double w[16];
    A += blockIdx.x * sa;
    double v = 0.0;
    for (int i = threadIdx.x; i < s; i += blockDim.x) v += A[i + (size_t)i * lda];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += w[k];
        out[blockIdx.x] = factor * t;
    }
}

// C_b (m x n) = alpha op(A_b) op(B_b) + beta D_b with op(X) = X or X^T (TA, TB);
// op(A): m x kk.  Column-major, grid (32-column tiles, 32-row tiles, matrix of
// the batch), strides in elements; D may be C.  One 16 x 16 quadrant of the
// tile a wave; bound by the latency of its loads (from the L2), so the 16
// loads of 32 inner indices are issued together, those of the next 32 before
// this one's matrix steps (s = 300: 15 us a product).
struct SmallMat {
    const double* p;
    int ld;
    size_t st;
};
template <bool TA, bool TB>
__global__ __launch_bounds__(256) void k_small_gemm(int m, int n, int kk, double alpha, SmallMat A, SmallMat B,
                                                    double beta, SmallMat D, double* __restrict__ C, int ldc,
                                                    size_t sc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
    const int i0 = blockIdx.y * 32 + (wave & 1) * 16, j0 = blockIdx.x * 32 + (wave >> 1) * 16;
    if (i0 >= m || j0 >= n) return;
    const double* a = A.p + blockIdx.z * A.st;
    const double* b = B.p + blockIdx.z * B.st;
    const int ai = min(i0 + lm, m - 1), bj = min(j0 + lm, n - 1);  // rows and columns past the end are not stored
    double av[2][8], bv[2][8];
    auto load = [&](int k0, int s) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + 4 * u + lk, kc = min(k, kk - 1);
            av[s][u] = TA ? a[kc + (size_t)ai * A.ld] : a[ai + (size_t)kc * A.ld];
            bv[s][u] = TB ? b[bj + (size_t)kc * B.ld] : b[kc + (size_t)bj * B.ld];
            if (k >= kk) av[s][u] = bv[s][u] = 0.0;
        }
    };
    d4_t acc = {0.0, 0.0, 0.0, 0.0};
    load(0, 0);
    for (int k0 = 0; k0 < kk; k0 += 64) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int k = k0 + 32 * s;
            if (k >= kk) break;
            if (k + 32 < kk) load(k + 32, 1 - s);
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s][u], bv[s][u], acc, 0, 0, 0);
        }
    }
    const int j = j0 + lm;
    if (j >= n) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = i0 + 4 * v + lk;
        if (i >= m) continue;
        double r = alpha * acc[v];
        if (beta != 0.0) r += beta * D.p[blockIdx.z * D.st + i + (size_t)j * D.ld];
        C[blockIdx.z * sc + i + (size_t)j * ldc] = r;
    }
}

// C[i, j] /= d[i] + d[j] (s x s): the solution of the Sylvester equation
// D X + X D = C for diagonal D.
__global__ void k_sylvester_diag(int s, const double* __restrict__ d, double* __restrict__ C, int ldc) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= s * s) return;
    const int i = id % s, j = id / s;
    C[i + (size_t)j * ldc] /= d[i] + d[j];
}

// out[i] = base[i] (0 when null) + sum_j w[j] V[i, j]^2 (V: n x k, ldv).
__global__ void k_weighted_squares(int n, int k, const double* __restrict__ V, int ldv, const double* __restrict__ w,
                                   const double* __restrict__ base, double* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = 0.0;
    for (int j = 0; j < k; ++j) {
        const double v = V[i + (size_t)j * ldv];
        acc += w[j] * v * v;
    }
    out[i] = (base ? base[i] : 0.0) + acc;
}

__global__ void k_scale_rows(int s, int t, const double* __restrict__ d, double* __restrict__ B, int ldb) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= s * t) return;
    const int i = id % s, j = id / s;
    B[i + (size_t)j * ldb] *= d[i];
}

}  // namespace

void gram(Ctx* ctx, DenseWork& w, int n, int s1, int s2, const double* X, int ldx, const double* Y,
          int ldy, double* C, int ldc, bool bf16) {
    if (!bf16 && s2 <= 16 * kWideMaxCT) {
        const int ct = ceil_div(s2, 16), rtt = ceil_div(s1, 16);
        const int nrb = ceil_div(rtt, 8), rt = ceil_div(rtt, nrb);
        int cus = 0;
        HINV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
        // about one workgroup a compute unit (the staging takes most of the
        // LDS), chunks of at least 256 rows in whole K steps
        int nsplit = std::max(1, std::min(ceil_div(cus, nrb), ceil_div(n, 256)));
        const int chunk = ceil_div(ceil_div(n, nsplit), kWideKC) * kWideKC;
        nsplit = ceil_div(n, chunk);
        w.part.ensure((size_t)nsplit * s1 * s2);
        const size_t shm = sizeof(double) * 2 * kWideKC * wide_ld(ct);
        const int self = X == Y && ldx == ldy && s1 <= s2;
        const dim3 g(nrb, nsplit);
        const double flops = 2.0 * n * s1 * s2;
        switch (ct) {
#define HINV_WIDE(c) \
    case c: launch_gram_wide<c>(ctx, flops, g, shm, n, s1, s2, chunk, rt, self, X, ldx, Y, ldy, w.part.get()); break;
            HINV_WIDE(1) HINV_WIDE(2) HINV_WIDE(3) HINV_WIDE(4) HINV_WIDE(5) HINV_WIDE(6) HINV_WIDE(7) HINV_WIDE(8)
            HINV_WIDE(9) HINV_WIDE(10) HINV_WIDE(11) HINV_WIDE(12) HINV_WIDE(13) HINV_WIDE(14) HINV_WIDE(15)
            default: launch_gram_wide<16>(ctx, flops, g, shm, n, s1, s2, chunk, rt, self, X, ldx, Y, ldy, w.part.get());
#undef HINV_WIDE
        }
        HINV_LAUNCH_CHECK();
        k_gram_reduce<<<ceil_div(s1 * s2, 64), 64 * kRedLanes, 0, ctx->stream>>>(s1, s2, nsplit, w.part.get(), C,
                                                                                ldc);
        HINV_LAUNCH_CHECK();
        return;
    }
    const int blocks = ((s1 + kBlk - 1) / kBlk) * ((s2 + kBlk - 1) / kBlk);
    // K split: about 2048 workgroups, chunks of at least 256 rows (a multiple
    // of the 16-row matrix-core step)
    int nsplit = std::max(1, std::min(ceil_div(2048, blocks), ceil_div(n, 256)));
    const int chunk = ceil_div(ceil_div(n, nsplit), kGramKC) * kGramKC;  // a multiple of both kernels' K steps
    nsplit = ceil_div(n, chunk);
    w.part.ensure((size_t)nsplit * s1 * s2);
    const double flops = 2.0 * n * s1 * s2;
    if (bf16)
        timed_launch(ctx, kKGram, flops, k_gram_bf16, dim3(blocks, nsplit), dim3(64 * kBlkWaves), ctx->stream,
                     n, s1, s2, chunk, X, ldx, Y, ldy, w.part.get());
    else
        timed_launch(ctx, kKGram, flops, k_gram_f64, dim3(blocks, nsplit), dim3(64 * kBlkWaves), ctx->stream,
                     n, s1, s2, chunk, X, ldx, Y, ldy, w.part.get());
    HINV_LAUNCH_CHECK();
    k_gram_reduce<<<ceil_div(s1 * s2, 64), 64 * kRedLanes, 0, ctx->stream>>>(s1, s2, nsplit, w.part.get(), C,
                                                                            ldc);
    HINV_LAUNCH_CHECK();
}

void gemm_tall(Ctx* ctx, int n, int s, int t, double alpha, const double* X, int ldx,
               const double* B, int ldb, double beta, double* C, int ldc) {
    if (n <= 0 || t <= 0) return;
    const dim3 g(ceil_div(ceil_div(n, 16), kBlkWaves), ceil_div(t, kBlk));
    k_gemm_tall<<<g, 64 * kBlkWaves, 0, ctx->stream>>>(n, s, t, alpha, X, ldx, B, ldb, beta, C, ldc);
    HINV_LAUNCH_CHECK();
}

// Whether a one-workgroup kernel may stage `bytes` of dynamic LDS on the
// context's device (with room for its static LDS, at most 8 KB here).
bool lds_fits(Ctx* ctx, size_t bytes) {
    int v = 0;
    HINV_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, ctx->device));
    return bytes + 8192 <= (size_t)v;
}

bool cholesky_upper(Ctx* ctx, DenseWork& w, int nb, int s, double* A, int lda, size_t sa,
                    const double* shift) {
    if (nb <= 0) return true;
    w.flag.ensure(nb);
    w.tmp.ensure((size_t)nb * 2 * kFacB * kFacB);
    const int nblk = ceil_div(s, kFacB);
    for (int j = 0; j < nblk; ++j)
        k_cholesky_row<<<dim3(nblk - j, nb), 256, 0, ctx->stream>>>(s, j, A, lda, sa, shift, w.tmp.get(),
                                                                    w.flag.get());
    HINV_LAUNCH_CHECK();
    std::vector<int> bad(nb);
    HINV_HIP(hipMemcpyAsync(bad.data(), w.flag.get(), sizeof(int) * nb, hipMemcpyDeviceToHost, ctx->stream));
    HINV_HIP(hipStreamSynchronize(ctx->stream));
    for (int b : bad)
        if (b) return false;
    return true;
}

void tri_inverse_upper(Ctx* ctx, DenseWork& w, int nb, int s, const double* R, int ldr, size_t sr, double* Rinv,
                       int ldi, size_t si) {
    if (nb <= 0 || s <= 0) return;
    const int nblk = ceil_div(s, kFacB), ld = nblk * kFacB + 2;
    k_tri_inverse_diag<<<dim3(nblk, nb), 64, 0, ctx->stream>>>(s, R, ldr, sr, Rinv, ldi, si);
    HINV_LAUNCH_CHECK();
    if (nblk == 1) return;
    const size_t shm = sizeof(double) * kFacB * ld;  // 129 KB at the largest s, 512
    k_tri_inverse_cols<<<dim3(nblk, nb), 256, shm, ctx->stream>>>(s, R, ldr, sr, Rinv, ldi, si, ld);
    HINV_LAUNCH_CHECK();
}

void sym_eig(Ctx* ctx, DenseWork& w, int nb, int s, double* T, int ldt, size_t st, double* S, int lds, size_t ss,
             double* lam, size_t sl) {
    if (s > 512) fail(HINV_EINVAL, "eigenproblem larger than 512");
    if (nb <= 0 || s <= 0) return;
    const size_t s2 = (size_t)s * s;
    const int sp = ceil_div(s, kJacT) * kJacT;
    const size_t sp2 = (size_t)sp * sp, shm = sizeof(double) * 2 * s2;
    w.part.ensure(nb * (3 * sp2 + s));
    double* lam_u = w.part.get() + nb * 3 * sp2;
    constexpr int kMaxSweeps = 40;
    // lam_u and the columns of V, sorted
    auto sorted = [&](const double* V, int ldv, size_t sv) {
        k_eig_permute<<<dim3(ceil_div(s * s, 256), nb), 256, 0, ctx->stream>>>(s, lam_u, s, V, ldv, sv, S, lds, ss,
                                                                                lam, sl);
        HINV_LAUNCH_CHECK();
    };
    if (jacobi_one_group(nb, s) && lds_fits(ctx, shm)) {
        double* Stmp = w.part.get();
        k_jacobi_lds<<<nb, 1024, shm, ctx->stream>>>(s, T, ldt, st, Stmp, s, s2, kMaxSweeps);
        HINV_LAUNCH_CHECK();
        k_diag_copy<<<dim3(ceil_div(s, 256), nb), 256, 0, ctx->stream>>>(s, T, ldt, st, lam_u, s);
        HINV_LAUNCH_CHECK();
        sorted(Stmp, s, s2);
        return;
    }
    const int np = sp / kJacT, nsteps = sp / kJacB - 1;
    const size_t q1 = (size_t)np * kJacT * kJacT, p1 = (size_t)np * np * 2;
    w.rot.ensure(nb * (2 * q1 + p1 + 1));
    w.flag.ensure(nb);
    double* const Q[2] = {w.rot.get(), w.rot.get() + nb * q1};
    double* part = Q[1] + nb * q1;
    double* prev = part + nb * p1;
    // T alternates between two buffers (the next rotations are found while the
    // tiles are written), S is rotated in place
    double* const Tb[2] = {w.part.get(), w.part.get() + nb * sp2};
    double* Tp = Tb[0];
    double* Sp = Tb[1] + nb * sp2;
    int* done = w.flag.get();
    hipStream_t q = ctx->stream;
    k_jacobi_init<<<dim3(ceil_div(sp * sp, 256), nb), 256, 0, q>>>(s, sp, T, ldt, st, Tp, Sp, done, prev);
    HINV_LAUNCH_CHECK();
    std::vector<int> hd(nb);
    k_jacobi_step<<<dim3(np, nb), 256, 0, q>>>(sp, -1, 0, Tb[0], nullptr, nullptr, Q[0], Q[0], nullptr, 0, done);
    HINV_LAUNCH_CHECK();
    int cur = 0;
    for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
        for (int t = 0; t < nsteps; ++t) {
            k_jacobi_step<<<dim3(np + 2 * np * np, nb), 256, 0, q>>>(sp, t, (t + 1) % nsteps, Tb[cur], Tb[1 - cur], Sp,
                                                                     Q[cur], Q[1 - cur], part, t == nsteps - 1, done);
            cur = 1 - cur;
        }
        HINV_LAUNCH_CHECK();
        k_jacobi_check<<<nb, 256, 0, q>>>(np, part, prev, done);
        HINV_LAUNCH_CHECK();
        // A dense matrix takes about ten sweeps at s = 64, thirteen at 300: the first
        // ones are enqueued without asking (a finished matrix skips them)
        if (sweep < 4) continue;
        HINV_HIP(hipMemcpyAsync(hd.data(), done, sizeof(int) * nb, hipMemcpyDeviceToHost, q));
        HINV_HIP(hipStreamSynchronize(q));
        if (std::all_of(hd.begin(), hd.end(), [](int v) { return v != 0; })) break;
    }
    // One Newton-Schulz step V = S (3 I - S^T S) / 2 takes the rounding of the
    // thousands of rotations out of S, and the Rayleigh quotients of T with V
    // out of the eigenvalues: at s = 300 orthogonality 1.3e-13 -> 1.8e-15, error
    // of the eigenvalues relative to the largest 1.2e-13 -> 7e-16.
    w.tmp.ensure(nb * sp2);
    double* V = w.tmp.get();
    const dim3 gs(ceil_div(s, 32), ceil_div(s, 32), nb);
    const SmallMat none{nullptr, 0, 0}, mS{Sp, sp, sp2}, mG{Tp, sp, sp2};
    k_small_gemm<true, false><<<gs, 256, 0, q>>>(s, s, s, 1.0, mS, mS, 0.0, none, Tp, sp, sp2);
    k_small_gemm<false, false><<<gs, 256, 0, q>>>(s, s, s, -0.5, mS, mG, 1.5, mS, V, sp, sp2);
    k_small_gemm<false, false><<<gs, 256, 0, q>>>(s, s, s, 1.0, SmallMat{T, ldt, st}, SmallMat{V, sp, sp2}, 0.0, none,
                                                  Tp, sp, sp2);
    k_rayleigh<<<dim3(s, nb), 64, 0, q>>>(s, V, Tp, sp, sp2, lam_u, s);
    HINV_LAUNCH_CHECK();
    sorted(V, sp, sp2);
}

void scaled_trace(Ctx* ctx, int nb, int s, const double* A, int lda, size_t sa, double factor, double* out) {
    if (nb <= 0) return;
    k_scaled_trace<<<nb, 1024, 0, ctx->stream>>>(s, A, lda, sa, factor, out);
    HINV_LAUNCH_CHECK();
}

void small_gemm(Ctx* ctx, bool ta, bool tb, int m, int n, int kk, double alpha, const double* A, int lda,
                const double* B, int ldb, double beta, double* C, int ldc) {
    if (m * n == 0) return;
    const dim3 g(ceil_div(n, 32), ceil_div(m, 32), 1);
    const SmallMat a{A, lda, 0}, b{B, ldb, 0}, c{C, ldc, 0};
    auto run = [&](auto kern) { kern<<<g, 256, 0, ctx->stream>>>(m, n, kk, alpha, a, b, beta, c, C, ldc, 0); };
    if (ta)
        run(tb ? k_small_gemm<true, true> : k_small_gemm<true, false>);
    else
        run(tb ? k_small_gemm<false, true> : k_small_gemm<false, false>);
    HINV_LAUNCH_CHECK();
}

void sylvester_diag(Ctx* ctx, int s, const double* d, double* C, int ldc) {
    if (s == 0) return;
    k_sylvester_diag<<<ceil_div((long)s * s, 256), 256, 0, ctx->stream>>>(s, d, C, ldc);
    HINV_LAUNCH_CHECK();
}

void weighted_squares(Ctx* ctx, int n, int k, const double* V, int ldv, const double* w, const double* base,
                      double* out) {
    k_weighted_squares<<<ceil_div(n, 256), 256, 0, ctx->stream>>>(n, k, V, ldv, w, base, out);
    HINV_LAUNCH_CHECK();
}

void scale_rows(Ctx* ctx, int s, int t, const double* d, double* B, int ldb) {
    if (s * t == 0) return;
    k_scale_rows<<<ceil_div(s * t, 256), 256, 0, ctx->stream>>>(s, t, d, B, ldb);
    HINV_LAUNCH_CHECK();
}

}  // namespace hinv
