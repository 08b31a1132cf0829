// Fused multigrid V-cycle and PCG kernels (included by solver.hip only).
//
// V-cycle, per level above the bottom (N_l > kBottomN), two kernels on wave rows
// (waverow.h):
//   k_down: x2 = S(b) (two Chebyshev steps from zero), r = b - A x2, b_coarse = P^T r
//   k_up:   x = x2 + P x_coarse, then two Chebyshev steps on A x = b
// or, with few columns, several coarse levels a launch on LDS tiles (k_down2,
// k_up_chain), and one kernel for all levels with N_l <= kBottomN (one workgroup
// per column, in FP32, the coarsest level solved with its dense inverse).
// PCG reductions: every workgroup writes its partial sum, and each workgroup of
// the next launch that needs the total sums the column's partials in a fixed order.
#pragma once

#include "grid.h"
#include "solver.h"

namespace hinv {

// Workgroup barrier for data exchanged through LDS.  __syncthreads() also
// orders global memory, so every wave first waits for all of its outstanding
// global loads; no kernel here exchanges data through global memory within a
// launch (each reads buffers that only earlier launches write), so with this
// barrier loads issued before it stay in flight across it and their latency
// overlaps the staging and reductions that follow.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kTFSmall = 16, kTFWide = 18;  // tile sides of the r^T z partials of few columns
constexpr int kTPair = 4;      // k_down2: level-C tile side
constexpr int kPairMaxN = 256;  // k_down2 pairs levels whose finer one has N_l <= this
constexpr int kTFChain = 16;   // k_up_chain: level-0 tile side
constexpr int kChainLen = 4;   // k_up_chain: levels a launch (measured: 4 > 2 at N = 1024)
constexpr int kFewCols = 8;    // calls below this many columns are latency bound
constexpr int kBottomN = 32;   // levels with N_l <= kBottomN run in the bottom kernel
constexpr int kBottomLevels = 3;  // at most (N_l = 32, 16, 8)

// Chebyshev degree-2 coefficients passed to the smoothing kernels.
struct ChebCoef {
    double inv_theta, theta, cA, cB, c1;  // pre: x = cA d0 + cB D^-1 r1; post: (1 + c1) d0 + cB D^-1 r1
};

// In-kernel reductions: every workgroup writes one partial sum per column to
// part[col * stride + blk]; a later kernel (after the kernel boundary, so no
// fences are needed) sums them in a fixed order.
// First phase: this thread's strided share of nblk >= 1 partials, the first
// kShareLoads per thread loaded without branches (clamped index, dropped
// afterwards), so that they are in flight together with the caller's other
// loads (a loop waits for each load it accumulates); more partials than
// kShareLoads per thread follow in a loop.  Summed in index order.
constexpr int kShareLoads = 4;
__device__ inline double partial_share(const double* part, int col, int stride, int nblk) {
    const double* p = part + (size_t)col * stride;
    const int t = threadIdx.x, nt = blockDim.x;
    double v[kShareLoads];
#pragma unroll
    for (int k = 0; k < kShareLoads; ++k) v[k] = p[min(t + k * nt, nblk - 1)];
    double s = t < nblk ? v[0] : 0.0;
#pragma unroll
    for (int k = 1; k < kShareLoads; ++k)
        if (t + k * nt < nblk) s += v[k];
    for (int b = t + kShareLoads * nt; b < nblk; b += nt) s += p[b];
    return s;
}

// Index i clamped into the mesh [0, N]: loads are issued without a branch, at a
// valid node for every slot, and the off-mesh ones dropped afterwards (a load
// inside a branch makes the wave wait for it there).
__device__ inline int clamp_node(int i, int N) { return min(max(i, 0), N); }

// A value the same in every lane of the wave, moved to a scalar register:
// integer division runs on the vector unit, and its result would otherwise
// keep the addresses formed from it in vector registers.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Waves of the workgroup as a uniform value (read once, outside the
// single-thread code that sums the per-wave slots).
__device__ inline int group_waves() { return __builtin_amdgcn_readfirstlane((int)(blockDim.x >> 6)); }

// Sum of the first nw of 16 wave slots in LDS, in index order (all reads are
// issued together).
__device__ inline double slot_sum(const double* ps, int nw) {
    double q[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) q[w] = ps[w];
    double t = q[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) t = w < nw ? t + q[w] : t;
    return t;
}

// Second phase: the workgroup total of the shares, returned to every thread
// (each sums the wave slots itself: one barrier).  The slots of a call stay
// in use until the workgroup's next barrier.
__device__ inline double share_total(double s) {
    __shared__ __attribute__((aligned(16))) double ps[16];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) ps[threadIdx.x >> 6] = s;
    lds_barrier();
    return slot_sum(ps, group_waves());
}

// Workgroup total of the partials in the order in which a workgroup of bd
// threads (a multiple of 64, at most 1024) would take it (partial_share,
// then share_total), whatever the size of this one: the shares of bd virtual
// threads, summed wave by wave.  vt_first issues this thread's first loads.
constexpr int kVtMax = 4;  // virtual threads a thread of a 256-thread workgroup stands for
struct VtShare {
    double v[kVtMax];
};
__device__ inline VtShare vt_first(const double* part, int col, int stride, int nblk) {
    const double* p = part + (size_t)col * stride;
    VtShare s;
#pragma unroll
    for (int k = 0; k < kVtMax; ++k) s.v[k] = p[min((int)(threadIdx.x + k * blockDim.x), nblk - 1)];
    return s;
}
// on: thread 0's reading of the column's flag, returned to every thread (one
// decision for the workgroup where the launch may clear the flag).
__device__ inline double vt_total(VtShare s, const double* part, int col, int stride, int nblk, int bd, int& on) {
    __shared__ __attribute__((aligned(16))) double ps[16];
    __shared__ int flag;
    if (threadIdx.x == 0) flag = on;
    const double* p = part + (size_t)col * stride;
#pragma unroll
    for (int k = 0; k < kVtMax; ++k) {
        const int vt = threadIdx.x + k * blockDim.x;
        if (k * (int)blockDim.x >= bd) break;  // uniform
        double t = vt < nblk && vt < bd ? s.v[k] : 0.0;
        if (vt < bd)
            for (int b = vt + bd; b < nblk; b += bd) t += p[b];
        t = wave_sum(t);
        if ((threadIdx.x & 63) == 0) ps[vt >> 6] = t;
    }
    lds_barrier();
    on = uniform(flag);
    return slot_sum(ps, bd >> 6);
}

// Partial-sum buffers of the PCG inner products ([ncols][stride] each).
struct PcgRed {
    double* rz;
    double* pq;
    double* rr;
    int stride;
    int nrz;  // number of partials of r^T z (workgroups, or tiles, of the last V-cycle kernel)
    int npq;  // number of partials of p^T q (workgroups of the apply kernel)
    int nrr;  // number of partials of r^T r (workgroups of the kernel that updates r)
    int per;  // node blocks of 256 per workgroup: sets the threads of the linear vector kernels
    int chunk;  // consecutive nodes per workgroup of the linear vector kernels (<= kVecNodes threads)
};

// Threads per workgroup of the linear PCG vector kernels: 256 per node block up to
// 1024, so a workgroup covers its 256 per nodes in at most kVecNodes passes.
__host__ __device__ inline int vec_threads(int per) { return per >= 4 ? 1024 : 256 * per; }
constexpr int kVecNodes = 4;

// Workgroup sum with its own LDS slot; result valid in thread 0.
__device__ inline double group_sum(double v) {
    __shared__ __attribute__((aligned(16))) double part[16];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    lds_barrier();
    return threadIdx.x < 64 ? slot_sum(part, group_waves()) : 0.0;
}

// The same with the first kShareLoads partials of each of V virtual threads a
// thread loaded ahead (more of them follow in a loop).
template <int V>
struct VtRest {
    double v[V][kShareLoads];
};
template <int V>
__device__ inline VtRest<V> vt_rest(const double* part, int col, int stride, int nblk, int bd) {
    const double* p = part + (size_t)col * stride;
    VtRest<V> s;
#pragma unroll
    for (int h = 0; h < V; ++h)
#pragma unroll
        for (int k = 0; k < kShareLoads; ++k)
            s.v[h][k] = p[min((int)(threadIdx.x + h * blockDim.x) + k * bd, nblk - 1)];
    return s;
}
template <int V>
__device__ inline double vt_rest_total(const VtRest<V>& s, const double* part, int col, int stride, int nblk, int bd) {
    __shared__ __attribute__((aligned(16))) double ps[16];
    const double* p = part + (size_t)col * stride;
#pragma unroll
    for (int h = 0; h < V; ++h) {
        if (h * (int)blockDim.x >= bd) break;  // uniform
        const int vt = threadIdx.x + h * blockDim.x;
        double t = vt < nblk ? s.v[h][0] : 0.0;
#pragma unroll
        for (int k = 1; k < kShareLoads; ++k)
            if (vt + k * bd < nblk) t += s.v[h][k];
        for (int b = vt + kShareLoads * bd; b < nblk; b += bd) t += p[b];
        t = wave_sum(t);
        if ((threadIdx.x & 63) == 0) ps[vt >> 6] = t;
    }
    lds_barrier();
    return slot_sum(ps, bd >> 6);
}

// alpha of a column from its r^T z and p^T q (0 on breakdown); the lead
// workgroup records the iteration and stops a column that broke down.
__device__ inline double pcg_alpha(double rz, double pq, ColState* st, int* act, bool lead) {
    const double alpha = pq > 0.0 ? rz / pq : 0.0;
    if (lead && threadIdx.x == 0) {
        st->rz = rz;
        st->pq = pq;
        st->alpha = alpha;
        st->its += 1.0;
        if (!(pq > 0.0)) *act = 0;
    }
    return alpha;
}

// Convergence test in the first kernel after the PCG step: r^T r is summed
// from its partials (share: this thread's part of them, loaded ahead by the
// caller); a column at its tolerance stops (every workgroup reaches the same
// decision; the lead workgroup records it).  The launch does not read act: a
// column that had stopped before still has the r^T r it stopped with, and one
// that never ran (or broke down) costs a cycle on vectors nothing reads.
__device__ inline bool column_done_share(double share, const PcgRed& red, int col, const ColState* st, int* act,
                                         bool lead) {
    const double rr = share_total(share);
    const ColState& c = st[col];
    const bool done = rr <= c.tol2 * c.bb;
    if (lead && threadIdx.x == 0 && done) act[col] = 0;
    return done;
}

// Flag of a column through the scalar cache, for launches that do not write
// the flags (a scalar load is not queued behind the vector loads).
__device__ inline int column_on(const int* act, int col) {
    if (!act) return 1;
    return *reinterpret_cast<const __attribute__((address_space(4))) int*>(reinterpret_cast<uintptr_t>(act + col));
}

// XCD-aware tile order.  The hardware hands consecutive workgroups to the
// eight XCDs in turn, so in the plain order the tiles next to a tile (which
// read its halo rows) run on other XCDs and fetch those rows into their own
// L2 again.  Here the j-th workgroup of XCD x (dispatch index h = 8 j + x)
// takes logical tile x P + j with P = floor(T / 8) of the T workgroups: each
// XCD sweeps a contiguous run of tiles in row-major order (x fastest, then y,
// then the column block), so left/right and most upper/lower halos come from
// its own L2.  The last T - 8 P workgroups keep the plain order.  A
// bijection of [0, T); returns the logical (x, y, z) of this workgroup.
// The grid's extents with the reciprocals of the two divisions (an integer
// division costs ~40 instructions of a latency-bound kernel's start):
// (n + 1/2) / d lies at least 1 / (2 d) from an integer and the product errs by
// far less, so the truncation is exact.
struct TileMap {
    int X, XY, T;
    double inv_x, inv_xy;
    __host__ explicit TileMap(dim3 g)
        : X(g.x), XY(g.x * g.y), T(g.x * g.y * g.z), inv_x(1.0 / g.x), inv_xy(1.0 / ((double)g.x * g.y)) {}
};
__device__ inline int fast_div(int n, double inv) { return uniform((int)(((double)n + 0.5) * inv)); }

__device__ inline int3 xcd_tile(const TileMap& g) {
    const int h = blockIdx.x + g.X * blockIdx.y + g.XY * blockIdx.z;
    const int P = g.T >> 3;
    const int L = h < 8 * P ? (h & 7) * P + (h >> 3) : h;
    const int z = fast_div(L, g.inv_xy), r = L - z * g.XY, y = fast_div(r, g.inv_x);
    return make_int3(r - y * g.X, y, z);
}

}  // namespace hinv

#include "waverow.h"

namespace hinv {

// ------------------------------------------------- two levels a launch ---
// Few columns make the coarse levels latency bound: a launch there costs
// ~4.5 us however small its level.  k_down2 does the down steps of two
// consecutive levels F (N) and M (N/2) in one launch, k_up_chain the up
// steps of up to kChainMax levels: each workgroup recomputes the coarser
// values its tile needs on a larger tile (redundant work on the halo instead
// of more launches).  The arithmetic per node is that of k_down / k_up, so
// the cycle's result is the same bit for bit.

// Grid: (tiles over level-C x, tiles over level-C y, column blocks), C = N/4.
// Level-C tile [K0, K0+kT) x [L0, L0+kT) needs b_M on level-M nodes
// [2 K0 - 3, 2 K1 + 3] (the k_down tile of width MW = 2 kT + 5), which in
// turn needs b_F on the level-F tile of width FW = 2 MW + 5.  Writes x2_F and
// x2_M, and b_M (read again by the up step of level M) on the nodes the tile
// owns, and b_C on the level-C tile.
template <typename T, class Op, int kT, int NT>
__global__ __launch_bounds__(NT) void k_down2(Op opF_, Op opM_, const T* __restrict__ bF, T* __restrict__ xF,
                                               int ldF, T* __restrict__ bM, T* __restrict__ xM, int ldM,
                                               T* __restrict__ bC, int ldC, int dirichlet,
                                               int* __restrict__ act, ChebCoef cc, PcgRed red,
                                               ColState* __restrict__ st, int check, int nc, int cb, TileMap tm) {
    constexpr int MW = 2 * kT + 5, FW = 2 * MW + 5, NM = MW * MW, NF = FW * FW;
    constexpr bool NE = kNorthEast<Op>;
    __shared__ T fb[NF], fx[NF], fr[NF];
    __shared__ T fc[NE ? NF : 1], fe[NF], fn[NF], fdv[NF], fg[NE ? NF : 1];
    __shared__ T mb[NM], mx[NM], mr[NM];
    __shared__ T mc[NE ? NM : 1], me[NM], mn[NM], mdv[NM], mg[NE ? NM : 1];
    const TileStencil<T> tsF{fc, fe, fn, fg, fdv}, tsM{mc, me, mn, mg, mdv};
    const int Nf = opF_.N, Nf1 = Nf + 1, Nm = Nf / 2, Nm1 = Nm + 1, Nc = Nm / 2, Nc1 = Nc + 1;
    const int3 tb = xcd_tile(tm);
    const int K0 = tb.x * kT, L0 = tb.y * kT;
    const int K1 = min(K0 + kT - 1, Nc), L1 = min(L0 + kT - 1, Nc);
    const int mox = 2 * K0 - 3, moy = 2 * L0 - 3;  // level-M coordinates of local (0, 0)
    const int fox = 2 * mox - 3, foy = 2 * moy - 3;  // level-F coordinates of local (0, 0)
    // owned nodes: level M [2 K0, 2 K1 + 1], level F [2 i0, 2 i1 + 1] of those
    const int mi0 = 2 * K0, mj0 = 2 * L0, mi1 = min(2 * K1 + 1, Nm), mj1 = min(2 * L1 + 1, Nm);
    const int fi0 = 2 * mi0, fj0 = 2 * mj0, fi1 = min(2 * mi1 + 1, Nf), fj1 = min(2 * mj1 + 1, Nf);
    const T inv_theta = (T)cc.inv_theta, cA = (T)cc.cA, cB = (T)cc.cB;
    constexpr int E = (NF + NT - 1) / NT;
    const void* staged = nullptr;
    const int c_end = min(nc, (tb.z + 1) * cb);
    for (int col = tb.z * cb; col < c_end; ++col) {
        if (!check && !column_on(act, col)) continue;
        const double rr_share = check ? partial_share(red.rr, col, red.stride, red.nrr) : 0.0;
        const auto& opF = opF_.at(col);
        const auto& opM = opM_.at(col);
        const T* bcol = bF + (size_t)col * ldF;
        T vb[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = threadIdx.x + NT * e;
            const int i = fox + t % FW, j = foy + t / FW;
            vb[e] = (t < NF && i >= 0 && i <= Nf && j >= 0 && j <= Nf) ? bcol[j * Nf1 + i] : (T)0;
        }
        lds_barrier();  // the previous column's LDS reads are done
        if (instance_key(opF) != staged) {
            stage_stencil<FW, NT>(opF, tsF, fox, foy);
            stage_stencil<MW, NT>(opM, tsM, mox, moy);
            staged = instance_key(opF);
        }
        if (check && column_done_share(rr_share, red, col, st, act, tb.x == 0 && tb.y == 0)) continue;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = threadIdx.x + NT * e;
            if (t < NF) fb[t] = vb[e];
        }
        lds_barrier();
        // level F: d0 = D^-1 b / theta; x2 = cA d0 + cB D^-1 (b - A d0) on
        // local [1, FW-1)^2 (owned nodes to global); residual on [2, FW-2)^2
        for (int t = threadIdx.x; t < NF; t += blockDim.x) fr[t] = fdv[t] * fb[t] * inv_theta;
        lds_barrier();
        {
            T* xcol = xF + (size_t)col * ldF;
            constexpr int W = FW - 2;
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int il = 1 + t % W, jl = 1 + t / W, l = jl * FW + il;
                const T v = cA * fr[l] + cB * fdv[l] * (fb[l] - tile_apply<NE>(tsF, FW, l, fr));
                fx[l] = v;
                const int i = fox + il, j = foy + jl;
                if (i >= fi0 && i <= fi1 && j >= fj0 && j <= fj1) xcol[j * Nf1 + i] = v;
            }
        }
        lds_barrier();
        {
            constexpr int W = FW - 4;
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int l = (2 + t / W) * FW + 2 + t % W;
                const T v = fb[l] - tile_apply<NE>(tsF, FW, l, fx);
                fr[l] = fdv[l] != (T)0 ? v : (T)0;
            }
        }
        lds_barrier();
        // P^T onto the whole level-M tile: b_M, zero off the mesh and on
        // Dirichlet rows; owned nodes to global
        {
            T* bcol2 = bM + (size_t)col * ldM;
            auto res = [&](int i, int j) { return fr[(j - foy) * FW + (i - fox)]; };
            for (int t = threadIdx.x; t < NM; t += blockDim.x) {
                const int I = mox + t % MW, J = moy + t / MW;
                T v = 0;
                if (I >= 0 && I <= Nm && J >= 0 && J <= Nm && !(dirichlet && (J == 0 || J == Nm))) {
                    const int i = 2 * I, j = 2 * J;
                    T sm = 0;
                    if (i > 0) sm += res(i - 1, j);
                    if (i < Nf) sm += res(i + 1, j);
                    if (j > 0) sm += res(i, j - 1);
                    if (j < Nf) sm += res(i, j + 1);
                    if (i < Nf && j < Nf) sm += res(i + 1, j + 1);
                    if (i > 0 && j > 0) sm += res(i - 1, j - 1);
                    v = res(i, j) + (T)0.5 * sm;
                }
                if (I >= mi0 && I <= mi1 && J >= mj0 && J <= mj1) bcol2[J * Nm1 + I] = v;
                mb[t] = v;
            }
        }
        lds_barrier();
        // level M: the same three steps on the level-M tile
        for (int t = threadIdx.x; t < NM; t += blockDim.x) mr[t] = mdv[t] * mb[t] * inv_theta;
        lds_barrier();
        {
            T* xcol = xM + (size_t)col * ldM;
            constexpr int W = MW - 2;
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int il = 1 + t % W, jl = 1 + t / W, l = jl * MW + il;
                const T v = cA * mr[l] + cB * mdv[l] * (mb[l] - tile_apply<NE>(tsM, MW, l, mr));
                mx[l] = v;
                const int I = mox + il, J = moy + jl;
                if (I >= mi0 && I <= mi1 && J >= mj0 && J <= mj1) xcol[J * Nm1 + I] = v;
            }
        }
        lds_barrier();
        {
            constexpr int W = MW - 4;
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int l = (2 + t / W) * MW + 2 + t % W;
                const T v = mb[l] - tile_apply<NE>(tsM, MW, l, mx);
                mr[l] = mdv[l] != (T)0 ? v : (T)0;
            }
        }
        lds_barrier();
        // P^T onto the level-C tile
        T* bccol = bC + (size_t)col * ldC;
        const int cw = K1 - K0 + 1, ch = L1 - L0 + 1;
        auto res = [&](int I, int J) { return mr[(J - moy) * MW + (I - mox)]; };
        for (int t = threadIdx.x; t < cw * ch; t += blockDim.x) {
            const int K = K0 + t % cw, L = L0 + t / cw;
            T v = 0;
            if (!(dirichlet && (L == 0 || L == Nc))) {
                const int I = 2 * K, J = 2 * L;
                T sm = 0;
                if (I > 0) sm += res(I - 1, J);
                if (I < Nm) sm += res(I + 1, J);
                if (J > 0) sm += res(I, J - 1);
                if (J < Nm) sm += res(I, J + 1);
                if (I < Nm && J < Nm) sm += res(I + 1, J + 1);
                if (I > 0 && J > 0) sm += res(I - 1, J - 1);
                v = res(I, J) + (T)0.5 * sm;
            }
            bccol[L * Nc1 + K] = v;
        }
    }
}

// Up steps of NL consecutive levels 0 (finest of the chain) .. NL-1 in one
// launch.  Grid: (tiles over level-0 x, tiles over level-0 y, column blocks).
// Level 0 is the k_up tile: the output tile O of kTF x kTF nodes at local
// [2, kTF+2) of a tile of width W_0 = kTF + 4 whose every node forms
// x2 + P x_1.  The level-(k+1) values that prolongation reads are the nodes
// [floor(o_k / 2), ceil((o_k + W_k - 1) / 2)] (o_k: the tile's origin), at
// most (W_k + 1) / 2 + 1 of them per side; they are the output region of the
// level-(k+1) up step on a tile two nodes wider on each side, so
// o_{k+1} = floor(o_k / 2) - 2 and W_{k+1} = (W_k + 1) / 2 + 5.  The widths
// settle at 11, so the redundant work per level stays bounded (kTF = 16:
// 20, 15, 13, 12, 11, ...); each level still adds its passes to the
// workgroup's latency.  Every input (b and x2 of each level,
// the level-NL correction x_C, the operator rows) is loaded at the start; the
// levels then run coarse to fine in LDS.  Writes x of level 0 on O only (the
// coarser x are used by nothing else).
template <int kTF>
constexpr int chain_width(int k) {
    int w = kTF + 4;
    for (int i = 0; i < k; ++i) w = (w + 1) / 2 + 5;
    return w;
}
template <int kTF>
constexpr int chain_offset(int k) {
    int s = 0;
    for (int i = 0; i < k; ++i) s += chain_width<kTF>(i) * chain_width<kTF>(i);
    return s;
}
constexpr int kChainMax = kChainLen;  // levels a chain may hold

template <typename T, class Op>
struct ChainArgs {
    Op op[kChainMax];
    const T* b[kChainMax];
    const T* x2[kChainMax];
    int ld[kChainMax];
    T* x;         // level-0 output
    const T* xc;  // level-NL correction (from the level below the chain)
    int ldc;
};

// Row of node (i, j) in the tile-stencil form (zero off the mesh), same
// arithmetic as stage_stencil.
template <typename T>
struct TileRow {
    T c, e, n, g, dv;
};
// The loads are issued without a branch, at the node clamped into the mesh
// (chain_load zeroes the row off the mesh): a load inside a branch makes the
// wave wait for it, and with it for every load issued before.
template <typename T>
__device__ inline TileRow<T> tile_row(const OpA<T>& op, int i, int j) {
    const int N = op.N, N1 = N + 1, k = clamp_node(j, N) * N1 + clamp_node(i, N);
    return TileRow<T>{(T)0, -op.wE[k], -op.wN[k], (T)0, op.dinv[k]};  // diagonal: tile_center
}
template <typename T, class OpK>
__device__ inline TileRow<T> tile_row(const OpK& op, int i, int j) {
    const int N = op.N;
    const KARow<T>& r = op.rows[ka_class(clamp_node(i, N), clamp_node(j, N), N)];
    return TileRow<T>{r.c, r.e, r.n, r.ne, r.dinv};
}

// Level k of the chain (then k - 1, ..., 0): x2 + P x_{k+1} (except on the
// coarsest level, whose P x_C came with the loads), d0, then x in place
// (level 0: to global on O).
template <typename T, class Op, int kTF, int NL, int k>
__device__ inline void chain_step(const ChainArgs<T, Op>& a, const int* ox, const int* oy, T* sx, T* sd,
                                  const T* sb, const TileStencil<T>& ts, int dirichlet, const ChebCoef& cc,
                                  int i0, int i1, int j0, int j1, int col) {
    constexpr int W = chain_width<kTF>(k), off = chain_offset<kTF>(k), NN = W * W;
    constexpr bool NE = kNorthEast<Op>;
    const TileStencil<T> st{NE ? ts.c + off : ts.c, ts.e + off, ts.n + off, NE ? ts.g + off : ts.g, ts.dv + off};
    T* x = sx + off;
    T* d = sd + off;
    const T* b = sb + off;
    const T inv_theta = (T)cc.inv_theta, theta = (T)cc.theta, cB = (T)cc.cB, c1 = (T)cc.c1;
    if constexpr (k < NL - 1) {
        constexpr int W1 = chain_width<kTF>(k + 1), off1 = chain_offset<kTF>(k + 1);
        const T* x1 = sx + off1;
        const int N = a.op[k].N, ox1 = ox[k + 1], oy1 = oy[k + 1];
        for (int t = threadIdx.x; t < NN; t += blockDim.x) {
            const int i = ox[k] + t % W, j = oy[k] + t / W;
            if (i >= 0 && i <= N && j >= 0 && j <= N && !(dirichlet && (j == 0 || j == N))) {
                const int I = i >> 1, J = j >> 1;
                const T p0 = x1[(J - oy1) * W1 + (I - ox1)];
                x[t] += ((i | j) & 1) ? (T)0.5 * (p0 + x1[(J + (j & 1) - oy1) * W1 + (I + (i & 1) - ox1)]) : p0;
            }
        }
        lds_barrier();
    }
    {
        constexpr int Wi = W - 2;
        for (int t = threadIdx.x; t < Wi * Wi; t += blockDim.x) {
            const int l = (1 + t / Wi) * W + 1 + t % Wi;
            d[l] = st.dv[l] * (b[l] - tile_apply<NE>(st, W, l, x)) * inv_theta;
        }
    }
    lds_barrier();
    if constexpr (k > 0) {
        // x on [2, W-2)^2 in place of x2 + P x (each node reads only its own entry)
        constexpr int Wi = W - 4;
        for (int t = threadIdx.x; t < Wi * Wi; t += blockDim.x) {
            const int l = (2 + t / Wi) * W + 2 + t % Wi;
            const T dk = d[l];
            const T r1 = theta * dk * tile_center<NE>(st, W, l) - tile_apply<NE>(st, W, l, d);
            x[l] = x[l] + ((T)1 + c1) * dk + cB * st.dv[l] * r1;
        }
        lds_barrier();
        chain_step<T, Op, kTF, NL, k - 1>(a, ox, oy, sx, sd, sb, ts, dirichlet, cc, i0, i1, j0, j1, col);
    } else {
        const int N1 = a.op[0].N + 1;
        T* xcol = a.x + (size_t)col * a.ld[0];
        const int w = i1 - i0 + 1, h = j1 - j0 + 1;
        for (int t = threadIdx.x; t < w * h; t += blockDim.x) {
            const int i = i0 + t % w, j = j0 + t / w;
            const int l = (j - oy[0]) * W + (i - ox[0]);
            const T dk = d[l];
            const T r1 = theta * dk * tile_center<NE>(st, W, l) - tile_apply<NE>(st, W, l, d);
            xcol[j * N1 + i] = x[l] + ((T)1 + c1) * dk + cB * st.dv[l] * r1;
        }
    }
}

// Loads of level k of the chain (then k + 1, ...), kept in registers until
// every level's loads are issued, then stored to LDS: b, x2 (plus P x_C on
// the coarsest level) and, when stage is set, the operator rows.
template <typename T, class Op, int kTF, int NL, int NT, int k>
__device__ inline void chain_load(const ChainArgs<T, Op>& a, const int* ox, const int* oy, int dirichlet, int col,
                                  bool stage, T* sx, T* sb, const TileStencil<T>& ts) {
    constexpr int W = chain_width<kTF>(k), off = chain_offset<kTF>(k), NN = W * W, E = (NN + NT - 1) / NT;
    constexpr bool NE = kNorthEast<Op>;
    const Op& op = a.op[k];
    const int N = op.N;
    // every load at a node clamped into the mesh, without a branch (a load
    // inside a branch waits there, and with it every load issued before it);
    // off-mesh and off-tile slots are dropped at the LDS stores
    T vb[E], vx[E], pc0[E], pc1[E];
    TileRow<T> vr[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = threadIdx.x + NT * e;
        const int i = ox[k] + t % W, j = oy[k] + t / W;
        const size_t g = (size_t)col * a.ld[k] + (size_t)clamp_node(j, N) * (N + 1) + clamp_node(i, N);
        vb[e] = a.b[k][g];
        vx[e] = a.x2[k][g];
        if constexpr (k == NL - 1) {
            // P x_C operands: the coarse node (i/2, j/2) and the far coarse
            // end of the fine edge through (i, j)
            const int Nc = N / 2, ic = clamp_node(i, N), jc = clamp_node(j, N), I = ic >> 1, J = jc >> 1;
            const T* xcc = a.xc + (size_t)col * a.ldc;
            pc0[e] = xcc[J * (Nc + 1) + I];
            pc1[e] = xcc[min(J + (jc & 1), Nc) * (Nc + 1) + min(I + (ic & 1), Nc)];
        }
        // rows loaded whether or not this column stages them (few-column
        // cycles: the next columns of a workgroup find them in cache)
        vr[e] = tile_row<T>(op.at(col), i, j);
    }
    if constexpr (k + 1 < NL) chain_load<T, Op, kTF, NL, NT, k + 1>(a, ox, oy, dirichlet, col, stage, sx, sb, ts);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = threadIdx.x + NT * e;
        if (t < NN) {
            const int i = ox[k] + t % W, j = oy[k] + t / W;
            const bool in = i >= 0 && i <= N && j >= 0 && j <= N;
            const bool fr = in && !(dirichlet && (j == 0 || j == N));
            T v = fr ? vx[e] : (T)0;
            // x2 + P x_C on the coarsest level of the chain: the coarse node
            // when i and j are even, else the mean of the edge's two ends
            if constexpr (k == NL - 1)
                if (fr) v += ((i | j) & 1) ? (T)0.5 * (pc0[e] + pc1[e]) : pc0[e];
            sb[off + t] = in ? vb[e] : (T)0;
            sx[off + t] = v;
            if (stage) {
                const TileRow<T> r = in ? vr[e] : TileRow<T>{};
                if constexpr (NE) ts.c[off + t] = r.c;
                ts.e[off + t] = r.e;
                ts.n[off + t] = r.n;
                if constexpr (NE) ts.g[off + t] = r.g;
                ts.dv[off + t] = r.dv;
            }
        }
    }
}

template <typename T, class Op, int kTF, int NL, int NT>
__global__ __launch_bounds__(NT) void k_up_chain(ChainArgs<T, Op> a, int dirichlet, const int* __restrict__ act,
                                                 ChebCoef cc, int nc, int cb, TileMap tm) {
    static_assert(kTF % 2 == 0 && NL >= 2 && NL <= kChainMax, "chain shape");
    constexpr int NA = chain_offset<kTF>(NL);  // nodes of all the chain's tiles
    constexpr bool NE = kNorthEast<Op>;
    __shared__ T sx[NA], sd[NA], sb[NA];
    __shared__ T tc[NE ? NA : 1], te[NA], tn[NA], tdv[NA], tg[NE ? NA : 1];
    const TileStencil<T> ts{tc, te, tn, tg, tdv};
    const int3 tb = xcd_tile(tm);
    const int i0 = tb.x * kTF, j0 = tb.y * kTF;
    const int i1 = min(i0 + kTF - 1, a.op[0].N), j1 = min(j0 + kTF - 1, a.op[0].N);
    int ox[NL], oy[NL];
    ox[0] = i0 - 2;
    oy[0] = j0 - 2;
#pragma unroll
    for (int k = 1; k < NL; ++k) {
        ox[k] = (ox[k - 1] >> 1) - 2;  // floor(o / 2) - 2
        oy[k] = (oy[k - 1] >> 1) - 2;
    }
    const void* staged = nullptr;
    const int c_end = min(nc, (tb.z + 1) * cb);
    for (int col = tb.z * cb; col < c_end; ++col) {
        if (!column_on(act, col)) continue;
        const void* key = instance_key(a.op[0].at(col));
        lds_barrier();  // the previous column's LDS reads are done
        chain_load<T, Op, kTF, NL, NT, 0>(a, ox, oy, dirichlet, col, key != staged, sx, sb, ts);
        staged = key;
        lds_barrier();
        chain_step<T, Op, kTF, NL, NL - 1>(a, ox, oy, sx, sd, sb, ts, dirichlet, cc, i0, i1, j0, j1, col);
    }
}

// -------------------------------------------------------------- bottom ---
// All levels with N_l <= kBottomN (at most three: 32, 16, 8) for one column in
// one workgroup of 1024 threads.  The bottom computes in FP32 whatever the
// solve's precision: it is the coarse correction of a preconditioner, so its
// rounding changes the preconditioner slightly but no result (the PCG and the
// refinement test residuals of the solve's own precision).  b and x are global
// level-Lb vectors of the solve's precision TV.
// One workgroup does ~18 short phases between barriers, so what counts is the
// instructions and LDS reads of a phase: a thread owns the same nodes of each
// level throughout and keeps their operator rows, right-hand sides and
// positions in registers; LDS holds the two vectors that neighbours read.  N = 32..8,
// state operator: 8.3 us with rows, diagonals and positions formed anew in each
// phase, 5.8 with them in registers (prior 9.4 -> 6.1).
struct BottomArgs {
    int nlev;                           // levels handled here (the last is the coarsest)
    int N[kBottomLevels];
    const float* wE[kBottomLevels];     // state operator coefficients (unused for the prior)
    const float* wN[kBottomLevels];
    const float* dinv[kBottomLevels];
    const float* cinv;                  // dense inverse of the coarsest level
    int nc;                             // its size
    KARow<float> ka[kBottomLevels][9];  // prior operator rows of each level
    // stacked instances (cpi = 0: one instance): column c belongs to instance
    // c / cpi, whose state coefficients of level l start cs[l] elements further,
    // whose coarse inverse starts cinv_stride further and whose prior rows of
    // level l are karows[l][9 inst .. 9 inst + 8]
    int cpi;
    long long cs[kBottomLevels];
    long long cinv_stride;
    const KARow<float>* karows[kBottomLevels];
};

// q / d for 0 <= q < 2^22 and d >= 1 by a float reciprocal: (q + 1/2) / d lies
// at least 1 / (2 d) from an integer and the float product errs by less than
// 2^-23 (q / d) < 1 / (2 d), so the truncation is exact (integer division is a
// long instruction sequence on the vector ALU).
__device__ inline int small_div(int q, float inv_d) { return (int)(((float)q + 0.5f) * inv_d); }

// The cycle of one column.  Each level lies in LDS with a ring of zeros (padded
// width N_l + 3), so the stencil applies without boundary branches; Dirichlet
// rows are masked by their zero inverse diagonal.  Node slots of a thread:
// nodes t and t + 1024 of level 0, node t of levels 1 and 2.
template <int KIND>
struct BottomCycle {
    static constexpr bool PRIOR = KIND == kOpPrior;
    static constexpr int NT = 1024, LV = kBottomLevels, NS = LV + 1, S = 12, kCU = 8;
    static constexpr int PN = (kBottomN + 3) * (kBottomN + 3) + (kBottomN / 2 + 3) * (kBottomN / 2 + 3) + 11 * 11;
    static_assert(kBottomN == 32 && LV == 3 && (kBottomN + 1) * (kBottomN + 1) <= 2 * NT, "node slots");
    struct Row {
        float c, e, w, n, s, ne, sw, dv;
    };
    int L;  // the coarsest level, solved with its dense inverse
    int Nl[LV], Pl[LV], po[LV];
    int sp[NS], si[NS], sj[NS];  // padded position (-1 past the level), (i, j)
    Row rw[NS];
    float bl[NS];  // right-hand sides
    int cr, cpart, nc;
    float cv[kCU];  // the thread's part of the dense inverse
    static __device__ int level(int s) { return s < 2 ? 0 : s - 1; }

    template <class F>
    __device__ __forceinline__ void load(const BottomArgs& a, int inst, F rhs) {
        const int nlev = a.nlev;
        L = nlev - 1;
        int p = 0;
#pragma unroll
        for (int l = 0; l < LV; ++l) {
            Nl[l] = l < nlev ? a.N[l] : 0;
            Pl[l] = Nl[l] + 3;
            po[l] = p;
            p += Pl[l] * Pl[l];
        }
        // ---- this thread's nodes: padded position (-1 past the level), (i, j),
        // operator row, right-hand side rhs(q); every global load issued here
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int l = level(s), q = threadIdx.x + (s == 1 ? NT : 0), N = Nl[l], N1 = N + 1;
            const bool in = l < nlev && q < N1 * N1;
            const int jq = small_div(q, 1.0f / (float)N1);
            const int i = in ? q - jq * N1 : 0, j = in ? jq : 0;
            si[s] = i;
            sj[s] = j;
            sp[s] = in ? po[l] + (j + 1) * Pl[l] + i + 1 : -1;
            bl[s] = 0.0f;
            rw[s] = Row{};
            if (!in) continue;
            if constexpr (PRIOR) {
                const int c = ka_class(i, j, N);
                const KARow<float> r = a.cpi ? a.karows[l][9 * inst + c] : a.ka[l][c];
                rw[s] = Row{r.c, r.e, r.w, r.n, r.s, r.ne, r.sw, r.dinv};
            } else {
                const long long at = a.cpi ? inst * a.cs[l] : 0;
                const float* pE = a.wE[l] + at;
                const float* pN = a.wN[l] + at;
                const float vE = pE[q], vW = pE[i > 0 ? q - 1 : q], vN = pN[q], vS = pN[j > 0 ? q - N1 : q];
                Row& r = rw[s];
                r.e = -vE;
                r.w = i > 0 ? -vW : 0.0f;
                r.n = -vN;
                r.s = j > 0 ? -vS : 0.0f;
                r.c = -(r.e + r.w + r.n + r.s);
                r.dv = (a.dinv[l] + at)[q];
            }
            if (l == 0) bl[s] = rhs(q);
        }
        // the thread's part of the dense coarse inverse
        const float* ci = a.cinv + (a.cpi ? inst * a.cinv_stride : 0);
        cr = threadIdx.x / S;
        cpart = threadIdx.x % S;
        nc = a.nc;
#pragma unroll
        for (int u = 0; u < kCU; ++u) {
            const int c = cpart + u * S;
            cv[u] = (cr < nc && c < nc) ? ci[cr * nc + c] : 0.0f;
        }
    }

    // From bl of level 0 to x in sx[sp[0]], sx[sp[1]] (written and to be read
    // by their own threads); sx and sw hold zeros off the nodes, and a barrier
    // has to lie between earlier reads of them and the call.
    __device__ __forceinline__ void run(const ChebCoef& cc, float* sx, float* sw, float* sbc, float* tmp) {
        const float inv_theta = (float)cc.inv_theta, theta = (float)cc.theta, cA = (float)cc.cA, cB = (float)cc.cB,
                    c1 = (float)cc.c1;
        // d0 of the first smoothing step (or the right-hand side of the dense solve)
#pragma unroll
        for (int s = 0; s < 2; ++s)
            if (sp[s] >= 0) {
                sw[sp[s]] = rw[s].dv * bl[s] * inv_theta;
                if (L == 0 && s == 0) sbc[threadIdx.x] = bl[s];
            }
        lds_barrier();
        // (A x)_p at padded position p of level l
        auto apply = [&](const Row& r, int P, int p, const float* x) -> float {
            if constexpr (PRIOR)
                return r.c * x[p] + r.e * x[p + 1] + r.w * x[p - 1] + r.n * x[p + P] + r.s * x[p - P] +
                       r.ne * x[p + P + 1] + r.sw * x[p - P - 1];
            else  // the diagonal's product is the rounded one of the sum
                return __builtin_fmaf(r.e, x[p + 1], r.c * x[p]) + r.w * x[p - 1] + r.n * x[p + P] + r.s * x[p - P];
        };
        // ---- down
#pragma unroll
        for (int l = 0; l < LV - 1; ++l) {
            if (l >= L) break;
            const int P = Pl[l];
            const int s0 = l == 0 ? 0 : l + 1, s1 = l + 2;
            // x2 = cA d0 + cB D^-1 (b - A d0), d0 in sw
#pragma unroll
            for (int s = s0; s < s1; ++s) {
                const int p = sp[s];
                if (p < 0) continue;
                const float ad = apply(rw[s], P, p, sw);
                sx[p] = cA * sw[p] + cB * rw[s].dv * (bl[s] - ad);
            }
            lds_barrier();
            // residual b - A x2 on the free nodes, into sw
#pragma unroll
            for (int s = s0; s < s1; ++s) {
                const int p = sp[s];
                if (p < 0) continue;
                const float v = bl[s] - apply(rw[s], P, p, sx);
                sw[p] = rw[s].dv != 0.0f ? v : 0.0f;
            }
            lds_barrier();
            // restriction P^T to level l + 1, and its first smoothing correction d0
            {
                const int sc = l + 2, pc = sp[sc];
                if (pc >= 0) {
                    const int f = po[l] + (2 * sj[sc] + 1) * P + 2 * si[sc] + 1;
                    const float dvc = rw[sc].dv;
                    float v = 0.0f;
                    if (dvc != 0.0f)
                        v = sw[f] + 0.5f * (sw[f - 1] + sw[f + 1] + sw[f - P] + sw[f + P] + sw[f + P + 1] + sw[f - P - 1]);
                    bl[sc] = v;
                    sw[pc] = dvc * v * inv_theta;
                    if (l + 1 == L) sbc[threadIdx.x] = v;
                }
            }
            lds_barrier();
        }
        // ---- coarsest: dense inverse, S threads per row (entries prefetched in cv)
        if (cr < nc) {
            float s = 0.0f;
#pragma unroll
            for (int u = 0; u < kCU; ++u) {
                const int c = cpart + u * S;
                if (c < nc) s += cv[u] * sbc[c];
            }
            tmp[threadIdx.x] = s;
        }
        lds_barrier();
        {
            const int s0 = sp[0], s2 = sp[2], s3 = sp[3], p = L == 0 ? s0 : (L == 1 ? s2 : s3);
            if ((int)threadIdx.x < nc) {
                float s = 0.0f;
                for (int part = 0; part < S; ++part) s += tmp[threadIdx.x * S + part];
                sx[p] = s;
            }
        }
        lds_barrier();
        // ---- up
#pragma unroll
        for (int l = LV - 2; l >= 0; --l) {
            if (l >= L) continue;
            const int P = Pl[l], Pc = Pl[l + 1];
            const int s0 = l == 0 ? 0 : l + 1, s1 = l + 2;
            // x += P x_coarse on the free nodes
#pragma unroll
            for (int s = s0; s < s1; ++s) {
                const int p = sp[s];
                if (p < 0 || rw[s].dv == 0.0f) continue;
                const int i = si[s], j = sj[s], I = i >> 1, J = j >> 1;
                const int ca0 = po[l + 1] + (J + 1) * Pc + I + 1;
                const int ca1 = po[l + 1] + (J + 1 + (j & 1)) * Pc + I + 1 + (i & 1);
                sx[p] += ((i | j) & 1) ? 0.5f * (sx[ca0] + sx[ca1]) : sx[ca0];
            }
            lds_barrier();
            // d0 = D^-1 (b - A x) / theta
#pragma unroll
            for (int s = s0; s < s1; ++s) {
                const int p = sp[s];
                if (p < 0) continue;
                const float ax = apply(rw[s], P, p, sx);
                sw[p] = rw[s].dv * (bl[s] - ax) * inv_theta;
            }
            lds_barrier();
            // x += (1 + c1) d0 + cB D^-1 r1 with r1 = theta D d0 - A d0
#pragma unroll
            for (int s = s0; s < s1; ++s) {
                const int p = sp[s];
                if (p < 0) continue;
                const float ad = apply(rw[s], P, p, sw);
                const float dk = sw[p];
                const float r1 = theta * dk * rw[s].c - ad;
                sx[p] += (1.0f + c1) * dk + cB * rw[s].dv * r1;
            }
            if (l > 0) lds_barrier();  // level 0 is read back by its own threads
        }
    }
};

// x_top = V-cycle(b_top) for every column (blockIdx.x = column).  When rv is
// given (the bottom is the whole hierarchy), sum_k rv_k x_k is written as the
// single partial of r^T z.
template <typename TV, int KIND>
__global__ __launch_bounds__(1024) void k_bottom(BottomArgs a, const TV* __restrict__ bg, TV* __restrict__ xg,
                                                 int ld, int* __restrict__ act, ChebCoef cc,
                                                 const TV* __restrict__ rv, PcgRed red,
                                                 ColState* __restrict__ st, int check) {
    using BC = BottomCycle<KIND>;
    constexpr int NT = BC::NT, PN = BC::PN;
    const int col = blockIdx.x;
    if (!check && !column_on(act, col)) return;
    // the convergence test's partials load together with the level data
    // below; the test itself follows the loads
    const double rr_share = check ? partial_share(red.rr, col, red.stride, red.nrr) : 0.0;
    __shared__ float sx[PN], sw[PN], sbc[81], tmp[NT];
    BC c;
    c.load(a, a.cpi ? uniform(col / a.cpi) : 0, [&](int q) { return (float)bg[(size_t)col * ld + q]; });
    // ---- LDS: zeros everywhere (the rings stay zero)
    for (int q = threadIdx.x; q < PN; q += NT) sx[q] = sw[q] = 0.0f;
    if (check) {
        if (column_done_share(rr_share, red, col, st, act, true)) return;  // its barrier follows the zeros
    } else {
        lds_barrier();
    }
    c.run(cc, sx, sw, sbc, tmp);
    double dot = 0.0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = threadIdx.x + NT * s;
        if (c.sp[s] >= 0) {
            const TV v = (TV)sx[c.sp[s]];
            xg[(size_t)col * ld + q] = v;
            if (rv) dot += (double)v * (double)rv[(size_t)col * ld + q];
        }
    }
    if (rv) {
        const double sm = group_sum(dot);
        if (threadIdx.x == 0) red.rz[(size_t)col * red.stride] = sm;
    }
}

// ------------------------------------------------------------------ PCG ---
// The linear kernels (few columns):
// workgroup blockIdx.x covers nodes [chunk x, chunk (x + 1)) of column
// blockIdx.y with vec_threads(per) threads, at most kVecNodes nodes a thread.

// p_new = z + beta p_old with beta = (r^T z) / rz_old (p_new = z on the first
// iteration, FIRST), q = A p_new = A z + beta A p_old, partials of p_new^T q;
// and x += alpha p_old, the step of the iteration before (p_old is read here
// anyway; the refinement step adds the last iteration's).
// The loads of the r^T z partials and of the thread's nodes (z and p_old at
// the stencil points, the operator rows) are issued before any of them is
// used, so their latencies overlap: all at once where the registers allow,
// else node by node with apply_window() nodes in flight (FP64 rows would spill).
// Node k = j (N + 1) + i is split by a double reciprocal: (k + 1/2) / (N + 1)
// lies at least 1 / (2 (N + 1)) from an integer and the product errs by far
// less, so the truncation is exact.  Workgroup 0 records r^T z for the finest
// k_down, which forms alpha from it and reads one value instead of the partials.
// The operator form the apply kernel combines with: the state operator as it
// is, the prior operators through their rows staged in LDS.
template <class OpT>
struct ApplyForm {
    using type = OpT;
    static constexpr bool kTable = false;
};
template <typename T>
struct ApplyForm<OpKA<T>> {
    using type = OpKALds<T>;
    static constexpr bool kTable = true;
};
template <typename T>
struct ApplyForm<OpKARef<T>> {
    using type = OpKALds<T>;
    static constexpr bool kTable = true;
};

template <class OpT>
constexpr int apply_window() {
    constexpr size_t b = sizeof(typename OpT::Row) + 2 * sizeof(typename OpT::Nb);  // loaded bytes per node
    return b <= 64 ? 4 : (b <= 112 ? 3 : 2);
}

// A workgroup of NT threads does the work of bd = vec_threads(per) of them:
// thread t stands for the virtual threads t and t + NT (bd = 2 NT; or one, bd =
// NT), and the sums are taken in the order of the bd.  Half of the waves with
// twice the nodes each: at N = 1024 a column's ~500 workgroups fit the
// registers of the 256 compute units in one round instead of two.  The
// node window is what 128 registers hold.  1024^2, one column, state operator
// (64 bytes a node with the step of x): 16.1 us = 4.2 TB/s (17.1 without x, at
// 1024 threads).
template <typename T, class Op, bool FIRST, int NT>
__global__ __launch_bounds__(NT, 4) void k_pcg_apply_few(Op op_, const T* __restrict__ z, const T* __restrict__ p_old,
                                                      T* __restrict__ p_new, T* __restrict__ q, T* __restrict__ x,
                                                      int ld, const int* __restrict__ act, ColState* __restrict__ st,
                                                      PcgRed red, TileMap tm) {
    constexpr int kHalves = 2, SL = kHalves * kVecNodes;  // node slots of a thread
    // node blocks in XCD-aware order: the rows above and below a block's
    // nodes belong to blocks on the same XCD
    const int3 tb = xcd_tile(tm);
    const int col = tb.y, bx = tb.x;
    const auto& op = op_.at(col);  // operator of the instance owning this column
    if (!column_on(act, col)) return;
    const int N = op.N, N1 = N + 1, n = N1 * N1;
    const int bd = vec_threads(red.per), halves = bd / NT;
    const bool need_rz = !FIRST || bx == 0;  // uniform in the workgroup
    VtRest<kHalves> srz;
    if (need_rz) srz = vt_rest<kHalves>(red.rz, col, red.stride, red.nrz, bd);
    const double rz_old = FIRST ? 1.0 : st[col].rz;
    const T alpha = FIRST ? (T)0 : (T)st[col].alpha;
    const T* zc = z + (size_t)col * ld;
    const T* pc = p_old + (size_t)col * ld;
    const T* xc = x + (size_t)col * ld;
    const int k0 = bx * red.chunk, k1 = min(n, k0 + red.chunk);
    const double inv_n1 = 1.0 / N1;
    using Form = ApplyForm<std::decay_t<decltype(op)>>;
    using OpT = typename Form::type;
    __shared__ KARow<T> krows[Form::kTable ? 9 : 1];
    __shared__ __attribute__((aligned(16))) double slots[16];
    OpT sop;
    if constexpr (Form::kTable)
        sop = OpT{N, krows};
    else
        sop = op;
    constexpr int W = apply_window<OpT>();
    typename OpT::Row rw[W];
    typename OpT::Nb vz[W], vp[W];
    T xk[W];
    // slot s: node of virtual thread t + NT (s mod halves), pass s / halves
    auto node = [&](int s, int& i, int& j) {
        const int e = halves == 2 ? s >> 1 : s, h = halves == 2 ? s & 1 : 0;
        const int k = k0 + e * bd + h * NT + (int)threadIdx.x;
        j = (int)(((double)k + 0.5) * inv_n1);
        i = k - j * N1;
        return k;
    };
    auto used = [&](int s) {  // uniform: some thread's node lies in the chunk
        const int e = halves == 2 ? s >> 1 : s, h = halves == 2 ? s & 1 : 0;
        return e < kVecNodes && k0 + e * bd + h * NT < k1;
    };
    auto load = [&](int s) {
        if (!used(s)) return;
        int i, j;
        const int k = min(node(s, i, j), k1 - 1);
        j = (int)(((double)k + 0.5) * inv_n1);
        i = k - j * N1;
        rw[s % W] = sop.row(i, j, k);
        vz[s % W] = sop.gather(i, j, k, zc);
        if constexpr (!FIRST) {
            vp[s % W] = sop.gather(i, j, k, pc);
            xk[s % W] = xc[k];
        }
    };
#pragma unroll
    for (int s = 0; s < W; ++s) load(s);
    if constexpr (Form::kTable) {
        // rows staged after the node loads are issued (waiting for them then
        // waits for nothing those loads would not)
        if (threadIdx.x < 9) krows[threadIdx.x] = ka_row(op, threadIdx.x);
    }
    T beta = 0;
    if (need_rz) {
        const double rz = vt_rest_total<kHalves>(srz, red.rz, col, red.stride, red.nrz, bd);
        if (!FIRST) beta = (T)(rz / rz_old);
        if (bx == 0 && threadIdx.x == 0) st[col].rz_new = rz;
    } else if constexpr (Form::kTable) {
        lds_barrier();
    }
    double dot[kHalves] = {0.0, 0.0};
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        if (!used(s)) continue;
        int i, j;
        const int k = node(s, i, j);
        if (k < k1) {
            const bool fr = sop.is_free(i, j);
            const T zk = vz[s % W].c;
            T az = fr ? sop.combine(i, j, rw[s % W], vz[s % W]) : (T)0;
            T pn = zk, v = az;
            const size_t o = (size_t)col * ld + k;
            if constexpr (!FIRST) {
                const T pk = vp[s % W].c;
                const T ap = fr ? sop.combine(i, j, rw[s % W], vp[s % W]) : (T)0;
                pn = zk + beta * pk;
                v = az + beta * ap;
                x[o] = xk[s % W] + alpha * pk;
            }
            p_new[o] = pn;
            q[o] = v;
            dot[halves == 2 ? s & 1 : 0] += (double)pn * (double)v;
        }
        __builtin_amdgcn_sched_barrier(0);  // keeps the window: no later load moves above
        if (s + W < SL) load(s + W);
    }
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
        if (h >= halves) break;
        const double sm = wave_sum(dot[h]);
        if ((threadIdx.x & 63) == 0) slots[(h * NT + (int)threadIdx.x) >> 6] = sm;
    }
    lds_barrier();
    if (threadIdx.x == 0) red.pq[(size_t)col * red.stride + bx] = slot_sum(slots, bd >> 6);
}

// A node's stencil values from a padded LDS vector (row width P).
template <typename T>
__device__ inline typename OpA<T>::Nb lds_nb(const typename OpA<T>::Nb*, const T* v, int P) {
    return {v[0], v[1], v[-1], v[P], v[-P]};
}
template <typename T>
__device__ inline KANb<T> lds_nb(const KANb<T>*, const T* v, int P) {
    return {v[0], v[1], v[-1], v[P], v[-P], v[P + 1], v[-P - 1]};
}

// Hierarchies whose levels all run in the bottom kernel (N <= kBottomN): a
// whole refinement pass of a column in one launch, one workgroup: the scaled
// inner right-hand side (first pass: r64 = b on the free rows and |b|), the PCG
// of precision T, x64 += |r| d, r64 = b - A x64 in FP64 and the column's state.
// r, x and p stay in the registers of the nodes' threads, z and p lie in padded
// LDS for the operator, and an iteration is the V-cycle's ~18 phases and three
// sums: ~6.8 us at N = 32 in FP64 where three launches (cycle, apply, update)
// took ~16.  The six small launches of a pass around the PCG took ~23 us more.
struct SmallPass {
    const double* b;
    int ldb;
    double *x64, *r64, *partial, *colnorm;
    int ld, nblk;  // nblk: partials of |r64|^2 a column has (the first one is the sum)
    int* oact;
    double rtol, tol_floor;
    int first;
};

// Outer state of a column with |r64|^2 = s: whether it goes on, |r64|, and the
// inner tolerance (squared) of the next pass.
__device__ inline bool outer_state(double s, double obb, double rtol, double tol_floor, double& norm, double& tol2) {
    norm = sqrt(s);
    if (!(isfinite(s) && isfinite(obb) && s > rtol * rtol * obb && s > 0.0)) return false;
    double t = 0.5 * rtol * sqrt(obb / s);
    if (t < tol_floor) t = tol_floor;
    tol2 = t * t;
    return true;
}

template <typename T, int KIND, class Op, class Op64>
__global__ __launch_bounds__(1024) void k_pcg_small(BottomArgs a, Op op_, Op64 op64_, SmallPass ps,
                                                    ColState* __restrict__ st, ChebCoef cc, int max_iter) {
    using BC = BottomCycle<KIND>;
    constexpr int NT = BC::NT, PN = BC::PN, W = kBottomN + 3;
    const int col = blockIdx.x;
    if (!ps.first && !column_on(ps.oact, col)) {
        if (threadIdx.x == 0) st[col].its = 0.0;
        return;
    }
    __shared__ float sx[PN], sw[PN], sbc[81], tmp[NT];
    __shared__ T sz[W * W], sp[W * W];
    __shared__ __attribute__((aligned(16))) double slots[2][16];
    const auto& op = op_.at(col);
    const auto& op64 = op64_.at(col);
    using Form = ApplyForm<std::decay_t<decltype(op)>>;
    using OpT = typename Form::type;
    __shared__ KARow<T> krows[Form::kTable ? 9 : 1];
    OpT sop;
    using Op64T = typename ApplyForm<std::decay_t<decltype(op64)>>::type;
    constexpr bool kWide = sizeof(T) == 8;  // the PCG's vectors and rows serve the FP64 residual too
    __shared__ KARow<double> krows64[Form::kTable && !kWide ? 9 : 1];
    __shared__ double sx64[kWide ? 1 : W * W];
    Op64T sop64;
    if constexpr (Form::kTable) {
        sop = OpT{op.N, krows};
        if (threadIdx.x < 9) krows[threadIdx.x] = ka_row(op, threadIdx.x);
        if constexpr (kWide) {
            sop64 = sop;
        } else {
            sop64 = Op64T{op64.N, krows64};
            if (threadIdx.x < 9) krows64[threadIdx.x] = ka_row(op64, threadIdx.x);
        }
    } else {
        sop = op;
        sop64 = op64;
    }
    BC c;
    c.load(a, a.cpi ? uniform(col / a.cpi) : 0, [](int) { return 0.0f; });
    const int P = c.Pl[0];
    const size_t co = (size_t)col * ps.ld;
    const double* bc = ps.b + (size_t)col * ps.ldb;
    typename OpT::Row row[2];
    double r6[2] = {0.0, 0.0};
    T rk[2], xk[2] = {0, 0}, pk[2] = {0, 0};
    bool fr[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = threadIdx.x + NT * s;
        rk[s] = 0;
        fr[s] = false;
        if (c.sp[s] < 0) continue;
        row[s] = sop.row(c.si[s], c.sj[s], q);
        fr[s] = sop.is_free(c.si[s], c.sj[s]);
        r6[s] = ps.first ? (fr[s] ? bc[q] : 0.0) : ps.r64[co + q];
    }
    for (int q = threadIdx.x; q < PN; q += NT) sx[q] = sw[q] = 0.0f;
    for (int q = threadIdx.x; q < W * W; q += NT) {
        sz[q] = sp[q] = (T)0;
        if constexpr (!kWide) sx64[q] = 0.0;
    }
    int par = 0;
    auto total = [&](double v) {  // in every thread; one barrier
        v = wave_sum(v);
        par ^= 1;
        if ((threadIdx.x & 63) == 0) slots[par][threadIdx.x >> 6] = v;
        lds_barrier();
        return slot_sum(slots[par], NT / 64);
    };
    double obb, norm, stop = 0.0;
    if (ps.first) {
        const double s2 = total(r6[0] * r6[0] + r6[1] * r6[1]);
        obb = s2;
        if (!outer_state(s2, s2, ps.rtol, ps.tol_floor, norm, stop)) {  // b = 0 or not finite: x = 0
#pragma unroll
            for (int s = 0; s < 2; ++s)
                if (c.sp[s] >= 0) {
                    ps.x64[co + threadIdx.x + NT * s] = 0.0;
                    ps.r64[co + threadIdx.x + NT * s] = r6[s];
                }
            if (threadIdx.x < ps.nblk) ps.partial[(size_t)col * ps.nblk + threadIdx.x] = threadIdx.x ? 0.0 : s2;
            if (threadIdx.x == 0) {
                st[col].obb = st[col].rr = s2;
                st[col].its = 0.0;
                ps.oact[col] = 0;
                ps.colnorm[col] = norm;
            }
            return;
        }
    } else {
        obb = st[col].obb;
        norm = ps.colnorm[col];
        stop = st[col].tol2;
    }
    const double inv_norm = 1.0 / norm;
#pragma unroll
    for (int s = 0; s < 2; ++s) rk[s] = (T)(r6[s] * inv_norm);
    double rz_old = 1.0, rz = 0.0, pq = 0.0, alpha = 0.0;
    bool off = false;
    int it = 0;
    while (it < max_iter) {
#pragma unroll
        for (int s = 0; s < 2; ++s) c.bl[s] = (float)rk[s];
        // LDS addresses and scaled coefficients are formed anew each iteration:
        // kept across it they would take the registers of the vectors
#pragma unroll
        for (int s = 0; s < BC::NS; ++s)
            asm volatile("" : "+v"(c.sp[s]), "+v"(c.si[s]), "+v"(c.sj[s]), "+v"(c.rw[s].c), "+v"(c.rw[s].dv));
        lds_barrier();  // the last reads of sx and sw are done
        c.run(cc, sx, sw, sbc, tmp);
        double d = 0.0;
        T zk[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            zk[s] = c.sp[s] >= 0 ? (T)sx[c.sp[s]] : (T)0;
            if (c.sp[s] >= 0) sz[c.sp[s]] = zk[s];
            d += (double)zk[s] * (double)rk[s];
        }
        rz = total(d);
        const T beta = it ? (T)(rz / rz_old) : (T)0, a_last = (T)alpha;
        T qk[2];
        d = 0.0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            qk[s] = 0;
            if (c.sp[s] < 0) continue;
            using Nb = typename OpT::Nb;
            const T az = fr[s] ? sop.combine(c.si[s], c.sj[s], row[s], lds_nb((const Nb*)nullptr, sz + c.sp[s], P)) : (T)0;
            const T ap = fr[s] ? sop.combine(c.si[s], c.sj[s], row[s], lds_nb((const Nb*)nullptr, sp + c.sp[s], P)) : (T)0;
            xk[s] += a_last * pk[s];
            pk[s] = zk[s] + beta * pk[s];
            qk[s] = az + beta * ap;
            d += (double)pk[s] * (double)qk[s];
        }
        pq = total(d);  // and every read of sp is done
        ++it;
        alpha = pq > 0.0 ? rz / pq : 0.0;
        rz_old = rz;
        d = 0.0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (c.sp[s] >= 0) sp[c.sp[s]] = pk[s];
            rk[s] -= (T)alpha * qk[s];
            d += (double)rk[s] * (double)rk[s];
        }
        off = !(pq > 0.0);
        if (off) break;  // uniform
        off = total(d) <= stop;
        if (off) break;
    }
    // x64 += |r| d with d the inner solution, the last step included
    double* const sv = kWide ? (double*)sz : sx64;
    double x6[2], bk[2];
    typename Op64T::Row row64[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (c.sp[s] < 0) continue;
        const int q = threadIdx.x + NT * s;
        x6[s] = ps.first ? 0.0 : ps.x64[co + q];
        bk[s] = bc[q];
        row64[s] = sop64.row(c.si[s], c.sj[s], q);
        const T d = xk[s] + (T)alpha * pk[s];
        x6[s] += norm * (double)d;
        sv[c.sp[s]] = x6[s];  // earlier reads lie before the last sum's barrier
        ps.x64[co + q] = x6[s];
    }
    lds_barrier();
    double v2 = 0.0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (c.sp[s] < 0) continue;
        using Nb = typename Op64T::Nb;
        const double v =
            fr[s] ? bk[s] - sop64.combine(c.si[s], c.sj[s], row64[s], lds_nb((const Nb*)nullptr, sv + c.sp[s], P)) : 0.0;
        ps.r64[co + threadIdx.x + NT * s] = v;
        v2 += v * v;
    }
    const double s2 = total(v2);
    if (threadIdx.x < ps.nblk) ps.partial[(size_t)col * ps.nblk + threadIdx.x] = threadIdx.x ? 0.0 : s2;
    if (threadIdx.x == 0) {
        double tol2 = stop;
        const bool on = outer_state(s2, obb, ps.rtol, ps.tol_floor, norm, tol2);
        st[col].obb = obb;
        st[col].rr = s2;
        st[col].its = it;
        st[col].tol2 = tol2;
        ps.oact[col] = on ? 1 : 0;
        ps.colnorm[col] = norm;
    }
}

}  // namespace hinv
