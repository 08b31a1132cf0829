// Quadratic (P2) state space: operator, two-level PCG, observation, gradient
// and Hessian-output kernels (see p2.h).
#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

#include "grid.h"
#include "p2.h"
#include "problem.h"

namespace hinv {

namespace {

inline dim3 grid2(int n, int nc) { return dim3(ceil_div(n, kBlock), nc); }

// Fine-grid offset (dx, dy) in [0, 2]^2 of local dof j of triangle s of a cell.
__host__ __device__ inline void p2_offset(int s, int j, int& dx, int& dy) {
    // lower: a (0,0) r (2,0) b (2,2) | mid(a,r) (1,0) mid(r,b) (2,1) mid(a,b) (1,1)
    // upper: a (0,0) r (0,2) b (2,2) | mid(a,r) (0,1) mid(r,b) (1,2) mid(a,b) (1,1)
    constexpr int lx[6] = {0, 2, 2, 1, 2, 1}, ly[6] = {0, 0, 2, 0, 1, 1};
    dx = s == 0 ? lx[j] : ly[j];
    dy = s == 0 ? ly[j] : lx[j];
}

// Local dof of triangle s at cell offset (dx, dy), or -1.
__device__ inline int p2_local(int s, int dx, int dy) {
    if (s == 1) {  // the upper triangle mirrors the lower one across the diagonal
        const int t = dx;
        dx = dy;
        dy = t;
    }
    // lower triangle: dy <= dx
    if (dy > dx) return -1;
    constexpr int tab[3][3] = {{0, 3, 1}, {-1, 5, 4}, {-1, -1, 2}};  // [dy][dx]
    return tab[dy][dx];
}

__device__ inline int p2_dof(int side, int ci, int cj, int s, int j) {
    int dx, dy;
    p2_offset(s, j, dx, dy);
    return (2 * cj + dy) * side + 2 * ci + dx;
}

// Visits the triangles that hold fine node (I, J): f(ci, cj, s, local dof).
template <class F>
__device__ inline void p2_for_triangles(int N, int I, int J, F f) {
    const int ci0 = I > 0 ? max(0, (I - 1) / 2) : 0, ci1 = min(N - 1, I / 2);
    const int cj0 = J > 0 ? max(0, (J - 1) / 2) : 0, cj1 = min(N - 1, J / 2);
    for (int cj = cj0; cj <= cj1; ++cj)
        for (int ci = ci0; ci <= ci1; ++ci)
            for (int s = 0; s < 2; ++s) {
                const int loc = p2_local(s, I - 2 * ci, J - 2 * cj);
                if (loc >= 0) f(ci, cj, s, loc);
            }
}

// Partial sums (n.. per column: one a workgroup, or one when they are summed
// in a launch of their own) and the smoother's coefficients.
struct P2Red {
    double *pq, *rr, *rz;
    int npq, nrr, nrz;
};
struct P2Cheb {
    double inv_theta, c1, c2;
};

template <typename T>
__device__ inline T* colp(T* p, int ld) {
    return p + (size_t)blockIdx.y * ld;
}

// Row (I, J) of A_2 on the values x(dx, dy) at the node's offsets and the
// triangle coefficients c(s, di, dj) of the cells (I/2 + di, J/2 + dj).  On
// legs 1 the quadratic element couples a vertex to the other vertex (1/6) and
// the midpoint (-2/3) of each leg it lies on, a leg's midpoint to itself (8/3),
// the leg's ends (-2/3) and the diagonal's midpoint (-4/3), and nothing else:
// 9 points for a vertex row, 5 for the others.
template <class X, class C>
__device__ __forceinline__ double p2_row(int I, int J, X x, C c) {
    constexpr double k13 = 1.0 / 3.0, k23 = 2.0 / 3.0, k43 = 4.0 / 3.0, k83 = 8.0 / 3.0;
    const double x0 = x(0, 0);
    if (I & 1) {
        const double xs = x(0, -1), xn = x(0, 1), xw = x(-1, 0), xe = x(1, 0), cl = c(0, 0, 0);
        if (J & 1) return cl * (k83 * x0 - k43 * (xs + xe)) + c(1, 0, 0) * (k83 * x0 - k43 * (xw + xn));
        const double t = k83 * x0 - k23 * (xw + xe);
        return cl * (t - k43 * xn) + c(1, 0, -1) * (t - k43 * xs);
    }
    const double cu = c(1, 0, 0), cw = c(0, -1, 0);
    const double xw = x(-1, 0), xe = x(1, 0), xs = x(0, -1), xn = x(0, 1);
    if (J & 1) {
        const double t = k83 * x0 - k23 * (xs + xn);
        return cu * (t - k43 * xe) + cw * (t - k43 * xw);
    }
    const double cd = c(1, 0, -1);
    const double e = c(0, 0, 0) + cd, w = cw + c(1, -1, -1), n = cu + cw, so = cd + c(0, -1, -1);
    return 0.5 * (e * (x0 + k13 * x(2, 0) - k43 * xe) + w * (x0 + k13 * x(-2, 0) - k43 * xw) +
                  n * (x0 + k13 * x(0, 2) - k43 * xn) + so * (x0 + k13 * x(0, -2) - k43 * xs));
}

// Coefficient of triangle s of cell (ci, cj), 0 outside the mesh.
__device__ __forceinline__ double p2_coef(int N, const double* __restrict__ cT, int ci, int cj, int s) {
    const bool in = ci >= 0 && cj >= 0 && ci < N && cj < N;
    return in ? cT[2 * (cj * N + ci) + s] : 0.0;
}

// y = scale K[coef] x on the free rows, 0 on the Dirichlet rows.  mhat: the
// coefficient is s_T = (c_T/3) sum mhat over the triangle's vertices, per
// column.  ldx = 0: the same x for every column.
template <bool SENS>
__global__ void k_p2_apply(int N, const double* __restrict__ cT, const double* __restrict__ mhat, int ldm,
                           const double* __restrict__ x, int ldx, double scale, double* __restrict__ y, int ldy) {
    const int side = 2 * N + 1, ns = side * side;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= ns) return;
    const int J = k / side, I = k - J * side;
    double v = 0.0;
    if (J > 0 && J < 2 * N) {
        const double* xc = x + (size_t)blockIdx.y * ldx;
        const double* mh = SENS ? colp(mhat, ldm) : nullptr;
        // neighbours outside the mesh meet a zero coefficient
        auto xv = [&](int dx, int dy) { return xc[min(max(J + dy, 0), 2 * N) * side + min(max(I + dx, 0), 2 * N)]; };
        auto cv = [&](int s, int di, int dj) {
            const int ci = (I >> 1) + di, cj = (J >> 1) + dj;
            double c = p2_coef(N, cT, ci, cj, s);
            if constexpr (SENS) {
                if (ci >= 0 && ci < N && cj >= 0 && cj < N) {
                    int ka, kr, kb;
                    tri_nodes(N, ci, cj, s, ka, kr, kb);
                    c = c * (1.0 / 3.0) * (mh[ka] + mh[kr] + mh[kb]);
                }
            }
            return c;
        };
        v = scale * p2_row(I, J, xv, cv);
    }
    colp(y, ldy)[k] = v;
}

// 1 / diag(A_2) on the free rows, 0 on the Dirichlet rows.
__global__ void k_p2_dinv(int N, P2Elem el, const double* __restrict__ cT, double* __restrict__ dinv) {
    const int side = 2 * N + 1, ns = side * side;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= ns) return;
    const int J = k / side, I = k - J * side;
    double dg = 0.0;
    p2_for_triangles(N, I, J, [&](int ci, int cj, int s, int loc) {
        dg += cT[2 * (cj * N + ci) + s] * el.K[s][loc][loc];
    });
    dinv[k] = (J > 0 && J < 2 * N && dg > 0.0) ? 1.0 / dg : 0.0;
}

__global__ void k_p2_top(int N, double* __restrict__ u) {
    const int side = 2 * N + 1;
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I < side) u[(size_t)(2 * N) * side + I] = 1.0;
}

// ---- the solver's three kernels -------------------------------------------
// A workgroup owns V x V P1 vertices with four nodes each: (2i, 2j) and the
// ones right, above and diagonally above.  What the stages of a kernel need of
// the neighbours' nodes is computed again in LDS (the stencil reaches two
// nodes), so a PCG iteration is three launches around the P1 V-cycle where one
// launch a vector operation took twenty: a 129 x 129 grid is all latency.
// Measured at 64^2, one column: 2.98 -> 0.85 ms a full Hessian
// action; tiles of 16 x 16 vertices were slower or equal at every size up
// to 1024^2 x 1 and 64^2 x 50 (50 columns: 1.64 against 1.96 ms).
struct P2Tile {
    static constexpr int V = kP2Tile;
    static constexpr int D = 2 * V + 7;      // nodes 2 i0 - 4 .. 2 (i0 + V) + 2
    static constexpr int Z = 2 * V + 3;      // nodes 2 i0 - 2 .. 2 (i0 + V)
    static constexpr int C = V + 3;          // cells i0 - 2 .. i0 + V
    static constexpr int SD = (D * D + 255) / 256, SZ = (Z * Z + 255) / 256, SO = (4 * V * V + 255) / 256;
    int N, i0, j0;
    __device__ P2Tile(int N_) : N(N_), i0(blockIdx.x * V), j0(blockIdx.y * V) {}
    __device__ bool free_node(int I, int J) const { return I >= 0 && I <= 2 * N && J > 0 && J < 2 * N; }
    __device__ bool owned(int I, int J) const {
        return I >= 2 * i0 && I < 2 * (i0 + V) && I <= 2 * N && J >= 2 * j0 && J < 2 * (j0 + V) && J <= 2 * N;
    }
    // node of item id of a square of side w around the tile
    __device__ void node(int id, int w, int& I, int& J) const {
        const int h = (w - 2 * V + 1) / 2, jj = id / w;  // D: 4, Z: 2, 2 V + 1: 1, 2 V: 0
        I = 2 * i0 - h + id - jj * w;
        J = 2 * j0 - h + jj;
    }
    __device__ int at(int I, int J) const { return (J - 2 * j0 + 4) * D + I - 2 * i0 + 4; }
    __device__ void load_coef(const double* __restrict__ cT, double* cs) const {
        for (int id = threadIdx.x; id < 2 * C * C; id += 256) {
            const int s = id & 1, t = id >> 1, cj = t / C, ci = t - cj * C;
            cs[id] = p2_coef(N, cT, i0 - 2 + ci, j0 - 2 + cj, s);
        }
    }
    // row (I, J) on the values a (indexed by at) and the coefficients cs
    __device__ double row(int I, int J, const double* a, const double* cs) const {
        const double* ap = a + at(I, J);
        const double* cp = cs + 2 * (((J >> 1) - j0 + 2) * C + (I >> 1) - i0 + 2);
        return p2_row(
            I, J, [&](int dx, int dy) { return ap[dy * D + dx]; },
            [&](int s, int di, int dj) { return cp[2 * (dj * C + di) + s]; });
    }
};

// Sum of n partials in a fixed order, in every thread (256 threads).
__device__ __forceinline__ double p2_total(const double* __restrict__ part, int n) {
    __shared__ double ws[4];
    double v = 0.0;
    for (int b = threadIdx.x; b < n; b += 256) v += part[b];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (ws[0] + ws[1]) + (ws[2] + ws[3]);
    __syncthreads();
    return v;
}

__device__ __forceinline__ void p2_partial(double v, double* part) {
    const double s = block_sum(v);
    if (threadIdx.x == 0) part[(size_t)blockIdx.z * gridDim.x * gridDim.y + blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// The PCG step x += alpha p, r <- r - alpha q (r_in -> r_out; alpha = rz / pq,
// no step for pq <= 0) with its r^T r, then the cycle's way down: z = two
// Chebyshev-Jacobi steps from zero, rc = P^T (r - A z) (P1 vertex: its own
// value plus half of the midpoints of the edges at it), 0 on the P1 Dirichlet
// rows.  FIRST: r = b on the free rows, x = 0.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_p2_down(int N, const double* __restrict__ cT,
                                                 const double* __restrict__ dinv, const double* __restrict__ r_in,
                                                 int ldr, double* __restrict__ r_out, const double* __restrict__ p,
                                                 const double* __restrict__ q, double* __restrict__ x, int ldx,
                                                 double* __restrict__ z, double* __restrict__ rc, int ldc,
                                                 P2Red red, P2Cheb ch, P2Col* __restrict__ st, int cur,
                                                 const int* __restrict__ act) {
    using T = P2Tile;
    constexpr int V = T::V;
    const int col = blockIdx.z;
    const bool on = FIRST || act[col];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) st[col].on = on;
    if (!on) return;
    const T t(N);
    const int side = 2 * N + 1, ns = side * side;
    __shared__ double cs[2 * T::C * T::C], sr[T::D * T::D], sd[T::D * T::D], sa[T::D * T::D], sz[T::D * T::D];
    const double* rin = r_in + (size_t)col * ldr;
    const size_t o = (size_t)col * ns;
    double rv[T::SD], qv[T::SD], dv[T::SD], pv[T::SD], xv[T::SD];
#pragma unroll
    for (int u = 0; u < T::SD; ++u) {
        const int id = min((int)threadIdx.x + 256 * u, T::D * T::D - 1);
        int I, J;
        t.node(id, T::D, I, J);
        const bool fr = t.free_node(I, J);
        const int k = fr ? J * side + I : side;
        rv[u] = rin[k];
        dv[u] = fr ? dinv[k] : 0.0;
        if (!FIRST) {
            qv[u] = q[o + k];
            pv[u] = xv[u] = 0.0;
            if (t.owned(I, J)) {
                pv[u] = p[o + k];
                xv[u] = x[(size_t)col * ldx + k];
            }
        }
    }
    t.load_coef(cT, cs);
    double alpha = 0.0;
    if (!FIRST) {
        const double pq = p2_total(red.pq + (size_t)col * red.npq, red.npq);
        alpha = pq > 0.0 ? st[col].rz[cur] / pq : 0.0;
    }
    double rr = 0.0;
#pragma unroll
    for (int u = 0; u < T::SD; ++u) {
        const int id = threadIdx.x + 256 * u;
        if (id >= T::D * T::D) break;
        int I, J;
        t.node(id, T::D, I, J);
        const bool fr = t.free_node(I, J);
        double v = fr ? rv[u] : 0.0;
        if (!FIRST && fr) v -= alpha * qv[u];
        if (t.owned(I, J)) {
            const int k = J * side + I;
            r_out[o + k] = v;
            if (FIRST)
                x[(size_t)col * ldx + k] = 0.0;
            else if (fr)
                x[(size_t)col * ldx + k] = xv[u] + alpha * pv[u];
            rr += v * v;
        }
        sr[id] = v;
        sd[id] = dv[u];
        sa[id] = dv[u] * v * ch.inv_theta;
    }
    __syncthreads();
    for (int id = threadIdx.x; id < T::Z * T::Z; id += 256) {
        int I, J;
        t.node(id, T::Z, I, J);
        const int a = t.at(I, J);
        double v = 0.0;
        if (t.free_node(I, J)) v = sa[a] + (ch.c1 * sa[a] + ch.c2 * sd[a] * (sr[a] - t.row(I, J, sa, cs)));
        sz[a] = v;
        if (t.owned(I, J)) z[o + J * side + I] = v;
    }
    __syncthreads();
    constexpr int R = 2 * V + 1;
    for (int id = threadIdx.x; id < R * R; id += 256) {
        int I, J;
        t.node(id, R, I, J);
        const int a = t.at(I, J);
        sa[a] = t.free_node(I, J) ? sr[a] - t.row(I, J, sz, cs) : 0.0;
    }
    __syncthreads();
    for (int id = threadIdx.x; id < V * V; id += 256) {
        const int i = t.i0 + id % V, j = t.j0 + id / V;
        if (i > N || j > N) continue;
        const double* a = sa + t.at(2 * i, 2 * j);
        constexpr int D = T::D;
        const double v = a[0] + 0.5 * (((a[-1] + a[1]) + (a[-D] + a[D])) + (a[D + 1] + a[-D - 1]));
        rc[(size_t)col * ldc + j * (N + 1) + i] = j > 0 && j < N ? v : 0.0;
    }
    p2_partial(rr, red.rr);
}

// The convergence test, then the cycle's way up: z + P e, and two
// Chebyshev-Jacobi steps from it on the residual; z_out with its r^T z.
__global__ __launch_bounds__(256) void k_p2_up(int N, const double* __restrict__ cT, const double* __restrict__ dinv,
                                               const double* __restrict__ r, const double* __restrict__ z,
                                               const double* __restrict__ e, int lde, double* __restrict__ z_out,
                                               P2Red red, P2Cheb ch, P2Col* __restrict__ st, double tol2, int first,
                                               int* __restrict__ act) {
    using T = P2Tile;
    constexpr int V = T::V;
    const int col = blockIdx.z;
    if (!st[col].on) return;  // not act: this launch clears it
    const T t(N);
    const int side = 2 * N + 1, ns = side * side, N1 = N + 1;
    __shared__ double cs[2 * T::C * T::C], sr[T::D * T::D], sd[T::D * T::D], sa[T::D * T::D], sz[T::D * T::D];
    const size_t o = (size_t)col * ns;
    const double* ec = e + (size_t)col * lde;
    double rv[T::SD], dv[T::SD], zv[T::SD], e0[T::SD], e1[T::SD];
#pragma unroll
    for (int u = 0; u < T::SD; ++u) {
        const int id = min((int)threadIdx.x + 256 * u, T::D * T::D - 1);
        int I, J;
        t.node(id, T::D, I, J);
        const bool fr = t.free_node(I, J);
        I = fr ? I : 0;
        J = fr ? J : 1;
        const int k = J * side + I;
        rv[u] = fr ? r[o + k] : 0.0;
        dv[u] = fr ? dinv[k] : 0.0;
        // the P1 function at the node: even coordinates give one vertex,
        // odd ones the two ends of the edge
        const double a = ec[(J >> 1) * N1 + (I >> 1)], b = ec[((J + 1) >> 1) * N1 + ((I + 1) >> 1)];
        zv[u] = fr ? z[o + k] : 0.0;
        e0[u] = fr ? a : 0.0;
        e1[u] = fr ? b : 0.0;
    }
    t.load_coef(cT, cs);
    // column state: the first pass sets |b|^2; a column ends when |r| <= tol |b|
    // or is not a number.  Every workgroup decides alike from the same sum.
    const double rr = p2_total(red.rr + (size_t)col * red.nrr, red.nrr);
    const double bb = first ? rr : st[col].bb;
    const bool done = first ? !(rr > 0.0 && rr < INFINITY) : !(rr > tol2 * bb);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        st[col].rr = rr;
        if (first) st[col].bb = rr;
        st[col].its += first ? 0 : 1;
        if (done) act[col] = st[col].live = 0;
    }
    if (done) return;
#pragma unroll
    for (int u = 0; u < T::SD; ++u) {
        const int id = threadIdx.x + 256 * u;
        if (id >= T::D * T::D) break;
        sr[id] = rv[u];
        sd[id] = dv[u];
        sz[id] = zv[u] + 0.5 * (e0[u] + e1[u]);
    }
    __syncthreads();
    double rs[T::SZ];
#pragma unroll
    for (int u = 0; u < T::SZ; ++u) {
        const int id = threadIdx.x + 256 * u;
        if (id >= T::Z * T::Z) break;
        int I, J;
        t.node(id, T::Z, I, J);
        const int a = t.at(I, J);
        rs[u] = t.free_node(I, J) ? sr[a] - t.row(I, J, sz, cs) : 0.0;
        sa[a] = sd[a] * rs[u] * ch.inv_theta;
    }
    __syncthreads();
    double rz = 0.0;
#pragma unroll
    for (int u = 0; u < T::SZ; ++u) {
        const int id = threadIdx.x + 256 * u;
        if (id >= T::Z * T::Z) break;
        int I, J;
        t.node(id, T::Z, I, J);
        if (!t.owned(I, J)) continue;
        const int a = t.at(I, J);
        double v = 0.0;
        if (t.free_node(I, J))
            v = sz[a] + sa[a] + (ch.c1 * sa[a] + ch.c2 * sd[a] * (rs[u] - t.row(I, J, sa, cs)));
        z_out[o + J * side + I] = v;
        rz += sr[a] * v;
    }
    p2_partial(rz, red.rz);
}

// p = z + beta p_old, beta = rz / rz_old (first: p = z), q = A p, p^T q.
__global__ __launch_bounds__(256) void k_p2_dir(int N, const double* __restrict__ cT, const double* __restrict__ z,
                                                const double* __restrict__ p_old, double* __restrict__ p,
                                                double* __restrict__ q, P2Red red, P2Col* __restrict__ st, int cur,
                                                int first, const int* __restrict__ act) {
    using T = P2Tile;
    constexpr int V = T::V;
    const int col = blockIdx.z;
    if (!act[col]) return;
    const T t(N);
    const int side = 2 * N + 1, ns = side * side;
    __shared__ double cs[2 * T::C * T::C], sp[T::D * T::D];
    const size_t o = (size_t)col * ns;
    double zv[T::SZ], pv[T::SZ];
#pragma unroll
    for (int u = 0; u < T::SZ; ++u) {
        const int id = min((int)threadIdx.x + 256 * u, T::Z * T::Z - 1);
        int I, J;
        t.node(id, T::Z, I, J);
        const bool fr = t.free_node(I, J);
        const int k = fr ? J * side + I : side;
        zv[u] = fr ? z[o + k] : 0.0;
        pv[u] = fr && !first ? p_old[o + k] : 0.0;
    }
    t.load_coef(cT, cs);
    const double rz = p2_total(red.rz + (size_t)col * red.nrz, red.nrz);
    const double beta = first ? 0.0 : rz / st[col].rz[1 - cur];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) st[col].rz[cur] = rz;
#pragma unroll
    for (int u = 0; u < T::SZ; ++u) {
        const int id = threadIdx.x + 256 * u;
        if (id >= T::Z * T::Z) break;
        int I, J;
        t.node(id, T::Z, I, J);
        const double v = first ? zv[u] : zv[u] + beta * pv[u];
        sp[t.at(I, J)] = v;
        if (t.owned(I, J)) p[o + J * side + I] = v;
    }
    __syncthreads();
    double pq = 0.0;
    for (int id = threadIdx.x; id < 4 * V * V; id += 256) {
        int I, J;
        t.node(id, 2 * V, I, J);
        if (!t.owned(I, J)) continue;
        const double v = t.free_node(I, J) ? t.row(I, J, sp, cs) : 0.0;
        q[o + J * side + I] = v;
        pq += sp[t.at(I, J)] * v;
    }
    p2_partial(pq, red.pq);
}

__global__ __launch_bounds__(256) void k_p2_finish(const double* __restrict__ part, int n, double* __restrict__ out) {
    const double v = p2_total(part + (size_t)blockIdx.x * n, n);
    if (threadIdx.x == 0) out[blockIdx.x] = v;
}

__global__ void k_p2_start(int nc, P2Col* __restrict__ st) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < nc) st[c] = P2Col{0.0, 0.0, {0.0, 0.0}, 0, 1, 1};
}

__global__ void k_p2_zero(int ns, double* __restrict__ x, int ld) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < ns) colp(x, ld)[k] = 0.0;
}

// u_T^T K_T w_T of triangle (ci, cj, s)
__device__ inline double p2_form(const P2Elem& el, int side, int ci, int cj, int s, const double* u,
                                 const double* w) {
    double uv[6], wv[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const int d = p2_dof(side, ci, cj, s, j);
        uv[j] = u[d];
        wv[j] = w[d];
    }
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        double t = 0.0;
#pragma unroll
        for (int b = 0; b < 6; ++b) t += el.K[s][a][b] * wv[b];
        acc += uv[a] * t;
    }
    return acc;
}

// g_v = sum_{T ni v} (c_T/3) u_T^T K p_T
__global__ void k_p2_grad(int N, P2Elem el, const double* __restrict__ cT, const double* __restrict__ u,
                          const double* __restrict__ p, double* __restrict__ g) {
    const int N1 = N + 1, side = 2 * N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int j = k / N1, i = k - j * N1;
    double acc = 0.0;
    for_incident_triangles(N, i, j, [&](int ci, int cj, int s, int) {
        acc += cT[2 * (cj * N + ci) + s] * (1.0 / 3.0) * p2_form(el, side, ci, cj, s, u, p);
    });
    g[k] = acc;
}

// (H mhat)_v without the prior: sum_{T ni v} (c_T/3) [u K phat + uhat K p + (1/3) sum_T mhat u K p]
// (Gauss-Newton: the first term only)
__global__ void k_p2_hess_out(int N, P2Elem el, const double* __restrict__ cT, const double* __restrict__ u,
                              const double* __restrict__ p, const double* __restrict__ uh, int ldu,
                              const double* __restrict__ ph, int ldp, const double* __restrict__ mh, int ldm,
                              double* __restrict__ out, int ldo, int gn, const double* __restrict__ add,
                              int ldadd) {
    const int N1 = N + 1, side = 2 * N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int j = k / N1, i = k - j * N1;
    const double* uhc = colp(uh, ldu);
    const double* phc = colp(ph, ldp);
    const double* mhc = colp(mh, ldm);
    double acc = 0.0;
    for_incident_triangles(N, i, j, [&](int ci, int cj, int s, int) {
        double v = p2_form(el, side, ci, cj, s, u, phc);
        if (!gn) {
            int ka, kr, kb;
            tri_nodes(N, ci, cj, s, ka, kr, kb);
            v += p2_form(el, side, ci, cj, s, uhc, p);
            v += (1.0 / 3.0) * (mhc[ka] + mhc[kr] + mhc[kb]) * p2_form(el, side, ci, cj, s, u, p);
        }
        acc += cT[2 * (cj * N + ci) + s] * (1.0 / 3.0) * v;
    });
    if (add) acc = colp(add, ldadd)[k] + acc;
    colp(out, ldo)[k] = acc;
}

// Observation point o in cell (i, j), triangle as for P1 (lower when the
// local x offset is >= the local y offset), barycentric (lam_a, lam_r, lam_b);
// the six P2 basis values there.
__global__ void k_p2_obs_setup(int N, int q, const double* __restrict__ xy, int* __restrict__ node,
                               double* __restrict__ w) {
    const int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= q) return;
    const int side = 2 * N + 1;
    const double x = xy[2 * o] * N, y = xy[2 * o + 1] * N;
    int i = (int)floor(x), j = (int)floor(y);
    i = i < 0 ? 0 : (i > N - 1 ? N - 1 : i);
    j = j < 0 ? 0 : (j > N - 1 ? N - 1 : j);
    const double xi = x - i, ze = y - j;
    const int s = xi >= ze ? 0 : 1;
    const double la = s == 0 ? 1.0 - xi : 1.0 - ze;
    const double lr = s == 0 ? xi - ze : ze - xi;
    const double lb = s == 0 ? ze : xi;
    const double psi[6] = {la * (2.0 * la - 1.0), lr * (2.0 * lr - 1.0), lb * (2.0 * lb - 1.0),
                           4.0 * la * lr,         4.0 * lr * lb,         4.0 * la * lb};
    for (int a = 0; a < 6; ++a) {
        node[6 * o + a] = p2_dof(side, i, j, s, a);
        w[6 * o + a] = psi[a];
    }
}

__global__ void k_p2_obs_gather(int q, const int* __restrict__ node, const double* __restrict__ w,
                                const double* __restrict__ u, int ldu, const double* __restrict__ d,
                                double* __restrict__ out, int ldo) {
    const int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= q) return;
    const double* uc = colp(u, ldu);
    double v = 0.0;
    for (int a = 0; a < 6; ++a) v += w[6 * o + a] * uc[node[6 * o + a]];
    if (d) v -= d[o];
    colp(out, ldo)[o] = v;
}

// y[dof] += scale (B^T v)[dof] over the dofs touched by observations (CSR, fixed order)
__global__ void k_p2_obs_scatter(int nt, const int* __restrict__ tnode, const int* __restrict__ tptr,
                                 const int* __restrict__ tent, const double* __restrict__ w,
                                 const double* __restrict__ v, int ldv, double scale, double* __restrict__ y,
                                 int ldy) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const double* vc = colp(v, ldv);
    double s = 0.0;
    for (int e = tptr[t]; e < tptr[t + 1]; ++e) {
        const int ent = tent[e];
        s += w[ent] * vc[ent / 6];
    }
    colp(y, ldy)[tnode[t]] += scale * s;
}

}  // namespace

// ---------------------------------------------------------------- host ---
P2Elem p2_element() {
    // cell with legs 1; lower: a (0,0), r (1,0), b (1,1); upper: a (0,0), r (0,1), b (1,1).
    // Barycentric gradients: lower lam_a = 1 - x, lam_r = x - y, lam_b = y;
    // upper lam_a = 1 - y, lam_r = y - x, lam_b = x.  Area 1/2.
    const double G[2][3][2] = {{{-1, 0}, {1, -1}, {0, 1}}, {{0, -1}, {-1, 1}, {1, 0}}};
    const int ev[3][2] = {{0, 1}, {1, 2}, {0, 2}};  // local edges of the midpoint dofs
    P2Elem el{};
    for (int s = 0; s < 2; ++s)
        for (int qp = 0; qp < 3; ++qp) {
            double lam[3] = {0, 0, 0};
            lam[ev[qp][0]] = lam[ev[qp][1]] = 0.5;
            double g[6][2];
            for (int v = 0; v < 3; ++v)
                for (int d = 0; d < 2; ++d) g[v][d] = (4.0 * lam[v] - 1.0) * G[s][v][d];
            for (int e = 0; e < 3; ++e) {
                const int v = ev[e][0], w = ev[e][1];
                for (int d = 0; d < 2; ++d) g[3 + e][d] = 4.0 * (lam[w] * G[s][v][d] + lam[v] * G[s][w][d]);
            }
            for (int a = 0; a < 6; ++a)
                for (int b = 0; b < 6; ++b)
                    el.K[s][a][b] += (0.5 / 3.0) * (g[a][0] * g[b][0] + g[a][1] * g[b][1]);
        }
    return el;
}

namespace {
// Largest eigenvalue of D^-1/2 K D^-1/2 of the element (power iteration on a
// 6 x 6 matrix whose spectrum is nonnegative).  A = sum c_T K_T and
// D = sum c_T diag(K_T) give x^T A x <= mu x^T D x for all x, so mu bounds the
// spectrum of D^-1 A_2 from above.
double element_bound(const P2Elem& el) {
    double mu = 0.0;
    for (int s = 0; s < 2; ++s) {
        double M[6][6];
        for (int a = 0; a < 6; ++a)
            for (int b = 0; b < 6; ++b) M[a][b] = el.K[s][a][b] / std::sqrt(el.K[s][a][a] * el.K[s][b][b]);
        double v[6] = {1, -0.7, 0.4, -0.9, 0.6, -0.3}, lam = 0.0;
        for (int it = 0; it < 500; ++it) {
            double w[6] = {0, 0, 0, 0, 0, 0}, nw = 0.0;
            for (int a = 0; a < 6; ++a)
                for (int b = 0; b < 6; ++b) w[a] += M[a][b] * v[b];
            for (int a = 0; a < 6; ++a) nw += w[a] * w[a];
            nw = std::sqrt(nw);
            for (int a = 0; a < 6; ++a) v[a] = w[a] / nw;
            lam = nw;
        }
        mu = std::max(mu, lam);
    }
    return mu;
}
}  // namespace

P2Space::P2Space(Ctx* ctx, int N_) : N(N_), side(2 * N_ + 1), ns((2 * N_ + 1) * (2 * N_ + 1)), ctx_(ctx) {
    el_ = p2_element();
    lmax_ = element_bound(el_) * 1.0001;  // power iteration converges from below
    dinv_.ensure(ns);
}

void P2Space::set_coefficient(const double* cT) {
    cT_ = cT;
    k_p2_dinv<<<ceil_div(ns, kBlock), kBlock, 0, ctx_->stream>>>(N, el_, cT, dinv_.get());
    HINV_LAUNCH_CHECK();
}

void P2Space::apply(int nc, const double* x, int ldx, double* y, int ldy, double scale) {
    if (!cT_) fail(HINV_ESTATE, "P2 operator used before its coefficient was set");
    k_p2_apply<false><<<grid2(ns, nc), kBlock, 0, ctx_->stream>>>(N, cT_, nullptr, 0, x, ldx, scale, y, ldy);
    HINV_LAUNCH_CHECK();
}

void P2Space::sens(int nc, const double* mhat, int ldm, const double* w, double scale, double* y, int ldy) {
    if (!cT_) fail(HINV_ESTATE, "P2 operator used before its coefficient was set");
    k_p2_apply<true><<<grid2(ns, nc), kBlock, 0, ctx_->stream>>>(N, cT_, mhat, ldm, w, 0, scale, y, ldy);
    HINV_LAUNCH_CHECK();
}

void P2Space::set_top(double* u) {
    k_p2_top<<<ceil_div(side, kBlock), kBlock, 0, ctx_->stream>>>(N, u);
    HINV_LAUNCH_CHECK();
}

void P2Space::forward_rhs(double* rhs) {
    ensure(1);
    double* uD = z_.get();
    k_p2_zero<<<ceil_div(ns, kBlock), kBlock, 0, ctx_->stream>>>(ns, uD, ns);
    HINV_LAUNCH_CHECK();
    set_top(uD);
    apply(1, uD, ns, rhs, ns, -1.0);
}

void P2Space::ensure(int nc) {
    if (nc <= cap_) return;
    cap_ = 0;  // until every buffer is there
    const size_t len = (size_t)ns * nc;
    for (auto* b : {&r_, &r2_, &z_, &z2_, &p_, &p2_, &q_v_}) b->ensure(len);
    const int nt = ceil_div(N + 1, kP2Tile);
    part_.ensure(3 * (size_t)(nt * nt + 1) * nc);
    st_.ensure(nc);
    if (hst_) (void)hipHostFree(hst_);
    hst_ = nullptr;
    HINV_HIP(hipHostMalloc((void**)&hst_, sizeof(P2Col) * nc, hipHostMallocDefault));
    cap_ = nc;
}

P2Space::~P2Space() {
    if (hst_) (void)hipHostFree(hst_);
}

constexpr int kFirstRun = 16;  // a solve to 1e-10 takes 8 or 9 iterations from 4^2 to 256^2

int& P2Space::last_its(int nc, double rtol) {
    const long long key = 64LL * nc + std::min(63, std::max(0, (int)std::lround(-std::log10(rtol))));
    for (auto& kv : last_its_)
        if (kv.first == key) return kv.second;
    last_its_.push_back({key, 8});
    return last_its_.back().second;
}

// PCG with the two-level cycle: degree-2 Chebyshev-Jacobi on [lmax / 4, lmax]
// from zero, P^T of the residual through one V-cycle of the P1 hierarchy, P
// back, and the same smoother again from the corrected iterate.  An iteration
// is k_p2_dir, k_p2_down, the V-cycle and k_p2_up, which tests the column; the
// host enqueues as many iterations as the last such solve took, at most
// kFirstRun, before it first looks (launches for finished columns return at
// once, but are launches all the same).
void P2Space::run_solve(int nc, const double* b, int ldb, double* x, int ldx, Hierarchy& coarse, double rtol,
                          int max_iter) {
    hipStream_t s = ctx_->stream;
    const double hi = lmax_, lo = 0.25 * lmax_;
    const double theta = 0.5 * (hi + lo), dl = 0.5 * (hi - lo), sigma1 = theta / dl;
    const double rho0 = 1.0 / sigma1, rho1 = 1.0 / (2.0 * sigma1 - rho0);
    const P2Cheb ch{1.0 / theta, rho1 * rho0, 2.0 * rho1 / dl};
    const int nt = ceil_div(N + 1, kP2Tile), nblk = nt * nt, n1 = (N + 1) * (N + 1);
    const dim3 g(nt, nt, nc);
    const bool fold = nblk > kP2MaxParts;
    double* part[3];
    double* tot = part_.get() + 3 * (size_t)nblk * nc;  // folded sums
    for (int i = 0; i < 3; ++i) part[i] = part_.get() + (size_t)i * nblk * nc;
    // what the kernels write (one partial a workgroup) and read
    const P2Red w{part[0], part[1], part[2], nblk, nblk, nblk};
    const P2Red rd = fold ? P2Red{tot, tot + nc, tot + 2 * nc, 1, 1, 1} : w;
    auto finish = [&](int i) {
        if (!fold) return;
        k_p2_finish<<<nc, 256, 0, s>>>(part[i], nblk, tot + (size_t)i * nc);
        HINV_LAUNCH_CHECK();
    };
    // kernels read sums of the earlier ones and write their own
    const P2Red rdown{rd.pq, w.rr, w.rz, rd.npq, w.nrr, w.nrz}, rup{w.pq, rd.rr, w.rz, w.npq, rd.nrr, w.nrz},
        rdir{w.pq, w.rr, rd.rz, w.npq, w.nrr, rd.nrz};
    coarse.cycle_prepare(nc);
    int* act = coarse.cycle_active();
    double* rc = coarse.cycle_in();
    const double* e = coarse.cycle_out();
    double *R[2] = {r_.get(), r2_.get()}, *P[2] = {p_.get(), p2_.get()};
    k_p2_start<<<ceil_div(nc, 64), 64, 0, s>>>(nc, st_.get());
    HINV_LAUNCH_CHECK();
    const bool timing = ctx_->timer.any_on();
    std::vector<KernelTimer::Mark> marks;  // around the V-cycle of each iteration
    auto cycle = [&](int it) {
        finish(1);
        if (timing) marks.push_back(ctx_->timer.mark());
        coarse.cycle(nc);
        if (timing) marks.push_back(ctx_->timer.mark());
        k_p2_up<<<g, 256, 0, s>>>(N, cT_, dinv_.get(), R[it & 1], z_.get(), e, n1, z2_.get(), rup, ch, st_.get(),
                                     rtol * rtol, it == 0, act);
        HINV_LAUNCH_CHECK();
        finish(2);
    };
    // the first kernel zeroes x and reads b around the nodes of a tile, so
    // columns of b and x that may overlap are solved from a copy of b
    const auto at = [](const void* p) { return reinterpret_cast<uintptr_t>(p); };
    if (at(x + (size_t)ldx * nc) > at(b) && at(b + (size_t)ldb * nc) > at(x)) {
        dev_copy(ctx_, ns, nc, b, ldb, R[1], ns);
        b = R[1];
        ldb = ns;
    }
    k_p2_down<true><<<g, 256, 0, s>>>(N, cT_, dinv_.get(), b, ldb, R[0], nullptr, nullptr, x, ldx, z_.get(), rc,
                                         n1, rdown, ch, st_.get(), 0, act);
    HINV_LAUNCH_CHECK();
    cycle(0);
    int it = 0;
    auto run = [&](int to) {
        for (; it < to; ++it) {
            const int cur = it & 1;
            k_p2_dir<<<g, 256, 0, s>>>(N, cT_, z2_.get(), P[1 - cur], P[cur], q_v_.get(), rdir, st_.get(), cur,
                                          it == 0, act);
            HINV_LAUNCH_CHECK();
            finish(0);
            k_p2_down<false><<<g, 256, 0, s>>>(N, cT_, dinv_.get(), R[cur], ns, R[1 - cur], P[cur], q_v_.get(), x,
                                                  ldx, z_.get(), rc, n1, rdown, ch, st_.get(), cur, act);
            HINV_LAUNCH_CHECK();
            cycle(it + 1);
        }
    };
    run(std::min({max_iter, kFirstRun, last_its(nc, rtol)}));
    for (;;) {
        HINV_HIP(hipMemcpyAsync(hst_, st_.get(), sizeof(P2Col) * nc, hipMemcpyDeviceToHost, s));
        HINV_HIP(hipStreamSynchronize(s));
        int live = 0;
        for (int c = 0; c < nc; ++c) live += hst_[c].live;
        if (!live || it >= max_iter) break;
        run(std::min(max_iter, it + 2));
    }
    // the V-cycle of iteration i ran for the columns that took i steps
    for (size_t i = 0; 2 * i < marks.size(); ++i) {
        int ran = 0;
        for (int c = 0; c < nc; ++c) ran += hst_[c].its >= (int)i;
        for (int k : {kclass_for(kKDown, nc), kclass_for(kKUp, nc), (int)kKBottom})
            ctx_->timer.cut(marks[2 * i], marks[2 * i + 1], k, (double)ran / nc);
    }
}

void P2Space::solve(int nc, const double* b, int ldb, double* x, int ldx, Hierarchy& coarse, double rtol,
                    int max_iter, SolveStats* st) {
    if (!cT_) fail(HINV_ESTATE, "P2 solve before the coefficient was set");
    if (nc <= 0) return;
    ensure(nc);
    run_solve(nc, b, ldb, x, ldx, coarse, rtol, max_iter);
    double worst = 0.0;
    bool finite = true;
    int its = 0, live = 0;
    for (int c = 0; c < nc; ++c) {
        const P2Col& h = hst_[c];
        if (!std::isfinite(h.bb) || !std::isfinite(h.rr)) finite = false;
        its = std::max(its, h.its);
        live += h.live;
        if (!(h.bb > 0.0)) continue;
        const double rel = std::sqrt(h.rr / h.bb);
        if (!std::isfinite(rel)) finite = false;
        else worst = std::max(worst, rel);
    }
    if (live == 0 && finite) last_its(nc, rtol) = std::max(1, its);
    if (!finite) worst = std::numeric_limits<double>::quiet_NaN();
    if (st) {
        st->solves += nc;
        st->iterations += its;
        st->refinements += 1;
        if (std::isnan(worst) || worst > st->max_relres) st->max_relres = worst;
        st->converged = st->converged && live == 0 && finite;
    }
}

void P2Space::grad(const double* u, const double* p, double* g) {
    const int n1 = (N + 1) * (N + 1);
    k_p2_grad<<<ceil_div(n1, kBlock), kBlock, 0, ctx_->stream>>>(N, el_, cT_, u, p, g);
    HINV_LAUNCH_CHECK();
}

void P2Space::hess_out(int nc, bool gn, const double* u, const double* p, const double* uh, int ldu,
                       const double* ph, int ldp, const double* mh, int ldm, double* out, int ldo,
                       const double* add, int ldadd) {
    const int n1 = (N + 1) * (N + 1);
    k_p2_hess_out<<<grid2(n1, nc), kBlock, 0, ctx_->stream>>>(N, el_, cT_, u, p, uh, ldu, ph, ldp, mh, ldm, out,
                                                              ldo, gn ? 1 : 0, add, ldadd);
    HINV_LAUNCH_CHECK();
}

void P2Space::set_observations(int q, const double* xy_dev) {
    q_ = q;
    if (q == 0) return;
    hipStream_t s = ctx_->stream;
    obs_node_.ensure(6 * (size_t)q);
    obs_w_.ensure(6 * (size_t)q);
    k_p2_obs_setup<<<ceil_div(q, kBlock), kBlock, 0, s>>>(N, q, xy_dev, obs_node_.get(), obs_w_.get());
    HINV_LAUNCH_CHECK();
    // transpose structure: dof -> list of (6 o + a), from the device's dof indices
    std::vector<int> hn(6 * (size_t)q);
    HINV_HIP(hipMemcpyAsync(hn.data(), obs_node_.get(), sizeof(int) * 6 * q, hipMemcpyDeviceToHost, s));
    HINV_HIP(hipStreamSynchronize(s));
    std::vector<int> order(6 * (size_t)q);
    for (int e = 0; e < 6 * q; ++e) order[e] = e;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return hn[a] < hn[b]; });
    std::vector<int> tn, tp, te;
    for (int e = 0; e < 6 * q; ++e) {
        const int nd = hn[order[e]];
        if (tn.empty() || tn.back() != nd) {
            tn.push_back(nd);
            tp.push_back(e);
        }
        te.push_back(order[e]);
    }
    tp.push_back(6 * q);
    n_touch_ = (int)tn.size();
    t_node_.ensure(tn.size());
    t_ptr_.ensure(tp.size());
    t_ent_.ensure(te.size());
    HINV_HIP(hipMemcpyAsync(t_node_.get(), tn.data(), sizeof(int) * tn.size(), hipMemcpyHostToDevice, s));
    HINV_HIP(hipMemcpyAsync(t_ptr_.get(), tp.data(), sizeof(int) * tp.size(), hipMemcpyHostToDevice, s));
    HINV_HIP(hipMemcpyAsync(t_ent_.get(), te.data(), sizeof(int) * te.size(), hipMemcpyHostToDevice, s));
    HINV_HIP(hipStreamSynchronize(s));
}

void P2Space::observe(int nc, const double* u, int ldu, const double* d, double* out, int ldo) {
    if (q_ == 0) return;
    k_p2_obs_gather<<<grid2(q_, nc), kBlock, 0, ctx_->stream>>>(q_, obs_node_.get(), obs_w_.get(), u, ldu, d, out,
                                                                ldo);
    HINV_LAUNCH_CHECK();
}

void P2Space::observe_adjoint(int nc, const double* v, int ldv, double scale, double* y, int ldy) {
    if (q_ == 0) return;
    k_p2_obs_scatter<<<grid2(n_touch_, nc), kBlock, 0, ctx_->stream>>>(n_touch_, t_node_.get(), t_ptr_.get(),
                                                                       t_ent_.get(), obs_w_.get(), v, ldv, scale, y,
                                                                       ldy);
    HINV_LAUNCH_CHECK();
}

}  // namespace hinv
