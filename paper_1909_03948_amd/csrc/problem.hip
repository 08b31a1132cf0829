// Operations of the Poisson coefficient-inversion problem on the device.
//
//   forward         A(m)_FF u_F = -A(m)_FD u_D          (Sec. 5.1, Eq. eq:poisson_weak)
//   cost            1/2 sigma^-2 |B u - d|^2 + 1/2 (m - m_pr)^T R (m - m_pr)
//                                                        (Sec. 5.1, Eq. eq:cost-elliptic)
//   adjoint         A_FF p_F = -[B^T (B u - d)]_F / sigma^2              (App. A, eq:firstadj)
//   gradient        g_v = [R (m - m_pr)]_v + sum_{T ni v} (c_T / 3) |T| grad u . grad p
//                                                        (App. A, eq:firstcontrol)
//   inc. forward    A_FF uhat_F = -[K[s] u]_F, s_T = (c_T/3) sum_{w in T} mhat_w
//                                                        (App. A, eq:incrementals1)
//   inc. adjoint    A_FF phat_F = -[B^T B uhat / sigma^2 + K[s] p]_F  (eq:incrementals2)
//   Hessian         (H mhat)_v = sum_{T ni v} (c_T/3) |T| (grad u . grad phat + grad uhat . grad p)
//                    + sum_{T ni v} (c_T/9) (sum_{w in T} mhat_w) |T| grad u . grad p [+ R mhat]
//                                                        (eq:incrementals3)
//   prior           R = K_A M^-1 K_A, R^-1 = K_A^-1 M K_A^-1           (Sec. 5.1, Sec. 2.3)
//   prior draw      m_pr + K_A^-1 C_M eta, C_M C_M^T = M  (Sec. 4.3.1, App. C)
//
// c_T = exp((m_a + m_r + m_b) / 3) (centroid rule); K[s] is the stiffness with
// per-triangle coefficient s_T, a five-point stencil on this mesh.
#include <algorithm>

#include "grid.h"
#include "problem.h"

namespace hinv {

namespace {

inline dim3 grid2(int n, int nc) { return dim3(ceil_div(n, kBlock), nc); }

template <typename T>
__device__ inline T* colp(T* p, int ld) {
    return p + (size_t)blockIdx.y * ld;
}

// ---------------------------------------------------------- observations ---
// Point (x, y) lies in cell (i, j) = (min(floor(x N), N-1), min(floor(y N), N-1)),
// local offsets xi = x N - i, zeta = y N - j.  Lower triangle when xi >= zeta:
// P1 weights (1 - xi, xi - zeta, zeta) on (k(i,j), k(i+1,j), k(i+1,j+1));
// upper: (1 - zeta, zeta - xi, xi) on (k(i,j), k(i,j+1), k(i+1,j+1)).
__global__ void k_obs_setup(int N, int q, const double* __restrict__ xy, int* __restrict__ node,
                            double* __restrict__ w) {
    const int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= q) return;
    const double x = xy[2 * o] * N, y = xy[2 * o + 1] * N;
    int i = (int)floor(x), j = (int)floor(y);
    i = i < 0 ? 0 : (i > N - 1 ? N - 1 : i);
    j = j < 0 ? 0 : (j > N - 1 ? N - 1 : j);
    const double xi = x - i, ze = y - j;
    node[3 * o] = knode(i, j, N);
    node[3 * o + 2] = knode(i + 1, j + 1, N);
    if (xi >= ze) {
        node[3 * o + 1] = knode(i + 1, j, N);
        w[3 * o] = 1.0 - xi;
        w[3 * o + 1] = xi - ze;
        w[3 * o + 2] = ze;
    } else {
        node[3 * o + 1] = knode(i, j + 1, N);
        w[3 * o] = 1.0 - ze;
        w[3 * o + 1] = ze - xi;
        w[3 * o + 2] = xi;
    }
}

// out[o] = (B u)_o - d_o (d may be null).
__global__ void k_obs_gather(int q, const int* __restrict__ node, const double* __restrict__ w,
                             const double* __restrict__ u, int ldu, const double* __restrict__ d,
                             double* __restrict__ out, int ldo) {
    const int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= q) return;
    const double* uc = colp(u, ldu);
    double v = w[3 * o] * uc[node[3 * o]] + w[3 * o + 1] * uc[node[3 * o + 1]] +
               w[3 * o + 2] * uc[node[3 * o + 2]];
    if (d) v -= d[o];
    colp(out, ldo)[o] = v;
}

// y[node] += scale * (B^T v)[node] over the nodes touched by observations (CSR, fixed order).
__global__ void k_obs_scatter(int nt, const int* __restrict__ tnode, const int* __restrict__ tptr,
                              const int* __restrict__ tent, const double* __restrict__ w,
                              const double* __restrict__ v, int ldv, double scale,
                              double* __restrict__ y, int ldy) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const double* vc = colp(v, ldv);
    double s = 0.0;
    for (int e = tptr[t]; e < tptr[t + 1]; ++e) {
        const int ent = tent[e];
        s += w[ent] * vc[ent / 3];
    }
    colp(y, ldy)[tnode[t]] += scale * s;
}

// ----------------------------------------------------- state equation ---
// -A_FD u_D with u_D = 0 on y = 0 and 1 on y = 1: only row j = N-1 couples to
// the top boundary, through its north edge weight.
__global__ void k_forward_rhs(int N, const double* __restrict__ wN, double* __restrict__ rhs) {
    const int N1 = N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int j = k / N1;
    rhs[k] = (j == N - 1) ? wN[k] : 0.0;
}

__global__ void k_set_top(int N, double* __restrict__ u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= N) u[knode(i, N, N)] = 1.0;
}

// Per-triangle sensitivity coefficient s_T = (c_T/3)(mhat_a + mhat_r + mhat_b).
__device__ inline double sens_coef(int N, const double* cT, const double* mh, int ci, int cj, int s) {
    if (ci < 0 || ci >= N || cj < 0 || cj >= N) return 0.0;
    int ka, kr, kb;
    tri_nodes(N, ci, cj, s, ka, kr, kb);
    return cT[2 * (cj * N + ci) + s] * (1.0 / 3.0) * (mh[ka] + mh[kr] + mh[kb]);
}

// y[:,c] = scale * (K[s(mhat[:,c])] w)_k on free rows, 0 on Dirichlet rows.
// w is one full state-space vector (its Dirichlet values take part).
template <int C>
__global__ void k_sens(int N, int nc, const double* __restrict__ cT, const double* __restrict__ mhat,
                       int ldm, const double* __restrict__ w, double scale, double* __restrict__ y,
                       int ldy) {
    const int N1 = N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int j = k / N1, i = k - j * N1, col0 = blockIdx.y * C;
    const bool fr = j > 0 && j < N;
    if (fr) {
        // Straight-line form: the six triangles around C = (i, j), as in the
        // Hessian output kernel; a triangle outside the mesh (i = 0 or N)
        // reads C in place of its missing nodes and has weight 0, so every
        // load is issued before the first product.  Each edge takes the mean
        // of the coefficients of its two triangles, in the order E, W, N, S.
        const bool e = i < N, wv = i > 0;
        const int kE = e ? k + 1 : k, kW = wv ? k - 1 : k, kN = k + N1, kS = k - N1;
        const int kNE = e ? k + N1 + 1 : k, kSW = wv ? k - N1 - 1 : k;
        const int c0 = j * N + i;  // cell (i, j)
        const double fe = e ? 1.0 : 0.0, fw = wv ? 1.0 : 0.0;
        const double t1 = fe * cT[e ? 2 * c0 : 0], t2 = fe * cT[e ? 2 * c0 + 1 : 0];
        const double t3 = fw * cT[wv ? 2 * (c0 - 1) : 0], t4 = fe * cT[e ? 2 * (c0 - N) + 1 : 0];
        const double t5 = fw * cT[wv ? 2 * (c0 - N - 1) : 0], t6 = fw * cT[wv ? 2 * (c0 - N - 1) + 1 : 0];
        const double wk = w[k], wE = w[kE], wW = w[kW], wN = w[kN], wS = w[kS];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int col = min(col0 + c, nc - 1);  // past the end: the last column again
            const double* mh = mhat + (size_t)col * ldm;
            const double mC = mh[k], mE = mh[kE], mN = mh[kN], mNE = mh[kNE], mW = mh[kW], mS = mh[kS],
                         mSW = mh[kSW];
            double v = 0.0;
            const double s1 = t1 * (1.0 / 3.0) * (mC + mE + mNE);   // (C, E, NE)
            const double s2 = t2 * (1.0 / 3.0) * (mC + mN + mNE);   // (C, N, NE)
            const double s3 = t3 * (1.0 / 3.0) * (mW + mC + mN);    // (W, C, N)
            const double s4 = t4 * (1.0 / 3.0) * (mS + mC + mE);    // (S, C, E)
            const double s5 = t5 * (1.0 / 3.0) * (mSW + mS + mC);   // (SW, S, C)
            const double s6 = t6 * (1.0 / 3.0) * (mSW + mW + mC);   // (SW, W, C)
            if (e) v += 0.5 * (s1 + s4) * (wk - wE);
            if (wv) v += 0.5 * (s3 + s6) * (wk - wW);
            v += 0.5 * (s2 + s3) * (wk - wN);
            v += 0.5 * (s4 + s5) * (wk - wS);
            v *= scale;
            y[(size_t)col * ldy + k] = v;
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) y[(size_t)min(col0 + c, nc - 1) * ldy + k] = 0.0;
}

// Hessian output without the prior term (see file header).  gn drops the
// terms that carry the adjoint p.
template <int C>
__global__ void k_hess_out(int N, int nc, const double* __restrict__ cT, const double* __restrict__ u,
                           const double* __restrict__ p, const double* __restrict__ uh, int ldu,
                           const double* __restrict__ ph, int ldp, const double* __restrict__ mh,
                           int ldm, double* __restrict__ out, int ldo, int gn,
                           const double* __restrict__ add, int ldadd) {
    const int N1 = N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int j = k / N1, i = k - j * N1;
    // The six triangles around node C = (i, j) (cells split along the SW-NE
    // diagonal), in the order the sum takes them:
    //   cell (i, j):         (C, E, NE), (C, N, NE)
    //   cell (i - 1, j):     (W, C, N)       cell (i, j - 1): (S, C, E)
    //   cell (i - 1, j - 1): (SW, S, C), (SW, W, C)
    // A triangle outside the mesh reads C in place of its missing nodes and
    // has weight 0, so every load is issued before the first product.
    const bool e = i < N, w = i > 0, nn = j < N, sd = j > 0;
    const int kE = e ? k + 1 : k, kW = w ? k - 1 : k, kN = nn ? k + N1 : k, kS = sd ? k - N1 : k;
    const int kNE = e && nn ? k + N1 + 1 : k, kSW = w && sd ? k - N1 - 1 : k;
    const int c0 = j * N + i;  // cell (i, j)
    const double w1 = e && nn ? 1.0 : 0.0, w3 = w && nn ? 1.0 : 0.0, w4 = e && sd ? 1.0 : 0.0,
                 w5 = w && sd ? 1.0 : 0.0;
    const double t1 = w1 * cT[e && nn ? 2 * c0 : 0], t2 = w1 * cT[e && nn ? 2 * c0 + 1 : 0];
    const double t3 = w3 * cT[w && nn ? 2 * (c0 - 1) : 0], t4 = w4 * cT[e && sd ? 2 * (c0 - N) + 1 : 0];
    const double t5 = w5 * cT[w && sd ? 2 * (c0 - N - 1) : 0], t6 = w5 * cT[w && sd ? 2 * (c0 - N - 1) + 1 : 0];
    const int nd[7] = {k, kE, kN, kNE, kW, kS, kSW};  // C E N NE W S SW
    double vu[7], vp[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        vu[q] = u[nd[q]];
        vp[q] = gn ? 0.0 : p[nd[q]];
    }
#pragma unroll
    for (int cc = 0; cc < C; ++cc) {
        const int col = min((int)blockIdx.y * C + cc, nc - 1);  // past the end: the last column again
        const double* uhc = uh + (size_t)col * ldu;
        const double* phc = ph + (size_t)col * ldp;
        const double* mhc = mh + (size_t)col * ldm;
        double vph[7], vuh[7], vmh[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            vph[q] = phc[nd[q]];
            vuh[q] = gn ? 0.0 : uhc[nd[q]];
            vmh[q] = gn ? 0.0 : mhc[nd[q]];
        }
        const double addv = add ? add[(size_t)col * ldadd + k] : 0.0;
        auto tri = [&](int a, int r, int b) {
            double v = tri_form(vu[a], vu[r], vu[b], vph[a], vph[r], vph[b]);
            if (!gn) {
                v += tri_form(vuh[a], vuh[r], vuh[b], vp[a], vp[r], vp[b]);
                v += (1.0 / 3.0) * (vmh[a] + vmh[r] + vmh[b]) * tri_form(vu[a], vu[r], vu[b], vp[a], vp[r], vp[b]);
            }
            return v;
        };
        constexpr int O = 0, E = 1, NN = 2, NE = 3, W = 4, S = 5, SW = 6;
        double acc = 0.0;
        acc += t1 * (1.0 / 3.0) * tri(O, E, NE);
        acc += t2 * (1.0 / 3.0) * tri(O, NN, NE);
        acc += t3 * (1.0 / 3.0) * tri(W, O, NN);
        acc += t4 * (1.0 / 3.0) * tri(S, O, E);
        acc += t5 * (1.0 / 3.0) * tri(SW, S, O);
        acc += t6 * (1.0 / 3.0) * tri(SW, W, O);
        if (add) acc = addv + acc;  // the prior term, as the accumulating apply adds it
        out[(size_t)col * ldo + k] = acc;
    }
}

// g_v = sum_{T ni v} (c_T/3) |T| grad u . grad p  (data part of the gradient).
__global__ void k_grad(int N, const double* __restrict__ cT, const double* __restrict__ u,
                       const double* __restrict__ p, double* __restrict__ g) {
    const int N1 = N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int i = k % N1, j = k / N1;
    double acc = 0.0;
    for_incident_triangles(N, i, j, [&](int ci, int cj, int s, int) {
        int a, r, b;
        tri_nodes(N, ci, cj, s, a, r, b);
        acc += cT[2 * (cj * N + ci) + s] * (1.0 / 3.0) * tri_form(u[a], u[r], u[b], p[a], p[r], p[b]);
    });
    g[k] = acc;
}

// (C_M eta)_v: every edge midpoint of a triangle carries one normal with
// quadrature weight |T|/3 and basis value 1/2 at both edge ends, so the
// entry of C_M is sqrt(|T|/3) / 2 = h / (2 sqrt 6).  Edges in (a, r, b) order:
// e0 = (a, r), e1 = (r, b), e2 = (a, b).
__global__ void k_mass_factor(int N, const double* __restrict__ eta, int lde,
                              double* __restrict__ out, int ldo) {
    const int N1 = N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int i = k % N1, j = k / N1;
    const double* ec = colp(eta, lde);
    double acc = 0.0;
    for_incident_triangles(N, i, j, [&](int ci, int cj, int s, int role) {
        const int t = 2 * (cj * N + ci) + s;
        // a: e0, e2;  r: e0, e1;  b: e1, e2
        const int ea = role == 2 ? 1 : 0;
        const int eb = role == 1 ? 1 : 2;
        acc += ec[3 * t + ea] + ec[3 * t + eb];
    });
    colp(out, ldo)[k] = acc * (0.5 / (N * sqrt(6.0)));
}

// y = op x + beta y (FP64, all rows of the prior / mass operator).
__global__ void k_prior_apply(OpKA<double> op, const double* __restrict__ x, int ldx,
                              double* __restrict__ y, int ldy, double beta) {
    const int N1 = op.N + 1;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N1 * N1) return;
    const int i = k % N1, j = k / N1;
    const double* xc = colp(x, ldx);
    double v = op.apply(i, j, k, [&](int, int, int kk) { return xc[kk]; });
    double* yc = colp(y, ldy);
    if (beta != 0.0) v += beta * yc[k];
    yc[k] = v;
}

// Chebyshev iteration for M x = b with the Jacobi-scaled spectrum in [1/2, 2]
// (x = 0, r = b, d = D^-1 b / theta; then per step r <- r - M d, x <- x + d,
// d <- c1 d + c2 D^-1 r), kMassSteps steps per launch.  A wave holds r, d and
// x of 64 columns and R rows in registers, one column a lane: east and west
// neighbours come through lane shifts, north and south ones are the next
// registers, and only the first and last row of a wave pass through LDS (one
// barrier a step).  The 8 waves of a workgroup stack to 8 R rows; a halo of
// kMassSteps nodes around the owned ones absorbs the wrong values that move
// in from the cut by one node a step.
// Bound by FP64 arithmetic in batches and by the chain of steps for few
// columns.  With r and d in LDS tiles (12 LDS accesses and two barriers a node
// and step) R mhat = K M^-1 K mhat took 2309 us at 512^2 x 64 and 228 / 70 us for
// one column of 1024^2 / 256^2, here 946 and 92 / 30.
constexpr int kMassSteps = 12, kMassWaves = 8;
constexpr int kMassOwnX = 64 - 2 * kMassSteps;
// R: 4 while the launch is one round of short chains, 8 (less halo a node)
// from 160 workgroups on: R mhat of 256^2 x 1 takes 31 / 40 us with R = 4 / 8
// (49 workgroups of the larger kind), 512^2 x 1 (169) 60 / 49, 512^2 x 64
// 1882 / 903 (16 and 20 rows spill under the 128 registers of two workgroups a
// compute unit: 4583 / 6860).
constexpr int kMassRowsFew = 4, kMassRowsMany = 8;
constexpr int mass_own_y(int R) { return kMassWaves * R - 2 * kMassSteps; }
struct MassSteps {
    double c1[kMassSteps], c2[kMassSteps];
};

template <int R>
__global__ __launch_bounds__(64 * kMassWaves, 4) void k_cheb_mass(OpKA<double> op, const double* __restrict__ b, int ldb,
                                                               double* __restrict__ x, double* __restrict__ r_io,
                                                               double* __restrict__ d_io, int ld, MassSteps cs,
                                                               int first, int last, double inv_theta) {
    __shared__ KARow<double> rows[10];  // by node class; 9: a node off the mesh
    __shared__ double edge[2][kMassWaves][2][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = op.N, N1 = N + 1;
    const int i = blockIdx.x * kMassOwnX - kMassSteps + lane;
    const int jt = blockIdx.y * mass_own_y(R) - kMassSteps, j0 = jt + wave * R;
    const size_t co = (size_t)blockIdx.z * ld;
    if (threadIdx.x < 10) rows[threadIdx.x] = threadIdx.x < 9 ? op.rows[threadIdx.x] : KARow<double>{};
    const bool in_x = i >= 0 && i <= N;
    const int ic = min(max(i, 0), N);
    const int cx = in_x ? (i == 0 ? 1 : (i == N ? 2 : 0)) : 9;
    const bool own_x = in_x && lane >= kMassSteps && lane < 64 - kMassSteps;
    // this lane's owned rows: [q0, q1)
    const int q0 = max(jt + kMassSteps - j0, 0), q1 = min(min(jt + kMassWaves * R - kMassSteps, N1) - j0, R);
    double r[R], d[R], xs[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int k = min(max(j0 + q, 0), N) * N1 + ic;
        if (first) {
            r[q] = b[(size_t)blockIdx.z * ldb + k];
            d[q] = 0.0;
            xs[q] = 0.0;
        } else {
            r[q] = r_io[co + k];
            d[q] = d_io[co + k];
            xs[q] = q >= q0 && q < q1 ? x[co + k] : 0.0;
        }
    }
    __syncthreads();
    const KARow<double> m = rows[cx];
    auto row_class = [&](int j) { return cx == 9 || j < 0 || j > N ? 9 : cx + (j == 0 ? 3 : (j == N ? 6 : 0)); };
    // a wave without rows on or beyond the mesh's edges has its coefficients in registers
    const bool plain = j0 > 0 && j0 + R <= N;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int j = j0 + q;
        if (!in_x || j < 0 || j > N) r[q] = d[q] = 0.0;
        if (first) d[q] = rows[row_class(j)].dinv * r[q] * inv_theta;
    }
    for (int st = 0; st < kMassSteps; ++st) {
        double(*e)[2][64] = edge[st & 1];
        e[wave][0][lane] = d[0];
        e[wave][1][lane] = d[R - 1];
        __syncthreads();
        const double up = wave + 1 < kMassWaves ? e[wave + 1][0][lane] : 0.0;
        double below = wave > 0 ? e[wave - 1][1][lane] : 0.0;
        const double c1 = cs.c1[st], c2 = cs.c2[st];
        double below_w = lane_west(below), at_e = lane_east(d[0]);
        auto sweep = [&](auto plain_rows) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const double at = d[q], above = q + 1 < R ? d[q + 1] : up;
                const double at_w = lane_west(at), above_e = lane_east(above);
                KARow<double> c;
                if constexpr (decltype(plain_rows)::value)
                    c = m;
                else
                    c = rows[row_class(j0 + q)];
                const double Md = c.c * at + c.e * at_e + c.w * at_w + c.n * above + c.s * below + c.ne * above_e +
                                  c.sw * below_w;
                r[q] -= Md;
                xs[q] += at;
                d[q] = c1 * at + c2 * c.dinv * r[q];
                below = at;
                below_w = at_w;
                at_e = above_e;
            }
        };
        if (plain)
            sweep(std::true_type{});
        else
            sweep(std::false_type{});
    }
    if (!own_x) return;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (q < q0 || q >= q1) continue;
        const size_t k = co + (size_t)(j0 + q) * N1 + i;
        x[k] = xs[q];
        if (!last) {
            r_io[k] = r[q];
            d_io[k] = d[q];
        }
    }
}

__global__ void k_add_scalar(int n, double v, double* __restrict__ x, int ld) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) colp(x, ld)[k] += v;
}

__global__ void k_axpby(int n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) y[k] = a * x[k] + b * y[k];
}

__global__ void k_fill(int n, double v, double* __restrict__ y) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) y[k] = v;
}

__global__ void k_copy(int n, const double* __restrict__ x, int ldx, double* __restrict__ y, int ldy) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) colp(y, ldy)[k] = colp(x, ldx)[k];
}

__global__ void k_dot_partial(int n, const double* __restrict__ a, int lda,
                              const double* __restrict__ b, int ldb, double* __restrict__ partial) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (k < n) v = colp(a, lda)[k] * colp(b, ldb)[k];
    const double s = block_sum(v);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

__global__ void k_dot_finish(const double* __restrict__ partial, int nblk, double* __restrict__ out) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) v += partial[(size_t)blockIdx.x * nblk + b];
    const double s = block_sum(v);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// ------------------------------------------------------------ white noise ---
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds of two 64x64
// multiplications with Weyl-sequence key increments.
__device__ inline void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
    for (int r = 0; r < 10; ++r) {
        const uint64_t hi0 = __umul64hi(M0, c[0]), lo0 = M0 * c[0];
        const uint64_t hi1 = __umul64hi(M1, c[2]), lo1 = M1 * c[2];
        const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
        k0 += W0;
        k1 += W1;
    }
}

// Box-Muller on one word pair: u1 in (0, 1], u2 in [0, 1).
__device__ inline void box_muller(uint64_t w0, uint64_t w1, double& z0, double& z1) {
    const double u1 = ((double)(w0 >> 11) + 1.0) * 0x1.0p-53;
    const double u2 = (double)(w1 >> 11) * 0x1.0p-53;
    const double r = sqrt(-2.0 * log(u1));
    double s, c;
    sincospi(2.0 * u2, &s, &c);
    z0 = r * c;
    z1 = r * s;
}

// eta[:, s] for samples first .. first+ns-1: sample S takes the stream words
// [S L, (S+1) L), word w from counter block w / 4 + 1 (L = 6 N^2, 4 | L).
__global__ void k_white_noise(int L, uint64_t seed, uint64_t stream, long long first,
                              double* __restrict__ eta, int ld) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;  // block within the sample
    if (4 * b >= L) return;
    const unsigned long long blk = (unsigned long long)(first + blockIdx.y) * (L / 4) + b + 1;
    uint64_t c[4] = {blk, 0, 0, 0};
    philox4x64_10(c, seed, stream);
    double* e = eta + (size_t)blockIdx.y * ld + 4 * b;
    box_muller(c[0], c[1], e[0], e[1]);
    box_muller(c[2], c[3], e[2], e[3]);
}

__global__ void k_zero_cols(int n, double* __restrict__ x, int ld) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) colp(x, ld)[k] = 0.0;
}

// Columns that share a thread's reading of the coefficient and of the fields at
// the linearization point in k_sens and k_hess_out, from kShareMin columns on
// (bound by bandwidth there; below, more threads hide the latency better).
// 1024^2 x 61: k_sens 703 us a column a thread, 479 with four; k_hess_out
// (Gauss-Newton) 754 and 521.
constexpr int kShareCols = 4, kShareMin = 8;
void launch_sens(hipStream_t s, int N, int n, int nc, const double* cT, const double* mhat, int ldm, const double* w,
                 double* y, int ldy) {
    if (nc >= kShareMin)
        k_sens<kShareCols><<<grid2(n, ceil_div(nc, kShareCols)), kBlock, 0, s>>>(N, nc, cT, mhat, ldm, w, -1.0, y, ldy);
    else
        k_sens<1><<<grid2(n, nc), kBlock, 0, s>>>(N, nc, cT, mhat, ldm, w, -1.0, y, ldy);
}

OpKA<double> prior_op(int N, const PriorParams& pp) { return make_prior_op<double>(N, pp); }

// The mass matrix as a prior operator (gamma = 0, delta = 1, beta = 0).
OpKA<double> mass_op(int N) { return make_prior_op<double>(N, PriorParams{0.0, 1.0, 0.0}); }

// Chebyshev iteration count for M: error factor 2 (1/3)^K = 7.1e-12 at K = 24,
// below the 1e-10 relative residual every PDE solve runs to (32 steps, to
// 2e-15, cost a fourth more in every application of R).
constexpr int kMassCheb = 24;
static_assert(kMassCheb % kMassSteps == 0, "mass Chebyshev steps come in whole launches");

}  // namespace

// ----------------------------------------------------------- vector ops ---
void dev_dots(Ctx* ctx, int n, int nc, const double* a, int lda, const double* b, int ldb,
              double* host_out) {
    const int nblk = ceil_div(n, kBlock);
    ctx->red.ensure((size_t)nblk * nc + nc);
    k_dot_partial<<<grid2(n, nc), kBlock, 0, ctx->stream>>>(n, a, lda, b, ldb, ctx->red.get());
    HINV_LAUNCH_CHECK();
    double* out = ctx->red.get() + (size_t)nblk * nc;
    k_dot_finish<<<nc, kBlock, 0, ctx->stream>>>(ctx->red.get(), nblk, out);
    HINV_LAUNCH_CHECK();
    // through pinned memory: a pageable destination adds a staging copy to
    // every read-back of the Newton-CG loop
    if (!ctx->host_red) HINV_HIP(hipHostMalloc((void**)&ctx->host_red, sizeof(double) * Ctx::kHostRed,
                                               hipHostMallocDefault));
    for (int c0 = 0; c0 < nc; c0 += Ctx::kHostRed) {
        const int m = std::min(Ctx::kHostRed, nc - c0);
        HINV_HIP(hipMemcpyAsync(ctx->host_red, out + c0, sizeof(double) * m, hipMemcpyDeviceToHost, ctx->stream));
        HINV_HIP(hipStreamSynchronize(ctx->stream));
        std::memcpy(host_out + c0, ctx->host_red, sizeof(double) * m);
    }
}

void dev_dot_to(Ctx* ctx, int n, const double* a, const double* b, double* out) {
    const int nblk = ceil_div(n, kBlock);
    ctx->red.ensure((size_t)nblk + 1);
    k_dot_partial<<<grid2(n, 1), kBlock, 0, ctx->stream>>>(n, a, n, b, n, ctx->red.get());
    HINV_LAUNCH_CHECK();
    k_dot_finish<<<1, kBlock, 0, ctx->stream>>>(ctx->red.get(), nblk, out);
    HINV_LAUNCH_CHECK();
}

double dev_dot(Ctx* ctx, int n, const double* a, const double* b) {
    double r;
    dev_dots(ctx, n, 1, a, n, b, n, &r);
    return r;
}

void dev_axpby(Ctx* ctx, int n, double a, const double* x, double b, double* y) {
    k_axpby<<<ceil_div(n, kBlock), kBlock, 0, ctx->stream>>>(n, a, x, b, y);
    HINV_LAUNCH_CHECK();
}

void dev_copy(Ctx* ctx, int n, int nc, const double* x, int ldx, double* y, int ldy) {
    if (nc <= 0) return;
    k_copy<<<grid2(n, nc), kBlock, 0, ctx->stream>>>(n, x, ldx, y, ldy);
    HINV_LAUNCH_CHECK();
}

void dev_fill(Ctx* ctx, int n, double v, double* y) {
    k_fill<<<ceil_div(n, kBlock), kBlock, 0, ctx->stream>>>(n, v, y);
    HINV_LAUNCH_CHECK();
}

// -------------------------------------------------------------- problem ---
Problem::Problem(Ctx* c, const hinv_problem_desc& desc)
    : ctx(c), N(desc.N), n((desc.N + 1) * (desc.N + 1)), q(desc.q), gamma(desc.gamma),
      delta(desc.delta), m_prior(desc.m_prior), sigma(desc.sigma), precision(desc.precision),
      rtol(desc.rtol), max_iter(desc.max_iter > 0 ? desc.max_iter : 200) {
    beta = std::isnan(desc.beta) ? std::sqrt(gamma * delta) / 1.42 : desc.beta;
    PriorParams pp{gamma, delta, beta};
    if (desc.theta1 > 0.0) {
        // Theta = theta1 v v^T + theta2 w w^T, v = (sin a, cos a), w = (cos a, -sin a):
        // the s.p.d. tensor with the eigenvalues and directions Sec. 5.1 states
        const double sa = std::sin(desc.alpha), ca = std::cos(desc.alpha);
        pp.t11 = desc.theta1 * sa * sa + desc.theta2 * ca * ca;
        pp.t12 = (desc.theta1 - desc.theta2) * sa * ca;
        pp.t22 = desc.theta1 * ca * ca + desc.theta2 * sa * sa;
    }
    prior = pp;
    deg = desc.state_degree == 2 ? 2 : 1;
    ns = deg == 2 ? (2 * N + 1) * (2 * N + 1) : n;
    HA = std::make_unique<Hierarchy>(ctx, kOpState, N, pp);
    HK = std::make_unique<Hierarchy>(ctx, kOpPrior, N, pp);
    if (deg == 2) S2 = std::make_unique<P2Space>(ctx, N);
    m_lin.ensure(n);
    u_lin.ensure(ns);
    p_lin.ensure(ns);
    hipStream_t s = ctx->stream;
    if (q > 0) {
        obs_xy.ensure(2 * (size_t)q);
        obs_w.ensure(3 * (size_t)q);
        obs_node.ensure(3 * (size_t)q);
        d.ensure(q);
        HINV_HIP(hipMemcpyAsync(obs_xy.get(), desc.obs_xy, sizeof(double) * 2 * q, hipMemcpyHostToDevice, s));
        k_obs_setup<<<ceil_div(q, kBlock), kBlock, 0, s>>>(N, q, obs_xy.get(), obs_node.get(), obs_w.get());
        HINV_LAUNCH_CHECK();
        // transpose structure: node -> list of (3 o + a), built from the device's node indices
        std::vector<int> hn(3 * (size_t)q);
        HINV_HIP(hipMemcpyAsync(hn.data(), obs_node.get(), sizeof(int) * 3 * q, hipMemcpyDeviceToHost, s));
        HINV_HIP(hipStreamSynchronize(s));
        std::vector<int> order(3 * (size_t)q);
        for (int e = 0; e < 3 * q; ++e) order[e] = e;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return hn[a] < hn[b]; });
        std::vector<int> tn, tp, te;
        for (int e = 0; e < 3 * q; ++e) {
            const int nd = hn[order[e]];
            if (tn.empty() || tn.back() != nd) {
                tn.push_back(nd);
                tp.push_back(e);
            }
            te.push_back(order[e]);
        }
        tp.push_back(3 * q);
        n_touch = (int)tn.size();
        t_node.ensure(tn.size());
        t_ptr.ensure(tp.size());
        t_ent.ensure(te.size());
        HINV_HIP(hipMemcpyAsync(t_node.get(), tn.data(), sizeof(int) * tn.size(), hipMemcpyHostToDevice, s));
        HINV_HIP(hipMemcpyAsync(t_ptr.get(), tp.data(), sizeof(int) * tp.size(), hipMemcpyHostToDevice, s));
        HINV_HIP(hipMemcpyAsync(t_ent.get(), te.data(), sizeof(int) * te.size(), hipMemcpyHostToDevice, s));
        HINV_HIP(hipStreamSynchronize(s));
        if (S2) S2->set_observations(q, obs_xy.get());
        set_data(desc.d_obs, sigma);
    }
}

void Problem::set_data(const double* d_host, double sig) {
    if (sig > 0) sigma = sig;
    if (q == 0) return;
    hipStream_t s = ctx->stream;
    if (d_host) {
        HINV_HIP(hipMemcpyAsync(d.get(), d_host, sizeof(double) * q, hipMemcpyHostToDevice, s));
        HINV_HIP(hipStreamSynchronize(s));
    } else {
        k_fill<<<ceil_div(q, kBlock), kBlock, 0, s>>>(q, 0.0, d.get());
        HINV_LAUNCH_CHECK();
    }
}

double* Problem::scratch(int which, int nc) {
    if (which < 0 || which >= kScratch) fail(HINV_EINVAL, "internal: scratch index out of range");
    if (nc > cap_) {
        cap_ = 0;  // until every buffer is there
        for (auto& w : w_) w.release();
        for (auto& w : w_) w.ensure((size_t)std::max(n, ns) * nc);
        cap_ = nc;
    }
    return w_[which].get();
}

double* Problem::obs_scratch(int nc) {
    if (nc > qcap_) {
        qcap_ = 0;
        wq_.ensure((size_t)std::max(q, 1) * nc);
        qcap_ = nc;
    }
    return wq_.get();
}

void Problem::set_state(const double* m) {
    HA->set_state_coefficient(m);
    if (S2) S2->set_coefficient(HA->coefficient());
}

void Problem::state_solve(int nc, const double* b, int ldb, double* x, int ldx, double tol, SolveStats* st,
                          double accept) {
    if (S2)
        S2->solve(nc, b, ldb, x, ldx, *HA, tol, max_iter, st);
    else
        HA->solve(nc, b, ldb, x, ldx, precision, tol, max_iter, st, accept);
}

void Problem::state_apply(int nc, const double* x, int ldx, double* y, int ldy) {
    if (S2)
        S2->apply(nc, x, ldx, y, ldy, 1.0);
    else
        HA->apply(nc, x, ldx, y, ldy);
}

void Problem::forward(const double* m, double* u, SolveStats* st) {
    hipStream_t s = ctx->stream;
    set_state(m);
    ha_is_lin = false;
    double* rhs = scratch(0, 1);
    if (S2) {
        S2->forward_rhs(rhs);
        state_solve(1, rhs, ns, u, ns, rtol, st);
        S2->set_top(u);
        return;
    }
    k_forward_rhs<<<ceil_div(n, kBlock), kBlock, 0, s>>>(N, HA->weightsN(), rhs);
    HINV_LAUNCH_CHECK();
    HA->solve(1, rhs, n, u, n, precision, rtol, max_iter, st);
    k_set_top<<<ceil_div(N + 1, kBlock), kBlock, 0, s>>>(N, u);
    HINV_LAUNCH_CHECK();
}

void Problem::observe(const double* u, int ldu, int nc, double* out, int ldo, bool minus_data) {
    if (q == 0) return;
    if (S2) {
        S2->observe(nc, u, ldu, minus_data ? d.get() : nullptr, out, ldo);
        return;
    }
    k_obs_gather<<<grid2(q, nc), kBlock, 0, ctx->stream>>>(q, obs_node.get(), obs_w.get(), u, ldu,
                                                           minus_data ? d.get() : nullptr, out, ldo);
    HINV_LAUNCH_CHECK();
}

void Problem::cost(const double* m, const double* u, double* misfit, double* reg) {
    double mis = 0.0;
    if (q > 0) {
        double* r = obs_scratch(1);
        observe(u, ns, 1, r, q, true);
        double ss;
        dev_dots(ctx, q, 1, r, q, r, q, &ss);
        mis = 0.5 * ss / (sigma * sigma);
    }
    double* dm = scratch(0, 1);
    double* Rdm = scratch(1, 1);
    dev_copy(ctx, n, 1, m, n, dm, n);
    k_add_scalar<<<ceil_div(n, kBlock), kBlock, 0, ctx->stream>>>(n, -m_prior, dm, n);
    HINV_LAUNCH_CHECK();
    prior_apply(1, dm, n, Rdm, n);
    *misfit = mis;
    *reg = 0.5 * dev_dot(ctx, n, dm, Rdm);
}

void Problem::gradient(const double* m, const double* u, double* p, double* g, SolveStats* st) {
    hipStream_t s = ctx->stream;
    set_state(m);
    ha_is_lin = false;
    double* rhs = scratch(0, 1);
    k_fill<<<ceil_div(ns, kBlock), kBlock, 0, s>>>(ns, 0.0, rhs);
    HINV_LAUNCH_CHECK();
    if (q > 0) {
        double* r = obs_scratch(1);
        observe(u, ns, 1, r, q, true);
        if (S2) {
            S2->observe_adjoint(1, r, q, -1.0 / (sigma * sigma), rhs, ns);
        } else {
            k_obs_scatter<<<ceil_div(n_touch, kBlock), kBlock, 0, s>>>(
                n_touch, t_node.get(), t_ptr.get(), t_ent.get(), obs_w.get(), r, q,
                -1.0 / (sigma * sigma), rhs, n);
            HINV_LAUNCH_CHECK();
        }
    }
    state_solve(1, rhs, ns, p, ns, rtol, st);
    if (S2) {
        S2->grad(u, p, g);
    } else {
        k_grad<<<ceil_div(n, kBlock), kBlock, 0, s>>>(N, HA->coefficient(), u, p, g);
        HINV_LAUNCH_CHECK();
    }
    double* dm = scratch(1, 1);
    dev_copy(ctx, n, 1, m, n, dm, n);
    k_add_scalar<<<ceil_div(n, kBlock), kBlock, 0, s>>>(n, -m_prior, dm, n);
    HINV_LAUNCH_CHECK();
    prior_apply(1, dm, n, g, n, /*accumulate=*/true);
}

void Problem::linearize(const double* m, const double* u, const double* p) {
    dev_copy(ctx, n, 1, m, n, m_lin.get(), n);
    dev_copy(ctx, ns, 1, u, ns, u_lin.get(), ns);
    dev_copy(ctx, ns, 1, p, ns, p_lin.get(), ns);
    set_state(m_lin.get());
    ha_is_lin = true;
    linearized = true;
    ++lin_version;
}

void Problem::ensure_lin_hierarchy() {
    if (!linearized) fail(HINV_ESTATE, "Hessian action before hinv_linearize");
    if (!ha_is_lin) {
        set_state(m_lin.get());
        ha_is_lin = true;
    }
}

// Right-hand side -[C(u) mhat]_F of the incremental forward problem.
void Problem::inc_forward_rhs(int nc, const double* mhat, int ldm, double* rhs, int ldr) {
    ensure_lin_hierarchy();
    if (S2) {
        S2->sens(nc, mhat, ldm, u_lin.get(), -1.0, rhs, ldr);
        return;
    }
    launch_sens(ctx->stream, N, n, nc, HA->coefficient(), mhat, ldm, u_lin.get(), rhs, ldr);
    HINV_LAUNCH_CHECK();
}

// Right-hand side -[B^T B uhat / sigma^2 + C(p) mhat]_F of the incremental
// adjoint problem (Gauss-Newton drops C(p) mhat).
void Problem::inc_adjoint_rhs(int nc, bool gn, const double* mhat, int ldm, const double* uhat,
                              int ldu, double* rhs, int ldr) {
    ensure_lin_hierarchy();
    hipStream_t s = ctx->stream;
    if (S2) {
        // the scale 0 zeroes the column under Gauss-Newton
        S2->sens(nc, mhat, ldm, p_lin.get(), gn ? 0.0 : -1.0, rhs, ldr);
        if (q > 0) {
            double* Bu = obs_scratch(nc);
            observe(uhat, ldu, nc, Bu, q, false);
            S2->observe_adjoint(nc, Bu, q, -1.0 / (sigma * sigma), rhs, ldr);
        }
        return;
    }
    if (gn)
        k_zero_cols<<<grid2(n, nc), kBlock, 0, s>>>(n, rhs, ldr);
    else
        launch_sens(s, N, n, nc, HA->coefficient(), mhat, ldm, p_lin.get(), rhs, ldr);
    HINV_LAUNCH_CHECK();
    if (q > 0) {
        double* Bu = obs_scratch(nc);
        observe(uhat, ldu, nc, Bu, q, false);
        k_obs_scatter<<<grid2(n_touch, nc), kBlock, 0, s>>>(n_touch, t_node.get(), t_ptr.get(),
                                                            t_ent.get(), obs_w.get(), Bu, q,
                                                            -1.0 / (sigma * sigma), rhs, ldr);
        HINV_LAUNCH_CHECK();
    }
}

// Hessian action from the incremental states (and R mhat for the full modes).
void Problem::hess_output(int mode, int nc, const double* mhat, int ldm, const double* uh, int ldu,
                          const double* ph, int ldp, double* out, int ldo, const double* rm) {
    const bool gn = mode == HINV_HESS_GN_FULL || mode == HINV_HESS_GN_MISFIT;
    const bool with_prior = mode == HINV_HESS_FULL || mode == HINV_HESS_GN_FULL;
    if (S2) {
        S2->hess_out(nc, gn, u_lin.get(), p_lin.get(), uh, ldu, ph, ldp, mhat, ldm, out, ldo,
                     with_prior ? rm : nullptr, n);
        if (with_prior && !rm) prior_apply(nc, mhat, ldm, out, ldo, true);
        return;
    }
    auto run = [&](auto kern, int C) {
        kern<<<grid2(n, ceil_div(nc, C)), kBlock, 0, ctx->stream>>>(
            N, nc, HA->coefficient(), u_lin.get(), p_lin.get(), uh, ldu, ph, ldp, mhat, ldm, out, ldo, gn ? 1 : 0,
            with_prior ? rm : nullptr, n);
    };
    if (nc >= kShareMin)
        run(k_hess_out<kShareCols>, kShareCols);
    else
        run(k_hess_out<1>, 1);
    HINV_LAUNCH_CHECK();
    if (with_prior && !rm) prior_apply(nc, mhat, ldm, out, ldo, true);
}

hipStream_t Problem::side_stream() {
    if (!side_) {
        HINV_HIP(hipStreamCreateWithFlags(&side_, hipStreamNonBlocking));
        HINV_HIP(hipEventCreateWithFlags(&ev_fork_, hipEventDisableTiming));
        HINV_HIP(hipEventCreateWithFlags(&ev_join_, hipEventDisableTiming));
    }
    return side_;
}

Problem::~Problem() {
    if (side_) {
        (void)hipStreamSynchronize(side_);
        (void)hipEventDestroy(ev_fork_);
        (void)hipEventDestroy(ev_join_);
        (void)hipStreamDestroy(side_);
    }
}

void Problem::inc_forward(int nc, const double* mhat, int ldm, double* uhat, int ldu, SolveStats* st,
                          double tol) {
    double* rhs = scratch(0, nc);
    inc_forward_rhs(nc, mhat, ldm, rhs, ns);
    // a tighter goal still accepts the problem's tolerance at the rounding floor
    state_solve(nc, rhs, ns, uhat, ldu, tol > 0 ? tol : rtol, st, rtol);
}

void Problem::inc_adjoint(int nc, bool gn, const double* mhat, int ldm, const double* uhat, int ldu,
                          double* phat, int ldp, SolveStats* st) {
    double* rhs = scratch(0, nc);
    inc_adjoint_rhs(nc, gn, mhat, ldm, uhat, ldu, rhs, ns);
    state_solve(nc, rhs, ns, phat, ldp, rtol, st);
}

void Problem::hessian(int mode, int nc, const double* mhat, int ldm, double* out, int ldo,
                      SolveStats* st) {
    const bool gn = mode == HINV_HESS_GN_FULL || mode == HINV_HESS_GN_MISFIT;
    const bool with_prior = mode == HINV_HESS_FULL || mode == HINV_HESS_GN_FULL;
    scratch(0, nc);
    double* uh = scratch(1, nc);
    double* ph = scratch(2, nc);
    // R mhat does not depend on the two solves: it runs on the side stream
    // meanwhile (its own scratch 3-9), joined before the output kernel adds it
    double* rm = nullptr;
    if (with_prior) {
        rm = scratch(9, nc);
        hipStream_t side = side_stream();
        HINV_HIP(hipEventRecord(ev_fork_, ctx->stream));
        HINV_HIP(hipStreamWaitEvent(side, ev_fork_, 0));
        prior_apply(nc, mhat, ldm, rm, n, false, side);
        HINV_HIP(hipEventRecord(ev_join_, side));
    }
    // joined also when a solve throws: the context's stream hands out again
    // what the side stream still works on
    struct Join {
        hipStream_t s;
        hipEvent_t ev;
        ~Join() {
            if (ev) (void)hipStreamWaitEvent(s, ev, 0);
        }
    };
    {
        const Join join{ctx->stream, with_prior ? ev_join_ : nullptr};
        // the P2 state solves in FP64 PCG: no chained tightening
        inc_forward(nc, mhat, ldm, uh, ns, st, S2 ? rtol : chained_first_rtol(precision, nc, rtol));
        inc_adjoint(nc, gn, mhat, ldm, uh, ns, ph, ns, st);
    }
    hess_output(mode, nc, mhat, ldm, uh, ns, ph, ns, out, ldo, rm);
}

void Problem::mass_apply(int nc, const double* x, int ldx, double* y, int ldy) {
    k_prior_apply<<<grid2(n, nc), kBlock, 0, ctx->stream>>>(mass_op(N), x, ldx, y,
                                                            ldy, 0.0);
    HINV_LAUNCH_CHECK();
}

void Problem::mass_solve(int nc, const double* b, int ldb, double* x, int ldx, hipStream_t s, double* ws) {
    // Chebyshev iteration (no inner products) on the Jacobi-scaled consistent
    // mass matrix, whose spectrum lies in [1/2, 2] for P1 triangles.
    if (!s) s = ctx->stream;
    const OpKA<double> M = mass_op(N);
    const double lo = 0.5, hi = 2.0;
    const double theta = 0.5 * (hi + lo), dl = 0.5 * (hi - lo), sigma1 = theta / dl;
    const size_t blk = (size_t)n * nc;
    double* r = ws ? ws : scratch(5, nc);
    double* d = ws ? ws + blk : scratch(6, nc);
    if (ldx != n) fail(HINV_EINVAL, "mass_solve needs a packed output");
    if (nc > 65535) fail(HINV_EINVAL, "mass_solve: at most 65535 columns per call");
    const int tx = ceil_div(N + 1, kMassOwnX);
    auto tiles = [&](int R) { return ceil_div(N + 1, mass_own_y(R)); };
    const bool many = (long long)tx * tiles(kMassRowsMany) * nc >= 160;
    double rho = 1.0 / sigma1;
    constexpr int launches = kMassCheb / kMassSteps;
    static_assert(launches <= 2, "a launch in the middle would read its neighbours' new r and d");
    for (int launch = 0; launch < launches; ++launch) {
        MassSteps cs;
        for (int st = 0; st < kMassSteps; ++st) {
            const double rho_n = 1.0 / (2.0 * sigma1 - rho);
            cs.c1[st] = rho_n * rho;
            cs.c2[st] = 2.0 * rho_n / dl;
            rho = rho_n;
        }
        auto run = [&](auto kern, int R) {
            kern<<<dim3(tx, tiles(R), nc), 64 * kMassWaves, 0, s>>>(M, b, ldb, x, r, d, n, cs, launch == 0,
                                                                    launch == launches - 1, 1.0 / theta);
        };
        if (many)
            run(k_cheb_mass<kMassRowsMany>, kMassRowsMany);
        else
            run(k_cheb_mass<kMassRowsFew>, kMassRowsFew);
        HINV_LAUNCH_CHECK();
    }
}

void Problem::prior_apply(int nc, const double* x, int ldx, double* y, int ldy, bool accumulate,
                          hipStream_t s, double* ws) {
    if (!s) s = ctx->stream;
    const OpKA<double> K = prior_op(N, prior);
    const size_t blk = (size_t)n * nc;
    double* t1 = ws ? ws : scratch(3, nc);
    double* t2 = ws ? ws + blk : scratch(4, nc);
    k_prior_apply<<<grid2(n, nc), kBlock, 0, s>>>(K, x, ldx, t1, n, 0.0);
    HINV_LAUNCH_CHECK();
    mass_solve(nc, t1, n, t2, n, s, ws ? ws + 2 * blk : nullptr);
    k_prior_apply<<<grid2(n, nc), kBlock, 0, s>>>(K, t2, n, y, ldy, accumulate ? 1.0 : 0.0);
    HINV_LAUNCH_CHECK();
}

void Problem::prior_solve(int nc, const double* x, int ldx, double* y, int ldy, SolveStats* st) {
    double* t1 = scratch(3, nc);
    double* t2 = scratch(4, nc);
    HK->solve(nc, x, ldx, t1, n, precision, rtol, max_iter, st);
    mass_apply(nc, t1, n, t2, n);
    HK->solve(nc, t2, n, y, ldy, precision, rtol, max_iter, st);
}

void Problem::white_noise(uint64_t seed, uint64_t stream, long long first, int ns, double* eta,
                          int ld) {
    const int L = 6 * N * N;
    k_white_noise<<<dim3(ceil_div(L / 4, kBlock), ns), kBlock, 0, ctx->stream>>>(L, seed, stream, first,
                                                                                  eta, ld);
    HINV_LAUNCH_CHECK();
}

void Problem::prior_sample(int ns, const double* eta, int ldeta, double* out, int ldo,
                           bool add_mean, SolveStats* st) {
    double* t = scratch(3, ns);
    k_mass_factor<<<grid2(n, ns), kBlock, 0, ctx->stream>>>(N, eta, ldeta, t, n);
    HINV_LAUNCH_CHECK();
    HK->solve(ns, t, n, out, ldo, precision, rtol, max_iter, st);
    if (add_mean) {
        k_add_scalar<<<grid2(n, ns), kBlock, 0, ctx->stream>>>(n, m_prior, out, ldo);
        HINV_LAUNCH_CHECK();
    }
}

}  // namespace hinv
