// One-level V-cycle kernels on wave rows (included by mgkernels.h).
//
// A wave owns a strip of the level 64 nodes wide (lane = column) and marches
// over a segment of its rows.  Every vector it needs of a row lives in one
// register: the east and west neighbours come from the adjacent lanes (DPP
// wave shifts), the north and south ones from the rows kept of the march, so
// the sweeps of a level run back to back as a pipeline over rows with no LDS
// traffic and no workgroup barrier.  Rows are loaded kCH at a time, the next
// kCH while the current ones are worked on.
//
// The arithmetic per node and its order are those of the tile kernels of
// several levels (k_down2, k_up_chain), so one or several levels a launch
// give the same cycle bit for bit.
//
// Batches are bound by HBM bandwidth, few columns by the latency of one pass.
// Against LDS tiles with a halo and a launch of its own for the PCG step, finest
// level: 1024^2 x 61 (FP32) down 240 us and step 175 us -> 211 us together,
// up 221 -> 132, apply 229 -> 214 (it now also moves x: 24 bytes a node at
// 7.2 TB/s, partly from the last-level cache); one column (FP64) of 1024^2 down
// 16.2 and step 10.6 -> 11.9 us together, up 12.2 -> 9.8, of 256^2 down 6.4 and
// step 3.8 -> 6.0, up 4.4 -> 4.2.
#pragma once

#include "grid.h"
#include "solver.h"

namespace hinv {

constexpr int kMarchWaves = 4;  // waves of a workgroup
// Nodes a wave owns of the 64 lanes: the down step needs the residual one
// node around its fine nodes, x2 two and b three (58 fine nodes, 29 coarse
// ones); the up step needs x2 + P x_c two nodes around its own (60).
constexpr int kDownOwn = 29, kUpOwn = 60;

// Rows a chunk (loaded together) and coarse rows a segment: calls of few
// columns take at most kLatencyRows coarse rows, i.e. two chunks, both loaded
// at the start, and aim at kLatencyWaves waves a compute unit; batches small
// chunks (few registers, many waves) and one of the kBatchRows lengths, timed
// at the first call of a shape (longer segments re-read fewer halo rows, shorter
// ones give small meshes enough waves).  C = 2 columns a wave share the state
// operator's coefficients and are picked by the same timing.
// Batches of at most kShortWaves waves a compute unit at 5 rows are bound by the
// march's length: they are timed at 5, 2 and 1 rows, one column a wave.
// Gauss-Newton action at 5 / 2 / 1 rows: 64^2 x 8 (0.4 waves) 768 / 676 / 641 us,
// 128^2 x 24 (3.7) 1147 / 1065 / 1141, 256^2 x 12 (6.1) 1630 / 1538 / 1632;
// past the line 128^2 x 70 (10.7) 1555 / 1697 / 1927, 64^2 x 220 (12) 1348 /
// 1508 / 1733.
constexpr int kLatencyChunk = 8, kLatencyRows = 5, kLatencyWaves = 6;
constexpr int kBatchChunk = 4;
constexpr int kBatchRows[] = {13, 29, 5, 2, 1}, kShortRows = 5, kShortWaves = 8;

// Rows of a row pipeline: a segment of len coarse rows of the down step takes
// 2 len + 5 rows, one of len fine rows of the up step len + 4.
struct March {
    int strips, segs, len;
    int cpi;   // columns per instance
    int many;  // several instances
    double inv_strips;
};

// A vector read through a buffer descriptor: row offset in a scalar register,
// lane offset in one 32-bit vector register shared by every row in flight
// (64-bit vector addresses took half of the registers), and reads past the
// end return 0.
template <typename V>
struct BufRef {
    __amdgpu_buffer_rsrc_t r;
    __device__ BufRef() {}
    __device__ BufRef(const V* p, long long count)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<V*>(p), 0, (unsigned)min(count * (long long)sizeof(V), 0xffffffffLL),
                                              0x00020000)) {}
    // element row + ic
    __device__ V get(int row, unsigned ic) const {
        if constexpr (sizeof(V) == 4)
            return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, ic * 4u, (unsigned)row * 4u, 0));
        else
            return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, ic * 8u, (unsigned)row * 8u, 0));
    }
};
// Element ic of a row behind a uniform pointer.
template <typename V>
__device__ inline void row_put(V* row, unsigned ic, V v) {
    *reinterpret_cast<V*>(reinterpret_cast<char*>(row) + (unsigned)(ic * (unsigned)sizeof(V))) = v;
}

// One row of the operator at the lane's node.
template <typename T>
struct LaneRow {
    T c{}, e{}, w{}, n{}, s{}, ne{}, sw{}, dv{};
};

// (A v) at the lane's node from the rows below, at and above it.
template <bool NE, typename T>
__device__ inline T lane_apply(const LaneRow<T>& r, T below, T at, T above) {
    T a = r.c * at + r.e * lane_east(at) + r.w * lane_west(at) + r.n * above + r.s * below;
    if constexpr (NE) a += r.ne * lane_east(above) + r.sw * lane_west(below);
    return a;
}

// Loads of the operator along the march: kCH rows of the state operator's
// coefficients; the prior operator loads nothing (its rows depend on the node
// class only: row 0 throughout in a wave of interior nodes, else read from
// the class table in LDS, whose entry 9 is a zero row for nodes off the mesh).
template <class Op, int CH>
struct RowLoads {
    struct Src {
        __device__ explicit Src(const Op&) {}
    };
    __device__ void load(const Src&, int, unsigned, int) {}
    template <bool UNI, typename T>
    __device__ LaneRow<T> row(const Op& op, const KARow<T>* tab, int, int i, int j, bool in, T) const {
        if constexpr (UNI) {
            const KARow<T>& r = op.rows[0];
            return LaneRow<T>{r.c, r.e, r.w, r.n, r.s, r.ne, r.sw, r.dinv};
        } else {
            const KARow<T>& r = tab[in ? ka_class(i, j, op.N) : 9];
            return LaneRow<T>{r.c, r.e, r.w, r.n, r.s, r.ne, r.sw, r.dinv};
        }
    }
};
template <typename T, int CH>
struct RowLoads<OpA<T>, CH> {
    struct Src {
        BufRef<T> e, n, d;
        __device__ explicit Src(const OpA<T>& o) {
            const long long cnt = (long long)(o.N + 1) * (o.N + 1);
            e = BufRef<T>(o.wE, cnt);
            n = BufRef<T>(o.wN, cnt);
            d = BufRef<T>(o.dinv, cnt);
        }
    };
    T we[CH], wn[CH], dv[CH];
    // the row whose first node is rowbase (clamped into the mesh), at column ic
    __device__ void load(const Src& s, int e, unsigned ic, int rowbase) {
        we[e] = s.e.get(rowbase, ic);
        wn[e] = s.n.get(rowbase, ic);
        dv[e] = s.d.get(rowbase, ic);
    }
    // below: the north coupling of row j - 1
    template <bool UNI>
    __device__ LaneRow<T> row(const OpA<T>&, const KARow<T>*, int e, int, int, bool in, T below) const {
        LaneRow<T> r;
        r.e = in ? -we[e] : (T)0;
        r.n = in ? -wn[e] : (T)0;
        r.dv = in ? dv[e] : (T)0;
        r.w = lane_west(r.e);
        r.s = below;
        r.c = -r.e + -r.n + -r.w + -r.s;
        return r;
    }
};

// Columns of a block that run (inactive ones read a running column's data and
// store nothing).
template <int C>
struct ColBlock {
    int col[C];
    bool on[C];
};

// Alternates two row chunks: the loads of one are in flight while the other is
// worked on; chunk 0 is already being loaded into m.A.
// ONE: the rows fit chunk A alone.
template <bool ONE, class M, class W>
__device__ __forceinline__ void march_chunks(M& m, W work) {
    if constexpr (ONE) {
        work(m.A, 0);
        return;
    }
    for (int ch = 0; ch < m.chunks; ch += 2) {
        if (ch + 1 < m.chunks) m.load(m.B, ch + 1);
        work(m.A, ch);
        if (ch + 1 < m.chunks) {
            if (ch + 2 < m.chunks) m.load(m.A, ch + 2);
            work(m.B, ch + 1);
        }
    }
}

// ---------------------------------------------------------- down, one wave ---
// UNI (a template argument of run): every row and lane of the wave is a node
// strictly inside the mesh, so nothing is masked.
// UPD: b is the PCG residual before the iteration's step, r = b - alpha q is
// formed where it is needed and written to rn on the wave's own nodes.
template <typename T, class Op, typename TB, int CH, int C, bool UPD>
struct DownMarch {
    static constexpr bool NE = kNorthEast<Op>;
    struct Chunk {
        TB vb[C][CH], vq[UPD ? C : 1][UPD ? CH : 1];
        RowLoads<Op, CH> ro;
    };
    const Op& op;
    const TB* __restrict__ b;
    const TB* __restrict__ q;
    int ld, I0, J0, J1, i, js, rows, chunks;
    unsigned ic;
    ColBlock<C> cb;
    BufRef<TB> bb[C], qb[UPD ? C : 1];
    typename RowLoads<Op, CH>::Src src;
    Chunk A, B;
    __device__ __forceinline__ DownMarch(const Op& o, const TB* b_, const TB* q_, int ld_, int strip, int seg, int H)
        : op(o), b(b_), q(q_), ld(ld_), src(o) {
        const int N = op.N;
        I0 = strip * kDownOwn;
        J0 = seg * H;
        J1 = min(J0 + H - 1, N / 2);
        i = 2 * I0 - 3 + (int)(threadIdx.x & 63);
        js = 2 * J0 - 3;
        ic = (unsigned)clamp_node(i, N);
        rows = 2 * (J1 - J0) + 7;
        chunks = (rows + CH - 1) / CH;
    }
    // the block's columns: cnt of them from col0 (the last one repeated)
    __device__ __forceinline__ void bind(int col0, int cnt) {
        const long long n = (long long)(op.N + 1) * (op.N + 1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            cb.col[c] = col0 + min(c, cnt - 1);
            bb[c] = BufRef<TB>(b + (size_t)cb.col[c] * ld, n);
            if constexpr (UPD) qb[c] = BufRef<TB>(q + (size_t)cb.col[c] * ld, n);
        }
    }
    __device__ bool inside() const {
        return 2 * I0 - 3 >= 1 && 2 * I0 + 60 <= op.N - 1 && js >= 1 && js + chunks * CH <= op.N;
    }
    __device__ __forceinline__ void load(Chunk& k, int ch) {
        const int N = op.N, N1 = N + 1;
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int base = clamp_node(js + ch * CH + e, N) * N1;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                k.vb[c][e] = bb[c].get(base, ic);
                if constexpr (UPD) k.vq[c][e] = qb[c].get(base, ic);
            }
            k.ro.load(src, e, ic, base);
        }
    }
    // alpha, rn, rr (the lane's part of r^T r) with UPD only
    template <bool UNI>
    __device__ __forceinline__ void run(const KARow<T>* tab, T* __restrict__ x, T* __restrict__ bc, int ldc,
                                        int dirichlet, const ChebCoef& cc, const TB* alpha, TB* __restrict__ rn,
                                        double* rr) {
        const int lane = threadIdx.x & 63;
        const int N = op.N, N1 = N + 1, Nc = N / 2, Nc1 = Nc + 1;
        const bool inx = i >= 0 && i <= N;
        const bool ownx = lane >= 3 && lane < 3 + 2 * kDownOwn && i <= N;
        const int I = I0 + ((lane - 3) >> 1);
        const bool ownc = (lane & 1) && lane >= 3 && lane < 3 + 2 * kDownOwn && I <= Nc;
        const int oj1 = min(2 * J1 + 1, N);
        const T inv_theta = (T)cc.inv_theta, cA = (T)cc.cA, cB = (T)cc.cB;
        // per column: b, d0 and x2 of the last rows, residuals of the last two
        T b1[C]{}, b2[C]{}, d1[C]{}, d2[C]{}, x2[C]{}, x3[C]{}, r3[C]{}, r4[C]{};
        LaneRow<T> R1, R2;
        march_chunks<false>(*this, [&](const Chunk& k, int ch) {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                if (!(e & 1) && ch * CH + e >= rows) return;
                const int j = js + ch * CH + e;  // odd for even e
                const bool in = UNI || (inx && (unsigned)j <= (unsigned)N);
                const LaneRow<T> R0 = k.ro.template row<UNI>(op, tab, e, i, j, in, R1.n);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    TB bv = k.vb[c][e];
                    if constexpr (UPD) {
                        bv = bv - alpha[c] * k.vq[c][e];
                        if (j >= 2 * J0 && j <= oj1 && cb.on[c]) {
                            TB* rr_row = rn + (size_t)cb.col[c] * ld + j * N1;
                            if (ownx) {
                                row_put(rr_row, ic, bv);
                                rr[c] += (double)bv * (double)bv;
                            }
                        }
                    }
                    const T b0 = in ? (T)bv : (T)0;
                    const T d0 = R0.dv * b0 * inv_theta;
                    // x2 of row j - 1
                    const T x1 = cA * d1[c] + cB * R1.dv * (b1[c] - lane_apply<NE>(R1, d2[c], d1[c], d0));
                    if (j - 1 >= 2 * J0 && j - 1 <= oj1 && cb.on[c]) {
                        T* xr = x + (size_t)cb.col[c] * ld + (j - 1) * N1;
                        if (ownx) row_put(xr, ic, x1);
                    }
                    // residual of row j - 2, zero off the free nodes
                    const T rv = b2[c] - lane_apply<NE>(R2, x3[c], x2[c], x1);
                    const T r2 = R2.dv != (T)0 ? rv : (T)0;
                    if (!(e & 1)) {
                        // P^T at coarse row (j - 3) / 2, fine row j - 3
                        const int J = (j - 3) >> 1;
                        if (J >= J0 && J <= J1 && cb.on[c]) {
                            T sm = lane_west(r3[c]);
                            sm += lane_east(r3[c]);
                            sm += r4[c];
                            sm += r2;
                            sm += lane_east(r2);
                            sm += lane_west(r4[c]);
                            const T v = r3[c] + (T)0.5 * sm;
                            T* br = bc + (size_t)cb.col[c] * ldc + J * Nc1;
                            if (ownc) row_put(br, (unsigned)I, dirichlet && (J == 0 || J == Nc) ? (T)0 : v);
                        }
                    }
                    b2[c] = b1[c];
                    b1[c] = b0;
                    d2[c] = d1[c];
                    d1[c] = d0;
                    x3[c] = x2[c];
                    x2[c] = x1;
                    r4[c] = r3[c];
                    r3[c] = r2;
                }
                R2 = R1;
                R1 = R0;
            }
        });
    }
};

// ------------------------------------------------------------ up, one wave ---
template <typename T, class Op, typename TB, typename TX, int CH, int C>
struct UpMarch {
    static constexpr bool NE = kNorthEast<Op>;
    static_assert(CH % 2 == 0, "rows come in pairs");
    struct Chunk {
        TB vb[C][CH];
        T vx[C][CH], pc[C][CH / 2 + 1], pf[C][CH / 2 + 1];
        RowLoads<Op, CH> ro;
    };
    const Op& op;
    const TB* __restrict__ b;
    const T* __restrict__ x2;
    const T* __restrict__ xc;
    int ld, ldc, i0, j0, j1, i, js, rows, chunks;
    unsigned ic, I, If;
    ColBlock<C> cb;
    BufRef<TB> bb[C];
    BufRef<T> xb[C], cr[C];
    typename RowLoads<Op, CH>::Src src;
    Chunk A, B;
    // columns from i0_ (even; lane 2), the R rows from j0_ (even)
    __device__ __forceinline__ UpMarch(const Op& o, const TB* b_, const T* x2_, const T* xc_, int ld_, int ldc_, int i0_, int j0_,
                                       int R)
        : op(o), b(b_), x2(x2_), xc(xc_), ld(ld_), ldc(ldc_), i0(i0_), j0(j0_), src(o) {
        const int N = op.N;
        j1 = min(j0 + R - 1, N);
        i = i0 - 2 + (int)(threadIdx.x & 63);
        js = j0 - 2;
        ic = (unsigned)clamp_node(i, N);
        I = (unsigned)clamp_node(i >> 1, N / 2);
        If = (unsigned)clamp_node((i + 1) >> 1, N / 2);
        rows = j1 - j0 + 5;
        chunks = (rows + CH - 1) / CH;
    }
    __device__ __forceinline__ void bind(int col0, int cnt) {
        const long long n = (long long)(op.N + 1) * (op.N + 1), nc = (long long)(op.N / 2 + 1) * (op.N / 2 + 1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            cb.col[c] = col0 + min(c, cnt - 1);
            bb[c] = BufRef<TB>(b + (size_t)cb.col[c] * ld, n);
            xb[c] = BufRef<T>(x2 + (size_t)cb.col[c] * ld, n);
            cr[c] = BufRef<T>(xc + (size_t)cb.col[c] * ldc, nc);
        }
    }
    __device__ bool inside() const {
        return i0 - 2 >= 1 && i0 + 61 <= op.N - 1 && js >= 1 && js + chunks * CH <= op.N;
    }
    __device__ __forceinline__ void load(Chunk& k, int ch) {
        const int N = op.N, N1 = N + 1, Nc = N / 2, Nc1 = Nc + 1;
        const int jb = js + ch * CH;
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int base = clamp_node(jb + e, N) * N1;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                k.vb[c][e] = bb[c].get(base, ic);
                k.vx[c][e] = xb[c].get(base, ic);
            }
            k.ro.load(src, e, ic, base);
        }
        // the coarse rows that prolongation reads: the coarse node at or west
        // of the lane's column and the one at or east of it
#pragma unroll
        for (int e = 0; e < CH / 2 + 1; ++e) {
            const int base = clamp_node((jb >> 1) + e, Nc) * Nc1;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                k.pc[c][e] = cr[c].get(base, I);
                k.pf[c][e] = cr[c].get(base, If);
            }
        }
    }
    // out(c, j, v, bv): x = v at (i, j) of block column c, where b = bv
    // (called by every lane, for the rows j0 .. j1 of running columns)
    template <bool UNI, bool ONE, class F>
    __device__ __forceinline__ void run(const KARow<T>* tab, int dirichlet, const ChebCoef& cc, F out) {
        const int lane = threadIdx.x & 63;
        const int N = op.N;
        const bool inx = i >= 0 && i <= N;
        const bool odd = lane & 1;  // column i is odd
        const T inv_theta = (T)cc.inv_theta, theta = (T)cc.theta, cB = (T)cc.cB, c1 = (T)cc.c1;
        T b1[C]{}, x1[C]{}, xx2[C]{}, d2[C]{}, d3[C]{};
        TB rb1[C]{}, rb2[C]{};
        LaneRow<T> R1, R2;
        march_chunks<ONE>(*this, [&](const Chunk& k, int ch) {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                if (!(e & 1) && ch * CH + e >= rows) return;
                const int j = js + ch * CH + e;  // parity of e
                const bool in = UNI || (inx && (unsigned)j <= (unsigned)N);
                const bool fr = in && !(!UNI && dirichlet && (j == 0 || j == N));
                const LaneRow<T> R0 = k.ro.template row<UNI>(op, tab, e, i, j, in, R1.n);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    // x2 + P x_c: the coarse node when i and j are even, else the
                    // mean of the two coarse ends of the fine edge through (i, j)
                    const T p0 = k.pc[c][e / 2], p1 = k.pf[c][e / 2 + (e & 1)];
                    const T pr = (e & 1) || odd ? (T)0.5 * (p0 + p1) : p0;
                    const T x0 = fr ? k.vx[c][e] + pr : (T)0;
                    const T b0 = in ? (T)k.vb[c][e] : (T)0;
                    // d0 of row j - 1
                    const T d1 = R1.dv * (b1[c] - lane_apply<NE>(R1, xx2[c], x1[c], x0)) * inv_theta;
                    // x of row j - 2
                    const T dk = d2[c];
                    const T rr = theta * dk * R2.c - lane_apply<NE>(R2, d3[c], dk, d1);
                    const T v = xx2[c] + ((T)1 + c1) * dk + cB * R2.dv * rr;
                    if (j - 2 >= j0 && j - 2 <= j1 && cb.on[c]) out(c, j - 2, v, rb2[c]);
                    b1[c] = b0;
                    rb2[c] = rb1[c];
                    rb1[c] = k.vb[c][e];
                    xx2[c] = x1[c];
                    x1[c] = x0;
                    d3[c] = d2[c];
                    d2[c] = d1;
                }
                R2 = R1;
                R1 = R0;
            }
        });
    }
};

// --------------------------------------------------- PCG apply, one wave ---
// Rows of p_new = z + beta p_old and q = A z + beta A p_old; lanes 1 .. 62 own
// their nodes.  The operator has the PCG's precision.
constexpr int kApplyOwn = 62;
template <class Op, int CH>
struct ApplyLoads {
    struct Src {
        __device__ explicit Src(const Op&) {}
    };
    __device__ void load(const Src&, int, unsigned, int) {}
};
template <typename T, int CH>
struct ApplyLoads<OpA<T>, CH> {
    struct Src {
        BufRef<T> e, n;
        __device__ explicit Src(const OpA<T>& o) {
            const long long cnt = (long long)(o.N + 1) * (o.N + 1);
            e = BufRef<T>(o.wE, cnt);
            n = BufRef<T>(o.wN, cnt);
        }
    };
    T we[CH], wn[CH];
    __device__ void load(const Src& s, int e, unsigned ic, int rowbase) {
        we[e] = s.e.get(rowbase, ic);
        wn[e] = s.n.get(rowbase, ic);
    }
};

template <typename T, class Op, int CH, int C, bool FIRST>
struct ApplyMarch {
    static constexpr bool NE = kNorthEast<Op>;
    static constexpr int CP = FIRST ? 1 : C, CHP = FIRST ? 1 : CH;
    struct Chunk {
        T vz[C][CH], vp[CP][CHP], vx[CP][CHP];
        ApplyLoads<Op, CH> ro;
    };
    const Op& op;
    int i, j0, j1, js, rows, chunks;
    unsigned ic;
    ColBlock<C> cb;
    BufRef<T> zb[C], pb[CP], xb[CP];
    typename ApplyLoads<Op, CH>::Src src;
    Chunk A, B;
    __device__ __forceinline__ ApplyMarch(const Op& o, int strip, int seg, int R) : op(o), src(o) {
        const int N = op.N;
        j0 = seg * R;
        j1 = min(j0 + R - 1, N);
        js = j0 - 1;
        i = strip * kApplyOwn - 1 + (int)(threadIdx.x & 63);
        ic = (unsigned)clamp_node(i, N);
        rows = j1 - j0 + 3;
        chunks = (rows + CH - 1) / CH;
    }
    __device__ __forceinline__ void bind(const T* z, const T* p, const T* x, int ld, int col0, int cnt) {
        const long long n = (long long)(op.N + 1) * (op.N + 1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            cb.col[c] = col0 + min(c, cnt - 1);
            zb[c] = BufRef<T>(z + (size_t)cb.col[c] * ld, n);
            if constexpr (!FIRST) {
                pb[c] = BufRef<T>(p + (size_t)cb.col[c] * ld, n);
                xb[c] = BufRef<T>(x + (size_t)cb.col[c] * ld, n);
            }
        }
    }
    __device__ __forceinline__ void load(Chunk& k, int ch) {
        const int N = op.N, N1 = N + 1;
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const int base = clamp_node(js + ch * CH + e, N) * N1;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                k.vz[c][e] = zb[c].get(base, ic);
                if constexpr (!FIRST) {
                    k.vp[c][e] = pb[c].get(base, ic);
                    k.vx[c][e] = xb[c].get(base, ic);
                }
            }
            k.ro.load(src, e, ic, base);
        }
    }
    // out(c, j, p, q, x): the column's new p, q and x at (i, j), called by
    // every lane for the rows j0 .. j1 of running columns
    __device__ bool inside() const {
        return i - (int)(threadIdx.x & 63) >= 1 && i - (int)(threadIdx.x & 63) + 63 <= op.N - 1 && js >= 1 &&
               js + chunks * CH <= op.N;
    }
    template <bool UNI, class F>
    __device__ __forceinline__ void run(const KARow<T>* tab, const T* beta, const T* alpha, F out) {
        const int N = op.N;
        T z1[C]{}, z2[C]{}, p1[C]{}, p2[C]{}, x1[C]{};
        T we1{}, wn1{}, wn2{};
        march_chunks<false>(*this, [&](const Chunk& k, int ch) {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                if (ch * CH + e >= rows) return;
                const int j = js + ch * CH + e, jc = j - 1;  // jc: the row whose products are complete
                T we0{}, wn0{};
                if constexpr (!NE) {
                    we0 = k.ro.we[e];
                    wn0 = k.ro.wn[e];
                }
                T ww{};
                if constexpr (!NE) ww = lane_west(we1);
                const bool fr = UNI || (i >= 0 && i <= N && op.is_free(i, jc));
                auto product = [&](T vm, T v, T vp) -> T {
                    if constexpr (NE) {
                        const KANb<T> nb{v, lane_east(v), lane_west(v), vp, vm, lane_east(vp), lane_west(vm)};
                        if constexpr (UNI)
                            return ka_combine(op.rows[0], nb);
                        else
                            return ka_combine(tab[ka_class(i, jc, N)], nb);
                    } else {
                        const typename Op::Nb nb{v, lane_east(v), lane_west(v), vp, vm};
                        return op.combine(i, jc, typename Op::Row{we1, ww, wn1, wn2}, nb);
                    }
                };
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const T z0 = k.vz[c][e];
                    T p0{}, x0{};
                    if constexpr (!FIRST) {
                        p0 = k.vp[c][e];
                        x0 = k.vx[c][e];
                    }
                    if (jc >= j0 && cb.on[c]) {
                        T az = product(z2[c], z1[c], z0), ap{};
                        az = fr ? az : (T)0;
                        T pn = z1[c], qn = az, xn{};
                        if constexpr (!FIRST) {
                            ap = product(p2[c], p1[c], p0);
                            ap = fr ? ap : (T)0;
                            pn = z1[c] + beta[c] * p1[c];
                            qn = az + beta[c] * ap;
                            xn = x1[c] + alpha[c] * p1[c];
                        }
                        out(c, jc, pn, qn, xn);
                    }
                    z2[c] = z1[c];
                    z1[c] = z0;
                    if constexpr (!FIRST) {
                        p2[c] = p1[c];
                        p1[c] = p0;
                        x1[c] = x0;
                    }
                }
                wn2 = wn1;
                wn1 = wn0;
                we1 = we0;
            }
        });
    }
};

// Class table of the prior operator in LDS with a zero row for nodes off the
// mesh (entry 9); the state operator needs none.
template <typename T, class Op>
__device__ inline void stage_rows(const Op& op, KARow<T>* tab) {
    if constexpr (kNorthEast<Op>) {
        if (threadIdx.x < 9) tab[threadIdx.x] = ka_row(op, threadIdx.x);
        if (threadIdx.x == 9) tab[9] = KARow<T>{};
    }
}

// Columns of column block z: blocks of C columns within an instance.
template <int C>
__device__ inline int block_columns(const March& m, int z, int& col0) {
    const int bpi = (m.cpi + C - 1) / C, inst = m.many ? uniform(z / bpi) : 0, k = z - inst * bpi;
    col0 = inst * m.cpi + k * C;
    return min(C, m.cpi - k * C);
}

// --------------------------------------------------------------- k_down ---
// x2 = S(b) (two Chebyshev steps from zero), r = b - A x2, b_coarse = P^T r.
// Grid: (workgroups of a column block, 1, column blocks); the waves of a
// column block take its strips x segments, strips first.  b may be of a wider
// type TB than the level's vectors (the finest level of an FP64 PCG).
// UPD (finest level inside the PCG): b is the residual before the iteration's
// step; alpha is formed from the partials of p^T q, b <- b - alpha q goes to rn
// and its partials of b^T b to red.rr (the next level down tests them).
// check: the launch first tests the columns' convergence (red.rr).
template <typename T, class Op, typename TB, int CH, int C, bool UPD>
__global__ __launch_bounds__(64 * kMarchWaves) void k_down(Op op_, const TB* __restrict__ b, const TB* __restrict__ q,
                                                           TB* __restrict__ rn, T* __restrict__ x, int ld,
                                                           T* __restrict__ bc, int ldc, int dirichlet,
                                                           int* __restrict__ act, ChebCoef cc, PcgRed red,
                                                           ColState* __restrict__ st, int check, March m,
                                                           TileMap tm) {
    __shared__ KARow<T> tab[kNorthEast<Op> ? 10 : 1];
    __shared__ double part[C][kMarchWaves];
    const int3 tb = xcd_tile(tm);
    int col0;
    const int cnt = block_columns<C>(m, tb.z, col0);
    const auto& op = op_.at(col0);
    // waves past the last segment take part in the barriers alone
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), item = tb.x * kMarchWaves + wave;
    const int it = min(item, m.strips * m.segs - 1), seg = fast_div(it, m.inv_strips), strip = it - seg * m.strips;
    DownMarch<T, std::decay_t<decltype(op)>, TB, CH, C, UPD> w(op, b, q, ld, strip, seg, m.len);
    w.bind(col0, cnt);
    // the partials and the first rows are in flight together (few columns:
    // also with the flags that say whether the column still runs)
    constexpr bool kAhead = CH == kLatencyChunk;
    double share[C]{}, rz[C]{};
    VtShare vt[C];
    int live[C]{};
    const int bd = kAhead ? vec_threads(red.per) : (int)blockDim.x;
    if constexpr (kAhead) w.load(w.A, 0);
    bool any = false;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        // UPD: the lead workgroup clears act[col] on a breakdown while others
        // read it, so thread 0 reads it for the workgroup (vt_total)
        w.cb.on[c] = c < cnt && (UPD || check || column_on(act, col0 + c));
        if constexpr (UPD && !kAhead) w.cb.on[c] = w.cb.on[c] && __syncthreads_or(act[col0 + c]);
        any = any || w.cb.on[c];
        if (!w.cb.on[c]) continue;
        if (check) share[c] = partial_share(red.rr, col0 + c, red.stride, red.nrr);
        if constexpr (UPD) {
            live[c] = act[col0 + c];
            vt[c] = vt_first(red.pq, col0 + c, red.stride, red.npq);
            rz[c] = st[col0 + c].rz_new;
        }
    }
    if (!any) return;
    if constexpr (!kAhead) w.load(w.A, 0);
    stage_rows(op, tab);
    TB alpha[C]{};
    if (check || UPD) {
        any = false;
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (w.cb.on[c]) {
                if constexpr (UPD) {
                    const double pq = vt_total(vt[c], red.pq, col0 + c, red.stride, red.npq, bd, live[c]);
                    if (live[c]) {
                        alpha[c] = (TB)pcg_alpha(rz[c], pq, st + col0 + c, act + col0 + c, tb.x == 0);
                        if (!(pq > 0.0)) w.cb.on[c] = false;
                    } else {
                        w.cb.on[c] = false;
                    }
                } else if (column_done_share(share[c], red, col0 + c, st, act, tb.x == 0)) {
                    w.cb.on[c] = false;
                }
                any = any || w.cb.on[c];
                if (c + 1 < C) lds_barrier();  // the LDS slots of the sum are reused by the next column
            }
        if (!any) return;
    } else if constexpr (kNorthEast<Op>) {
        lds_barrier();
    }
    double rr[C]{};
    if (item < m.strips * m.segs) {
        if (w.inside())
            w.template run<true>(tab, x, bc, ldc, dirichlet, cc, alpha, rn, rr);
        else
            w.template run<false>(tab, x, bc, ldc, dirichlet, cc, alpha, rn, rr);
    }
    if constexpr (UPD) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const double s = wave_sum(rr[c]);
            if ((threadIdx.x & 63) == 0) part[c][wave] = s;
        }
        lds_barrier();
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (threadIdx.x == 0 && w.cb.on[c]) {
                double s = 0.0;
                for (int v = 0; v < kMarchWaves; ++v) s += part[c][v];
                red.rr[(size_t)(col0 + c) * red.stride + tb.x] = s;
            }
    }
}

// ----------------------------------------------------------------- k_up ---
// x = x2 + P x_coarse, then two Chebyshev steps on A x = b; with rz set the
// workgroup's part of sum_k b_k x_k (the PCG inner product r^T z).  b may be of
// a wider type TB and the output x of a wider type TX than the level's
// vectors.  Grid as k_down.
template <typename T, class Op, typename TB, typename TX, int CH, int C>
__global__ __launch_bounds__(64 * kMarchWaves) void k_up(Op op_, const TB* __restrict__ b, const T* __restrict__ x2,
                                                         TX* __restrict__ x, int ld, const T* __restrict__ xc, int ldc,
                                                         int dirichlet, const int* __restrict__ act, ChebCoef cc,
                                                         int rz, PcgRed red, March m, TileMap tm) {
    __shared__ KARow<T> tab[kNorthEast<Op> ? 10 : 1];
    __shared__ double part[C][kMarchWaves];
    const int3 tb = xcd_tile(tm);
    int col0;
    const int cnt = block_columns<C>(m, tb.z, col0);
    const auto& op = op_.at(col0);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), item = tb.x * kMarchWaves + wave;
    const int it = min(item, m.strips * m.segs - 1), seg = fast_div(it, m.inv_strips), strip = it - seg * m.strips;
    UpMarch<T, std::decay_t<decltype(op)>, TB, TX, CH, C> w(op, b, x2, xc, ld, ldc, strip * kUpOwn, seg * m.len, m.len);
    constexpr bool kAhead = CH == kLatencyChunk;  // see k_down
    bool any = false;
    w.bind(col0, cnt);
    if constexpr (kAhead) w.load(w.A, 0);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        w.cb.on[c] = c < cnt && column_on(act, col0 + c);
        any = any || w.cb.on[c];
    }
    if (!any) return;
    if constexpr (!kAhead) w.load(w.A, 0);
    if constexpr (kNorthEast<Op>) {
        stage_rows(op, tab);
        lds_barrier();
    }
    double dots[C]{};
    if (item < m.strips * m.segs) {
        const int lane = threadIdx.x & 63, N = op.N;
        const bool own = lane >= 2 && lane < 2 + kUpOwn && w.i <= N;
        auto out = [&](int c, int j, T v, TB bv) {
            TX* xr = x + (size_t)w.cb.col[c] * ld + j * (N + 1);
            if (own) {
                row_put(xr, w.ic, (TX)v);
                if (rz) dots[c] += (double)v * (double)bv;
            }
        };
        if (w.inside())
            w.template run<true, false>(tab, dirichlet, cc, out);
        else
            w.template run<false, false>(tab, dirichlet, cc, out);
    }
    if (!rz) return;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double s = wave_sum(dots[c]);
        if ((threadIdx.x & 63) == 0) part[c][wave] = s;
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (threadIdx.x == 0 && w.cb.on[c]) {
            double s = 0.0;
            for (int v = 0; v < kMarchWaves; ++v) s += part[c][v];
            red.rz[(size_t)(col0 + c) * red.stride + tb.x] = s;
        }
}

// The finest up step of few columns, with r^T z in a fixed order that does not
// depend on how the waves split the mesh: one partial per TF x TF tile, summed
// over the tile's nodes as 256 threads in row-major order would (two-level:
// 64 values by a butterfly, then the groups in turn).  FP64 results keep their
// last bit whatever the wave shapes (FP32 solves round alpha and beta to FP32
// and do not notice).  A workgroup covers kUpTiles tiles side by side; its
// waves take a quarter of the rows each, all of whose loads are in flight at
// once, and hand x and b to the sum through LDS.
// Grid: (tile groups, tile rows, columns).
constexpr int kUpTiles = 3, kUpFewChunk = 10;
template <typename T, class Op, typename TB, typename TX, int TF>
__global__ __launch_bounds__(64 * kMarchWaves) __attribute__((amdgpu_waves_per_eu(4))) void k_up_few(Op op_, const TB* __restrict__ b, const T* __restrict__ x2,
                                                             TX* __restrict__ x, int ld, const T* __restrict__ xc,
                                                             int ldc, int dirichlet, const int* __restrict__ act,
                                                             ChebCoef cc, PcgRed red, TileMap tm) {
    constexpr int OW = kUpTiles * TF, NT = 64 * kMarchWaves;
    constexpr int R1 = TF / kMarchWaves / 2 * 2, R0 = TF - (kMarchWaves - 1) * R1;  // rows of wave 0, of the others
    static_assert(OW + 4 <= 64 && R0 + 4 <= kUpFewChunk && TF % 2 == 0, "tile shape");
    __shared__ KARow<T> tab[kNorthEast<Op> ? 10 : 1];
    __shared__ T xs[TF][OW];
    __shared__ TB bs[TF][OW];
    __shared__ double part[kUpTiles][NT / 64];
    const int3 tb = xcd_tile(tm);
    const int col = tb.z;
    const auto& op = op_.at(col);
    const int N = op.N, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = tb.x * OW, j0 = tb.y * TF, jw = wave == 0 ? 0 : R0 + (wave - 1) * R1;
    UpMarch<T, std::decay_t<decltype(op)>, TB, TX, kUpFewChunk, 1> w(op, b, x2, xc, ld, ldc, i0, j0 + jw,
                                                                     wave == 0 ? R0 : R1);
    w.bind(col, 1);
    w.cb.on[0] = true;
    w.load(w.A, 0);
    if (!column_on(act, col)) return;
    if constexpr (kNorthEast<Op>) {
        stage_rows(op, tab);
        lds_barrier();
    }
    {
        const bool own = lane >= 2 && lane < 2 + OW && w.i <= N;
        auto out = [&](int, int j, T v, TB bv) {
            TX* xr = x + (size_t)col * ld + j * (N + 1);
            if (own) {
                row_put(xr, w.ic, (TX)v);
                xs[j - j0][lane - 2] = v;
                bs[j - j0][lane - 2] = bv;
            }
        };
        if (w.inside())
            w.template run<true, true>(tab, dirichlet, cc, out);
        else
            w.template run<false, true>(tab, dirichlet, cc, out);
    }
    lds_barrier();
    const int h = min(TF, N + 1 - j0);
    double s[kUpTiles];
#pragma unroll
    for (int q = 0; q < kUpTiles; ++q) {
        const int wd = min(TF, N + 1 - (i0 + q * TF));  // width of tile q (none past the mesh)
        s[q] = 0.0;
        if (wd > 0)
            for (int t = threadIdx.x; t < wd * h; t += NT) {
                const int jj = t / wd, ii = q * TF + t - jj * wd;
                s[q] += (double)xs[jj][ii] * (double)bs[jj][ii];
            }
    }
#pragma unroll
    for (int q = 0; q < kUpTiles; ++q) {
        const double t = wave_sum(s[q]);
        if (lane == 0) part[q][wave] = t;
    }
    lds_barrier();
    const int tiles = (N + TF) / TF;  // tiles a mesh row (N + 1 nodes)
    if (threadIdx.x < kUpTiles && tb.x * kUpTiles + (int)threadIdx.x < tiles) {
        double t = 0.0;
        for (int v = 0; v < NT / 64; ++v) t += part[threadIdx.x][v];
        red.rz[(size_t)col * red.stride + tb.y * tiles + tb.x * kUpTiles + threadIdx.x] = t;
    }
}

// ------------------------------------------------------------ k_pcg_apply ---
// The PCG apply of batches (see k_pcg_apply_few for what it does).  Grid as
// k_down: strips of kApplyOwn columns, segments of m.len rows.
template <typename T, class Op, bool FIRST, int CH, int C>
__global__ __launch_bounds__(64 * kMarchWaves) void k_pcg_apply(Op op_, const T* __restrict__ z,
                                                                const T* __restrict__ p_old, T* __restrict__ p_new,
                                                                T* __restrict__ q, T* __restrict__ x, int ld,
                                                                const int* __restrict__ act, ColState* __restrict__ st,
                                                                PcgRed red, March m, TileMap tm) {
    __shared__ KARow<T> tab[kNorthEast<Op> ? 10 : 1];
    __shared__ double part[C][kMarchWaves];
    const int3 tb = xcd_tile(tm);
    int col0;
    const int cnt = block_columns<C>(m, tb.z, col0);
    const auto& op = op_.at(col0);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), item = tb.x * kMarchWaves + wave;
    const int it = min(item, m.strips * m.segs - 1), seg = fast_div(it, m.inv_strips), strip = it - seg * m.strips;
    ApplyMarch<T, std::decay_t<decltype(op)>, CH, C, FIRST> w(op, strip, seg, m.len);
    bool any = false;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        w.cb.on[c] = c < cnt && column_on(act, col0 + c);
        any = any || w.cb.on[c];
    }
    if (!any) return;
    w.bind(z, p_old, x, ld, col0, cnt);
    const bool need_rz = !FIRST || tb.x == 0;  // uniform in the workgroup
    double share[C]{};
    T beta[C]{}, alpha[C]{};
    double rz_old[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (!w.cb.on[c]) continue;
        if (need_rz) share[c] = partial_share(red.rz, col0 + c, red.stride, red.nrz);
        rz_old[c] = FIRST ? 1.0 : st[col0 + c].rz;
        alpha[c] = FIRST ? (T)0 : (T)st[col0 + c].alpha;
    }
    w.load(w.A, 0);
    stage_rows(op, tab);
    if (need_rz) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (w.cb.on[c]) {
                const double rz = share_total(share[c]);
                if constexpr (!FIRST) beta[c] = (T)(rz / rz_old[c]);
                if (tb.x == 0 && threadIdx.x == 0) st[col0 + c].rz_new = rz;
                if (c + 1 < C) lds_barrier();
            }
    } else if constexpr (kNorthEast<Op>) {
        lds_barrier();
    }
    double dots[C]{};
    if (item < m.strips * m.segs) {
        const int lane = threadIdx.x & 63, N = op.N;
        const bool own = lane >= 1 && lane <= kApplyOwn && w.i <= N;
        auto out = [&](int c, int j, T pn, T qn, T xn) {
            const size_t o = (size_t)w.cb.col[c] * ld + j * (N + 1);
            if (own) {
                row_put(p_new + o, w.ic, pn);
                row_put(q + o, w.ic, qn);
                if constexpr (!FIRST) row_put(x + o, w.ic, xn);
                dots[c] += (double)pn * (double)qn;
            }
        };
        if (kNorthEast<Op> && w.inside())
            w.template run<kNorthEast<Op>>(tab, beta, alpha, out);
        else
            w.template run<false>(tab, beta, alpha, out);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double s = wave_sum(dots[c]);
        if ((threadIdx.x & 63) == 0) part[c][wave] = s;
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (threadIdx.x == 0 && w.cb.on[c]) {
            double s = 0.0;
            for (int v = 0; v < kMarchWaves; ++v) s += part[c][v];
            red.pq[(size_t)(col0 + c) * red.stride + tb.x] = s;
        }
}

}  // namespace hinv
