// Field kernels: the implicit B / explicit E step (Sec. III.B, eqs. "bnplus1",
// "enplus1", "EllipticB") and the high-order current line solve (Sec. III.C, eqs.
// "jj6d", "penta").  Mesh arrays are FP64, x fastest, periodic.
#include <new>

#include "pp_device.hpp"
#include "pp_fixed.hpp"
#include "pp_internal.hpp"

namespace pp {

// Threads of a field launch: a block of 256 threads covers rows of x-consecutive cells
// (a row of nx cells, padded to a power of two, several rows per block) or, for nx > 256, a
// 256-cell chunk of one row; the remaining indices j, k come from the row number.  All
// indices are 32-bit (a box has at most 2^30 cells).
struct FieldGeom {
    int n[3];
    int M;           // half-width of the first-derivative stencil (order / 2)
    int64_t nc;
    double a[3][3];  // a[axis][m-1] / d[axis]: first-derivative coefficients
    double L[3][11]; // Laplacian stencil per axis, offsets -R..R
    int R;           // Laplacian half-width 2M - 1
    int xchunks;     // 256-cell chunks per row (nx > 256), else 1
    int xbits;       // log2 of the padded row length inside a block (<= 8)
    int rows;        // ny * nz
    int rpb;         // rows per block
    int small;       // an axis shorter than the stencil reach: general wrap
    double inv_ny;   // 1 / ny (row -> j, k)
};

// the same without the stencils
struct CellGeom {
    int n[3];
    int small;
    int64_t nc;
    int xchunks, xbits, rows, rpb;
    double inv_ny;
    CellGeom() = default;
    explicit CellGeom(const FieldGeom& G)
        : n{G.n[0], G.n[1], G.n[2]}, small(G.small), nc(G.nc), xchunks(G.xchunks), xbits(G.xbits), rows(G.rows),
          rpb(G.rpb), inv_ny(G.inv_ny) {}
};

constexpr int FIELD_BS = 256;

// index o cells away from i on a periodic axis of n cells
__device__ __forceinline__ int nbw(int i, int o, int n, int small) {
    int j = i + o;
    if (small) {
        j %= n;
        return j < 0 ? j + n : j;
    }
    return j < 0 ? j + n : (j >= n ? j - n : j);
}

// cell of thread t in block b of a run's launch; false for padding threads
template <class GEOM>
__device__ __forceinline__ bool field_cell(const GEOM& G, int64_t b, int t, int& i, int& j, int& k) {
    const int xc = (int)(b % G.xchunks);
    const int64_t rb = b / G.xchunks;
    i = xc * FIELD_BS + (t & ((1 << G.xbits) - 1));
    const int64_t row = rb * G.rpb + (t >> G.xbits);
    if (i >= G.n[0] || row >= G.rows) return false;
    k = (int)floor(((double)row + 0.5) * G.inv_ny);
    j = (int)(row - (int64_t)k * G.n[1]);
    if (j < 0) {
        j += G.n[1];
        --k;
    } else if (j >= G.n[1]) {
        j -= G.n[1];
        ++k;
    }
    return true;
}

template <class GEOM>
__device__ __forceinline__ int lin(const GEOM& G, int i, int j, int k) { return i + G.n[0] * (j + G.n[1] * k); }

// up-shifted derivative along axis ax of f (values on integer nodes along ax) at cell (i,j,k):
// sum_m a_m (f[i+m] - f[i-m+1]) / d
__device__ __forceinline__ double dup(const FieldGeom& G, const double* __restrict__ f, int ax, int i, int j, int k) {
    const int c[3] = {i, j, k};
    double s = 0.0;
    for (int m = 1; m <= G.M; ++m) {
        int hi[3] = {i, j, k}, lo[3] = {i, j, k};
        hi[ax] = nbw(c[ax], m, G.n[ax], G.small);
        lo[ax] = nbw(c[ax], -m + 1, G.n[ax], G.small);
        s += G.a[ax][m - 1] * (f[lin(G, hi[0], hi[1], hi[2])] - f[lin(G, lo[0], lo[1], lo[2])]);
    }
    return s;
}

// down-shifted derivative: sum_m a_m (g[i+m-1] - g[i-m]) / d
__device__ __forceinline__ double ddn(const FieldGeom& G, const double* __restrict__ f, int ax, int i, int j, int k) {
    const int c[3] = {i, j, k};
    double s = 0.0;
    for (int m = 1; m <= G.M; ++m) {
        int hi[3] = {i, j, k}, lo[3] = {i, j, k};
        hi[ax] = nbw(c[ax], m - 1, G.n[ax], G.small);
        lo[ax] = nbw(c[ax], -m, G.n[ax], G.small);
        s += G.a[ax][m - 1] * (f[lin(G, hi[0], hi[1], hi[2])] - f[lin(G, lo[0], lo[1], lo[2])]);
    }
    return s;
}

// composed Laplacian (d- after d+) of f at (i,j,k)
__device__ __forceinline__ double lap(const FieldGeom& G, const double* __restrict__ f, int i, int j, int k) {
    const int nx = G.n[0], nxy = G.n[0] * G.n[1];
    const int rowx = nx * (j + G.n[1] * k);
    const int colyz = i + nxy * k;
    const int colzx = i + nx * j;
    double s = 0.0;
    for (int o = -G.R; o <= G.R; ++o) {
        s += G.L[0][o + G.R] * f[rowx + nbw(i, o, nx, G.small)];
        s += G.L[1][o + G.R] * f[colyz + nx * nbw(j, o, G.n[1], G.small)];
        s += G.L[2][o + G.R] * f[colzx + nxy * nbw(k, o, G.n[2], G.small)];
    }
    return s;
}

// Everything one field step of one run needs (the single-run launches pass it by value,
// the batched launches read a table of them).
struct FieldDesc {
    FieldGeom G;
    double* E;
    double* B;
    const double* J;
    double* Bn;  // copy of B^n
    double* Bw;  // relaxation partner
    double* Bx;  // a second one (see relax_arrays)
    double* R;   // right-hand side
    const double* omega;        // Chebyshev weights omega_k, k = 1..sweeps (device)
    const double* rho;          // charge density (Gauss-law filter)
    double rho_bg, ieps0, kappa;  // background density, 1/eps0, filter damping
    double cab, dt, cj;         // alpha beta s, dt, alpha c^2 mu0 dt^2   (s = c^2 dt^2)
    double al2s, gdiag;         // alpha^2 s, gamma / diagonal
    double al, be, c2dt, mu0;   // alpha, beta, c^2 dt, mu0
    int sweeps;
    int zc;                     // planes a block of the tiled kernels marches over; 0: a thread per cell
};

// Gauss-law filter pass, first half: r = div- E - (rho + rho_bg)/eps0 into R
__device__ __forceinline__ void gauss_res_body(const FieldDesc& D, int i, int j, int k) {
    const FieldGeom& G = D.G;
    const int q = lin(G, i, j, k);
    double dv = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) dv += ddn(G, D.E + c * G.nc, c, i, j, k);
    D.R[q] = dv - (D.rho[q] + D.rho_bg) * D.ieps0;
}

// second half: E_c += kappa d+_c r
__device__ __forceinline__ void gauss_corr_body(const FieldDesc& D, int i, int j, int k) {
    const FieldGeom& G = D.G;
    const int q = lin(G, i, j, k);
#pragma unroll
    for (int c = 0; c < 3; ++c) D.E[c * G.nc + q] += D.kappa * dup(G, D.R, c, i, j, k);
}

enum FieldPhase { PH_GAUSS_RES = 0, PH_GAUSS_CORR = 1 };

__global__ void __launch_bounds__(FIELD_BS) k_field(FieldDesc D, int phase) {
    int i, j, k;
    if (!field_cell(D.G, blockIdx.x, threadIdx.x, i, j, k)) return;
    if (phase == PH_GAUSS_RES)
        gauss_res_body(D, i, j, k);
    else
        gauss_corr_body(D, i, j, k);
}

// ---- the field step, tiled -------------------------------------------------------------
// A block owns a 32 x 8 column of cells in x-y of one component and marches over D.zc planes in
// z.  Each array a stencil reads streams through the block plane by plane: a thread keeps the
// values of its own column at the z offsets the stencil needs in registers, and where a stencil
// runs along x or y the block stages the plane and the ring around it in LDS.  A value then
// comes from memory about once per plane instead of once per tap.  The next plane's loads are
// in flight while the block works on the current one.  Single and batched runs take the same
// code, so a batched run gives the same bits as the run alone.
//
// A sweep is bound by memory in large boxes (256^3: 0.34 ms, 4.7 TB/s for the four arrays it
// cannot do without) and by latency in small ones, where short marches (D.zc, down to one plane
// with every load in flight at once) spread it over the GPU.  Boxes that leave most of a column's
// threads idle take a thread per cell instead (thin_box).  Tiles of 64x8, 32x16, 64x4 and 64x16
// took 0 to 14 % longer.  Whole field step, us, with each tap of the boxes below 1024 columns read
// through the caches and now: 256^3 5750 and 4510, 128^3 1520 and 608, 128x32x32 260 and 98,
// 512x256x1 243 and 107, 64x32x32 222 and 70.
constexpr int RX_TX = 32, RX_TY = 8, RX_ZC = 32;
constexpr int RX_BS = RX_TX * RX_TY;  // one thread per column of the tile

// Sweep k (1-based) of the Chebyshev-accelerated Jacobi iteration for (1 - al2s lap) x = rhs:
//   y = x_{k-1} + gamma (rhs - A x_{k-1}) / diag,   x_k = x_{k-2} + omega_k (y - x_{k-2}),
// x_0 = x_{-1} = B^n, omega_1 = 1.  The right-hand side's kernel reads B^n and its Laplacian
// already: it keeps the copy of B^n (Bn) and takes sweep 1 as well, into Bw.  The others
// alternate between two arrays such that the last one is B; an iterate shares the array of the
// one before last (each cell reads its own old value before writing it):
//   an even number of sweeps: even iterates in B, odd ones in Bw;
//   an odd number:            x_1 in Bw, then even iterates in Bx, odd ones in B.
__device__ __forceinline__ double* relax_array(const FieldDesc& D, int k) {
    if ((D.sweeps & 1) == 0) return (k & 1) ? D.Bw : D.B;
    if (D.sweeps == 1) return D.B;  // a single sweep is not taken with the right-hand side
    return k == 1 ? D.Bw : ((k & 1) ? D.B : D.Bx);
}

struct TileCtx {
    int comp, i0, j0, z0, z1, tx, ty, col, own, nxy, n2, small;
    bool valid;
};

// The entries around a tile that its x and y taps reach: H deep on each side, no corners.  A
// thread's share of them: LDS index (-1: none) and in-plane offset (periodic), the same for every
// plane.  HX or HY 0: no taps along that axis.
template <int HX, int HY>
struct Ring {
    static constexpr int W = RX_TX + 2 * HX, H = RX_TY + 2 * HY;
    static constexpr int NX = 2 * HX * RX_TY, NY = 2 * HY * RX_TX, NH = (NX + NY + RX_BS - 1) / RX_BS;
    int hl[NH], hg[NH];
    __device__ __forceinline__ void init(int i0, int j0, int n0, int n1) {
#pragma unroll
        for (int e = 0; e < NH; ++e) {
            const int h = threadIdx.x + RX_BS * e;
            int a, b;  // column and row, 0 at the first of the entries' rows and columns
            if (h < NX) {
                b = HY + h / (HX > 0 ? 2 * HX : 1);
                a = h % (HX > 0 ? 2 * HX : 1);
                a += a < HX ? 0 : RX_TX;
            } else {
                b = (h - NX) / RX_TX;
                b += b < HY ? 0 : RX_TY;
                a = HX + (h - NX) % RX_TX;
            }
            const bool ring = h < NX + NY;
            hl[e] = ring ? a + W * b : -1;
            hg[e] = ring ? wrap_near(i0 + a - HX, n0) + n0 * wrap_near(j0 + b - HY, n1) : 0;
        }
    }
    static __device__ __forceinline__ int own(int tx, int ty) { return (ty + HY) * W + tx + HX; }
};

// block b of a run's launch: component, column and planes
__device__ __forceinline__ void tile_ctx(const FieldGeom& G, int zc, int b, TileCtx& X) {
    const int n0 = G.n[0], n1 = G.n[1];
    const int nbx = (n0 + RX_TX - 1) / RX_TX, nby = (n1 + RX_TY - 1) / RX_TY, nbz = (G.n[2] + zc - 1) / zc;
    const int bx = b % nbx;
    b /= nbx;
    const int by = b % nby;
    b /= nby;
    const int bz = b % nbz;
    X.comp = b / nbz;
    X.i0 = bx * RX_TX;
    X.j0 = by * RX_TY;
    X.z0 = bz * zc;
    X.z1 = X.z0 + zc < G.n[2] ? X.z0 + zc : G.n[2];
    X.tx = threadIdx.x % RX_TX;
    X.ty = threadIdx.x / RX_TX;
    X.valid = X.i0 + X.tx < n0 && X.j0 + X.ty < n1;
    X.col = wrap_near(X.i0 + X.tx, n0) + n0 * wrap_near(X.j0 + X.ty, n1);  // idle threads load wrapped columns
    X.own = X.valid ? X.col : 0;
    X.nxy = n0 * n1;
    X.n2 = G.n[2];
    X.small = G.small;
}

// STREAM: what a phase touches once passes by the caches, which are left to the stencils' reads (see
// streams_past_cache).
template <bool STREAM>
__device__ __forceinline__ double load_once(const double* p) {
    if constexpr (STREAM)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <bool STREAM>
__device__ __forceinline__ void store_once(double v, double* p) {
    if constexpr (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Sweep k of one block: the loads are unconditional (the last plane reloads its own plane, a lane
// off the ring or the box reads entry 0), so that none waits at a branch before the plane that is
// computed meanwhile.
template <int R, bool STREAM>
__device__ __forceinline__ void relax_tile(const FieldDesc& D, int b, int k, double* pl) {
    constexpr int W = Ring<R, R>::W, NH = Ring<R, R>::NH;
    const FieldGeom& G = D.G;
    TileCtx X;
    Ring<R, R> g;
    tile_ctx(G, D.zc, b, X);
    g.init(X.i0, X.j0, G.n[0], G.n[1]);
    const int64_t co = (int64_t)X.comp * G.nc;
    double* out = gl(relax_array(D, k)) + co;
    const double* x = gl(k == 1 ? D.Bn : relax_array(D, k - 1)) + co;
    const double* pv = gl(k <= 2 ? D.Bn : relax_array(D, k - 2)) + co;
    const double* rhs = gl(D.R) + co;
    const double w = gl(D.omega)[k];
    const int nxy = X.nxy, own = X.own;
    double q[2 * R + 1], hv[NH];
#pragma unroll
    for (int t = 0; t <= 2 * R; ++t) q[t] = x[X.col + nxy * nbw(X.z0, t - R, X.n2, X.small)];
#pragma unroll
    for (int e = 0; e < NH; ++e) hv[e] = x[g.hg[e] + X.z0 * nxy];
    double rq = load_once<STREAM>(rhs + own + X.z0 * nxy);
    double pq = load_once<STREAM>(pv + own + X.z0 * nxy);
    const int c0 = g.own(X.tx, X.ty);
    for (int kz = X.z0; kz < X.z1; ++kz) {
        if (kz > X.z0) __syncthreads();  // the previous plane's LDS reads are done
        pl[c0] = q[R];
#pragma unroll
        for (int e = 0; e < NH; ++e)
            if (g.hl[e] >= 0) pl[g.hl[e]] = hv[e];
        __syncthreads();
        const bool more = kz + 1 < X.z1;
        const int kn = more ? kz + 1 : kz;
        double qn = 0.0, rn = 0.0, pn = 0.0;
        if (D.zc > 1) {
            qn = x[X.col + nxy * nbw(kn, R, X.n2, X.small)];
#pragma unroll
            for (int e = 0; e < NH; ++e) hv[e] = x[g.hg[e] + kn * nxy];
            rn = load_once<STREAM>(rhs + own + kn * nxy);
            pn = load_once<STREAM>(pv + own + kn * nxy);
        }
        if (X.valid) {
            double sl = 0.0;
#pragma unroll
            for (int o = -R; o <= R; ++o) {
                sl += G.L[0][o + R] * pl[c0 + o];
                sl += G.L[1][o + R] * pl[c0 + o * W];
                sl += G.L[2][o + R] * q[R + o];
            }
            const double xq = q[R];
            const double Ax = xq - D.al2s * sl;
            const double y = xq + (rq - Ax) * D.gdiag;
            store_once<STREAM>(pq + w * (y - pq), out + own + kz * nxy);
        }
        if (more) {
#pragma unroll
            for (int t = 0; t < 2 * R; ++t) q[t] = q[t + 1];
            q[2 * R] = qn;
            rq = rn;
            pq = pn;
        }
    }
}

// One array streamed through the planes: values at z offsets WLO..WHI of the thread's column
// around the current plane and, where the array has taps along x (HX deep) or y (HY), the plane
// and its ring staged in LDS.
template <int HX, int HY, int WLO, int WHI>
struct ZStream {
    static constexpr bool PLANE = HX > 0 || HY > 0;
    static constexpr int NW = WHI - WLO + 1;
    using G = Ring<HX, HY>;
    static constexpr int NH = PLANE ? G::NH : 1, LDS = PLANE ? G::W * G::H : 0;
    const double* f;
    double* pl;
    int c0;
    G g;
    double w[NW];
    double hv[NH];
    double wn;
    // lds: the next free part of the block's LDS
    __device__ __forceinline__ void init(const double* src, const TileCtx& X, const FieldGeom& F, double*& lds) {
        f = gl(src);
#pragma unroll
        for (int t = 0; t < NW; ++t) w[t] = f[X.col + X.nxy * nbw(X.z0, WLO + t, X.n2, X.small)];
        if constexpr (PLANE) {
            pl = lds;
            lds += LDS;
            c0 = G::own(X.tx, X.ty);
            g.init(X.i0, X.j0, F.n[0], F.n[1]);
#pragma unroll
            for (int e = 0; e < NH; ++e) hv[e] = f[g.hg[e] + X.z0 * X.nxy];
        }
    }
    __device__ __forceinline__ void stage() const {
        if constexpr (PLANE) {
            pl[c0] = w[-WLO];
#pragma unroll
            for (int e = 0; e < NH; ++e)
                if (g.hl[e] >= 0) pl[g.hl[e]] = hv[e];
        }
    }
    __device__ __forceinline__ void prefetch(int kz1, const TileCtx& X) {
        wn = f[X.col + X.nxy * nbw(kz1, WHI, X.n2, X.small)];
        if constexpr (PLANE) {
#pragma unroll
            for (int e = 0; e < NH; ++e) hv[e] = f[g.hg[e] + kz1 * X.nxy];
        }
    }
    __device__ __forceinline__ void shift() {
#pragma unroll
        for (int t = 0; t < NW - 1; ++t) w[t] = w[t + 1];
        w[NW - 1] = wn;
    }
    __device__ __forceinline__ double at(int o) const { return w[o - WLO]; }
    __device__ __forceinline__ double x(int o) const { return pl[c0 + o]; }
    __device__ __forceinline__ double y(int o) const { return pl[c0 + o * G::W]; }
};

// A stream for first differences along AX only (UP: as dtile)
template <int M, int AX, int UP>
using DStream = ZStream<AX == 0 ? M : 0, AX == 1 ? M : 0, AX == 2 ? UP - M : 0, AX == 2 ? M - 1 + UP : 0>;

// sum_m a_m (f[+m-1+UP] - f[-m+UP]) along axis AX (UP = 1: dup, UP = 0: ddn), from the staged
// plane (x, y) or the z window
template <int M, int AX, int UP>
__device__ __forceinline__ double dtile(const DStream<M, AX, UP>& st, const double* a) {
    double s = 0.0;
#pragma unroll
    for (int m = 1; m <= M; ++m) {
        const int hi = m - 1 + UP, lo = -m + UP;
        if constexpr (AX == 2)
            s += a[m - 1] * (st.at(hi) - st.at(lo));
        else if constexpr (AX == 1)
            s += a[m - 1] * (st.y(hi) - st.y(lo));
        else
            s += a[m - 1] * (st.x(hi) - st.x(lo));
    }
    return s;
}

// rhs = B + alpha beta s lap B - dt curl+ E + alpha c^2 mu0 dt^2 curl+ J   (B = B^n), B^n's copy and
// sweep 1
template <int M, int C, bool STREAM>
__device__ __forceinline__ void rhs_tiled_comp(const FieldDesc& D, const TileCtx& X, double* lds) {
    constexpr int R = 2 * M - 1;
    constexpr int d1 = (C + 1) % 3, d2 = (C + 2) % 3;
    const FieldGeom& G = D.G;
    ZStream<R, R, -R, R> sB;
    DStream<M, d1, 1> sEu, sJu;  // E_d2, J_d2 along d1
    DStream<M, d2, 1> sEv, sJv;  // E_d1, J_d1 along d2
    double* Bn = gl(D.Bn) + C * G.nc;
    double* x1 = D.sweeps > 1 ? gl(D.Bw) + C * G.nc : nullptr;
    const double w1 = gl(D.omega)[1];
    sB.init(D.B + C * G.nc, X, G, lds);
    sEu.init(D.E + d2 * G.nc, X, G, lds);
    sEv.init(D.E + d1 * G.nc, X, G, lds);
    sJu.init(D.J + d2 * G.nc, X, G, lds);
    sJv.init(D.J + d1 * G.nc, X, G, lds);
    for (int kz = X.z0; kz < X.z1; ++kz) {
        if (kz > X.z0) __syncthreads();  // the previous plane's LDS reads are done
        sB.stage();
        sEu.stage();
        sEv.stage();
        sJu.stage();
        sJv.stage();
        __syncthreads();
        const bool more = kz + 1 < X.z1;
        if (more) {
            sB.prefetch(kz + 1, X);
            sEu.prefetch(kz + 1, X);
            sEv.prefetch(kz + 1, X);
            sJu.prefetch(kz + 1, X);
            sJv.prefetch(kz + 1, X);
        }
        if (X.valid) {
            double lp = 0.0;
#pragma unroll
            for (int o = -R; o <= R; ++o) {
                lp += G.L[0][o + R] * sB.x(o);
                lp += G.L[1][o + R] * sB.y(o);
                lp += G.L[2][o + R] * sB.at(o);
            }
            const double curlE = dtile<M, d1, 1>(sEu, G.a[d1]) - dtile<M, d2, 1>(sEv, G.a[d2]);
            const double curlJ = dtile<M, d1, 1>(sJu, G.a[d1]) - dtile<M, d2, 1>(sJv, G.a[d2]);
            const double xq = sB.at(0);
            const double rq = xq + D.cab * lp - D.dt * curlE + D.cj * curlJ;
            const int64_t q = X.own + (int64_t)kz * X.nxy;
            store_once<STREAM>(rq, gl(D.R) + C * G.nc + q);
            store_once<STREAM>(xq, Bn + q);
            if (x1) {  // sweep 1
                const double Ax = xq - D.al2s * lp;
                const double y = xq + (rq - Ax) * D.gdiag;
                store_once<STREAM>(xq + w1 * (y - xq), x1 + q);
            }
        }
        if (more) {
            sB.shift();
            sEu.shift();
            sEv.shift();
            sJu.shift();
            sJv.shift();
        }
    }
}

// E += c^2 dt (curl- (alpha B' + beta B) - mu0 J)
template <int M, int C, bool STREAM>
__device__ __forceinline__ void update_E_tiled_comp(const FieldDesc& D, const TileCtx& X, double* lds) {
    constexpr int d1 = (C + 1) % 3, d2 = (C + 2) % 3;
    const FieldGeom& G = D.G;
    DStream<M, d1, 0> sBu, sNu;  // B_d2, Bn_d2 along d1
    DStream<M, d2, 0> sBv, sNv;  // B_d1, Bn_d1 along d2
    ZStream<0, 0, 0, 0> sE, sJ;
    sBu.init(D.B + d2 * G.nc, X, G, lds);
    sBv.init(D.B + d1 * G.nc, X, G, lds);
    sNu.init(D.Bn + d2 * G.nc, X, G, lds);
    sNv.init(D.Bn + d1 * G.nc, X, G, lds);
    sE.init(D.E + C * G.nc, X, G, lds);
    sJ.init(D.J + C * G.nc, X, G, lds);
    for (int kz = X.z0; kz < X.z1; ++kz) {
        if (kz > X.z0) __syncthreads();
        sBu.stage();
        sBv.stage();
        sNu.stage();
        sNv.stage();
        __syncthreads();
        const bool more = kz + 1 < X.z1;
        if (more) {
            sBu.prefetch(kz + 1, X);
            sBv.prefetch(kz + 1, X);
            sNu.prefetch(kz + 1, X);
            sNv.prefetch(kz + 1, X);
            sE.prefetch(kz + 1, X);
            sJ.prefetch(kz + 1, X);
        }
        if (X.valid) {
            const double cn = dtile<M, d1, 0>(sBu, G.a[d1]) - dtile<M, d2, 0>(sBv, G.a[d2]);
            const double co = dtile<M, d1, 0>(sNu, G.a[d1]) - dtile<M, d2, 0>(sNv, G.a[d2]);
            store_once<STREAM>(sE.at(0) + D.c2dt * (D.al * cn + D.be * co - D.mu0 * sJ.at(0)),
                               gl(D.E) + C * G.nc + X.own + (int64_t)kz * X.nxy);
        }
        if (more) {
            sBu.shift();
            sBv.shift();
            sNu.shift();
            sNv.shift();
            sE.shift();
            sJ.shift();
        }
    }
}

enum FieldKind { FK_RHS = 0, FK_RELAX = 1, FK_UPDATE_E = 2 };

// LDS of a phase (doubles): the Laplacian's plane, and the curl's planes of the component with the
// most (the one whose curl runs along x and y)
template <int M>
constexpr int field_lds(int kind) {
    constexpr int R = 2 * M - 1;
    constexpr int lap = Ring<R, R>::W * Ring<R, R>::H;
    constexpr int dx = DStream<M, 0, 1>::LDS, dy = DStream<M, 1, 1>::LDS;
    return kind == FK_RELAX ? lap : (kind == FK_RHS ? lap : 0) + 2 * (dx + dy);
}

// ---- the field step, a thread per cell and component ------------------------------------
// For boxes that the columns fit badly (see thin_box): every tap read through the caches, the
// sums in the tiled kernels' order.
template <int M, int UP>
__device__ __forceinline__ double dcell(const FieldGeom& G, const double* f, int ax, int i, int j, int k) {
    const int c[3] = {i, j, k};
    const int stride = ax == 0 ? 1 : (ax == 1 ? G.n[0] : G.n[0] * G.n[1]);
    const double* line = f + (lin(G, i, j, k) - c[ax] * stride);
    double s = 0.0;
#pragma unroll
    for (int m = 1; m <= M; ++m)
        s += G.a[ax][m - 1] * (line[nbw(c[ax], m - 1 + UP, G.n[ax], G.small) * stride] -
                               line[nbw(c[ax], -m + UP, G.n[ax], G.small) * stride]);
    return s;
}

template <int R>
__device__ __forceinline__ double lap_cell(const FieldGeom& G, const double* f, int i, int j, int k) {
    const int nx = G.n[0], nxy = G.n[0] * G.n[1];
    const double *fx = f + nx * (j + G.n[1] * k), *fy = f + (i + nxy * k), *fz = f + (i + nx * j);
    double s = 0.0;
#pragma unroll
    for (int o = -R; o <= R; ++o) {
        s += G.L[0][o + R] * fx[nbw(i, o, nx, G.small)];
        s += G.L[1][o + R] * fy[nx * nbw(j, o, G.n[1], G.small)];
        s += G.L[2][o + R] * fz[nxy * nbw(k, o, G.n[2], G.small)];
    }
    return s;
}

template <int M, int KIND>
__device__ __forceinline__ void field_cells(const FieldDesc& D, int b, int k) {
    constexpr int R = 2 * M - 1;
    const FieldGeom& G = D.G;
    const int blocks = G.xchunks * ((G.rows + G.rpb - 1) / G.rpb);
    const int C = b / blocks, d1 = C == 2 ? 0 : C + 1, d2 = C == 0 ? 2 : C - 1;
    int i, j, z;
    if (!field_cell(G, b - C * blocks, threadIdx.x, i, j, z)) return;
    const int64_t co = C * G.nc, q = co + lin(G, i, j, z);
    if constexpr (KIND == FK_RELAX) {
        const double* x = gl(k == 1 ? D.Bn : relax_array(D, k - 1)) + co;
        const double pq = gl(k <= 2 ? D.Bn : relax_array(D, k - 2))[q], xq = x[q - co], w = gl(D.omega)[k];
        const double Ax = xq - D.al2s * lap_cell<R>(G, x, i, j, z);
        const double y = xq + (gl(D.R)[q] - Ax) * D.gdiag;
        gl(relax_array(D, k))[q] = pq + w * (y - pq);
    } else if constexpr (KIND == FK_RHS) {
        const double *E1 = gl(D.E) + d1 * G.nc, *E2 = gl(D.E) + d2 * G.nc;
        const double *J1 = gl(D.J) + d1 * G.nc, *J2 = gl(D.J) + d2 * G.nc;
        const double* x = gl(D.B) + co;
        const double lp = lap_cell<R>(G, x, i, j, z);
        const double curlE = dcell<M, 1>(G, E2, d1, i, j, z) - dcell<M, 1>(G, E1, d2, i, j, z);
        const double curlJ = dcell<M, 1>(G, J2, d1, i, j, z) - dcell<M, 1>(G, J1, d2, i, j, z);
        const double xq = x[q - co];
        const double rq = xq + D.cab * lp - D.dt * curlE + D.cj * curlJ;
        gl(D.R)[q] = rq;
        gl(D.Bn)[q] = xq;
        if (D.sweeps > 1) {  // sweep 1
            const double Ax = xq - D.al2s * lp;
            const double y = xq + (rq - Ax) * D.gdiag;
            gl(D.Bw)[q] = xq + gl(D.omega)[1] * (y - xq);
        }
    } else {
        const double *B1 = gl(D.B) + d1 * G.nc, *B2 = gl(D.B) + d2 * G.nc;
        const double *N1 = gl(D.Bn) + d1 * G.nc, *N2 = gl(D.Bn) + d2 * G.nc;
        const double cn = dcell<M, 0>(G, B2, d1, i, j, z) - dcell<M, 0>(G, B1, d2, i, j, z);
        const double co_ = dcell<M, 0>(G, N2, d1, i, j, z) - dcell<M, 0>(G, N1, d2, i, j, z);
        gl(D.E)[q] = gl(D.E)[q] + D.c2dt * (D.al * cn + D.be * co_ - D.mu0 * gl(D.J)[q]);
    }
}

template <int M, int KIND>
__global__ void __launch_bounds__(FIELD_BS) k_field_cells(FieldDesc D, int k) {
    field_cells<M, KIND>(D, (int)blockIdx.x, k);
}

// block b of a run's launch of one phase (k: the sweep)
template <int M, int KIND, bool STREAM>
__device__ __forceinline__ void field_tile(const FieldDesc& D, int b, int k, double* lds) {
    if constexpr (KIND == FK_RELAX) {
        relax_tile<2 * M - 1, STREAM>(D, b, k, lds);
    } else {
        TileCtx X;
        tile_ctx(D.G, D.zc, b, X);
        if constexpr (KIND == FK_RHS) {
            if (X.comp == 0)
                rhs_tiled_comp<M, 0, STREAM>(D, X, lds);
            else if (X.comp == 1)
                rhs_tiled_comp<M, 1, STREAM>(D, X, lds);
            else
                rhs_tiled_comp<M, 2, STREAM>(D, X, lds);
        } else {
            if (X.comp == 0)
                update_E_tiled_comp<M, 0, STREAM>(D, X, lds);
            else if (X.comp == 1)
                update_E_tiled_comp<M, 1, STREAM>(D, X, lds);
            else
                update_E_tiled_comp<M, 2, STREAM>(D, X, lds);
        }
    }
}

// The launch order of a phase's blocks.  A sweep's blocks side by side on an XCD share the planes
// around them in its L2 (128^3: 47 us against 59).  In the other two phases a field is read for two
// components: in boxes large enough for marches (zc > 1) a tile's three blocks are launched one
// after the other on an XCD, which takes the tiles of a contiguous eighth of the box (E update
// 256^3 603 -> 503 us, 128^3 72 -> 64; right-hand side 128^3 107 -> 103 and 256^3 the same; the
// contiguous eighths without a tile's components together take 256^3 from 0.97 to 1.07 ms).
// Smaller boxes gain nothing from it (128x32x32: 97.5 us a step, 98.7 with it).
__host__ __device__ __forceinline__ bool components_together(int kind, int zc) { return kind != FK_RELAX && zc > 1; }

// Four workgroups a CU for the right-hand side, at 125 registers instead of 137 and three (256^3:
// 797 -> 779 us, 128^3 107 -> 103).
template <int M, int KIND, bool STREAM>
__global__ void __launch_bounds__(RX_BS, KIND == FK_RHS ? 4 : 1) k_field_tiles(FieldDesc D, int k, int blocks) {
    __shared__ double lds[field_lds<M>(KIND)];
    int b = (int)blockIdx.x;
    if (KIND == FK_RELAX) {
        b = (int)xcd_block(blockIdx.x, blocks);
    } else if (components_together(KIND, D.zc)) {
        const int tiles = blocks / 3, comp = (b >> 3) % 3;
        const int t = (int)xcd_block((b & 7) + 8 * (int64_t)(b / 24), tiles);
        b = t >= 0 ? comp * tiles + t : -1;
    }
    if (b >= 0) field_tile<M, KIND, STREAM>(D, b, k, lds);
}

// batched: block b belongs to run r with prefix[r] <= b < prefix[r+1] (prefix in blocks)
template <int KIND>
__global__ void __launch_bounds__(RX_BS) k_field_tiles_batch(const FieldDesc* __restrict__ T,
                                                             const int64_t* __restrict__ prefix, int nruns, int k) {
    __shared__ double lds[field_lds<3>(KIND)];
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, nruns, b);
    if (r < 0) return;
    const FieldDesc& D = T[r];
    if (KIND == FK_RELAX && (k > D.sweeps || (k == 1 && D.sweeps > 1))) return;
    const int lb = (int)(b - prefix[r]);
    if (D.zc == 0) return;  // k_field_cells_batch
    if (D.G.M == 3)
        field_tile<3, KIND, false>(D, lb, k, lds);
    else if (D.G.M == 2)
        field_tile<2, KIND, false>(D, lb, k, lds);
    else
        field_tile<1, KIND, false>(D, lb, k, lds);
}

// the same launch for the members with a thread per cell
template <int KIND>
__global__ void __launch_bounds__(FIELD_BS) k_field_cells_batch(const FieldDesc* __restrict__ T,
                                                                const int64_t* __restrict__ prefix, int nruns, int k) {
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, nruns, b);
    if (r < 0) return;
    const FieldDesc& D = T[r];
    if (D.zc != 0 || (KIND == FK_RELAX && (k > D.sweeps || (k == 1 && D.sweeps > 1)))) return;
    const int lb = (int)(b - prefix[r]);
    if (D.G.M == 3)
        field_cells<3, KIND>(D, lb, k);
    else if (D.G.M == 2)
        field_cells<2, KIND>(D, lb, k);
    else
        field_cells<1, KIND>(D, lb, k);
}

// One phase of a batch, nthin of whose n members take a thread per cell.
template <int KIND>
static void launch_field_batch(const FieldDesc* T, const int64_t* prefix, int n, int nthin, unsigned blocks, int k,
                               hipStream_t st) {
    if (nthin < n)
        hipLaunchKernelGGL(k_field_tiles_batch<KIND>, dim3(blocks), dim3(RX_BS), 0, st, T, prefix, n, k);
    if (nthin > 0)
        hipLaunchKernelGGL(k_field_cells_batch<KIND>, dim3(blocks), dim3(FIELD_BS), 0, st, T, prefix, n, k);
}

// The whole relaxation of a small box, a workgroup per component: the current iterate in LDS
// (two buffers, so one barrier a sweep), the one before last and the right-hand side in registers.
// A sweep by launch costs 3.4 us at least; here 4096 cells of the 2nd-order stencil take 1.3, but
// on one CU the work of a wider stencil or a larger box soon costs more than the launch it saves.
constexpr int RS_BS = 1024, RS_CELLS = 4 * RS_BS;

static bool relax_in_lds(const FieldGeom& G) { return G.nc * G.R <= RS_CELLS; }

template <int R>
__global__ void __launch_bounds__(RS_BS) k_relax_small(FieldDesc D) {
    constexpr int PER = (RS_CELLS / R + RS_BS - 1) / RS_BS;
    __shared__ double buf[2][PER * RS_BS];
    const FieldGeom& G = D.G;
    const int nc = (int)G.nc, n0 = G.n[0], n1 = G.n[1], n2 = G.n[2], nxy = n0 * n1;
    const int64_t co = (int64_t)blockIdx.x * G.nc;
    int k = D.sweeps > 1 ? 2 : 1;
    const double* x = (k == 1 ? D.Bn : relax_array(D, k - 1)) + co;
    double p[PER], rq[PER];
    int nb[PER][3][2 * R];  // LDS entries of the taps, the same in every sweep
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        const int q = threadIdx.x + c * RS_BS, qc = q < nc ? q : 0;
        buf[0][q] = x[qc];
        p[c] = D.Bn[co + qc];
        rq[c] = D.R[co + qc];
        const int kz = qc / nxy, r = qc - kz * nxy, j = r / n0, i = r - j * n0;
#pragma unroll
        for (int t = 0; t < 2 * R; ++t) {
            const int o = t < R ? t - R : t - R + 1;
            nb[c][0][t] = qc - i + nbw(i, o, n0, G.small);
            nb[c][1][t] = qc + (nbw(j, o, n1, G.small) - j) * n0;
            nb[c][2][t] = qc + (nbw(kz, o, n2, G.small) - kz) * nxy;
        }
    }
    for (int cur = 0; k <= D.sweeps; ++k, cur ^= 1) {
        const double w = D.omega[k];
        __syncthreads();
        const double* b = buf[cur];
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int q = threadIdx.x + c * RS_BS;  // entries past the box take part and are not kept
            const double xq = b[q];
            double sl = 0.0;
#pragma unroll
            for (int t = 0; t <= 2 * R; ++t)
#pragma unroll
                for (int ax = 0; ax < 3; ++ax)
                    sl += G.L[ax][t] * (t == R ? xq : b[nb[c][ax][t < R ? t : (t == R ? 0 : t - 1)]]);
            const double Ax = xq - D.al2s * sl;
            const double y = xq + (rq[c] - Ax) * D.gdiag;
            const double xn = p[c] + w * (y - p[c]);
            buf[cur ^ 1][q] = xn;
            p[c] = xq;
            if (k == D.sweeps && q < nc) D.B[co + q] = xn;
        }
    }
}

static void launch_relax_small(const FieldDesc& D, hipStream_t st) {
    if (D.G.R == 5)
        hipLaunchKernelGGL(k_relax_small<5>, dim3(3), dim3(RS_BS), 0, st, D);
    else if (D.G.R == 3)
        hipLaunchKernelGGL(k_relax_small<3>, dim3(3), dim3(RS_BS), 0, st, D);
    else
        hipLaunchKernelGGL(k_relax_small<1>, dim3(3), dim3(RS_BS), 0, st, D);
}

// Boxes whose four arrays of a sweep are far larger than the 256 MB of the last cache: they come from
// memory in every pass, and what is touched once only drives out what a neighbouring block reads
// again.  Field step with all accesses cached -> this, ms: 256^3 (1.6 GB) 4.77 -> 4.51, 192^3 2.07 -> 1.92
// and at 4th order 2.00 -> 1.79, 160^3 (393 MB) 1.265 -> 1.243.  Smaller boxes find part of the arrays in
// the cache: 152^3 (337 MB) 1.07 -> 1.23, 128^3 0.60 -> 0.68.
static bool streams_past_cache(const FieldGeom& G) { return 4 * 3 * G.nc * (int64_t)sizeof(double) > (352ll << 20); }

template <int KIND, bool STREAM>
static void launch_field_order(const FieldDesc& D, dim3 grid, unsigned blocks, int k, hipStream_t st) {
    if (D.G.M == 3)
        hipLaunchKernelGGL((k_field_tiles<3, KIND, STREAM>), grid, dim3(RX_BS), 0, st, D, k, (int)blocks);
    else if (D.G.M == 2)
        hipLaunchKernelGGL((k_field_tiles<2, KIND, STREAM>), grid, dim3(RX_BS), 0, st, D, k, (int)blocks);
    else
        hipLaunchKernelGGL((k_field_tiles<1, KIND, STREAM>), grid, dim3(RX_BS), 0, st, D, k, (int)blocks);
}

template <int KIND>
static void launch_field_tiles(const FieldDesc& D, unsigned blocks, int k, hipStream_t st) {
    if (D.zc == 0) {
        if (D.G.M == 3)
            hipLaunchKernelGGL((k_field_cells<3, KIND>), dim3(blocks), dim3(FIELD_BS), 0, st, D, k);
        else if (D.G.M == 2)
            hipLaunchKernelGGL((k_field_cells<2, KIND>), dim3(blocks), dim3(FIELD_BS), 0, st, D, k);
        else
            hipLaunchKernelGGL((k_field_cells<1, KIND>), dim3(blocks), dim3(FIELD_BS), 0, st, D, k);
        return;
    }
    const dim3 grid(KIND == FK_RELAX                  ? xcd_grid(blocks)
                    : components_together(KIND, D.zc) ? 3 * xcd_grid(blocks / 3)
                                                      : blocks);
    if (streams_past_cache(D.G))
        launch_field_order<KIND, true>(D, grid, blocks, k, st);
    else
        launch_field_order<KIND, false>(D, grid, blocks, k, st);
}

// Boxes that leave most of their columns' threads without a cell, or are only a few cells wide, so that a
// column's rows are partial lines: a thread per cell (the same in a batch as alone).  Field step, us, 32x8
// columns -> cells, orders 2 and 6: 2x300x300 387 -> 111 and 595 -> 245; 8x300x300 417 -> 237, 584 -> 500;
// 512x1x512 236 -> 98, 409 -> 275; 1000000x1x1 1498 -> 213, 3505 -> 788; 10x10x300 88 -> 69, 123 -> 94; on the
// other side of the line 512x2x512 at 4th and 6th order 374 and 469 against 376 and 529, 12x300x300 478 and 591
// against 617 and 887, 33x33x33 82 and 87 against 88 and 111.
static bool thin_box(const int n[3], int order) {
    const int64_t cells = (int64_t)n[0] * n[1];
    const int64_t threads = (int64_t)RX_BS * ((n[0] + RX_TX - 1) / RX_TX) * ((n[1] + RX_TY - 1) / RX_TY);
    return n[0] <= 8 || 5 * cells <= threads || (4 * cells <= threads && (order == 2 || n[2] <= 8));
}

// Planes per block: as many as leave the launch about 8 blocks per CU (its share of them in a
// batch of nruns), so that small boxes fill the GPU, and at most RX_ZC, where reading the
// stencil's planes above and below once per block costs little.  0: a thread per cell.
static int planes_per_block(const pp_run* r, int nruns) {
    const int* n = r->p.n;
    if (thin_box(n, r->p.field_order)) return 0;
    const int64_t cols = 3 * (int64_t)((n[0] + RX_TX - 1) / RX_TX) * ((n[1] + RX_TY - 1) / RX_TY);
    const int64_t zc = cols * n[2] * nruns / 2048;
    return (int)(zc < 1 ? 1 : (zc > RX_ZC ? RX_ZC : zc));
}

static void fd_coeffs(int order, double a[3]) {
    a[0] = a[1] = a[2] = 0.0;
    if (order == 2) {
        a[0] = 1.0;
    } else if (order == 4) {
        a[0] = 9.0 / 8.0;
        a[1] = -1.0 / 24.0;
    } else {
        // 6th order; the normalisation a + 3b + 5c = 1 fixes a = 75/64
        a[0] = 75.0 / 64.0;
        a[1] = -25.0 / 384.0;
        a[2] = 3.0 / 640.0;
    }
}

static FieldGeom make_geom(const pp_run* r) {
    FieldGeom G{};
    for (int d = 0; d < 3; ++d) G.n[d] = r->p.n[d];
    G.nc = r->g.ncell;
    G.M = r->p.field_order / 2;
    double a[3];
    fd_coeffs(r->p.field_order, a);
    for (int d = 0; d < 3; ++d)
        for (int m = 0; m < 3; ++m) G.a[d][m] = a[m] / r->p.d[d];
    G.R = r->lap_r;
    for (int d = 0; d < 3; ++d)
        for (int o = 0; o < 2 * G.R + 1; ++o) G.L[d][o] = r->lap[d][o];
    const int nx = G.n[0];
    if (nx >= FIELD_BS) {
        G.xbits = 8;
        G.xchunks = (nx + FIELD_BS - 1) / FIELD_BS;
        G.rpb = 1;
    } else {
        G.xbits = 0;
        while ((1 << G.xbits) < nx) ++G.xbits;
        G.xchunks = 1;
        G.rpb = FIELD_BS >> G.xbits;
    }
    G.rows = G.n[1] * G.n[2];
    G.inv_ny = 1.0 / G.n[1];
    G.small = 0;
    for (int d = 0; d < 3; ++d)
        if (G.n[d] < G.R || G.n[d] < G.M) G.small = 1;
    return G;
}

template <class GEOM>
static int64_t blocks_of(const GEOM& G) { return (int64_t)G.xchunks * ((G.rows + G.rpb - 1) / G.rpb); }

bool field_by_cells(const pp_run* r) { return thin_box(r->p.n, r->p.field_order); }

// Blocks of one phase of a run's field step, in a batch of nruns.
int64_t field_blocks(const pp_run* r, int nruns) {
    const int* n = r->p.n;
    const int zc = planes_per_block(r, nruns);
    if (zc == 0) return 3 * blocks_of(make_geom(r));
    return 3 * (int64_t)((n[0] + RX_TX - 1) / RX_TX) * ((n[1] + RX_TY - 1) / RX_TY) * ((n[2] + zc - 1) / zc);
}

// Host set-up of the field-step constants: the composed Laplacian stencil (d- after d+,
// identical as a stencil to d+ after d-), the true diagonal of A = 1 - alpha^2 s lap on this
// periodic grid, and the relaxation.  A is circulant, so the Jacobi iteration matrix
// G = 1 - A / diag has its spectrum in [g0, g1] = [1 - amax/diag, 1 - 1/diag] exactly (amax
// the largest eigenvalue of A, from the stencil's symbol).  The relaxation is Jacobi
// extrapolated by gamma = 2 / (2 - g0 - g1), which centres that interval on 0 with radius
// r = (g1 - g0) / (2 - g0 - g1), and accelerated by Chebyshev semi-iteration (Golub and
// Varga 1961): after m sweeps the error is multiplied by at most 1 / T_m(1/r) (T_m the
// Chebyshev polynomial) and the residual by at most amax / T_m(1/r); m is the smallest
// count for which that is <= relax_tol.
static void relax_setup(pp_run* r, double dt, pp_run::RelaxSet& S, double* om);

void field_setup(pp_run* r, double* consts) {
    double a[3];
    fd_coeffs(r->p.field_order, a);
    const int M = r->p.field_order / 2;
    const int R = 2 * M - 1;
    r->lap_r = R;
    for (int d = 0; d < 3; ++d) {
        for (int o = 0; o < 16; ++o) r->lap[d][o] = 0.0;
        const double id2 = 1.0 / (r->p.d[d] * r->p.d[d]);
        for (int m = 1; m <= M; ++m)
            for (int mp = 1; mp <= M; ++mp) {
                double cf = a[m - 1] * a[mp - 1] * id2;
                r->lap[d][(m + mp - 1) + R] += cf;
                r->lap[d][(m - mp) + R] -= cf;
                r->lap[d][(-m + mp) + R] -= cf;
                r->lap[d][(-m - mp + 1) + R] += cf;
            }
    }
    // Gauss-law filter damping: 1 / max over the grid's wave numbers of sum_d K_d^2, K_d the
    // symbol (2/d) sum_m a_m sin((m - 1/2) k) of the field-order first derivative
    double kmax2 = 0.0;
    for (int d = 0; d < 3; ++d) {
        const int N = r->p.n[d];
        double best = 0.0;
        for (int mm = 0; mm < N; ++mm) {
            const double k = 2.0 * M_PI * mm / N;
            double sym = 0.0;
            for (int l = 1; l <= M; ++l) sym += a[l - 1] * sin((l - 0.5) * k);
            sym *= 2.0 / r->p.d[d];
            best = sym * sym > best ? sym * sym : best;
        }
        kmax2 += best;
    }
    r->gauss_kappa = kmax2 > 0.0 ? 1.0 / kmax2 : 0.0;
    // relaxation constants for each drift size the run steps with
    const double drifts[3] = {r->p.dt, FR_DRIFT[0] * r->p.dt, FR_DRIFT[2] * r->p.dt};
    for (int k = 0; k < r->nrs; ++k) relax_setup(r, drifts[k], r->rs[k], consts + (r->rs[k].omega - r->consts));
    use_relax_set(r, 0);
    r->dt_kick = r->dt_drift = r->p.dt;
}

// Relaxation constants of one drift size dt (the operator depends on dt^2 only); om: its weights.
static void relax_setup(pp_run* r, double dt, pp_run::RelaxSet& S, double* om) {
    const int R = r->lap_r;
    const double s = r->p.c * r->p.c * dt * dt;
    const double al2s = r->p.alpha * r->p.alpha * s;
    double diag = 1.0, amax = 1.0, min_sym[3];
    for (int d = 0; d < 3; ++d) {
        const int N = r->p.n[d];
        double fold0 = 0.0;
        for (int o = -R; o <= R; ++o)
            if (((o % N) + N) % N == 0) fold0 += r->lap[d][o + R];
        diag -= al2s * fold0;
        double mn = 0.0;
        int same = -1;  // an axis before with the same stencil and length: the same minimum
        for (int e = 0; e < d; ++e)
            if (r->p.n[e] == N && r->p.d[e] == r->p.d[d]) same = e;
        for (int mm = 0; same < 0 && mm < N; ++mm) {
            double k = 2.0 * M_PI * mm / N, sym = 0.0, cs[16];
            for (int o = 0; o <= R; ++o) cs[o] = cos(o * k);  // cos(-o k) is the same value
            for (int o = -R; o <= R; ++o) sym += r->lap[d][o + R] * cs[o < 0 ? -o : o];
            if (sym < mn) mn = sym;
        }
        min_sym[d] = mn = same < 0 ? mn : min_sym[same];
        amax -= al2s * mn;
    }
    S.drift = dt;
    S.diagA = diag;
    const double g0 = 1.0 - amax / diag, g1 = 1.0 - 1.0 / diag;
    S.jac_rho = fmax(fabs(g0), fabs(g1));
    S.gamma = 2.0 / (2.0 - g0 - g1);
    const double rr = (g1 - g0) / (2.0 - g0 - g1);
    S.r = rr;
    // The paper relaxes until the residual is small (Sec. III.B).  After k sweeps the error is
    // reduced by at most 1/cosh(k acosh(1/r)) (Chebyshev); the residual rhs - A B_k = A e_k is
    // then reduced by at most that times the condition number of A, whose eigenvalues lie in
    // [1, amax] (1 - al2s lap with lap <= 0; the constant mode has eigenvalue 1).  The sweep
    // count is the smallest whose residual bound reaches relax_tol.
    const double kappa = amax;
    int sweeps = 1;
    double bound = 0.0;
    if (rr > 1e-300) {
        const double ac = acosh(1.0 / rr);
        for (sweeps = 1; sweeps < r->p.relax_max_iter; ++sweeps)
            if (kappa / cosh(sweeps * ac) <= r->p.relax_tol) break;
        bound = kappa / cosh(sweeps * ac);
    }
    S.sweeps = sweeps;
    S.bound = bound;
    S.converged = bound <= r->p.relax_tol;
    // omega_1 = 1, omega_2 = 1 / (1 - r^2/2), omega_{k+1} = 1 / (1 - r^2 omega_k / 4)
    const int n_om = r->p.relax_max_iter + 2;
    om[0] = 0.0;
    om[1] = 1.0;
    for (int k = 2; k < n_om; ++k) om[k] = k == 2 ? 1.0 / (1.0 - 0.5 * rr * rr) : 1.0 / (1.0 - 0.25 * rr * rr * om[k - 1]);
}

void use_relax_set(pp_run* r, int k) {
    const pp_run::RelaxSet& S = r->rs[k];
    r->diagA = S.diagA;
    r->jac_rho = S.jac_rho;
    r->relax_gamma = S.gamma;
    r->relax_r = S.r;
    r->jac_sweeps = S.sweeps;
    r->jac_bound = S.bound;
    r->jac_converged = S.converged;
    r->omega = S.omega;
    r->dt_drift = S.drift;
}

void field_desc(const pp_run* r, FieldDesc* D, int nruns) {
    D->G = make_geom(r);
    const double c2 = r->p.c * r->p.c, dt = r->dt_drift, s = c2 * dt * dt;
    const double al = r->p.alpha, be = 1.0 - al;
    const double mu0 = 1.0 / (r->p.eps0 * c2);
    D->E = r->mesh.E;
    D->B = r->mesh.B;
    D->J = r->mesh.J;
    D->Bn = r->Bn;
    D->Bw = r->Bw;
    D->Bx = r->J2;
    D->R = r->R;
    D->omega = r->omega;
    D->rho = r->rho;
    D->rho_bg = r->p.rho_background;
    D->ieps0 = 1.0 / r->p.eps0;
    D->kappa = r->gauss_kappa;
    D->cab = al * be * s;
    D->dt = dt;
    D->cj = al * c2 * mu0 * dt * dt;
    D->al2s = al * al * s;
    D->gdiag = r->relax_gamma / r->diagA;
    D->al = al;
    D->be = be;
    D->c2dt = c2 * dt;
    D->mu0 = mu0;
    D->sweeps = r->jac_sweeps;
    D->zc = planes_per_block(r, nruns);
}

size_t field_desc_size() { return sizeof(FieldDesc); }

hipError_t launch_field_step(pp_run* r) {
    FieldDesc D;
    field_desc(r, &D, 1);
    const unsigned blocks = (unsigned)field_blocks(r, 1);
    launch_field_tiles<FK_RHS>(D, blocks, 0, r->stream);
    if (relax_in_lds(D.G))
        launch_relax_small(D, r->stream);
    else
        for (int k = D.sweeps > 1 ? 2 : 1; k <= D.sweeps; ++k) launch_field_tiles<FK_RELAX>(D, blocks, k, r->stream);
    launch_field_tiles<FK_UPDATE_E>(D, blocks, 0, r->stream);
    note_relax_rhs(r);
    return hipGetLastError();
}

void note_relax_rhs(pp_run* r) {
    const double c2 = r->p.c * r->p.c, dt = r->dt_drift;
    r->rhs_valid = true;
    r->rhs_al2s = r->p.alpha * r->p.alpha * c2 * dt * dt;
}

// Residual of the relaxation actually reached (Sec. III.B: the paper relaxes to a residual):
// per cell and component r = R - (B - al2s lap B) with R the stored right-hand side, reduced
// to max |r| and max |R| (non-negative doubles compared as their bit patterns).
__device__ __forceinline__ void max_bits(double v, double* acc) {
    atomicMax((unsigned long long*)acc, (unsigned long long)__double_as_longlong(v));
}

__global__ void __launch_bounds__(FIELD_BS) k_relax_resid(FieldGeom G, const double* __restrict__ B,
                                                          const double* __restrict__ R, double al2s, double* acc) {
    __shared__ double red[2][FIELD_BS / 64];
    double rmax = 0.0, hmax = 0.0;
    int i, j, k;
    if (field_cell(G, blockIdx.x, threadIdx.x, i, j, k)) {
        const int q = lin(G, i, j, k);
        for (int c = 0; c < 3; ++c) {
            const double* x = B + c * G.nc;
            const double rhs = R[c * G.nc + q];
            const double Ax = x[q] - al2s * lap(G, x, i, j, k);
            rmax = fmax(rmax, fabs(rhs - Ax));
            hmax = fmax(hmax, fabs(rhs));
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        rmax = fmax(rmax, __shfl_xor(rmax, o));
        hmax = fmax(hmax, __shfl_xor(hmax, o));
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = rmax;
        red[1][threadIdx.x >> 6] = hmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < FIELD_BS / 64; ++w) {
            rmax = fmax(rmax, red[0][w]);
            hmax = fmax(hmax, red[1][w]);
        }
        max_bits(rmax, acc);
        max_bits(hmax, acc + 1);
    }
}

hipError_t launch_relax_resid(pp_run* r, double* acc) {
    const FieldGeom G = make_geom(r);
    hipLaunchKernelGGL(k_relax_resid, dim3((unsigned)blocks_of(G)), dim3(FIELD_BS), 0, r->stream, G,
                       (const double*)r->mesh.B, (const double*)r->R, r->rhs_al2s, acc);
    return hipGetLastError();
}

// Gauss-law filter of a run (after its field step): rho of the current positions, then the
// passes, each a residual launch and a correction launch.
hipError_t launch_gauss_filter(pp_run* r) {
    r->rhs_valid = false;  // the passes keep their residual in R
    hipError_t e = deposit_rho_all(r);
    if (e != hipSuccess) return e;
    FieldDesc D;
    field_desc(r, &D, 1);
    const dim3 grid((unsigned)blocks_of(D.G));
    for (int it = 0; it < r->p.gauss_filter_passes; ++it) {
        hipLaunchKernelGGL(k_field, grid, dim3(FIELD_BS), 0, r->stream, D, (int)PH_GAUSS_RES);
        hipLaunchKernelGGL(k_field, grid, dim3(FIELD_BS), 0, r->stream, D, (int)PH_GAUSS_CORR);
    }
    return hipGetLastError();
}

// Batched field step over n runs: table (device) of FieldDesc, prefix (device) of blocks.
hipError_t launch_field_step_batch(const void* table, const int64_t* prefix, int n, int nthin, int64_t total_blocks,
                                   int min_sweeps, int max_sweeps, hipStream_t st) {
    if (n == 0 || total_blocks == 0) return hipSuccess;
    const FieldDesc* T = (const FieldDesc*)table;
    const unsigned blocks = (unsigned)total_blocks;
    launch_field_batch<FK_RHS>(T, prefix, n, nthin, blocks, 0, st);
    for (int k = min_sweeps > 1 ? 2 : 1; k <= max_sweeps; ++k)
        launch_field_batch<FK_RELAX>(T, prefix, n, nthin, blocks, k, st);
    launch_field_batch<FK_UPDATE_E>(T, prefix, n, nthin, blocks, 0, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// High-order current: on a periodic line the paper's construction (solve T dJ = dJ2 for the
// differences, prefix-sum, keep the line mean) equals J_O = T^{-1} J_2, because the
// high-order down derivative factors as T applied after the second-order one and T keeps
// line means (its symbol is 1 at k = 0).  T^{-1} is circulant with exponentially decaying
// coefficients; it is applied as a convolution along each component's own axis.
// ---------------------------------------------------------------------------------------
struct LineArgs {
    CellGeom G;
    const double* coef[3];
    int len[3], off[3];
    // LDS form: W[c] lines of component c per block (a power of two, at most 64) and the
    // blocks of each component; W[0] == 0 selects the global-memory form
    int W[3];
    int64_t nb[3];
    const double* J2;
    // LDS form of a split run: the fixed-point current, read in J2's place and cleared for the
    // next step (nullptr: J2)
    FixedScale scale;
    unsigned long long* Jq;
    double* J;
};

// Global-memory form (lines too long for the LDS copy): one thread per cell, the stencil
// read through the caches.
__device__ __forceinline__ void line_body(const LineArgs& A, int64_t b) {
    int ijk[3];
    if (!field_cell(A.G, b, threadIdx.x, ijk[0], ijk[1], ijk[2])) return;
    const int nc = (int)A.G.nc;
    const int q = lin(A.G, ijk[0], ijk[1], ijk[2]);
    const int stride[3] = {1, A.G.n[0], A.G.n[0] * A.G.n[1]};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double* src = gl(A.J2) + (int64_t)c * nc;
        const int N = A.G.n[c];
        const int rowbase = q - ijk[c] * stride[c];
        double s = 0.0;
        int idx = ijk[c] + A.off[c];
        idx %= N;
        if (idx < 0) idx += N;
        for (int jj = 0; jj < A.len[c]; ++jj) {
            s += gl(A.coef[c])[jj] * src[rowbase + idx * stride[c]];
            if (++idx == N) idx = 0;
        }
        gl(A.J)[(int64_t)c * nc + q] = s;
    }
}

// LDS form.  A block takes W lines of one component along that component's axis, copies
// each line, extended by the stencil's wrap-around (ext = N + len - 1 values starting at
// offset off), into LDS with coalesced loads, then writes J[j] = sum_t coef[t] ext[j + t].
// x lines are rows (stored line by line, j fastest); y and z lines are taken W consecutive
// x at a time (stored with the W lines interleaved, x fastest), so loads and stores move
// whole rows or W-wide row segments.  A thread takes LINE_OUT consecutive outputs of a line, so
// an LDS value is read once per LINE_OUT outputs it enters; LINE_OUT is odd, so that the lanes of
// an x line, LINE_OUT values apart, fall on different banks.  256^3, 25 taps: 0.26 ms for the
// three components with the fixed-point current read and cleared (0.74 ms for the lines alone
// with one output per thread, and 0.19 for the passes that converted and cleared the current);
// 128x32x32: 12 us (23, and 12 for those passes and the scale's own launch).
constexpr int LINE_LDS_DOUBLES = 4608;  // 36 KiB: 16 lines of 256 cells plus the wrap-around
constexpr int LINE_BATCH = 8;           // loads per thread in flight while a block fills its lines
constexpr int LINE_OUT = 5;

typedef const __attribute__((address_space(4))) double const_f64;
typedef const __attribute__((address_space(1))) double glob_f64;
typedef __attribute__((address_space(1))) unsigned long long glob_u64;

// LINE_OUT outputs from x[0], x[step], ...; each sum in the order of the taps
__device__ __forceinline__ void line_taps(const double* x, int step, const_f64* cf, int len, double acc[LINE_OUT]) {
#pragma unroll
    for (int o = 0; o < LINE_OUT; ++o) acc[o] = 0.0;
    if (len < LINE_OUT) {
        for (int t = 0; t < len; ++t)
#pragma unroll
            for (int o = 0; o < LINE_OUT; ++o) acc[o] += cf[t] * x[(t + o) * step];
        return;
    }
#pragma unroll
    for (int t = 0; t < LINE_OUT - 1; ++t) {
        const double v = x[t * step];
#pragma unroll
        for (int o = 0; o <= t; ++o) acc[o] += cf[t - o] * v;
    }
    for (int t = LINE_OUT - 1; t < len; ++t) {
        const double v = x[t * step];
#pragma unroll
        for (int o = 0; o < LINE_OUT; ++o) acc[o] += cf[t - o] * v;
    }
#pragma unroll
    for (int t = 0; t < LINE_OUT - 1; ++t) {
        const double v = x[(len + t) * step];
#pragma unroll
        for (int o = t + 1; o < LINE_OUT; ++o) acc[o] += cf[len + t - o] * v;
    }
}

// element c of a kernel argument's array, without an address of it (which would move the
// arguments to scratch memory)
template <typename T>
__device__ __forceinline__ T arg3(const T a[3], int c) {
    return c == 0 ? a[0] : (c == 1 ? a[1] : a[2]);
}

__device__ __forceinline__ void line_lds_body(const LineArgs& A, int64_t b, double* e) {
    const CellGeom& G = A.G;
    int c = 0;
    if (b >= A.nb[0]) {
        b -= A.nb[0];
        c = 1;
        if (b >= A.nb[1]) {
            b -= A.nb[1];
            c = 2;
        }
    }
    if (c == 2 && b >= A.nb[2]) return;
    const int n0 = G.n[0], n1 = G.n[1];
    const int N = arg3(G.n, c), W = arg3(A.W, c), len = arg3(A.len, c), off = arg3(A.off, c);
    const int ext = N + len - 1;
    const int64_t nc = G.nc;
    double* dst = gl(A.J) + (int64_t)c * nc;
    // first line of the block and the line count / axis stride
    int64_t base0;
    int stride, nlines;
    if (c == 0) {
        const int64_t L0 = b * W;
        const int64_t rows = (int64_t)n1 * G.n[2];
        base0 = L0 * n0;
        stride = 1;
        nlines = (int)(rows - L0 < W ? rows - L0 : W);
    } else {
        const int nbx = (n0 + W - 1) / W;
        const int bx = (int)(b % nbx);
        const int64_t other = b / nbx;  // k for y lines, j for z lines
        const int i0 = bx * W;
        base0 = c == 1 ? i0 + (int64_t)n0 * n1 * other : i0 + (int64_t)n0 * other;
        stride = c == 1 ? n0 : n0 * n1;
        nlines = n0 - i0 < W ? n0 - i0 : W;
    }
    // line w starts at base0 + w * (x lines: n0, else 1); in LDS at w * ws, its values js apart
    const int64_t lstep = c == 0 ? n0 : 1;
    const int ws = c == 0 ? ext : 1, js = c == 0 ? 1 : W;
    // a thread stays on one line: 256 / W threads a line, neighbours along the memory order
    const int per_line = FIELD_BS / W;
    const int w = c == 0 ? (int)threadIdx.x / per_line : (int)threadIdx.x % W;
    const int j0 = c == 0 ? (int)threadIdx.x % per_line : (int)threadIdx.x / W;
    const bool live = w < nlines;
    const int64_t line = (int64_t)c * nc + base0 + (live ? w : 0) * lstep;
    // global memory (not generic) accesses, which the LDS stores need not wait behind
    glob_f64* gsrc = A.Jq ? (glob_f64*)A.Jq + line : (glob_f64*)A.J2 + line;
    const double inv = A.Jq ? 1.0 / fixed_scale(A.scale) : 1.0;  // exact: a power of two
    // LINE_BATCH loads per thread in flight before the first is stored; every lane loads (past the
    // end, its line's first value), so that no load waits at a branch
    for (int q0 = j0; q0 < ext; q0 += LINE_BATCH * per_line) {
        double v[LINE_BATCH];
#pragma unroll
        for (int t = 0; t < LINE_BATCH; ++t) {
            const int jj = q0 + t * per_line;
            v[t] = gsrc[(int64_t)wrap_near(off + (jj < ext ? jj : 0), N) * stride];
        }
#pragma unroll
        for (int t = 0; t < LINE_BATCH; ++t) {
            const int jj = q0 + t * per_line;
            if (jj < ext) e[w * ws + jj * js] = A.Jq ? (double)__double_as_longlong(v[t]) * inv : v[t];
        }
    }
    __syncthreads();
    if (A.Jq && live) {
        glob_u64* gq = (glob_u64*)A.Jq + line;
        for (int j = j0; j < N; j += per_line) gq[(int64_t)j * stride] = 0ull;
    }
    // the coefficients are the same for the whole block: read-only, uniform (scalar) loads
    const_f64* cf = (const_f64*)arg3(A.coef, c);
    const int chunks = (N + LINE_OUT - 1) / LINE_OUT;
    for (int k = j0; k < chunks; k += per_line) {
        // the last chunk starts earlier instead of running past the line
        const int j = k * LINE_OUT + LINE_OUT <= N ? k * LINE_OUT : (N > LINE_OUT ? N - LINE_OUT : 0);
        double acc[LINE_OUT];
        if (N >= LINE_OUT) {
            line_taps(e + w * ws + j * js, js, cf, len, acc);
        } else {
#pragma unroll
            for (int o = 0; o < LINE_OUT; ++o) {
                acc[o] = 0.0;
                if (o < N)
                    for (int t = 0; t < len; ++t) acc[o] += cf[t] * e[w * ws + (o + t) * js];
            }
        }
        if (!live) continue;
#pragma unroll
        for (int o = 0; o < LINE_OUT; ++o)
            if (j + o < N) dst[base0 + w * lstep + (int64_t)(j + o) * stride] = acc[o];
    }
}

__device__ __forceinline__ void line_any(const LineArgs& A, int64_t b, double* e) {
    if (A.W[0] > 0)
        line_lds_body(A, b, e);
    else
        line_body(A, b);
}

__global__ void __launch_bounds__(FIELD_BS) k_line_solve(LineArgs A) {
    __shared__ double e[LINE_LDS_DOUBLES];
    line_any(A, blockIdx.x, e);
}

__global__ void __launch_bounds__(FIELD_BS) k_line_solve_batch(const LineArgs* __restrict__ T,
                                                               const int64_t* __restrict__ prefix, int nruns) {
    __shared__ double e[LINE_LDS_DOUBLES];
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, nruns, b);
    if (r < 0) return;
    line_any(T[r], b - prefix[r], e);
}

// Host: coefficients of T^{-1} on a periodic line of N cells, by the discrete Fourier
// transform of 1 / T(k); truncated where they fall below 1e-16 of the centre value.  At most 127
// of them; 0 if there is no memory.
int line_setup_axis(int order, int N, double* coef_host, int* off) {
    double a[3];
    fd_coeffs(order, a);
    const int M = order / 2;
    double T[3] = {0, 0, 0};
    for (int l = 0; l < M; ++l)
        for (int m = l + 1; m <= M; ++m) T[l] += a[m - 1];
    double* symbol = new (std::nothrow) double[N];  // T(k)
    if (!symbol) return 0;
    for (int kk = 0; kk < N; ++kk) {
        double k = 2.0 * M_PI * kk / N;
        symbol[kk] = T[0];
        for (int l = 1; l < M; ++l) symbol[kk] += 2.0 * T[l] * cos(l * k);
    }
    // g(m) = 1/N sum_k cos(2 pi k m / N) / T(k), each worked out once
    double known[130];
    int nknown = 0;
    auto g = [&](int m) {
        for (; nknown <= m; ++nknown) {
            double s = 0.0;
            for (int kk = 0; kk < N; ++kk) s += cos(2.0 * M_PI * kk / N * nknown) / symbol[kk];
            known[nknown] = s / N;
        }
        return known[m];
    };
    // the coefficients decay geometrically down to the rounding noise of the sum (~1e-17);
    // keep them while two consecutive ones stand above 1e-16 of the centre value
    const double g0 = g(0);
    int Rr = 0;
    while (Rr < N / 2 && Rr < 63) {
        if (fabs(g(Rr + 1)) < 1e-16 * fabs(g0) && fabs(g(Rr + 2)) < 1e-16 * fabs(g0)) break;
        ++Rr;
    }
    if (2 * Rr + 1 >= N) {  // full circulant: offsets 0..N-1
        for (int m = 0; m < N; ++m) coef_host[m] = g(m);
        delete[] symbol;
        *off = 0;
        return N;
    }
    for (int m = -Rr; m <= Rr; ++m) coef_host[m + Rr] = g(m < 0 ? -m : m);
    delete[] symbol;
    *off = -Rr;
    return 2 * Rr + 1;
}

// Lines per block of each axis: as many as the LDS copy holds, fewer (down to 8, whole cache
// lines of the y and z rows) while a component has not two blocks per CU (its share of them in a
// batch of nruns).
static bool line_blocks_of(const pp_run* r, int nruns, int W[3], int64_t nb[3]) {
    const int64_t n0 = r->p.n[0];
    for (int d = 0; d < 3; ++d) {
        const int ext = r->p.n[d] + r->line[d].len - 1;
        W[d] = 64;
        while (W[d] > 1 && (int64_t)W[d] * ext > LINE_LDS_DOUBLES) W[d] >>= 1;
        if ((int64_t)W[d] * ext > LINE_LDS_DOUBLES) return false;
        auto blocks = [&] {
            return d == 0 ? ((int64_t)r->p.n[1] * r->p.n[2] + W[d] - 1) / W[d]
                          : ((n0 + W[d] - 1) / W[d]) * (d == 1 ? r->p.n[2] : r->p.n[1]);
        };
        while (W[d] > 8 && blocks() * nruns < 512) W[d] >>= 1;
        nb[d] = blocks();
    }
    return true;
}

bool line_reads_fixed(const pp_run* r) {
    int W[3];
    int64_t nb[3];
    return uses_line_solve(r) && r->Jq && line_blocks_of(r, 1, W, nb);
}

void line_desc(const pp_run* r, LineArgs* A, int nruns) {
    A->G = CellGeom(make_geom(r));
    for (int d = 0; d < 3; ++d) {
        A->coef[d] = r->line[d].coef;
        A->len[d] = r->line[d].len;
        A->off[d] = r->line[d].off;
    }
    A->Jq = nullptr;
    if (!line_blocks_of(r, nruns, A->W, A->nb)) {
        A->W[0] = 0;
        A->nb[0] = blocks_of(A->G);
        A->nb[1] = A->nb[2] = 0;
    } else if (r->Jq) {
        A->Jq = (unsigned long long*)r->Jq;
        A->scale = gpd32_scale(r);
    }
    A->J2 = r->J2;
    A->J = r->mesh.J;
}

size_t line_desc_size() { return sizeof(LineArgs); }

int64_t line_blocks(const pp_run* r, int nruns) {
    int W[3];
    int64_t nb[3];
    return line_blocks_of(r, nruns, W, nb) ? nb[0] + nb[1] + nb[2] : blocks_of(make_geom(r));
}

hipError_t launch_line_solve(pp_run* r) {
    LineArgs A;
    line_desc(r, &A, 1);
    hipLaunchKernelGGL(k_line_solve, dim3((unsigned)line_blocks(r, 1)), dim3(FIELD_BS), 0, r->stream, A);
    return hipGetLastError();
}

hipError_t launch_line_solve_batch(const void* table, const int64_t* prefix, int n, int64_t total_blocks, hipStream_t st) {
    if (n == 0 || total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_line_solve_batch, dim3((unsigned)total_blocks), dim3(FIELD_BS), 0, st, (const LineArgs*)table,
                       prefix, n);
    return hipGetLastError();
}

}  // namespace pp
