// FP64 diagnostics: kinetic energy and momentum per species, field energies, the charge
// density (eq. "rho2", same weights as the gather), the Gauss-law residual with the
// field-order divergence, the discrete continuity residual (eq. "cc1") and div B.
//
// Charge density of the split form, once the particles are stored tile by tile: one
// workgroup per tile adds the (O+1)^3 contributions q w W of each of its particles to an LDS
// block of the tile plus its support halo (1 node below, O above), in 64-bit fixed point
// (the contribution scaled by 2^e and rounded by one fused multiply-add with 1.5*2^52, whose
// bit pattern is added with an integer atomic; the node sum is the sign-extended low 51
// bits).  The block is then added to a global 64-bit accumulator, and a last pass writes
// rho = sum * 2^-e.  A particle found outside the tile it is stored with (after a push, before
// the sort) adds its rounded contributions straight to the global accumulator.  The result
// is the exact sum of the rounded contributions, whatever the order.  The FP64 form, and a
// split species never sorted, use one thread per particle with FP64 global atomics.
#include "pp_device.hpp"
#include "pp_internal.hpp"

namespace pp {

// accumulator slots (doubles) in r->dacc
enum {
    ACC_KIN = 0,                           // [PP_MAX_SPECIES]
    ACC_MOM = ACC_KIN + PP_MAX_SPECIES,    // [PP_MAX_SPECIES][3]
    ACC_UE = ACC_MOM + 3 * PP_MAX_SPECIES,
    ACC_UB,
    ACC_UEX,
    ACC_GAUSS,  // max, stored as the bits of a non-negative double
    ACC_CC,
    ACC_DIVB,
    ACC_RELAX,      // max |rhs - A B| of the last relaxation (bits of a non-negative double)
    ACC_RELAX_RHS,  // max |rhs|
    ACC_COUNT
};
// after the accumulators: the flag word (copied with them) and, device-only, 2^e of the
// fixed-point charge density and the partials
constexpr int ACC_FLAGS = ACC_COUNT;
constexpr int ACC_RHO_SCALE = ACC_COUNT + 1;
constexpr int ACC_PART = ACC_COUNT + 8;  // partials of the sums (ROW_COUNT rows)

__global__ void k_fill_f64(double* p, int64_t n, double v) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        p[q] = v;
}

hipError_t launch_fill(double* p, int64_t n, double v, hipStream_t st) {
    const int bs = 256;
    int64_t g = (n + bs - 1) / bs;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)g), dim3(bs), 0, st, p, n, v);
    return hipGetLastError();
}

// Sums and maxima over particles or cells: each workgroup writes its value of every row to the
// row's partials, and k_finish combines them in a fixed order (atomics on one address are served
// one after another, about 13 ns each: 5.2e6 particles' moments took 2 x 160 us that way).
// Partials of a row, the workgroups that a launch can have: 512 (two a CU) are enough where the caches
// hold the box, and cost a small run little memory; a large box needs the 4096 to wait for memory in
// enough places at once.  256^3, 64 particles per cell: residuals and moments 684 and 3180 us with 512,
// 340 and 2564 with 2048, 329 and 2500 with 4096.
static int part_max(int64_t ncell) { return (int)(ncell < 512 * 128 ? 512 : (ncell > 4096 * 128 ? 4096 : ncell / 128)); }
enum { ROW_SPECIES = 0, ROW_FIELD = 4 * PP_MAX_SPECIES, ROW_RESID = ROW_FIELD + 3, ROW_COUNT = ROW_RESID + 3 };

template <bool MAX>
__device__ __forceinline__ double join(double a, double b) {
    return MAX ? fmax(a, b) : a + b;
}

template <int NV, bool MAX>
__device__ __forceinline__ void write_partials(double v[NV], double* part, int row) {
    __shared__ double sh[NV][4];
#pragma unroll
    for (int a = 0; a < NV; ++a)
        for (int o = 32; o > 0; o >>= 1) v[a] = join<MAX>(v[a], __shfl_xor(v[a], o, 64));
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int a = 0; a < NV; ++a) sh[a][threadIdx.x >> 6] = v[a];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int a = 0; a < NV; ++a)
            part[(int64_t)a * row + blockIdx.x] =
                join<MAX>(join<MAX>(sh[a][0], sh[a][1]), join<MAX>(sh[a][2], sh[a][3]));
}

constexpr int DIAG_UNROLL = 4;

// workgroups of 256 threads for a sum over n entries: up to 1024 with a round of work each, and more if
// each has 64 rounds (128^3, 64 particles per cell: moments 323 us with 1024, 382 with 4096)
static unsigned sum_grid(int64_t n, int most) {
    const int64_t round = 256 * DIAG_UNROLL, rounds = (n + round - 1) / round;
    const int64_t g = rounds <= 1024 ? rounds : (rounds / 64 > 1024 ? rounds / 64 : 1024);
    return (unsigned)(g < 1 ? 1 : (g > most ? most : g));
}

// kinetic energy w V m u^2/(gamma + 1) (= w V m c^2 (gamma - 1)) and momentum w V m u of every
// species in one launch
struct MomentArgs {
    const void* u[PP_MAX_SPECIES][3];
    int64_t n[PP_MAX_SPECIES];
    double wVm[PP_MAX_SPECIES];
    int slot[PP_MAX_SPECIES];
    double ic;
    double* part;
    int row;  // entries of a row of partials
};

template <typename T>
__global__ void __launch_bounds__(256) k_moments(MomentArgs A) {
    const int s = blockIdx.y;
    const T* ux = (const T*)A.u[s][0];
    const T* uy = (const T*)A.u[s][1];
    const T* uz = (const T*)A.u[s][2];
    const int64_t n = A.n[s];
    const double ic = A.ic;
    double v[4] = {0, 0, 0, 0};
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t p0 = (int64_t)blockIdx.x * 256 + threadIdx.x; p0 < n; p0 += DIAG_UNROLL * step) {
        T x[DIAG_UNROLL], y[DIAG_UNROLL], z[DIAG_UNROLL];
#pragma unroll
        for (int k = 0; k < DIAG_UNROLL; ++k) {
            const int64_t p = p0 + k * step < n ? p0 + k * step : p0;
            x[k] = ux[p];
            y[k] = uy[p];
            z[k] = uz[p];
        }
#pragma unroll
        for (int k = 0; k < DIAG_UNROLL; ++k) {
            if (p0 + k * step >= n) break;
            const double a = (double)x[k], b = (double)y[k], c = (double)z[k];
            const double u2 = a * a + b * b + c * c;
            const double g = sqrt(1.0 + u2 * ic * ic);
            v[0] += u2 / (g + 1.0);
            v[1] += a;
            v[2] += b;
            v[3] += c;
        }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) v[a] *= A.wVm[s];
    write_partials<4, false>(v, A.part + (int64_t)(ROW_SPECIES + 4 * A.slot[s]) * A.row, A.row);
}

__global__ void __launch_bounds__(256) k_field_energy(const double* __restrict__ E, const double* __restrict__ B,
                                                      int64_t nc, double hV_eps0, double hV_imu0, double* part,
                                                      int row) {
    double v[3] = {0, 0, 0};
#pragma unroll 2
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nc; q += (int64_t)gridDim.x * blockDim.x) {
        double ex = E[q], ey = E[nc + q], ez = E[2 * nc + q];
        double bx = B[q], by = B[nc + q], bz = B[2 * nc + q];
        v[0] += ex * ex + ey * ey + ez * ez;
        v[1] += bx * bx + by * by + bz * bz;
        v[2] += ex * ex;
    }
    v[0] *= hV_eps0;
    v[1] *= hV_imu0;
    v[2] *= hV_eps0;
    write_partials<3, false>(v, part + (int64_t)ROW_FIELD * row, row);
}

// rho(node) += q w W(X - node), FP64, for either particle form
template <int O, typename T>
__global__ void __launch_bounds__(256) k_deposit_rho(int nx, int ny, int nz, const int32_t* __restrict__ cell,
                                                     const T* __restrict__ px, const T* __restrict__ py,
                                                     const T* __restrict__ pz, int64_t n, double qw, double* rho,
                                                     int split) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double X[3];
    if (split) {
        int32_t c = cell[p];
        if (c < 0 || c >= nx * ny * nz) return;
        int i = c % nx, r = c / nx, j = r % ny, k = r / ny;
        X[0] = i + (double)px[p];
        X[1] = j + (double)py[p];
        X[2] = k + (double)pz[p];
    } else {
        X[0] = (double)px[p];
        X[1] = (double)py[p];
        X[2] = (double)pz[p];
    }
    double w[3][O + 1];
    int i0[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) i0[d] = weights_abs<O>(X[d], w[d]);
    const int N[3] = {nx, ny, nz};
#pragma unroll
    for (int c = 0; c <= O; ++c) {
        int k = wrap(i0[2] + c, N[2]);
#pragma unroll
        for (int b = 0; b <= O; ++b) {
            int j = wrap(i0[1] + b, N[1]);
            double wzy = qw * w[2][c] * w[1][b];
#pragma unroll
            for (int a = 0; a <= O; ++a) {
                int i = wrap(i0[0] + a, N[0]);
                atomic_add_f64(rho + (int64_t)i + (int64_t)nx * (j + (int64_t)ny * k), wzy * w[0][a]);
            }
        }
    }
}

// ---- split form: tiled fixed-point charge deposit ------------------------------------------
struct Rho32Sp {
    const int32_t* start;  // tile starts of the stored order (ntiles + 1)
    const int32_t* cell;
    const float* pos[3];
    double qw;
};

// A workgroup deposits the particles stored in its tile's range; under a pending sort
// order that range holds the particles of the tile before their last push, which may have
// moved up to RHO_HALO cells out of it, so the LDS block covers that many cells around the
// tile (particles further away, only in flagged states, take global atomics).
constexpr int RHO_HALO = 2;

struct Rho32Args {
    int n[3], t[3], nt[3];
    int ext[3];   // LDS block extent per axis: t + 2 RHO_HALO + O + 1 (1 on a single-cell axis)
    int lo[3];    // nodes below the tile: RHO_HALO + 1 (0 on a single-cell axis)
    int halo[3];  // cells around the tile deposited in the block: RHO_HALO (0 on a single-cell axis)
    int64_t nc;
    double inv_n0, inv_n1;  // 1 / n[0], 1 / n[1]: a cell's row and plane without integer divisions
    int nsp;
    Rho32Sp sp[PP_MAX_SPECIES];
    unsigned long long* acc;  // nc, zero on entry
    const double* scale;      // 2^e
};

constexpr double RHO_MAGIC = 6755399441055744.0;  // 1.5 * 2^52
constexpr unsigned long long RHO_LOW51 = (1ull << 51) - 1ull;
constexpr long long RHO_BIT50 = 1ll << 50;

// sum of the rounded values held in the low 51 bits of a sum of bit patterns
__device__ __forceinline__ long long rho_fixed_sum(unsigned long long v) {
    return (long long)((v & RHO_LOW51) ^ (unsigned long long)RHO_BIT50) - RHO_BIT50;
}

// bit pattern of 1.5*2^52 + round(x), |x| < 2^50
__device__ __forceinline__ unsigned long long rho_pattern(double a, double b) {
    return (unsigned long long)__double_as_longlong(fma(a, b, RHO_MAGIC));
}

// 2^e with e = e0 - ceil(log2(N)), N the sum of the largest tile populations of the deposited
// species: a contribution is at most 2^(50 - ceil log2 N) and an LDS node sum at most 2^50 in
// magnitude.  The populations are those of the ranges that the particles lie in: under a pending
// sort order (mask pending) the order's before it (a cluster at a tile's corner that shares itself
// out among eight tiles leaves an eighth of its old tile's count in each).
__global__ void k_rho_scale(const int32_t* __restrict__ tile_max, unsigned mask, unsigned pending, int e0, double* scale) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    long long nb = 0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s)
        if (mask & (1u << s)) nb += tile_max[pending & (1u << s) ? PP_MAX_SPECIES + s : s];
    int lg = 0;
    while ((1ll << lg) < nb) ++lg;
    *scale = ldexp(1.0, e0 - lg);
}

// What a particle deposits: its weights and the first node of its support in the block; ok false:
// nothing there.
template <int O>
struct RhoWin {
    double w[3][O + 1];
    int base;
    bool ok;
};

// The block's strides.  Compile-time for the 4x4x4 tile (CUBE): rows of 12 words put the 16 cells of a
// plane, 16 lanes of a round, on different banks.  A single-cell axis has stride 0.
template <int O, bool CUBE>
struct RhoBlk {
    static constexpr int E = 4 + 2 * RHO_HALO + O + 1;
    static constexpr int sx = 1, sy = 12, sz = 12 * E, words = 12 * E * E;
    static_assert(E <= 12, "row padding");
    __device__ RhoBlk(const Rho32Args&) {}
};

template <int O>
struct RhoBlk<O, false> {
    int sx, sy, sz;
    __device__ RhoBlk(const Rho32Args& A) {
        sx = A.ext[0] == 1 ? 0 : 1;
        sy = A.ext[1] == 1 ? 0 : A.ext[0];
        sz = A.ext[2] == 1 ? 0 : A.ext[0] * A.ext[1];
    }
};

template <int O, class BL>
__device__ __forceinline__ void rho_window(const Rho32Args& A, const Rho32Sp& S, const BL& L, const int org[3], int32_t p,
                                           double v, RhoWin<O>& W) {
    const int32_t cell = S.cell[p];
    if (cell < 0 || (int64_t)cell >= A.nc) return;  // reported by the error flags
    // exact: (cell + 1/2) / n is at least 1/(2n) from an integer, and below 2^30
    const int row = (int)(((double)cell + 0.5) * A.inv_n0), gz = (int)(((double)row + 0.5) * A.inv_n1);
    const int g[3] = {cell - row * A.n[0], row - gz * A.n[1], gz};
    const float f[3] = {S.pos[0][p], S.pos[1][p], S.pos[2][p]};
    const float flo = O == 2 ? -0.5f : 0.0f;
    bool finite = true, in_block = true;
    int ll[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        finite = finite && fabsf(f[d]) <= 1048576.0f;  // false for NaN and Inf as well
        int l = g[d] - org[d];  // cell relative to the tile, nearest periodic image
        if (l >= A.t[d] + A.halo[d])
            l -= A.n[d];
        else if (l < -A.halo[d])
            l += A.n[d];
        ll[d] = l;
        in_block = in_block && l >= -A.halo[d] && l < A.t[d] + A.halo[d] && f[d] >= flo && f[d] < flo + 2.0f;
    }
    if (!finite) return;  // reported by the error flags
    int i0[3];
    if (in_block) {
        // support inside the block: nodes of cells -halo .. t + halo - 1 around the tile,
        // i.e. block indices 0 .. t + 2 halo + O
#pragma unroll
        for (int d = 0; d < 3; ++d) i0[d] = weights_abs<O>((double)(ll[d] + A.lo[d]) + (double)f[d], W.w[d]);
        W.base = i0[0] * L.sx + i0[1] * L.sy + i0[2] * L.sz;
        W.ok = true;
        return;
    }
    double w[3][O + 1];
#pragma unroll
    for (int d = 0; d < 3; ++d) i0[d] = weights_abs<O>((double)g[d] + (double)f[d], w[d]);
#pragma unroll
    for (int c = 0; c <= O; ++c) {
        const int k = wrap(i0[2] + c, A.n[2]);
#pragma unroll
        for (int b = 0; b <= O; ++b) {
            const int j = wrap(i0[1] + b, A.n[1]);
            const double vzy = v * w[2][c] * w[1][b];
#pragma unroll
            for (int a = 0; a <= O; ++a) {
                const int i = wrap(i0[0] + a, A.n[0]);
                const long long x = rho_fixed_sum(rho_pattern(vzy, w[0][a]));
                atomicAdd(A.acc + (int64_t)i + (int64_t)A.n[0] * (j + (int64_t)A.n[1] * k), (unsigned long long)x);
            }
        }
    }
}

// Charge of one particle, or of two on the same nodes (PAIR; v2 = 0: of the first alone): each
// contribution's pattern is rounded on its own, so that two of them summed before the atomic give
// the same exact sum as two atomics.
template <int O, class BL, bool PAIR>
__device__ __forceinline__ void rho_deposit(unsigned long long* blk, const BL& L, const RhoWin<O>& W1, const RhoWin<O>& W2,
                                            double v1, double v2) {
#pragma unroll
    for (int c = 0; c <= O; ++c)
#pragma unroll
        for (int b = 0; b <= O; ++b) {
            const double vzy1 = v1 * W1.w[2][c] * W1.w[1][b];
            const double vzy2 = PAIR ? v2 * W2.w[2][c] * W2.w[1][b] : 0.0;
            unsigned long long* row = blk + W1.base + c * L.sz + b * L.sy;
#pragma unroll
            for (int a = 0; a <= O; ++a) {
                unsigned long long bits = rho_pattern(vzy1, W1.w[0][a]);
                if (PAIR) bits += rho_pattern(vzy2, W2.w[0][a]);
                atomicAdd(row + a * L.sx, bits);
            }
        }
}

// Bound by the LDS atomics, 64 a cubic particle.  In the 4x4x4 tiles' storage order (chunks of 64
// pairs, see pp_sort.hip) lane l takes slots l and 64 + l of a chunk, two particles of a cell, whose
// supports are the same unless one of them has since left it: one atomic a node for both.  70x46x50,
// 1.03e7 particles, cubic: 169 us one by one with the strides read from the arguments, 128 now;
// 50x42x37, quadratic, after a push: 85 and 75.
template <int O, bool CUBE>
__global__ void __launch_bounds__(256) k_rho32(Rho32Args A) {
    extern __shared__ unsigned long long rho_blk[];
    const RhoBlk<O, CUBE> L(A);
    const uint32_t tile = blockIdx.x, trow = tile / (uint32_t)A.nt[0], layer = trow / (uint32_t)A.nt[1];
    const int org[3] = {(int)(tile - trow * (uint32_t)A.nt[0]) * A.t[0], (int)(trow - layer * (uint32_t)A.nt[1]) * A.t[1],
                        (int)layer * A.t[2]};
    int vol;
    if constexpr (CUBE)
        vol = L.words;
    else
        vol = A.ext[0] * A.ext[1] * A.ext[2];
    for (int q = threadIdx.x; q < vol; q += blockDim.x) rho_blk[q] = 0ull;
    __syncthreads();
    const double sc = *A.scale;
    for (int s = 0; s < A.nsp; ++s) {
        const Rho32Sp& S = A.sp[s];
        const double v = S.qw * sc;
        const int32_t start = S.start[tile], end = S.start[tile + 1];
        if constexpr (CUBE) {
            const int lane = threadIdx.x & 63;
            for (int32_t b = start + 128 * (int)(threadIdx.x >> 6); b < end; b += 128 * 4) {
                RhoWin<O> W1, W2;
                W1.ok = W2.ok = false;
                W1.base = W2.base = 0;
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int a = 0; a <= O; ++a) W2.w[d][a] = 0.0;  // finite where v2 = 0 leaves it out
                const int32_t p1 = b + lane, p2 = p1 + 64;
                if (p1 < end) rho_window<O>(A, S, L, org, p1, v, W1);
                if (p2 < end) rho_window<O>(A, S, L, org, p2, v, W2);
                const bool same = W1.ok && W2.ok && W1.base == W2.base;
                if (__any(same)) {
                    if (W1.ok) rho_deposit<O, RhoBlk<O, CUBE>, true>(rho_blk, L, W1, W2, v, same ? v : 0.0);
                } else if (W1.ok) {
                    rho_deposit<O, RhoBlk<O, CUBE>, false>(rho_blk, L, W1, W1, v, 0.0);
                }
                if (W2.ok && !same) rho_deposit<O, RhoBlk<O, CUBE>, false>(rho_blk, L, W2, W2, v, 0.0);
            }
        } else {
            for (int32_t p = start + threadIdx.x; p < end; p += blockDim.x) {
                RhoWin<O> W;
                W.ok = false;
                rho_window<O>(A, S, L, org, p, v, W);
                if (W.ok) rho_deposit<O, RhoBlk<O, CUBE>, false>(rho_blk, L, W, W, v, 0.0);
            }
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < vol; q += blockDim.x) {
        const long long x = rho_fixed_sum(rho_blk[q]);
        if (x == 0) continue;
        int a, b, c;
        if constexpr (CUBE) {  // the rows' padding holds nothing
            c = q / L.sz;
            b = (q - c * L.sz) / L.sy;
            a = q - c * L.sz - b * L.sy;
        } else {
            a = q % A.ext[0];
            b = (q / A.ext[0]) % A.ext[1];
            c = q / (A.ext[0] * A.ext[1]);
        }
        const int i = wrap_near(org[0] - A.lo[0] + a, A.n[0]);
        const int j = wrap_near(org[1] - A.lo[1] + b, A.n[1]);
        const int k = wrap_near(org[2] - A.lo[2] + c, A.n[2]);
        atomicAdd(A.acc + (int64_t)i + (int64_t)A.n[0] * (j + (int64_t)A.n[1] * k), (unsigned long long)x);
    }
}

__global__ void __launch_bounds__(256) k_rho_from_fixed(unsigned long long* __restrict__ acc, int64_t nc,
                                                        const double* __restrict__ scale, double* rho) {
    const double inv = 1.0 / *scale;  // exact: a power of two
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nc; q += (int64_t)gridDim.x * blockDim.x) {
        rho[q] = (double)(long long)acc[q] * inv;
        acc[q] = 0ull;
    }
}

struct DivGeom {
    int n[3];
    int64_t nc;
    int M;
    double a[3][3];  // a_m / d
    double inv_n0, inv_n1;  // 1 / n[0], 1 / n[1]
};

__device__ __forceinline__ int nbw(int i, int o, int n) {
    int j = i + o;
    while (j < 0) j += n;
    while (j >= n) j -= n;
    return j;
}

// down divergence of a face field at cell centre (i,j,k)
__device__ __forceinline__ double div_dn(const DivGeom& G, const double* F, int i, int j, int k) {
    const int c[3] = {i, j, k};
    double s = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
        const double* f = F + ax * G.nc;
        for (int m = 1; m <= G.M; ++m) {
            int hi[3] = {i, j, k}, lo[3] = {i, j, k};
            hi[ax] = nbw(c[ax], m - 1, G.n[ax]);
            lo[ax] = nbw(c[ax], -m, G.n[ax]);
            s += G.a[ax][m - 1] * (f[hi[0] + (int64_t)G.n[0] * (hi[1] + (int64_t)G.n[1] * hi[2])] -
                                   f[lo[0] + (int64_t)G.n[0] * (lo[1] + (int64_t)G.n[1] * lo[2])]);
        }
    }
    return s;
}

__device__ __forceinline__ double div_up(const DivGeom& G, const double* F, int i, int j, int k) {
    const int c[3] = {i, j, k};
    double s = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
        const double* f = F + ax * G.nc;
        for (int m = 1; m <= G.M; ++m) {
            int hi[3] = {i, j, k}, lo[3] = {i, j, k};
            hi[ax] = nbw(c[ax], m, G.n[ax]);
            lo[ax] = nbw(c[ax], -m + 1, G.n[ax]);
            s += G.a[ax][m - 1] * (f[hi[0] + (int64_t)G.n[0] * (hi[1] + (int64_t)G.n[1] * hi[2])] -
                                   f[lo[0] + (int64_t)G.n[0] * (lo[1] + (int64_t)G.n[1] * lo[2])]);
        }
    }
    return s;
}

// Gauss residual |div E - (rho + rho_bg)/eps0| and continuity residual
// |rho - rho_prev + dt div J|, max norms
__global__ void __launch_bounds__(256) k_residuals(DivGeom G, const double* __restrict__ E, const double* __restrict__ J,
                                                   const double* __restrict__ B, const double* __restrict__ rho,
                                                   const double* __restrict__ rho_prev, double rho_bg, double ieps0,
                                                   double dt, int want_rho, int have_prev, int want_divb, double* part,
                                                   int part_row) {
    double g = 0.0, cc = 0.0, db = 0.0;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < G.nc; q += (int64_t)gridDim.x * blockDim.x) {
        const int row = (int)(((double)q + 0.5) * G.inv_n0), k = (int)(((double)row + 0.5) * G.inv_n1);
        const int i = (int)q - row * G.n[0], j = row - k * G.n[1];
        if (want_rho) {
            g = fmax(g, fabs(div_dn(G, E, i, j, k) - (rho[q] + rho_bg) * ieps0));
            if (have_prev) cc = fmax(cc, fabs(rho[q] - rho_prev[q] + dt * div_dn(G, J, i, j, k)));
        }
        if (want_divb) db = fmax(db, fabs(div_up(G, B, i, j, k)));
    }
    double v[3] = {g, cc, db};
    write_partials<3, true>(v, part + (int64_t)ROW_RESID * part_row, part_row);
}

static void fd_coeffs(int order, double a[3]) {
    a[0] = a[1] = a[2] = 0.0;
    if (order == 2) {
        a[0] = 1.0;
    } else if (order == 4) {
        a[0] = 9.0 / 8.0;
        a[1] = -1.0 / 24.0;
    } else {
        a[0] = 75.0 / 64.0;
        a[1] = -25.0 / 384.0;
        a[2] = 3.0 / 640.0;
    }
}

template <typename T>
static void deposit_rho_species(pp_run* r, const Species& S) {
    const int bs = 256;
    const unsigned g = (unsigned)((S.n + bs - 1) / bs);
    const int split = r->p.precision == PP_PREC_FP32_SPLIT;
    const double qw = S.q * S.w;
    if (r->p.shape_order == 2)
        hipLaunchKernelGGL((k_deposit_rho<2, T>), dim3(g), dim3(bs), 0, r->stream, r->p.n[0], r->p.n[1], r->p.n[2],
                           (const int32_t*)S.cur.cell, (const T*)S.cur.pos[0], (const T*)S.cur.pos[1],
                           (const T*)S.cur.pos[2], S.n, qw, r->rho, split);
    else
        hipLaunchKernelGGL((k_deposit_rho<3, T>), dim3(g), dim3(bs), 0, r->stream, r->p.n[0], r->p.n[1], r->p.n[2],
                           (const int32_t*)S.cur.cell, (const T*)S.cur.pos[0], (const T*)S.cur.pos[1],
                           (const T*)S.cur.pos[2], S.n, qw, r->rho, split);
}

// Tiled charge deposit of the split species in mask (each stored tile by tile); writes rho.
static hipError_t launch_rho32(pp_run* r, unsigned mask) {
    Rho32Args A;
    const int O = r->p.shape_order;
    double qwmax = 0.0;
    unsigned pending = 0;
    A.nsp = 0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        if (!(mask & (1u << s))) continue;
        const Species& S = r->sp[s];
        Rho32Sp& D = A.sp[A.nsp++];
        // with a sort order pending, the buffers still follow the previous tile starts
        D.start = S.pending ? S.offsets_next : S.offsets;
        pending |= S.pending ? 1u << s : 0u;
        D.cell = (const int32_t*)S.cur.cell;
        for (int d = 0; d < 3; ++d) D.pos[d] = (const float*)S.cur.pos[d];
        D.qw = S.q * S.w;
        qwmax = fabs(D.qw) > qwmax ? fabs(D.qw) : qwmax;
    }
    int vol = 1;
    for (int d = 0; d < 3; ++d) {
        A.n[d] = r->p.n[d];
        A.t[d] = r->g.t[d];
        A.nt[d] = r->g.nt[d];
        const bool single = r->p.n[d] == 1;
        A.ext[d] = single ? 1 : r->g.t[d] + 2 * RHO_HALO + O + 1;
        A.lo[d] = single ? 0 : RHO_HALO + 1;
        A.halo[d] = single ? 0 : RHO_HALO;
        vol *= A.ext[d];
    }
    A.nc = r->g.ncell;
    A.inv_n0 = 1.0 / A.n[0];
    A.inv_n1 = 1.0 / A.n[1];
    A.acc = (unsigned long long*)r->Jq;  // free and zero between steps, and left so
    A.scale = r->dacc + ACC_RHO_SCALE;
    // every contribution is at most |q w| (the weights of a node are at most 1); a box of one cell, whose
    // node takes whole particles, needs a bit more to keep a sum of 2^50 below the sign
    int e0 = 50 - (int)ceil(log2(qwmax)) - (A.nc == 1 ? 1 : 0);
    if (e0 > 1000) e0 = 1000;
    hipLaunchKernelGGL(k_rho_scale, dim3(1), dim3(64), 0, r->stream, (const int32_t*)r->tile_max, mask, pending, e0,
                       r->dacc + ACC_RHO_SCALE);
    const bool cube = A.t[0] == 4 && A.t[1] == 4 && A.t[2] == 4 && A.ext[0] > 1 && A.ext[1] > 1 && A.ext[2] > 1;
    if (cube) vol = O == 2 ? RhoBlk<2, true>::words : RhoBlk<3, true>::words;
    const size_t lds = (size_t)vol * sizeof(unsigned long long);
    const dim3 grid((unsigned)r->g.ntiles);
    if (O == 2 && cube)
        hipLaunchKernelGGL((k_rho32<2, true>), grid, dim3(256), lds, r->stream, A);
    else if (O == 2)
        hipLaunchKernelGGL((k_rho32<2, false>), grid, dim3(256), lds, r->stream, A);
    else if (cube)
        hipLaunchKernelGGL((k_rho32<3, true>), grid, dim3(256), lds, r->stream, A);
    else
        hipLaunchKernelGGL((k_rho32<3, false>), grid, dim3(256), lds, r->stream, A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int64_t g = (A.nc + 255) / 256;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_rho_from_fixed, dim3((unsigned)g), dim3(256), 0, r->stream,
                       (unsigned long long*)r->Jq, A.nc, (const double*)(r->dacc + ACC_RHO_SCALE), r->rho);
    return hipGetLastError();
}

// rho of the current particle positions into r->rho.  Split species stored tile by tile
// (sorted, or pushed since the last sort) go through the tiled fixed-point deposit, which
// writes every node of rho; the others are added with FP64 atomics.
hipError_t deposit_rho_all(pp_run* r) {
    const int64_t nc = r->g.ncell;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    unsigned tiled = 0;
    if (split)
        for (int s = 0; s < PP_MAX_SPECIES; ++s) {
            const Species& S = r->sp[s];
            if (S.active && S.n > 0 && S.q * S.w != 0.0 && (S.sorted || S.ranked)) tiled |= 1u << s;
        }
    hipError_t e = tiled ? launch_rho32(r, tiled) : launch_fill(r->rho, nc, 0.0, r->stream);
    if (e != hipSuccess) return e;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        const Species& S = r->sp[s];
        if (!S.active || S.n == 0 || S.q * S.w == 0.0 || (tiled & (1u << s))) continue;
        if (split)
            deposit_rho_species<float>(r, S);
        else
            deposit_rho_species<double>(r, S);
    }
    return hipGetLastError();
}

// The partials of every row into the accumulators (zero rows whose partials were not written), and
// beside them the flag word (a double holds it exactly), cleared for the next call: one copy to
// the host takes all.
struct FinishArgs {
    const double* part;
    double* dacc;
    int32_t* flags;
    int stride;            // entries of a row of partials
    int count[ROW_COUNT];  // partials of each row
};

constexpr int FINISH_BS = 256;

// a workgroup per row
__global__ void __launch_bounds__(FINISH_BS) k_finish(FinishArgs A) {
    __shared__ double sh[FINISH_BS / 64];
    const int row = blockIdx.x;
    const bool mx = row >= ROW_RESID;
    auto joined = [&](double a, double b) { return mx ? fmax(a, b) : a + b; };
    double v = 0.0;
    for (int i = threadIdx.x; i < A.count[row]; i += FINISH_BS) v = joined(v, A.part[(int64_t)row * A.stride + i]);
    for (int o = 32; o > 0; o >>= 1) v = joined(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < FINISH_BS / 64; ++w) v = joined(v, sh[w]);
    int to;
    if (row < ROW_FIELD)
        to = row % 4 == 0 ? ACC_KIN + row / 4 : ACC_MOM + 3 * (row / 4) + row % 4 - 1;
    else
        to = row < ROW_RESID ? ACC_UE + row - ROW_FIELD : ACC_GAUSS + row - ROW_RESID;
    A.dacc[to] = v;
    if (row == 0) {
        A.dacc[ACC_FLAGS] = (double)*A.flags;
        *A.flags = 0;
    }
}

// Fills host_out[0..ACC_COUNT) with the accumulators and [ACC_COUNT] with the flag word.
hipError_t launch_diag(pp_run* r, uint32_t what, double* host_out) {
    const int bs = 256;
    const int64_t nc = r->g.ncell;
    // a pending sort order needs no move here: the moments are sums over every particle and
    // the charge deposit follows the tile starts of the buffers as they are
    hipError_t e = hipSuccess;
    FinishArgs F{};
    F.part = r->dacc + ACC_PART;
    F.dacc = r->dacc;
    F.flags = r->flags;
    double* part = r->dacc + ACC_PART;
    const int most = part_max(nc);
    F.stride = most;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    const double V = r->p.d[0] * r->p.d[1] * r->p.d[2];
    const double ic = 1.0 / r->p.c;
    if (what & PP_DIAG_MOMENTS) {
        MomentArgs A;
        unsigned ns = 0;
        int64_t nmax = 0;
        for (int s = 0; s < PP_MAX_SPECIES; ++s) {
            const Species& S = r->sp[s];
            if (!S.active || S.n == 0) continue;
            for (int d = 0; d < 3; ++d) A.u[ns][d] = S.cur.u[d];
            A.n[ns] = S.n;
            A.wVm[ns] = S.w * V * S.m;
            A.slot[ns] = s;
            nmax = S.n > nmax ? S.n : nmax;
            ++ns;
        }
        A.ic = ic;
        A.part = part;
        A.row = most;
        if (ns > 0) {
            const dim3 grid(sum_grid(nmax, most), ns);
            for (unsigned k = 0; k < ns; ++k)
                for (int a = 0; a < 4; ++a) F.count[ROW_SPECIES + 4 * A.slot[k] + a] = (int)grid.x;
            if (split)
                hipLaunchKernelGGL(k_moments<float>, grid, dim3(bs), 0, r->stream, A);
            else
                hipLaunchKernelGGL(k_moments<double>, grid, dim3(bs), 0, r->stream, A);
        }
    }
    if (what & PP_DIAG_FIELDS) {
        const double mu0 = 1.0 / (r->p.eps0 * r->p.c * r->p.c);
        hipLaunchKernelGGL(k_field_energy, dim3(sum_grid(nc, most)), dim3(bs), 0, r->stream, (const double*)r->mesh.E,
                           (const double*)r->mesh.B, nc, 0.5 * r->p.eps0 * V, 0.5 * V / mu0, part, most);
        for (int a = 0; a < 3; ++a) F.count[ROW_FIELD + a] = (int)sum_grid(nc, most);
    }
    const bool want_rho = (what & PP_DIAG_RHO) != 0;
    const bool want_divb = (what & PP_DIAG_DIVB) != 0;
    bool have_prev = false;
    if (want_rho) {
        e = deposit_rho_all(r);
        if (e != hipSuccess) return e;
        have_prev = r->rho_prev_step >= 0 && r->rho_prev_step == r->step - 1;
    }
    if (want_rho || want_divb) {
        DivGeom G;
        for (int d = 0; d < 3; ++d) G.n[d] = r->p.n[d];
        G.nc = nc;
        G.M = r->p.field_order / 2;
        G.inv_n0 = 1.0 / G.n[0];
        G.inv_n1 = 1.0 / G.n[1];
        double a[3];
        fd_coeffs(r->p.field_order, a);
        for (int d = 0; d < 3; ++d)
            for (int m = 0; m < 3; ++m) G.a[d][m] = a[m] / r->p.d[d];
        int64_t g = (nc + bs - 1) / bs;
        if (g > most) g = most;
        for (int a = 0; a < 3; ++a) F.count[ROW_RESID + a] = (int)g;
        hipLaunchKernelGGL(k_residuals, dim3((unsigned)g), dim3(bs), 0, r->stream, G, (const double*)r->mesh.E,
                           (const double*)r->mesh.J, (const double*)r->mesh.B, (const double*)r->rho,
                           (const double*)r->rho_prev, r->p.rho_background, 1.0 / r->p.eps0, r->dt_drift, want_rho ? 1 : 0,
                           have_prev ? 1 : 0, want_divb ? 1 : 0, part, most);
    }
    const bool want_relax = (what & PP_DIAG_RELAX) != 0 && r->rhs_valid;
    if (want_relax) {
        e = launch_fill(r->dacc + ACC_RELAX, 2, 0.0, r->stream);
        if (e != hipSuccess) return e;
        e = launch_relax_resid(r, r->dacc + ACC_RELAX);
        if (e != hipSuccess) return e;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finish, dim3(ROW_COUNT), dim3(FINISH_BS), 0, r->stream, F);
    e = hipMemcpyAsync(host_out, r->dacc, (ACC_COUNT + 1) * sizeof(double), hipMemcpyDeviceToHost, r->stream);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(r->stream);
    if (e != hipSuccess) return e;
    host_out[ACC_COUNT + 1] = have_prev ? 1.0 : 0.0;
    host_out[ACC_COUNT + 2] = want_relax ? 1.0 : 0.0;
    if (want_rho) {
        double* t = r->rho_prev;
        r->rho_prev = r->rho;
        r->rho = t;
        r->rho_prev_step = r->step;
    }
    return hipSuccess;
}

int diag_acc_count() { return ACC_COUNT; }
int64_t diag_buffer_count(int64_t ncell) { return ACC_PART + (int64_t)ROW_COUNT * part_max(ncell); }

}  // namespace pp
