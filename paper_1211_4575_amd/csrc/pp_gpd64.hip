// FP64 form of steps 1-3 (Sec. III): absolute FP64 positions and momenta.
//
// k_gpd64_tile takes the particles as the sort left them, binned by cell: a workgroup per tile of
// 64 cells with the tile's fields and current in LDS, and more workgroups for the tiles that hold
// far more particles than the mean.  In large boxes of few particles k_gpd64_sparse first lists the
// tiles that are worth a workgroup.  A particle that does not lie in its tile (its position written
// between the sort and the push) is taken by the lane that finds it.  Where a caller has had the
// arrays, so that there may be many, those are left to k_gpd64_deferred, and so are the particles of
// the tiles not listed.  k_gpd64 takes particles in any order (pushed again without a sort).  Both
// have one thread per particle, read the fields from and add the current to global memory.
#include "pp_device.hpp"
#include "pp_internal.hpp"

namespace pp {

struct Gpd64Args {
    int n[3];
    double d[3];      // cell size
    double dt, ic;    // drift time step (positions, current), 1/c
    double dtk;       // kick time step (momentum update)
    double h;         // q dt / m
    double krad;      // radiative cooling constant rad_tau q^2 / m (0: off)
    double fac[3];    // -q w d_c / dt, current prefactor per component
    int64_t np;
    // particle p of pos and u goes to slot q of pos_o and u_o: the same arrays and p = q, or, with
    // a sort order pending, the other buffers and p = perm[q]
    const int32_t* perm;
    int defer;  // particles out of their tile are left to k_gpd64_deferred
    const double* pos[3];
    const double* u[3];
    double* pos_o[3];
    double* u_o[3];
    const int64_t* id;  // tags that move along (nullptr: none, or in place)
    int64_t* id_o;
    // for the next sort (tiled kernel): particles per new bin whose words hold a rank, those whose words
    // hold the bin alone, rank word per slot
    int32_t* cnt;
    int32_t* named;
    int32_t* rank;
    const double* E;
    const double* B;
    double* J;
    int64_t ncell;
    int32_t* flags;
    int pusher;
    int direct;       // PP_CURRENT_DIRECT: eq. "jj2" instead of the Esirkepov current
    double qw;        // q w (direct current)
};

template <int O, int U>
__device__ __forceinline__ double gather1(const double* __restrict__ F, const int* ix, const int* iy, const int* iz,
                                          const double* wx, const double* wy, const double* wz, int nx, int nxy) {
    double acc = 0.0;
#pragma unroll U
    for (int c = 0; c <= O; ++c) {
        double accy = 0.0;
#pragma unroll U
        for (int b = 0; b <= O; ++b) {
            const double* row = F + (int64_t)iz[c] * nxy + (int64_t)iy[b] * nx;
            double s = 0.0;
#pragma unroll U
            for (int a = 0; a <= O; ++a) s += row[ix[a]] * wx[a];
            accy += s * wy[b];
        }
        acc += accy * wz[c];
    }
    return acc;
}

// new positions back into the box
__device__ __forceinline__ void gpd64_wrap(const Gpd64Args& A, double X[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double nd = (double)A.n[d];
        if (X[d] < 0.0) X[d] += nd;
        if (X[d] >= nd) X[d] -= nd;
    }
}

__device__ __forceinline__ void gpd64_store(const Gpd64Args& A, int64_t q, const double X[3], const V3<double>& u,
                                            double Xn[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) A.pos_o[d][q] = Xn[d] = X[d];
    A.u_o[0][q] = u.x;
    A.u_o[1][q] = u.y;
    A.u_o[2][q] = u.z;
}

// Particle p to slot q (its stored position also in Xn), anywhere in the box (and, as before it is wrapped, a period or more outside).  U
// unrolls the loops over nodes: O + 2 all of them, 1 none (few registers, for a rare path).
template <int O, int U>
__device__ __forceinline__ void gpd64_particle(const Gpd64Args& A, int64_t p, int64_t q, double Xn[3]) {
    const int nx = A.n[0], ny = A.n[1], nz = A.n[2];
    const int nxy = nx * ny;
    const int64_t nc = A.ncell;

    double X0[3] = {A.pos[0][p], A.pos[1][p], A.pos[2][p]};
    V3<double> u{A.u[0][p], A.u[1][p], A.u[2][p]};

    // weights: centred (nodes at integers) and staggered (nodes at i + 1/2) per axis
    double wc[3][O + 1], ws[3][O + 1];
    int ic0[3][O + 1], is0[3][O + 1];
#pragma unroll U
    for (int d = 0; d < 3; ++d) {
        const int nd = A.n[d];
        int c0 = weights_abs<O>(X0[d], wc[d]);
        int s0 = weights_abs<O>(X0[d] - 0.5, ws[d]);
#pragma unroll U
        for (int a = 0; a <= O; ++a) {
            ic0[d][a] = wrap(c0 + a, nd);
            is0[d][a] = wrap(s0 + a, nd);
        }
    }
    // eq. "pfields": E_x staggered along x, B_x staggered along y and z, cyclic
    V3<double> E, B;
    E.x = gather1<O, U>(A.E, is0[0], ic0[1], ic0[2], ws[0], wc[1], wc[2], nx, nxy);
    E.y = gather1<O, U>(A.E + nc, ic0[0], is0[1], ic0[2], wc[0], ws[1], wc[2], nx, nxy);
    E.z = gather1<O, U>(A.E + 2 * nc, ic0[0], ic0[1], is0[2], wc[0], wc[1], ws[2], nx, nxy);
    B.x = gather1<O, U>(A.B, ic0[0], is0[1], is0[2], wc[0], ws[1], ws[2], nx, nxy);
    B.y = gather1<O, U>(A.B + nc, is0[0], ic0[1], is0[2], ws[0], wc[1], ws[2], nx, nxy);
    B.z = gather1<O, U>(A.B + 2 * nc, is0[0], is0[1], ic0[2], ws[0], ws[1], wc[2], nx, nxy);

    const V3<double> um = u;
    if (A.pusher == PP_PUSH_BORIS)
        push_boris<double>(A.h, A.ic, E, B, u);
    else
        push_vay<double>(A.h, A.ic, E, B, u);
    if (A.krad != 0.0) rad_cool<double>(A.krad, A.dtk, A.ic, um, u);

    const double g = sqrt(1.0 + dot(u, u) * A.ic * A.ic);
    const double uu[3] = {u.x, u.y, u.z};
    double X1[3];
    int bad = 0;
#pragma unroll U
    for (int d = 0; d < 3; ++d) {
        X1[d] = X0[d] + A.dt * uu[d] / (g * A.d[d]);
        if (fabs(X1[d] - X0[d]) >= 1.0) bad |= PP_FLAG_CFL;
        if (!isfinite(X1[d]) || !isfinite(uu[d])) bad |= PP_FLAG_NONFINITE;
    }
    if (bad) {  // left as it was
        atomic_or_flag(A.flags, bad);
        gpd64_store(A, q, X0, um, Xn);
        return;
    }

    if (A.direct) {
        // direct current (eq. "jj2"): q w v_c W at J_c's staggered nodes, at the time-centred
        // position, with the gather's weights
        double Xm[3], wmc[3][O + 1], wms[3][O + 1];
        int imc[3][O + 1], ims[3][O + 1];
#pragma unroll U
        for (int d = 0; d < 3; ++d) {
            Xm[d] = 0.5 * (X0[d] + X1[d]);
            const int c0 = weights_abs<O>(Xm[d], wmc[d]);
            const int s0 = weights_abs<O>(Xm[d] - 0.5, wms[d]);
#pragma unroll U
            for (int a = 0; a <= O; ++a) {
                imc[d][a] = wrap(c0 + a, A.n[d]);
                ims[d][a] = wrap(s0 + a, A.n[d]);
            }
        }
#pragma unroll U
        for (int comp = 0; comp < 3; ++comp) {
            const double vq = A.qw * uu[comp] / g;
            double* Jc = A.J + comp * nc;
#pragma unroll U
            for (int c = 0; c <= O; ++c) {
                const int k = comp == 2 ? ims[2][c] : imc[2][c];
                const double wz = comp == 2 ? wms[2][c] : wmc[2][c];
#pragma unroll U
                for (int b = 0; b <= O; ++b) {
                    const int j = comp == 1 ? ims[1][b] : imc[1][b];
                    const double wzy = vq * wz * (comp == 1 ? wms[1][b] : wmc[1][b]);
#pragma unroll U
                    for (int a = 0; a <= O; ++a) {
                        const int i = comp == 0 ? ims[0][a] : imc[0][a];
                        const double v = wzy * (comp == 0 ? wms[0][a] : wmc[0][a]);
                        if (v != 0.0) atomic_add_f64(Jc + (int64_t)i + (int64_t)nx * (j + (int64_t)ny * k), v);
                    }
                }
            }
        }
    } else {
    // Esirkepov current (Sec. III.C) on the common window of O+2 centred nodes per axis
    double S0[3][O + 2], DS[3][O + 2];
    int base[3];
#pragma unroll U
    for (int d = 0; d < 3; ++d) {
        double w0[O + 1], w1[O + 1];
        int a0 = weights_abs<O>(X0[d], w0);
        int a1 = weights_abs<O>(X1[d], w1);
        int b = a0 < a1 ? a0 : a1;
        base[d] = b;
        int o0 = a0 - b, o1 = a1 - b;  // 0 or 1
#pragma unroll U
        for (int k = 0; k < O + 2; ++k) {
            int k0 = k - o0, k1 = k - o1;
            double s0 = (k0 >= 0 && k0 <= O) ? w0[k0 < 0 ? 0 : (k0 > O ? O : k0)] : 0.0;
            double s1 = (k1 >= 0 && k1 <= O) ? w1[k1 < 0 ? 0 : (k1 > O ? O : k1)] : 0.0;
            S0[d][k] = s0;
            DS[d][k] = s1 - s0;
        }
    }
    int idx[3][O + 2];
#pragma unroll U
    for (int d = 0; d < 3; ++d)
#pragma unroll U
        for (int k = 0; k < O + 2; ++k) idx[d][k] = wrap(base[d] + k, A.n[d]);

#pragma unroll U
    for (int comp = 0; comp < 3; ++comp) {
        const int d1 = comp == 0 ? 1 : (comp == 1 ? 2 : 0);
        const int d2 = comp == 0 ? 2 : (comp == 1 ? 0 : 1);
        double* Jc = A.J + comp * nc;
        const int strides[3] = {1, nx, nxy};
#pragma unroll U
        for (int b = 0; b < O + 2; ++b) {
#pragma unroll U
            for (int e = 0; e < O + 2; ++e) {
                double F = S0[d1][b] * S0[d2][e] + 0.5 * DS[d1][b] * S0[d2][e] + 0.5 * S0[d1][b] * DS[d2][e] +
                           DS[d1][b] * DS[d2][e] * (1.0 / 3.0);
                if (F == 0.0) continue;
                int64_t off = (int64_t)idx[d1][b] * strides[d1] + (int64_t)idx[d2][e] * strides[d2];
                double acc = 0.0;
#pragma unroll U
                for (int a = 0; a <= O; ++a) {  // the last prefix (a = O+1) vanishes
                    acc += DS[comp][a] * F;
                    double v = A.fac[comp] * acc;
                    if (v != 0.0) atomic_add_f64(Jc + off + (int64_t)idx[comp][a] * strides[comp], v);
                }
            }
        }
    }
    }
    (void)ny;
    (void)nz;

    gpd64_wrap(A, X1);
    gpd64_store(A, q, X1, u, Xn);
}

template <int O>
__global__ void __launch_bounds__(256) k_gpd64(Gpd64Args A) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double Xn[3];
    if (p < A.np) gpd64_particle<O, O + 2>(A, p, p, Xn);
}

// ---- tiled form ------------------------------------------------------------------------
// A particle of cell c has X in [c - 1/2, c + 1/2): its centred and staggered supports start at
// c - 2 or later and end at c + 2 (cubic) or c + 1 (quadratic); a step of less than a cell widens
// the current's window by one node each way.
constexpr int F64_LO = 2;
constexpr int f64_hi(int O) { return O - 1; }
constexpr int GPD64_BS = 256;
constexpr int32_t RANK_DEFERRED = -1;  // no bin has that number

struct Gpd64TileArgs {
    int t[3], tsh[3], nt[3];  // sides (powers of two) and their logarithms, tiles
    int64_t ntiles;
    int per_xcd;
    int parts;  // workgroups sharing a tile's particles of a species
    int split;  // nsp: a workgroup per species; 1: all of them in one
    int sext[3];  // destination-cell window per axis
    int heavy;    // rounds of 64 particles that a workgroup takes of a tile and species at most
    int helpers;  // blocks past the tiles' own: a chunk of a heavy tile's other rounds each
    int chunk;    // rounds of a chunk
    // a sparse box: the tiles to be taken, as found by k_gpd64_sparse (nullptr: all of them)
    int32_t* list;
    int32_t* list_count;  // zero before k_gpd64_sparse
    int few;              // particles of a tile that is not worth a place in the list
    int nsp;
    const int32_t* bins[PP_MAX_SPECIES];  // cell-bin starts of the sort (64 per tile)
    const int32_t* tile_max[PP_MAX_SPECIES];  // an upper bound of a tile's particles, from the sort
    Gpd64Args sp[PP_MAX_SPECIES];
};

// LDS extents and strides of a tile: compile-time for 4x4x4 and 8x8x1, runtime otherwise.  An
// axis of one cell is collapsed (extent 1, stride 0: every node of it is the same).  Rows of the
// current are padded so that the 16 lanes served together, one per cell of a 4x4 layer (or of two
// rows of 8), fall on 16 different pairs of banks.
template <int O, int TX, int TY, int TZ>
struct Tile64CT {
    static constexpr bool cz = TZ == 1;
    static constexpr int fex = TX + F64_LO + f64_hi(O), fey = TY + F64_LO + f64_hi(O);
    static constexpr int fez = cz ? 1 : TZ + F64_LO + f64_hi(O);
    static constexpr int cex = TX + F64_LO + f64_hi(O) + 2, cey = TY + F64_LO + f64_hi(O) + 2;
    static constexpr int cez = cz ? 1 : TZ + F64_LO + f64_hi(O) + 2;
    static constexpr int fsx = 1, fsy = fex, fsz = cz ? 0 : fex * fey;
    static constexpr int csx = 1, csy = cz ? 24 : 12, csz = cz ? 0 : csy * cey;
    static constexpr int fvol = fex * fey * fez, cvol = csy * cey * cez;
    static constexpr int frow = fex, fplane = fex * fey, crow = csy, cplane = csy * cey;
    static_assert(csy >= cex, "current row padding");
    __device__ Tile64CT(const Gpd64TileArgs&) {}
    // the counters of destination cells live in the rows' padding (a third workgroup per CU would
    // not fit with an array of their own)
    static constexpr int pad = 2 * (csy - cex);
    static_assert(pad * cey * cez * 3 >= (TX + 2 * DEST_HALO) * (TY + 2 * DEST_HALO) * (cz ? 1 : TZ + 2 * DEST_HALO),
                  "room for the counters");
    __device__ int32_t* slot(double* cur, int s) const {
        return (int32_t*)(cur + (s / pad) * csy + cex) + s % pad;
    }
};

template <int O>
struct Tile64RT {
    int fex, fey, fez, cex, cey, cez, fsx, fsy, fsz, csx, csy, csz, fvol, cvol, frow, fplane, crow, cplane;
    __device__ Tile64RT(const Gpd64TileArgs& A) {
        const int* n = A.sp[0].n;
        const int grow = F64_LO + f64_hi(O);
        fex = n[0] == 1 ? 1 : A.t[0] + grow;
        fey = n[1] == 1 ? 1 : A.t[1] + grow;
        fez = n[2] == 1 ? 1 : A.t[2] + grow;
        cex = n[0] == 1 ? 1 : A.t[0] + grow + 2;
        cey = n[1] == 1 ? 1 : A.t[1] + grow + 2;
        cez = n[2] == 1 ? 1 : A.t[2] + grow + 2;
        frow = fex;
        fplane = fex * fey;
        crow = cex;
        cplane = cex * cey;
        fsx = n[0] == 1 ? 0 : 1;
        csx = fsx;
        fsy = n[1] == 1 ? 0 : frow;
        csy = n[1] == 1 ? 0 : crow;
        fsz = n[2] == 1 ? 0 : fplane;
        csz = n[2] == 1 ? 0 : cplane;
        fvol = fplane * fez;
        cvol = cplane * cez;
    }
    __device__ int32_t* slot(double* cur, int s) const { return (int32_t*)(cur + 3 * cvol) + s; }
};

template <int O, class TL>
__device__ __forceinline__ double gather64(const double* F, const TL& L, int bx, int by, int bz, const double* wx,
                                           const double* wy, const double* wz) {
    const double* base = F + bx * L.fsx + by * L.fsy + bz * L.fsz;
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c <= O; ++c) {
        double accy = 0.0;
#pragma unroll
        for (int b = 0; b <= O; ++b) {
            double s = 0.0;
#pragma unroll
            for (int a = 0; a <= O; ++a) s += base[c * L.fsz + b * L.fsy + a * L.fsx] * wx[a];
            accy += s * wy[b];
        }
        acc += accy * wz[c];
    }
    return acc;
}

// bin (tile-major cell index) of cell c
__device__ __forceinline__ int32_t bin_of(const Gpd64TileArgs& A, const int c[3]) {
    int tile = 0, lc = 0, mul = 1, tmul = 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        tile += (c[d] >> A.tsh[d]) * tmul;
        lc += (c[d] & (A.t[d] - 1)) * mul;
        mul *= A.t[d];
        tmul *= A.nt[d];
    }
    return tile * TILE_CELLS + lc;
}

// rank word of a particle that only names its bin
__device__ __forceinline__ int32_t name_bin(const Gpd64Args& S, int32_t bin) {
    atomicAdd(&S.named[bin], 1);
    return (int32_t)(0x80000000u | (uint32_t)bin);
}

// cell of entry q of a tile's destination window (se: its extents)
__device__ __forceinline__ void window_cell(const Gpd64Args& G, const int org[3], const int se[3], int q, int c[3]) {
    const int z = q / (se[0] * se[1]), r = q - z * se[0] * se[1], y = r / se[0], x = r - y * se[0];
    c[0] = se[0] == 1 ? 0 : wrap_near(org[0] + x - DEST_HALO, G.n[0]);
    c[1] = se[1] == 1 ? 0 : wrap_near(org[1] + y - DEST_HALO, G.n[1]);
    c[2] = se[2] == 1 ? 0 : wrap_near(org[2] + z - DEST_HALO, G.n[2]);
}

__device__ __forceinline__ void lds_add_f64(double* p, double v) {
    __hip_atomic_fetch_add((__attribute__((address_space(3))) double*)p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Steps 1-3 of particle p of the tile whose first cell is org, to slot q (its stored position also
// in Xn); false when a support of it leaves the tile's block (nothing done then).
template <int O, class TL>
__device__ __forceinline__ bool gpd64_in_tile(const Gpd64Args& A, const TL& L, const int org[3], const int t[3],
                                              const double* fld, double* cur, int64_t p, int64_t q,
                                              double Xn[3]) {
    double X0[3] = {A.pos[0][p], A.pos[1][p], A.pos[2][p]};
    V3<double> u{A.u[0][p], A.u[1][p], A.u[2][p]};
    const int fe[3] = {L.fex, L.fey, L.fez};
    int org_p[3];  // the tile's first cell in the particle's period
    V3<double> E, B;
    {
        double wc[3][O + 1], ws[3][O + 1];
        int fc[3], fs[3];
        bool inside = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int v = (int)floor(X0[d] + 0.5) - org[d];
            org_p[d] = org[d] + (v >= t[d] ? A.n[d] : (v < 0 ? -A.n[d] : 0));
            fc[d] = weights_abs<O>(X0[d], wc[d]) - org_p[d] + F64_LO;
            fs[d] = weights_abs<O>(X0[d] - 0.5, ws[d]) - org_p[d] + F64_LO;
            if (A.n[d] > 1)
                inside = inside && fc[d] >= 0 && fs[d] >= 0 && fc[d] <= fe[d] - 1 - O && fs[d] <= fe[d] - 1 - O;
        }
        if (!inside) return false;
        // eq. "pfields"
        E.x = gather64<O>(fld + 0 * L.fvol, L, fs[0], fc[1], fc[2], ws[0], wc[1], wc[2]);
        E.y = gather64<O>(fld + 1 * L.fvol, L, fc[0], fs[1], fc[2], wc[0], ws[1], wc[2]);
        E.z = gather64<O>(fld + 2 * L.fvol, L, fc[0], fc[1], fs[2], wc[0], wc[1], ws[2]);
        B.x = gather64<O>(fld + 3 * L.fvol, L, fc[0], fs[1], fs[2], wc[0], ws[1], ws[2]);
        B.y = gather64<O>(fld + 4 * L.fvol, L, fs[0], fc[1], fs[2], ws[0], wc[1], ws[2]);
        B.z = gather64<O>(fld + 5 * L.fvol, L, fs[0], fs[1], fc[2], ws[0], ws[1], wc[2]);
    }
    const V3<double> um = u;
    if (A.pusher == PP_PUSH_BORIS)
        push_boris<double>(A.h, A.ic, E, B, u);
    else
        push_vay<double>(A.h, A.ic, E, B, u);
    if (A.krad != 0.0) rad_cool<double>(A.krad, A.dtk, A.ic, um, u);

    const double g = sqrt(1.0 + dot(u, u) * A.ic * A.ic);
    const double uu[3] = {u.x, u.y, u.z};
    double X1[3];
    int bad = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        X1[d] = X0[d] + A.dt * uu[d] / (g * A.d[d]);
        if (fabs(X1[d] - X0[d]) >= 1.0) bad |= PP_FLAG_CFL;
        if (!isfinite(X1[d]) || !isfinite(uu[d])) bad |= PP_FLAG_NONFINITE;
    }
    if (bad) {  // left as it was
        atomic_or_flag(A.flags, bad);
        gpd64_store(A, q, X0, um, Xn);
        return true;
    }

    const int cst[3] = {L.csx, L.csy, L.csz};
    if (A.direct) {
        // direct current (eq. "jj2") at the time-centred position
        double wmc[3][O + 1], wms[3][O + 1];
        int bc[3], bs[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double Xm = 0.5 * (X0[d] + X1[d]);
            bc[d] = (weights_abs<O>(Xm, wmc[d]) - org_p[d] + F64_LO + 1) * cst[d];
            bs[d] = (weights_abs<O>(Xm - 0.5, wms[d]) - org_p[d] + F64_LO + 1) * cst[d];
        }
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            const double vq = A.qw * uu[comp] / g;
            double* Jc = cur + comp * L.cvol + (comp == 0 ? bs[0] : bc[0]) + (comp == 1 ? bs[1] : bc[1]) +
                         (comp == 2 ? bs[2] : bc[2]);
            const double* wx = comp == 0 ? wms[0] : wmc[0];
            const double* wy = comp == 1 ? wms[1] : wmc[1];
            const double* wz = comp == 2 ? wms[2] : wmc[2];
#pragma unroll
            for (int c = 0; c <= O; ++c)
#pragma unroll
                for (int b = 0; b <= O; ++b) {
                    const double wzy = vq * wz[c] * wy[b];
#pragma unroll
                    for (int a = 0; a <= O; ++a) lds_add_f64(Jc + c * cst[2] + b * cst[1] + a * cst[0], wzy * wx[a]);
                }
        }
    } else {
        // Esirkepov current (Sec. III.C) on the common window of O + 2 centred nodes per axis;
        // along an axis where the old and new supports coincide its last node carries nothing
        double S0[3][O + 2], DS[3][O + 2];
        int off0 = 0;
        bool moved[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double w0[O + 1], w1[O + 1];
            const int a0 = weights_abs<O>(X0[d], w0), a1 = weights_abs<O>(X1[d], w1);
            const bool lo1 = a1 < a0, hi1 = a1 > a0;
#pragma unroll
            for (int k = 0; k < O + 2; ++k) {
                const double s0 = lo1 ? (k >= 1 ? w0[k >= 1 ? k - 1 : 0] : 0.0) : (k <= O ? w0[k <= O ? k : O] : 0.0);
                const double s1 = hi1 ? (k >= 1 ? w1[k >= 1 ? k - 1 : 0] : 0.0) : (k <= O ? w1[k <= O ? k : O] : 0.0);
                S0[d][k] = s0;
                DS[d][k] = s1 - s0;
            }
            moved[d] = lo1 || hi1;
            off0 += ((lo1 ? a1 : a0) - org_p[d] + F64_LO + 1) * cst[d];
        }
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            const int d1 = comp == 0 ? 1 : (comp == 1 ? 2 : 0);
            const int d2 = comp == 0 ? 2 : (comp == 1 ? 0 : 1);
            double* Jc = cur + comp * L.cvol + off0;
            double P[O + 1];  // prefix sums along the component's axis (the last, a = O + 1, vanishes)
            double acc = 0.0;
#pragma unroll
            for (int a = 0; a <= O; ++a) {
                acc += DS[comp][a];
                P[a] = acc * A.fac[comp];
            }
#pragma unroll
            for (int b = 0; b < O + 2; ++b) {
                if (b == O + 1 && !moved[d1]) continue;
#pragma unroll
                for (int e = 0; e < O + 2; ++e) {
                    if (e == O + 1 && !moved[d2]) continue;
                    const double F = S0[d1][b] * (S0[d2][e] + 0.5 * DS[d2][e]) +
                                     DS[d1][b] * (0.5 * S0[d2][e] + DS[d2][e] * (1.0 / 3.0));
                    double* Jn = Jc + b * cst[d1] + e * cst[d2];
#pragma unroll
                    for (int a = 0; a <= O; ++a) {
                        if (a == O && !moved[comp]) continue;
                        lds_add_f64(Jn + a * cst[comp], P[a] * F);
                    }
                }
            }
        }
    }
    gpd64_wrap(A, X1);
    gpd64_store(A, q, X1, u, Xn);
    return true;
}

// Rounds first .. last - 1 (a wavefront takes every step-th, from first + its number) of the particles
// of species s0 .. s1 - 1 in a tile.
struct TileWork {
    int64_t tile;
    int s0, s1;
    int32_t first, last, step;
};

__device__ __forceinline__ int32_t tile_rounds(const Gpd64TileArgs& A, int s, int64_t tile) {
    return (A.bins[s][(tile + 1) * TILE_CELLS] - A.bins[s][tile * TILE_CELLS] + 63) / 64;
}

// What the tiles' own workgroups leave of tiles past A.heavy rounds a part, in chunks of A.chunk rounds
// numbered through species and tiles: finds the given one (the same in every lane).  A chunk is ranked
// like a workgroup of its own: its counts are reserved in the destination cells as theirs are.
__device__ __forceinline__ bool heavy_chunk(const Gpd64TileArgs& A, int number, double* lds, TileWork& W) {
    uint64_t* words = (uint64_t*)lds;
    const int32_t own = A.heavy * A.parts;
    const int64_t ntiles = A.list ? *A.list_count : A.ntiles;
    auto tile_at = [&](int64_t i) { return A.list ? (int64_t)A.list[i] : i; };
    for (int s = 0; s < A.nsp; ++s) {
        if (*A.tile_max[s] <= 64 * (int64_t)own) continue;
        for (int64_t base = 0; base < ntiles; base += GPD64_BS) {
            const int64_t t = base + threadIdx.x;
            const uint64_t heavy = __ballot(t < ntiles && tile_rounds(A, s, tile_at(t < ntiles ? t : 0)) > own);
            if ((threadIdx.x & 63) == 0) words[threadIdx.x >> 6] = heavy;
            __syncthreads();
            for (int w = 0; w < GPD64_BS / 64; ++w) {
                uint64_t left = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)words[w]) |
                                (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(words[w] >> 32)) << 32;
                for (; left != 0; left &= left - 1) {
                    const int64_t tile = tile_at(base + 64 * w + __ffsll((unsigned long long)left) - 1);
                    const int32_t rounds = tile_rounds(A, s, tile);
                    const int n = (rounds - own + A.chunk - 1) / A.chunk;
                    if (number < n) {
                        const int32_t first = own + number * A.chunk;
                        W = TileWork{tile, s, s + 1, first, first + A.chunk, 4};
                        __syncthreads();
                        return true;
                    }
                    number -= n;
                }
            }
            __syncthreads();
        }
    }
    return false;
}

// What bounds it: the LDS, 384 reads of 8 bytes for the cubic gather and up to 300 additions of
// 8 bytes per particle (ds_add_f64 runs at 9 clocks per wavefront where the 64 lanes' addresses
// differ and at 193 where they coincide), against 300 global FP64 atomics of the untiled kernel.
// 1.05e6 particles of a 64x16x16 two-stream box, cubic: 0.275 ms against 8.70; 9.9e5 of a 45x38x29
// pair plasma: 0.354 against 6.67; 6.6e4 of a 16^3 box, quadratic: 0.031 against 0.252.
// A workgroup takes the particles of one tile (a part of them where the box has few tiles).
// They lie in cell order, so lane l of a wavefront walks the l-th 64th of them: the 64 lanes
// then sit in different cells, mostly one each, and their LDS additions fall on different
// addresses; the four wavefronts take neighbouring particles of each lane's range and share its
// cache lines.  It also moves the particles into a pending sort order and ranks them for the next
// sort: 0.29 ms with both for the 1.05e6 particles, where the histogram and the scatter of a
// counting sort took 0.22 besides.
template <int O, class TL>
__global__ void __launch_bounds__(GPD64_BS, 3) k_gpd64_tile(Gpd64TileArgs A) {
    extern __shared__ __align__(16) double lds64[];
    const TL L(A);
    // blocks by tile, then by part, then by species (in a small box), and the helpers last
    const uint32_t row_blocks = 8 * (uint32_t)A.per_xcd;
    const int brow = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / row_blocks));
    const int bspecies = __builtin_amdgcn_readfirstlane(brow / A.parts);
    const uint32_t b = blockIdx.x - (uint32_t)brow * row_blocks;
    int64_t tile = (b & 7) * (int64_t)A.per_xcd + (b >> 3);
    int s0 = A.split > 1 ? bspecies : 0, s1 = A.split > 1 ? s0 + 1 : A.nsp;
    int first = 4 * (brow - bspecies * A.parts), most = A.heavy * A.parts, step = 4 * A.parts;
    if (bspecies >= A.split) {
        TileWork W;
        if (!heavy_chunk(A, (int)(blockIdx.x - row_blocks * (uint32_t)(A.parts * A.split)), lds64, W)) return;
        tile = __builtin_amdgcn_readfirstlane((int)W.tile);
        s0 = __builtin_amdgcn_readfirstlane(W.s0);
        s1 = s0 + 1;
        first = __builtin_amdgcn_readfirstlane(W.first);
        most = __builtin_amdgcn_readfirstlane(W.last);
        step = 4;
    } else if (A.list) {
        if ((int)b >= *A.list_count) return;
        tile = __builtin_amdgcn_readfirstlane(A.list[b]);
    }
    if (tile >= A.ntiles) return;
    int any = 0;
    for (int s = s0; s < s1; ++s) any |= A.bins[s][(tile + 1) * TILE_CELLS] - A.bins[s][tile * TILE_CELLS];
    if (any == 0) return;
    const Gpd64Args& G = A.sp[0];
    const uint32_t row = (uint32_t)tile / (uint32_t)A.nt[0], layer = row / (uint32_t)A.nt[1];  // numbered in 32 bits
    const int org[3] = {(int)((uint32_t)tile - row * (uint32_t)A.nt[0]) * A.t[0],
                        (int)(row - layer * (uint32_t)A.nt[1]) * A.t[1], (int)layer * A.t[2]};
    double* fld = lds64;
    double* cur = lds64 + 6 * L.fvol;
    const int se[3] = {A.sext[0], A.sext[1], A.sext[2]};
    const int nslots = se[0] * se[1] * se[2];
    for (int q = threadIdx.x; q < 3 * L.cvol; q += GPD64_BS) cur[q] = 0.0;
    for (int q = threadIdx.x; q < nslots; q += GPD64_BS) *L.slot(cur, q) = 0;
    for (int q = threadIdx.x; q < L.fvol; q += GPD64_BS) {
        const int c = q / L.fplane, r = q - c * L.fplane, b = r / L.frow, a = r - b * L.frow;
        const int i = G.n[0] == 1 ? 0 : wrap_near(org[0] - F64_LO + a, G.n[0]);
        const int j = G.n[1] == 1 ? 0 : wrap_near(org[1] - F64_LO + b, G.n[1]);
        const int k = G.n[2] == 1 ? 0 : wrap_near(org[2] - F64_LO + c, G.n[2]);
        const int64_t g = (int64_t)i + (int64_t)G.n[0] * (j + (int64_t)G.n[1] * k);
        double v[6];
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            v[comp] = G.E[comp * G.ncell + g];
            v[comp + 3] = G.B[comp * G.ncell + g];
        }
#pragma unroll
        for (int comp = 0; comp < 6; ++comp) fld[comp * L.fvol + q] = v[comp];
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int s = s0; s < s1; ++s) {
        const Gpd64Args& S = A.sp[s];
        const int32_t start = A.bins[s][tile * TILE_CELLS], end = A.bins[s][(tile + 1) * TILE_CELLS];
        const int32_t per = (end - start + 63) / 64, last = per < most ? per : most;
        for (int32_t r = first + wave; r < last; r += step) {
            const int64_t q = start + (int64_t)lane * per + r;
            if (q >= end) continue;
            const int64_t p = S.perm ? S.perm[q] : q;
            double Xn[3];
            if (S.id) S.id_o[q] = S.id[p];
            if (!gpd64_in_tile<O, TL>(S, L, org, A.t, fld, cur, p, q, Xn)) {
                if (S.defer) {
                    S.rank[q] = RANK_DEFERRED;
                    continue;
                }
                gpd64_particle<O, 1>(S, p, q, Xn);
            }
            // rank among the particles bound for the new cell: in the tile's neighbourhood counted
            // in LDS, else in the cell's count itself
            int c[3], sl = 0, mul = 1;
            bool win = true;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                c[d] = nearest_cell(Xn[d], G.n[d]);
                int x = c[d] - org[d];
                x += x >= A.t[d] + DEST_HALO ? -G.n[d] : (x < -DEST_HALO ? G.n[d] : 0);
                x = se[d] == 1 ? 0 : x + DEST_HALO;
                win = win && x >= 0 && x < se[d];
                sl += x * mul;
                mul *= se[d];
            }
            int32_t rank = -1;
            if (win) rank = atomicAdd(L.slot(cur, sl), 1);
            if (win && rank < F64_RANKS) {
                rank |= sl << 20;
            } else {
                if (win) atomicSub(L.slot(cur, sl), 1);  // past the word's range: counted below instead
                rank = name_bin(S, bin_of(A, c));
            }
            S.rank[q] = rank;
        }
        // reserve the workgroup's range in each destination cell's count, then complete the ranks
        __syncthreads();
        for (int q = threadIdx.x; q < nslots; q += GPD64_BS) {
            int32_t* slot = L.slot(cur, q);
            if (*slot == 0) continue;
            int c[3];
            window_cell(G, org, se, q, c);
            *slot = atomicAdd(&S.cnt[bin_of(A, c)], *slot);
        }
        __syncthreads();
        for (int32_t r = first + wave; r < last; r += step) {
            const int64_t q = start + (int64_t)lane * per + r;
            if (q >= end) continue;
            const int32_t w = S.rank[q];
            if (w < 0) continue;  // names its bin, or deferred
            const int sl = w >> 20;
            const int32_t rank = *L.slot(cur, sl) + (w & 0xFFFFF);
            if (rank < F64_RANKS) {
                S.rank[q] = (sl << 20) | rank;
            } else {  // past the word's range (the sort takes F64_RANKS of the cell's count for ranked)
                int c[3];
                window_cell(G, org, se, sl, c);
                S.rank[q] = name_bin(S, bin_of(A, c));
            }
        }
        __syncthreads();
        for (int q = threadIdx.x; q < nslots; q += GPD64_BS) *L.slot(cur, q) = 0;
        __syncthreads();
    }
    for (int q = threadIdx.x; q < L.cvol; q += GPD64_BS) {  // by node: its place in the mesh serves three components
        const int c = q / L.cplane, r = q - c * L.cplane, b = r / L.crow, a = r - b * L.crow;
        if (a >= L.cex) continue;  // padding
        const double v[3] = {cur[q], cur[L.cvol + q], cur[2 * L.cvol + q]};
        const int i = G.n[0] == 1 ? 0 : wrap_near(org[0] - F64_LO - 1 + a, G.n[0]);
        const int j = G.n[1] == 1 ? 0 : wrap_near(org[1] - F64_LO - 1 + b, G.n[1]);
        const int k = G.n[2] == 1 ? 0 : wrap_near(org[2] - F64_LO - 1 + c, G.n[2]);
        double* J = G.J + (int64_t)i + (int64_t)G.n[0] * (j + (int64_t)G.n[1] * k);
#pragma unroll
        for (int comp = 0; comp < 3; ++comp)
            if (v[comp] != 0.0) atomic_add_f64(J + comp * G.ncell, v[comp]);
    }
}

// A sparse box, before the tile kernel: tiles of more than A.few particles go to its list, the particles
// of the others are left to k_gpd64_deferred.
__global__ void __launch_bounds__(256) k_gpd64_sparse(Gpd64TileArgs A) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int32_t n = 0;
    if (t < A.ntiles)
        for (int s = 0; s < A.nsp; ++s) n += A.bins[s][(t + 1) * TILE_CELLS] - A.bins[s][t * TILE_CELLS];
    const uint64_t dense = __ballot(n > A.few);
    const int lane = threadIdx.x & 63;
    int32_t first = 0;
    if (lane == 0 && dense != 0) first = atomicAdd(A.list_count, (int32_t)__popcll(dense));
    first = __shfl(first, 0, 64);
    if (dense >> lane & 1) {
        A.list[first + (int32_t)__popcll(dense & ((1ull << lane) - 1ull))] = (int32_t)t;
        return;
    }
    if (n == 0) return;
    for (int s = 0; s < A.nsp; ++s)
        for (int32_t q = A.bins[s][t * TILE_CELLS]; q < A.bins[s][(t + 1) * TILE_CELLS]; ++q) {
            A.sp[s].rank[q] = RANK_DEFERRED;
            if (A.sp[s].id) A.sp[s].id_o[q] = A.sp[s].id[A.sp[s].perm ? A.sp[s].perm[q] : q];
        }
}

// Steps 1-3 of the particles that the tile kernel left out, as k_gpd64, and the bins they go to: those
// that do not lie in their tile where pp_get_particles has handed out the positions since the sort, so
// that there may be many, and those of a sparse box's tiles of a few particles.  (The tile kernel takes
// a stray one itself, with its loops over nodes rolled up, which holds up a wavefront for 0.3 ms.)  All
// species in one launch; a workgroup packs what it finds in DEFER_BLOCK slots.
// 64x16x16, 5e5 particles, cubic, 1 % of them moved elsewhere by the caller: 1.56 ms -> 0.31 for both
// kernels, 4.0 by k_gpd64 for all; 16^3, 3e4: 0.35 -> 0.15 and 0.28.  All of them moved: 4.3, 4.2 by k_gpd64.
constexpr int DEFER_BLOCK = 256;

template <int O>
__global__ void __launch_bounds__(256) k_gpd64_deferred(Gpd64TileArgs T) {
    __shared__ int32_t slot[DEFER_BLOCK];
    __shared__ int32_t count;
    const Gpd64Args& A = T.sp[blockIdx.y];
    if (!A.defer) return;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * DEFER_BLOCK;
    for (int i = threadIdx.x; i < DEFER_BLOCK && base + i < A.np; i += 256)
        if (A.rank[base + i] == RANK_DEFERRED) slot[atomicAdd(&count, 1)] = (int32_t)(base + i);
    __syncthreads();
    for (int i = threadIdx.x; i < count; i += 256) {
        const int32_t q = slot[i];
        double Xn[3];
        gpd64_particle<O, O + 2>(A, A.perm ? A.perm[q] : q, q, Xn);
        const int c[3] = {nearest_cell(Xn[0], A.n[0]), nearest_cell(Xn[1], A.n[1]), nearest_cell(Xn[2], A.n[2])};
        A.rank[q] = name_bin(A, bin_of(T, c));
    }
}

static void gpd64_args(const pp_run* r, int s, double* J, Gpd64Args& A) {
    const Species& S = r->sp[s];
    for (int d = 0; d < 3; ++d) {
        A.n[d] = r->p.n[d];
        A.d[d] = r->p.d[d];
        A.pos[d] = (const double*)S.cur.pos[d];
        A.u[d] = (const double*)S.cur.u[d];
        A.pos_o[d] = (double*)(S.pending ? S.cur.pos_alt[d] : S.cur.pos[d]);
        A.u_o[d] = (double*)(S.pending ? S.cur.u_alt[d] : S.cur.u[d]);
        A.fac[d] = -S.q * S.w * r->p.d[d] / r->dt_drift;
    }
    A.dt = r->dt_drift;
    A.dtk = r->dt_kick;
    A.ic = 1.0 / r->p.c;
    A.h = S.q * r->dt_kick / S.m;
    A.krad = r->p.rad_tau * S.q * S.q / S.m;
    A.np = S.n;
    A.perm = S.pending ? S.perm : nullptr;
    A.defer = S.handed_out ? 1 : 0;
    A.id = S.pending ? S.cur.id : nullptr;
    A.id_o = S.pending ? S.cur.id_alt : nullptr;
    A.cnt = S.cell_cnt;
    A.named = S.cell_cnt + r->g.nbins;
    A.rank = S.rank;
    A.E = r->mesh.E;
    A.B = r->mesh.B;
    A.J = J;
    A.ncell = r->g.ncell;
    A.flags = r->flags;
    A.pusher = r->p.pusher;
    A.direct = r->p.current_scheme == PP_CURRENT_DIRECT ? 1 : 0;
    A.qw = S.q * S.w;
}

hipError_t launch_gpd64(pp_run* r, int s, double* J) {
    const Species& S = r->sp[s];
    if (S.n == 0) return hipSuccess;
    Gpd64Args A;
    gpd64_args(r, s, J, A);
    const int bs = 256;
    const int64_t nb = (S.n + bs - 1) / bs;
    if (r->p.shape_order == 2)
        hipLaunchKernelGGL(k_gpd64<2>, dim3((unsigned)nb), dim3(bs), 0, r->stream, A);
    else
        hipLaunchKernelGGL(k_gpd64<3>, dim3((unsigned)nb), dim3(bs), 0, r->stream, A);
    return hipGetLastError();
}

template <int O, class TL>
static void launch_tile(const Gpd64TileArgs& A, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL((k_gpd64_tile<O, TL>), dim3((unsigned)(8 * A.per_xcd * A.parts * A.split + A.helpers)), dim3(GPD64_BS),
                       lds, st, A);
}

// LDS bytes of a tile of the runtime-shaped kernel.
static size_t runtime_tile_lds(const pp_run* r) {
    size_t fv = 1, cv = 1;
    for (int d = 0; d < 3; ++d) {
        const int grow = F64_LO + f64_hi(r->p.shape_order);
        fv *= r->p.n[d] == 1 ? 1 : r->g.t[d] + grow;
        cv *= r->p.n[d] == 1 ? 1 : r->g.t[d] + grow + 2;
    }
    return (6 * fv + 3 * cv) * sizeof(double) + r->g.dest_slots() * sizeof(int32_t);
}

template <int O>
static hipError_t launch_tiles(pp_run* r, const Gpd64TileArgs& A) {
    const int* n = r->p.n;
    const int* t = A.t;
    if (n[0] > 1 && n[1] > 1 && n[2] > 1 && t[0] == 4 && t[1] == 4 && t[2] == 4) {
        using TL = Tile64CT<O, 4, 4, 4>;
        launch_tile<O, TL>(A, (6 * TL::fvol + 3 * TL::cvol) * sizeof(double), r->stream);
    } else if (n[0] > 1 && n[1] > 1 && n[2] == 1 && t[0] == 8 && t[1] == 8 && t[2] == 1) {
        using TL = Tile64CT<O, 8, 8, 1>;
        launch_tile<O, TL>(A, (6 * TL::fvol + 3 * TL::cvol) * sizeof(double), r->stream);
    } else {
        launch_tile<O, Tile64RT<O>>(A, runtime_tile_lds(r), r->stream);
    }
    return hipGetLastError();
}

// How the particles of np are shared out.  256 CUs hold three workgroups each.
// Few tiles: a workgroup per tile, species and part of its particles, with as many parts (two to eight) as
// make the workgroups resident at once, 768, where each has a wavefront's worth of particles.  Two
// species, cubic, time with parts of at least 256 particles and in powers of two -> this: 8^3, 8 per cell
// 47 -> 34 us; 16^3, 8 per cell 47 -> 43; 64x64 flat, 20 per cell 39 -> 32; 24^3, 16 per cell 194 -> 168.
// Past 384 tiles and species two parts of each would be more than one round.  Up to three species are then
// taken together by a workgroup, in parts of the tile's that make one: 64x16x16 (256 tiles, two species),
// four steps of a bunched two-stream plasma 2.69 -> 2.50 ms, at 8 and 32 per cell without bunches 101 -> 91 us
// and 281 -> 287; 168 tiles of three 181 -> 177; 196 of two 147 -> 152; one species the same.  With more of them
// walking through the species costs more than the second round: 100 tiles of four, 8 and 32 per cell, 85
// and 271 us -> 103 and 271, 60 tiles of eight 105 and 288 -> 177 and 331.
// Many tiles: all species of a tile in one workgroup, which stages the fields once, unless that
// leaves the last round of workgroups mostly empty: 45x38x29 (960 tiles, 768 and 192) 393 -> 352 us
// with a workgroup per species, but 32^3 (512, two a CU) 184 -> 202.
static void plan_workgroups(Gpd64TileArgs& A, int64_t np) {
    const int64_t units = A.ntiles * A.nsp;
    A.parts = 1;
    A.split = A.nsp;
    if (units <= 512) {
        if (units > 384 && A.nsp <= 3) A.split = 1;
        const int64_t n = A.split == 1 ? A.ntiles : units;
        A.parts = (int)(768 / n < 2 ? 2 : (768 / n > 8 ? 8 : 768 / n));
        while (A.parts > 1 && np < units * A.parts * 64) --A.parts;
        return;
    }
    const int64_t slots = A.ntiles <= 768 ? 256 : 768, filled = (A.ntiles + slots - 1) / slots * slots;
    if (A.ntiles > 2 * 768 || 10 * A.ntiles >= 9 * filled) A.split = 1;
}

// A tile that holds a good part of all particles (a bunch, a point source of tracers) would keep one
// workgroup busy while the rest of the GPU is done.  What a workgroup would have to take of it past
// A.heavy rounds -- 64, or four times the mean -- goes to workgroups of their own, a chunk of rounds each;
// there are as many as np particles can make chunks, and where the sort found no tile that heavy they
// end after one load.  1e6 particles in one cell of a 64^3 box, cubic: 191 ms -> 1.6 (53 with the untiled
// kernel); in eight tiles 12.3 -> 0.93; spread evenly 0.31 either way.  Chunks of 256 rounds: 3.4 ms and 2.0.
static void plan_helpers(Gpd64TileArgs& A, int64_t np) {
    const int64_t mean = np / (64 * A.ntiles * A.nsp * A.parts), chunk = np / (64 * 256);
    A.chunk = (int)(chunk > 64 ? chunk : 64);
    A.heavy = (int)(4 * mean > A.chunk ? 4 * mean : A.chunk);
    // a tile of c particles, past heavy >= chunk rounds, has fewer than c / 64 / chunk chunks to share
    A.helpers = np < 64 * (int64_t)A.heavy ? 0 : (int)(np / (64 * (int64_t)A.chunk)) + 1;
}

// All species whose particles lie as the sort left them, in one launch; *done has a bit for each
// (the others take launch_gpd64).
hipError_t launch_gpd64_tiles(pp_run* r, double* J, unsigned* done) {
    Gpd64TileArgs A{};
    *done = 0;
    if (runtime_tile_lds(r) > 65536) return hipSuccess;  // thin tiles with a halo past the default LDS limit
    int64_t np = 0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        const Species& S = r->sp[s];
        if (!S.active || !S.binned || S.n == 0) continue;
        A.bins[A.nsp] = S.offsets;
        A.tile_max[A.nsp] = r->tile_max + s;
        gpd64_args(r, s, J, A.sp[A.nsp++]);
        *done |= 1u << s;
        np += S.n;
    }
    if (A.nsp == 0) return hipSuccess;
    for (int d = 0; d < 3; ++d) {
        A.t[d] = r->g.t[d];
        A.tsh[d] = 0;
        while ((1 << A.tsh[d]) < A.t[d]) ++A.tsh[d];
        A.nt[d] = r->g.nt[d];
        A.sext[d] = r->g.dest_ext(d);
    }
    A.ntiles = r->g.ntiles;
    A.per_xcd = (int)((A.ntiles + 7) / 8);
    plan_workgroups(A, np);
    plan_helpers(A, np);
    // A sparse box.  A tile takes a workgroup about 25 ns of the whole GPU's time (15 if flat) and 10 more a
    // further species, and a launch over all tiles 0.8 each; a particle by itself takes 7 ns, but 0.15 ms at
    // least.  So the tiles are listed first, those of a few particles only where all particles together
    // are few.  Push and sort, us, a workgroup per tile -> this, and the untiled kernel with a counting sort:
    // 200^3, 1000 particles 394 -> 202 (370); 2e4 877 -> 541 (524); 1e5 2122 -> 1160 (1200); 128^3, 2e4 485 ->
    // 326 (316).  Up to 16384 tiles and from 3 particles per tile of one species on it gains nothing.
    if (sparse_box(A.ntiles, np, A.nsp)) {
        A.list = r->sort_cursor;  // the counting sort's, which runs elsewhere
        A.list_count = r->tile_count;
        A.few = np > 8192 ? (r->p.n[2] == 1 ? 1 + A.nsp : 2 + 3 * A.nsp / 2) : 0;
        const hipError_t e = launch_fill_i32(r->tile_count, 1, 0, r->stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_gpd64_sparse, dim3((unsigned)((A.ntiles + 255) / 256)), dim3(256), 0, r->stream, A);
        const int64_t most = np / (A.few + 1);  // entries of the list
        A.per_xcd = (int)(((most < A.ntiles ? most : A.ntiles) + 7) / 8);
        for (int k = 0; k < A.nsp && A.few > 0; ++k) A.sp[k].defer = 1;
    }
    hipError_t e = r->p.shape_order == 2 ? launch_tiles<2>(r, A) : launch_tiles<3>(r, A);
    int64_t longest = 0;
    for (int k = 0; k < A.nsp; ++k)
        if (A.sp[k].defer && A.sp[k].np > longest) longest = A.sp[k].np;
    if (e != hipSuccess || longest == 0) return e;
    const dim3 grid((unsigned)((longest + DEFER_BLOCK - 1) / DEFER_BLOCK), (unsigned)A.nsp);
    if (r->p.shape_order == 2)
        hipLaunchKernelGGL(k_gpd64_deferred<2>, grid, dim3(256), 0, r->stream, A);
    else
        hipLaunchKernelGGL(k_gpd64_deferred<3>, grid, dim3(256), 0, r->stream, A);
    return hipGetLastError();
}

}  // namespace pp
