// Split-precision form of steps 1-3 (Sec. III), tiled.  Particles: int32 cell index +
// FP32 offset inside the cell + FP32 proper velocity (the paper's integer cell + fraction
// storage, Sec. V.B).  The offset is measured from the nearest node (lo = -1/2) for quadratic
// weights and from the node below (lo = 0) for cubic weights and lies in [lo, lo + 1), so
// that the centred support starts one node below the cell; a particle whose last
// displacement, repeated (scaled by the ratio of the next drift to this one inside a
// composed step), would take it across the lower face of its cell is kept in the cell
// below with its offset in [lo + 1, lo + 2).  Then the current window of the next step
// (old and new support) starts 2 nodes below the cell for almost every particle.
// Particles are stored per tile in pairs of ranks, 64 pairs to a chunk of 128 slots (see
// pp_sort.hip): the 64 first and the 64 second particles of a chunk each sit in different
// cells of the tile, in a full round all 64 cells in order, so the 64 lanes of a wavefront
// touch 64 aligned stencils, which the padded LDS layout spreads over all banks.
//
// One workgroup (4 wavefronts; more in small boxes) per tile of 64 cells:
//   1. stage E and B of the tile plus a 2-node halo from the FP64 mesh into LDS as FP32;
//   2. each wavefront takes 64 or 128 consecutive particles at a time (coalesced stores,
//      loads through the pending order): gather (LDS) -> push (registers) -> move and renormalise the split
//      position -> Esirkepov current (registers) -> LDS accumulation of the tile's current
//      block (halo of 2 nodes below and O + 1 above);
//   3. flush the current block to the global accumulator with 64-bit integer atomics.
// For the next sort each particle also gets its rank among the particles of its new cell:
// an LDS counter per destination cell of the tile's neighbourhood hands out ranks inside
// the tile, and one global atomic per destination cell then reserves the tile's range in that
// cell's count; the sort adds the start of that range, kept per tile and cell.
// Current accumulation is exact 64-bit fixed point.  Each contribution P_a * F * fac is
// formed in FP64 by one fused multiply-add with the rounding constant 1.5*2^52, whose bit
// pattern is then (constant bits + round(contribution * 2^e)); that pattern is added to the
// LDS block with an integer atomic (integer LDS atomics run at full rate on gfx950, FP32 LDS
// atomics at a small fraction of it).  The constant's share of a node's sum only touches bit
// 51 and above, so the sum of the rounded contributions is the sign-extended low 51 bits,
// recovered when the block is flushed; the scale 2^e (from the largest particle count of any
// tile) keeps every node's sum below 2^50 in magnitude.  The global accumulator adds the
// recovered integers, so the current is the exact sum of the rounded contributions,
// independent of summation order (bitwise deterministic).  A workgroup takes all species of its
// tile or, up to a few thousand tiles, one (see launch_tiles32).
#include <type_traits>

#include "pp_device.hpp"
#include "pp_fixed.hpp"
#include "pp_internal.hpp"

namespace pp {

struct Sp32 {
    const int32_t* start;  // tile starts (ntiles + 1)
    int32_t* cnt;          // particles per cell of the new positions (for the next sort)
    int32_t* rank;         // rank word of each particle (for the next sort, see pp_sort.hip)
    int32_t* base;         // per tile and destination cell: the rank its particles start from
    // A sort leaves the new order as a permutation: slot q of the tile order holds the
    // particle at index perm[q] of the input arrays, and the kernel writes slot q of the
    // output arrays (it moves the particles as it updates them).  perm == nullptr: in place.
    const int32_t* perm;
    const int32_t* cell;
    const float* pos[3];
    const float* u[3];
    int32_t* cell_o;
    float* pos_o[3];
    float* u_o[3];
    const int64_t* id;  // tags moved with the permutation (nullptr: none or in place)
    int64_t* id_o;
    float h;        // q dt / m
    float krad;     // radiative cooling constant rad_tau q^2 / m (0: off)
    double fac[3];  // -q w d_c / dt
    double qw;      // q w (direct current)
};

struct Gpd32Args {
    int n[3];
    int t[3];
    int nt[3];
    int64_t ntiles;
    int64_t nc;
    float dt;   // drift: positions and current
    float dtk;  // kick: momentum update (radiative cooling included)
    float pred; // next drift / this drift: the next displacement expected from this one
    float inv_d[3];
    float ic;
    int pusher;
    int nsp;
    Sp32 sp[PP_MAX_SPECIES];
    const double* E;
    const double* B;
    unsigned long long* Jq;  // fixed-point current accumulator (3 * nc, zero on entry)
    FixedScale scale;
    int32_t* flags;
    int per_xcd;
    int direct;   // PP_CURRENT_DIRECT: eq. "jj2" instead of the Esirkepov current
};

constexpr int GPD32_BS = 256;  // threads of a workgroup (small boxes take more, see launch_tiles32)
constexpr int STAGE_NODES = 3;  // nodes whose fields a thread loads before the first wait
constexpr double ROUND_MAGIC = 6755399441055744.0;  // 1.5 * 2^52
constexpr unsigned long long LOW51 = (1ull << 51) - 1ull;
constexpr long long BIT50 = 1ll << 50;

// sum of rounded contributions held in the low 51 bits of an accumulated bit pattern
__device__ __forceinline__ long long fixed_sum(unsigned long long v) {
    return (long long)((v & LOW51) ^ (unsigned long long)BIT50) - BIT50;
}

// Padded row and plane strides (64-bit elements) of the current block.  The 64 lanes of a
// round hold one particle per cell, so an accumulation instruction touches 64 addresses laid
// out like the tile's cells.  A 64-bit LDS access covers a pair of the 32 banks and is served
// 16 lanes at a time; lanes 16g..16g+15 are the 4x4 cells of one z layer (or two x rows of
// a flat 8x8 tile), and a row stride of 12 (24) puts those 16 addresses on 16 different bank
// pairs.  A plane stride that is a multiple of 16 keeps a window moved by one z layer on its
// bank pairs.
constexpr int cur_row_444 = 12;
constexpr int cur_plane_444(int O) { return O == 2 ? 112 : 128; }
constexpr int cur_row_881 = 24;
// Row and plane strides (floats) of the field tile of a 4x4x4 tile.  The gather reads two
// neighbouring floats per lane, half a wavefront at a time: the windows of 32 particles, one per
// cell of two z layers and each up to a node off its cell, over 64 banks.  A row of 10 and planes
// one short of nine (eight) such rows collide least of the strides near the extents 9 and 81 (8
// and 64): 1.3 accesses a read for random offsets, against 1.6 with planes of 90 and 2.3 with 8
// and 64.  Quadratic, 50x42x37: 471 -> 446 us; cubic, 128^3: 11.31 -> 11.25 ms.  A plane's last row
// is not padded.
constexpr int fld_row_444 = 10;
constexpr int fld_plane_444(int O) { return O == 3 ? 89 : 79; }

// LDS layout of a tile: compile-time for the common shapes, runtime otherwise.  A
// single-cell axis is collapsed (extent 1, stride 0): every node offset maps to plane 0.
// The current block is indexed x + crow*y + cplane*z (padding entries stay zero).
template <int O, int TX, int TY, int TZ, bool CZ, bool PAIRS>
struct TileCT {
    static constexpr bool fixed_shape = true;
    static constexpr int tx = TX, ty = TY, tz = TZ;
    static constexpr int flox = FLD_LO, floy = FLD_LO, floz = CZ ? 0 : FLD_LO;
    static constexpr int clox = cur_lo(O), cloy = cur_lo(O), cloz = CZ ? 0 : cur_lo(O);
    static constexpr int fex = TX + FLD_LO + fld_hi(O), fey = TY + FLD_LO + fld_hi(O);
    static constexpr int fez = CZ ? 1 : TZ + FLD_LO + fld_hi(O);
    static constexpr int cex = TX + cur_lo(O) + cur_hi(O), cey = TY + cur_lo(O) + cur_hi(O);
    static constexpr int cez = CZ ? 1 : TZ + cur_lo(O) + cur_hi(O);
    // destination cells: the tile and DEST_HALO around it
    static constexpr int dex = TX + 2 * DEST_HALO, dey = TY + 2 * DEST_HALO, dez = CZ ? 1 : TZ + 2 * DEST_HALO;
    static constexpr bool f444 = TX == 4 && TY == 4 && TZ == 4 && !CZ;
    static constexpr int frow = f444 ? fld_row_444 : fex;
    static constexpr int fplane = f444 ? fld_plane_444(O) : frow * fey;
    static constexpr int fsx = 1, fsy = frow, fsz = CZ ? 0 : fplane;
    static constexpr bool t444 = TX == 4 && TY == 4 && TZ == 4 && !CZ;
    static constexpr bool t881 = TX == 8 && TY == 8 && CZ;
    static constexpr int crow = t444 ? cur_row_444 : (t881 ? cur_row_881 : cex);
    static constexpr int cplane = t444 ? cur_plane_444(O) : crow * cey;
    static_assert(crow >= cex, "current row padding");
    static_assert(cplane >= crow * cey, "current plane padding");
    static constexpr int csx = 1, csy = crow, csz = CZ ? 0 : cplane;
    static_assert(frow >= fex && fplane >= frow * (fey - 1) + fex, "field tile padding");
    static constexpr int fvol = fplane * fez, cvol = cplane * cez;
    // two particles per lane (the paired deposit) on cubic tiles; flat tiles keep one per
    // lane, whose smaller register set leaves room for more resident wavefronts
    static constexpr bool pairs = PAIRS;
    static constexpr bool flat = CZ;  // one field plane: the gather's z taps read the same nodes
    __device__ TileCT(const Gpd32Args&) {}
};

template <int O, bool PAIRS>
using Tile444 = TileCT<O, 4, 4, 4, false, PAIRS>;
template <int O>
using Tile881 = TileCT<O, 8, 8, 1, true, false>;

template <int O>
struct TileRT {
    static constexpr bool fixed_shape = false;
    static constexpr bool pairs = false;
    static constexpr bool flat = false;
    int tx, ty, tz;
    int flox, floy, floz, clox, cloy, cloz;
    int fex, fey, fez, cex, cey, cez, dex, dey, dez;
    int fsx, fsy, fsz, csx, csy, csz;
    int crow, cplane, frow, fplane;
    int fvol, cvol;
    __device__ TileRT(const Gpd32Args& A) {
        tx = A.t[0];
        ty = A.t[1];
        tz = A.t[2];
        const bool one[3] = {A.n[0] == 1, A.n[1] == 1, A.n[2] == 1};
        constexpr int fgrow = FLD_LO + fld_hi(O), cgrow = cur_lo(O) + cur_hi(O), dgrow = 2 * DEST_HALO;
        flox = one[0] ? 0 : FLD_LO;
        floy = one[1] ? 0 : FLD_LO;
        floz = one[2] ? 0 : FLD_LO;
        clox = one[0] ? 0 : cur_lo(O);
        cloy = one[1] ? 0 : cur_lo(O);
        cloz = one[2] ? 0 : cur_lo(O);
        fex = one[0] ? 1 : tx + fgrow;
        fey = one[1] ? 1 : ty + fgrow;
        fez = one[2] ? 1 : tz + fgrow;
        cex = one[0] ? 1 : tx + cgrow;
        cey = one[1] ? 1 : ty + cgrow;
        cez = one[2] ? 1 : tz + cgrow;
        dex = one[0] ? 1 : tx + dgrow;
        dey = one[1] ? 1 : ty + dgrow;
        dez = one[2] ? 1 : tz + dgrow;
        fsx = A.n[0] > 1 ? 1 : 0;
        frow = fex;
        fplane = fex * fey;
        fsy = A.n[1] > 1 ? frow : 0;
        fsz = A.n[2] > 1 ? fplane : 0;
        crow = cex;
        cplane = cex * cey;
        csx = A.n[0] > 1 ? 1 : 0;
        csy = A.n[1] > 1 ? crow : 0;
        csz = A.n[2] > 1 ? cplane : 0;
        fvol = fplane * fez;
        cvol = cplane * cez;
    }
};

// Lower end of the offset range of the split form (see the header).
template <int O>
__device__ __forceinline__ constexpr float off_lo() {
    return O == 2 ? -0.5f : 0.0f;
}

template <int O>
__device__ __forceinline__ bool offset_ok(float f) {
    return f >= off_lo<O>() && f < off_lo<O>() + 2.0f;
}

// weights of the centred and staggered node sets for offset f of a particle in cell c;
// returned base offsets are relative to c.
template <int O>
__device__ __forceinline__ void split_weights(float f, float* wc, int& bc, float* ws, int& bs) {
    if (O == 2) {
        const float cn = floorf(f + 0.5f);  // nearest node: 0 or 1
        weights_frac<2, float>(f - cn, wc);  // nodes c-1+cn .. c+1+cn
        bc = -1 + (int)cn;
        const float cs = floorf(f);  // nearest staggered node c+cs+1/2, cs in -1..1
        weights_frac<2, float>(f - 0.5f - cs, ws);
        bs = -1 + (int)cs;
    } else {
        const float fl = floorf(f);  // 0 or 1
        weights_frac<3, float>(f - fl, wc);  // nodes c-1+fl .. c+2+fl
        bc = -1 + (int)fl;
        const float y = f - 0.5f;  // position on the staggered lattice
        const float fy = floorf(y);  // -1, 0 or 1
        weights_frac<3, float>(y - fy, ws);
        bs = -1 + (int)fy;
    }
}

// centred weights of a position c + x, x in (-3/2, 3/2): first node offset and weights
template <int O>
__device__ __forceinline__ int centred_weights(float x, float* w) {
    if (O == 2) {
        float cn = floorf(x + 0.5f);
        weights_frac<2, float>(x - cn, w);
        return (int)cn - 1;
    } else {
        float f = floorf(x);
        weights_frac<3, float>(x - f, w);
        return (int)f - 1;
    }
}

typedef __attribute__((address_space(3))) const float lds_cfloat;

template <int O, class TL>
__device__ __forceinline__ float gather_comp(const float* __restrict__ F, const TL& L, int bx, int by, int bz,
                                             const float* wx, const float* wy, const float* wz) {
    lds_cfloat* base = (lds_cfloat*)(F + bz * L.fsz + by * L.fsy + bx * L.fsx);
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c <= O; ++c) {
        // one address per plane, kept opaque: the plane's nodes are then small immediate
        // offsets of it (LDS paired reads reach 255 words; the stencil spans more than that).
        // A flat tile has one plane, whose reads the compiler shares between the z taps.
        lds_cfloat* plane = base + c * L.fsz;
        if constexpr (!TL::flat) asm volatile("" : "+v"(plane));
        float accy = 0.f;
#pragma unroll
        for (int b = 0; b <= O; ++b) {
            float s = 0.f;
#pragma unroll
            for (int a = 0; a <= O; ++a) s += plane[b * L.fsy + a * L.fsx] * wx[a];
            accy += s * wy[b];
        }
        acc += accy * wz[c];
    }
    return acc;
}

// Rank of a particle among those bound for its destination cell: rel = destination cell
// relative to the tile origin (unwrapped), gcell = its linear index.  Inside the tile's
// window the rank comes from the LDS counter of that cell (slot << 20 | rank in the tile; the
// sort adds the cell's range start); otherwise from the global count directly (bit 31 set).
template <class TL>
__device__ __forceinline__ int32_t dest_rank(const Sp32& S, const TL& L, int32_t* slots, const int rel[3], int32_t gcell) {
    const int x = L.dex == 1 ? 0 : rel[0] + DEST_HALO, y = L.dey == 1 ? 0 : rel[1] + DEST_HALO;
    const int z = L.dez == 1 ? 0 : rel[2] + DEST_HALO;
    if ((unsigned)x < (unsigned)L.dex && (unsigned)y < (unsigned)L.dey && (unsigned)z < (unsigned)L.dez) {
        const int sl = x + L.dex * (y + L.dey * z);
        const int32_t r = atomicAdd(&slots[sl], 1);
        if (r < (1 << 20)) return (sl << 20) | r;
        atomicSub(&slots[sl], 1);  // past the word's range: counted below instead
    }
    return (int32_t)(0x80000000u | (uint32_t)atomicAdd(gl(S.cnt) + gcell, 1));
}

// What the charge-conserving deposit of one particle needs, kept in registers between its step
// and its deposit: the old offset, the new position relative to the old cell and the cell's
// place in the tile (the window is built from them at deposit time).
template <int O>
struct Win {
    float f[3], x1[3];
    int loc[3];
    bool dep;
};

// The Esirkepov window of a particle: S0 and DS = S1 - S0 on the O + 2 centred nodes per axis
// covering the old and the new support, the window's first node in the tile's current block,
// and which axes the supports differ on.
template <int O, class TL>
__device__ __forceinline__ void make_window(const TL& L, const Win<O>& W, float S0[3][O + 2], float DS[3][O + 2],
                                            int wb[3], int& moved) {
    const int clo[3] = {L.clox, L.cloy, L.cloz};
    moved = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        float w0[O + 1], w1[O + 1];
        const int a0 = centred_weights<O>(W.f[d], w0);
        const int a1 = centred_weights<O>(W.x1[d], w1);
        const bool lo1 = a1 < a0;  // the new support starts one node lower
        const bool hi1 = a1 > a0;
        const int bmin = lo1 ? a1 : a0;
#pragma unroll
        for (int kk = 0; kk < O + 2; ++kk) {
            // old weights sit at window offset (a0 - bmin), new at (a1 - bmin)
            const float s0 = lo1 ? (kk >= 1 ? w0[kk - 1 < O ? kk - 1 : O] : 0.f) : (kk <= O ? w0[kk <= O ? kk : O] : 0.f);
            const float s1 = hi1 ? (kk >= 1 ? w1[kk - 1 < O ? kk - 1 : O] : 0.f) : (kk <= O ? w1[kk <= O ? kk : O] : 0.f);
            S0[d][kk] = s0;
            DS[d][kk] = s1 - s0;
        }
        wb[d] = W.loc[d] + clo[d] + bmin;
        moved |= (lo1 || hi1) ? 1 << d : 0;
    }
}

// First node of a particle's window along axis d (as make_window), without the weights.
template <int O, class TL>
__device__ __forceinline__ int window_start(const TL& L, const Win<O>& W, int d) {
    const int clo[3] = {L.clox, L.cloy, L.cloz};
    const int a0 = O == 2 ? (int)floorf(W.f[d] + 0.5f) - 1 : (int)floorf(W.f[d]) - 1;
    const int a1 = O == 2 ? (int)floorf(W.x1[d] + 0.5f) - 1 : (int)floorf(W.x1[d]) - 1;
    return W.loc[d] + clo[d] + (a1 < a0 ? a1 : a0);
}

// What the particle step of one tile and species needs besides the arguments.
struct TileCtx {
    int org[3];
    uint32_t base_cell, nxy;  // of 32 bits as the particles' cell indices are
    const float* fld;
    unsigned long long* cur;
    int32_t* slots;
    double* facq;  // LDS: -q w d_c / dt per axis and q w (direct current), times the fixed-point scale
};

// The particle step of slot q (gather, push, move, renormalise, store, rank for the next sort;
// the direct current is deposited here).  For the charge-conserving current the window is left
// in W for the deposit (W.dep = false when the particle deposits nothing: left as it was, or
// the direct scheme).
template <int O, class TL>
__device__ __forceinline__ void step_particle(const Gpd32Args& A, const Sp32& S, const TL& L, const TileCtx& C,
                                              int32_t q, Win<O>& W, int& bad_all) {
    W.dep = false;
    const int n0 = A.n[0], n1 = A.n[1], n2 = A.n[2];
    const int32_t p = S.perm ? gl(S.perm)[q] : q;
    if (p < 0) {  // an empty slot (counts made inconsistent by flagged particles)
        gl(S.rank)[q] = -1;
        return;
    }
    const int32_t cell = gl(S.cell)[p];
    float f[3] = {gl(S.pos[0])[p], gl(S.pos[1])[p], gl(S.pos[2])[p]};
    V3<float> u{gl(S.u[0])[p], gl(S.u[1])[p], gl(S.u[2])[p]};
    if (S.id) gl(S.id_o)[q] = gl(S.id)[p];
    // a particle left as it is still moves to its slot when the kernel reorders
    auto keep = [&](const V3<float>& uk) {
        if (!S.perm) return;
        gl(S.cell_o)[q] = cell;
        gl(S.pos_o[0])[q] = f[0];
        gl(S.pos_o[1])[q] = f[1];
        gl(S.pos_o[2])[q] = f[2];
        gl(S.u_o[0])[q] = uk.x;
        gl(S.u_o[1])[q] = uk.y;
        gl(S.u_o[2])[q] = uk.z;
    };
    // position inside the tile: rel = li + n0 lj + n0 n1 lk with l < t, found by
    // comparisons (no division)
    uint32_t rel = (uint32_t)cell - C.base_cell;
    int lk = 0, lj = 0;
    if constexpr (TL::fixed_shape) {
#pragma unroll
        for (int k = 1; k < TL::tz; ++k) lk += rel >= k * C.nxy ? 1 : 0;
        rel -= lk * C.nxy;
#pragma unroll
        for (int k = 1; k < TL::ty; ++k) lj += rel >= (uint32_t)(k * n0) ? 1 : 0;
        rel -= lj * n0;
    } else {
        while (lk < L.tz - 1 && rel >= C.nxy) {
            rel -= C.nxy;
            ++lk;
        }
        while (lj < L.ty - 1 && rel >= (uint32_t)n0) {
            rel -= n0;
            ++lj;
        }
    }
    const int li = (int)rel;
    const int loc[3] = {li, lj, lk};
    const int* org = C.org;
    // the particle must lie in this tile (the cell index rebuilt from li, lj and lk is the stored one)
    const bool inside = rel < (uint32_t)L.tx && org[0] + li < n0 && org[1] + lj < n1 && org[2] + lk < n2;
    if (!inside) {  // not this tile's particle: left out of the next sort
        bad_all |= PP_FLAG_OUT_OF_TILE;
        keep(u);
        gl(S.rank)[q] = -1;
        return;
    }
    if (!offset_ok<O>(f[0]) || !offset_ok<O>(f[1]) || !offset_ok<O>(f[2])) {  // left as it is
        bad_all |= PP_FLAG_OUT_OF_TILE;
        keep(u);
        gl(S.rank)[q] = dest_rank<TL>(S, L, C.slots, loc, cell);
        return;
    }

    // gather (eq. "pfields") from the LDS field tile
    float wc[3][O + 1], ws[3][O + 1];
    int fc[3], fs[3];
    {
        const int flo[3] = {L.flox, L.floy, L.floz};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int bc, bs;
            split_weights<O>(f[d], wc[d], bc, ws[d], bs);
            fc[d] = loc[d] + flo[d] + bc;
            fs[d] = loc[d] + flo[d] + bs;
        }
    }
    const float* fld = C.fld;
    V3<float> E, B;
    E.x = gather_comp<O>(fld + 0 * L.fvol, L, fs[0], fc[1], fc[2], ws[0], wc[1], wc[2]);
    E.y = gather_comp<O>(fld + 1 * L.fvol, L, fc[0], fs[1], fc[2], wc[0], ws[1], wc[2]);
    E.z = gather_comp<O>(fld + 2 * L.fvol, L, fc[0], fc[1], fs[2], wc[0], wc[1], ws[2]);
    B.x = gather_comp<O>(fld + 3 * L.fvol, L, fc[0], fs[1], fs[2], wc[0], ws[1], ws[2]);
    B.y = gather_comp<O>(fld + 4 * L.fvol, L, fs[0], fc[1], fs[2], ws[0], wc[1], ws[2]);
    B.z = gather_comp<O>(fld + 5 * L.fvol, L, fs[0], fs[1], fc[2], ws[0], ws[1], wc[2]);

    const V3<float> um = u;
    if (A.pusher == PP_PUSH_BORIS)
        push_boris<float>(S.h, A.ic, E, B, u);
    else
        push_vay<float>(S.h, A.ic, E, B, u);
    if (S.krad != 0.0f) rad_cool<float>(S.krad, A.dtk, A.ic, um, u);

    const float ig = rsqrtf(1.0f + dot(u, u) * A.ic * A.ic);
    const float uu[3] = {u.x, u.y, u.z};
    float x1[3], dxs[3];
    int bad = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float dd = A.dt * uu[d] * ig * A.inv_d[d];
        if (!(fabsf(dd) < 1.0f)) bad |= isfinite(dd) ? PP_FLAG_CFL : PP_FLAG_NONFINITE;
        if (!isfinite(uu[d])) bad |= PP_FLAG_NONFINITE;
        x1[d] = f[d] + dd;  // new position relative to the old cell's node
        dxs[d] = dd;
    }
    if (bad) {  // left as it was before the push
        bad_all |= bad;
        keep(um);
        gl(S.rank)[q] = dest_rank<TL>(S, L, C.slots, loc, cell);
        return;
    }

    if (A.direct) {
        // direct current (eq. "jj2"): q w v_c W at J_c's staggered nodes, at the
        // time-centred offset f + dd/2 (its supports stay inside the block's halo)
        float wcm[3][O + 1], wsm[3][O + 1];
        int ncm[3], nsm[3];
        const int clo[3] = {L.clox, L.cloy, L.cloz};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int bc, bs;
            split_weights<O>(f[d] + 0.5f * dxs[d], wcm[d], bc, wsm[d], bs);
            ncm[d] = loc[d] + clo[d] + bc;
            nsm[d] = loc[d] + clo[d] + bs;
        }
        const int cst[3] = {L.csx, L.csy, L.csz};
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            unsigned long long* Jc = C.cur + comp * L.cvol;
            const double vq = C.facq[3] * (double)(uu[comp] * ig);
            const int n0x = comp == 0 ? nsm[0] : ncm[0];
            const int n0y = comp == 1 ? nsm[1] : ncm[1];
            const int n0z = comp == 2 ? nsm[2] : ncm[2];
            const float* wx = comp == 0 ? wsm[0] : wcm[0];
            const float* wy = comp == 1 ? wsm[1] : wcm[1];
            const float* wz = comp == 2 ? wsm[2] : wcm[2];
            if constexpr (TL::flat) {  // the z nodes are one: their contributions take one atomic, as in deposit_flat
#pragma unroll
                for (int b = 0; b <= O; ++b) {
                    unsigned long long sum[O + 1];
#pragma unroll
                    for (int c = 0; c <= O; ++c) {
                        const double wzy = vq * (double)(wz[c] * wy[b]);
#pragma unroll
                        for (int a = 0; a <= O; ++a) {
                            const double dq = fma(wzy, (double)wx[a], ROUND_MAGIC);
                            sum[a] = (c == 0 ? 0ull : sum[a]) + (unsigned long long)__double_as_longlong(dq);
                        }
                    }
#pragma unroll
                    for (int a = 0; a <= O; ++a) atomicAdd(Jc + (n0x + a) * cst[0] + (n0y + b) * cst[1], sum[a]);
                }
                continue;
            }
#pragma unroll
            for (int c = 0; c <= O; ++c) {
#pragma unroll
                for (int b = 0; b <= O; ++b) {
                    const double wzy = vq * (double)(wz[c] * wy[b]);
                    const int rowo = n0x * cst[0] + (n0y + b) * cst[1] + (n0z + c) * cst[2];
#pragma unroll
                    for (int a = 0; a <= O; ++a) {
                        const double dq = fma(wzy, (double)wx[a], ROUND_MAGIC);
                        atomicAdd(Jc + rowo + a * cst[0], (unsigned long long)__double_as_longlong(dq));
                    }
                }
            }
        }
    } else {
        // the charge-conserving current is deposited later, from these
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            W.f[d] = f[d];
            W.x1[d] = x1[d];
            W.loc[d] = loc[d];
        }
        W.dep = true;
    }

    // renormalise: new cell and offset in [lo, lo + 1), or in [lo + 1, lo + 2) in the
    // cell below when the next displacement (this one times the ratio of the next drift
    // to this one) would cross the lower face
    int nc3[3], shv[3];
    float fn[3];
    const int gc[3] = {org[0] + li, org[1] + lj, org[2] + lk};
    const float lo = off_lo<O>();
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        float sh = floorf(x1[d] - lo);
        float o = x1[d] - sh;
        // rounding can land the offset just outside the range: move it back in
        if (o < lo) {
            o += 1.0f;
            sh -= 1.0f;
        } else if (o >= lo + 1.0f) {
            o -= 1.0f;
            sh += 1.0f;
        }
        const float up = o + 1.0f;
        if (o + dxs[d] * A.pred < lo && up < lo + 2.0f) {
            o = up;
            sh -= 1.0f;
        }
        fn[d] = o;
        shv[d] = (int)sh;
        nc3[d] = wrap_near(gc[d] + (int)sh, A.n[d]);
    }
    const int32_t newcell = nc3[0] + n0 * (nc3[1] + n1 * nc3[2]);
    gl(S.cell_o)[q] = newcell;
    gl(S.pos_o[0])[q] = fn[0];
    gl(S.pos_o[1])[q] = fn[1];
    gl(S.pos_o[2])[q] = fn[2];
    gl(S.u_o[0])[q] = u.x;
    gl(S.u_o[1])[q] = u.y;
    gl(S.u_o[2])[q] = u.z;
    const int dst[3] = {li + shv[0], lj + shv[1], lk + shv[2]};
    gl(S.rank)[q] = dest_rank<TL>(S, L, C.slots, dst, newcell);
}

// sum over the four lanes of a quad (where all of them are active)
__device__ __forceinline__ unsigned long long quad_sum(unsigned long long v) {
#pragma unroll
    for (int step = 0; step < 2; ++step) {
        int lo = (int)v, hi = (int)(v >> 32);
        lo = step == 0 ? __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, true);
        hi = step == 0 ? __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, true);
        v += (unsigned long long)(unsigned)lo | (unsigned long long)(unsigned)hi << 32;
    }
    return v;
}

// Charge-conserving current of one particle (W1), or of two particles whose windows start at
// the same node of the block (W1 and W2, PAIR): per component the prefix sums of DS along the
// component's axis times the scaled factor, P_a, and for every transverse node pair the
// factor F = S0_1 (S0_2 + DS_2/2) + DS_1 (S0_2/2 + DS_2/3); each node then receives the bits
// of (1.5*2^52 + round(P_a F)) in one 64-bit integer atomic.  For a pair the two patterns,
// each rounded on its own, are added as integers before the one atomic, so the node gets the
// same exact fixed-point sum as from two atomics.  f2 != 0 marks lanes whose second particle
// deposits; on the others its prefix sums are zeros, so that its patterns are 1.5*2^52 itself,
// whose low 51 bits are zero (the caller keeps that particle's window state finite).
template <int O, class TL, bool PAIR>
__device__ __forceinline__ void deposit_cc(const TL& L, unsigned long long* cur, const Win<O>& P1, const double* facq1,
                                           const Win<O>& P2, const double* facq2, float f2) {
    float S0a[3][O + 2], DSa[3][O + 2], S0b[3][O + 2], DSb[3][O + 2];
    int wb[3], wb2[3], moved1, moved2 = 0;
    make_window<O, TL>(L, P1, S0a, DSa, wb, moved1);
    if (PAIR) make_window<O, TL>(L, P2, S0b, DSb, wb2, moved2);
    struct WinF {
        const float (*S0)[O + 2];
        const float (*DS)[O + 2];
    } W1{S0a, DSa}, W2{S0b, DSb};
    const int cst[3] = {L.csx, L.csy, L.csz};
    const bool use2 = PAIR && f2 != 0.0f;
    const int moved = use2 ? (moved1 | moved2) : moved1;
    bool in_quad = false;
    auto deposit = [&](auto quads) {
        constexpr bool QUADS = decltype(quads)::value;
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
        const int d1 = comp == 0 ? 1 : (comp == 1 ? 2 : 0);
        const int d2 = comp == 0 ? 2 : (comp == 1 ? 0 : 1);
        unsigned long long* Jc = cur + comp * L.cvol;
        const int off0 = wb[0] * L.csx + wb[1] * L.csy + wb[2] * L.csz;
        // prefix sums of DS along the component's own axis (the last one vanishes),
        // scaled to fixed-point units: P_a * fac * 2^e in FP64
        // A particle whose supports coincide along the component's axis contributes nothing
        // at the last node even when its partner's does: its last prefix sum is only the
        // rounding residue of a vanishing sum, which the single deposit leaves out too.
        const bool own1 = (moved1 >> comp) & 1, own2 = (moved2 >> comp) & 1;
        double Pq1[O + 1], Pq2[O + 1];
        float acc1 = 0.f, acc2 = 0.f;
#pragma unroll
        for (int a = 0; a <= O; ++a) {
            acc1 += W1.DS[comp][a];
            Pq1[a] = (a < O || own1) ? (double)acc1 * facq1[comp] : 0.0;
            if (PAIR) {  // zero for a second particle that deposits nothing
                acc2 += W2.DS[comp][a];
                Pq2[a] = (use2 && (a < O || own2)) ? (double)acc2 * facq2[comp] : 0.0;
            }
        }
        const bool m1 = (moved >> d1) & 1, m2 = (moved >> d2) & 1, mc = (moved >> comp) & 1;
        // Along an axis where the supports coincide the window's last node carries no
        // weight (its transverse factors are exactly zero) and the last prefix sum is
        // the rounding residue of a vanishing sum: those additions are left out.
#pragma unroll
        for (int bq = 0; bq < O + 2; ++bq) {
            if (bq == O + 1 && !m1) continue;
            const float g1 = W1.S0[d1][bq], h1 = W1.DS[d1][bq];
            const float g2 = PAIR ? W2.S0[d1][bq] : 0.f, h2 = PAIR ? W2.DS[d1][bq] : 0.f;
#pragma unroll
            for (int e = 0; e < O + 2; ++e) {
                if (e == O + 1 && !m2) continue;
                const double Fd1 = (double)(g1 * (W1.S0[d2][e] + 0.5f * W1.DS[d2][e]) +
                                            h1 * (0.5f * W1.S0[d2][e] + (1.0f / 3.0f) * W1.DS[d2][e]));
                double Fd2 = 0.0;
                if (PAIR)
                    Fd2 = (double)(g2 * (W2.S0[d2][e] + 0.5f * W2.DS[d2][e]) +
                                   h2 * (0.5f * W2.S0[d2][e] + (1.0f / 3.0f) * W2.DS[d2][e]));
                const int rowo = off0 + bq * cst[d1] + e * cst[d2];
#pragma unroll
                for (int a = 0; a <= O; ++a) {
                    if (a == O && !mc) continue;
                    // bits of (1.5*2^52 + round(P_a F fac 2^e)): see the header.  A pair
                    // adds its two patterns as integers: each contribution is rounded on its
                    // own, as by two atomics (a chained FMA would round the second one
                    // against the first, and a tie could then round the other way).
                    unsigned long long bits = (unsigned long long)__double_as_longlong(fma(Pq1[a], Fd1, ROUND_MAGIC));
                    if (PAIR) bits += (unsigned long long)__double_as_longlong(fma(Pq2[a], Fd2, ROUND_MAGIC));
                    if constexpr (QUADS) {
                        const unsigned long long sum = quad_sum(bits);
                        bits = in_quad ? sum : bits;
                        if (in_quad && (threadIdx.x & 3) != 0) continue;
                    }
                    atomicAdd(Jc + rowo + a * cst[comp], bits);
                }
            }
        }
    }
    };
    if constexpr (!PAIR && !TL::pairs && TL::fixed_shape) {
        // Half of the quads of neighbouring lanes on the same nodes: particles crowded into a cell or two,
        // whose additions to one address are served one after another.  A quad then adds its sum (of
        // patterns, each rounded on its own).  32^3, one cell with 2e4 or 1e6 particles: 2.5 ms
        // and 125 -> 0.83 and 42 (1.55 and 78 in pairs).
        const int key = (wb[0] * L.csx + wb[1] * L.csy + wb[2] * L.csz) * 8 + moved;
        const uint64_t same = __ballot(__builtin_amdgcn_mov_dpp(key, 0x00, 0xF, 0xF, true) == key);
        const uint64_t whole = same & same >> 1 & same >> 2 & same >> 3 & 0x1111111111111111ull;
        if (__popcll(whole) >= 8) {
            in_quad = whole >> (threadIdx.x & 60) & 1;
            deposit(std::true_type{});
            return;
        }
    }
    deposit(std::false_type{});
}

// The same for a flat tile, whose z nodes are all one: what a particle adds to a node of the block
// for the O + 2 nodes of its window along z is summed in a register, pattern by pattern (each
// contribution still rounded on its own, so the same exact sum), and takes one atomic.  A lane whose
// supports coincide along z adds the zeros of its last node where another lane's do not.
// Cubic, a particle that crosses no face: 40 atomics instead of 144, which had held the kernel to
// the LDS's rate.  512x256, 2 x 8.4e6 particles: 990 us with an atomic per contribution, 780 now.
template <int O, class TL>
__device__ __forceinline__ void deposit_flat(const TL& L, unsigned long long* cur, const Win<O>& P1, const double* facq) {
    float S0[3][O + 2], DS[3][O + 2];
    int wb[3], moved;
    make_window<O, TL>(L, P1, S0, DS, wb, moved);
    const bool mv[3] = {(moved & 1) != 0, (moved & 2) != 0, (moved & 4) != 0};
    const bool any_z = __any(mv[2]);
    const int cst[2] = {L.csx, L.csy};
    const int off0 = wb[0] * L.csx + wb[1] * L.csy;
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
        const int d1 = comp == 0 ? 1 : (comp == 1 ? 2 : 0);
        const int d2 = comp == 0 ? 2 : (comp == 1 ? 0 : 1);
        unsigned long long* Jc = cur + comp * L.cvol + off0;
        double Pq[O + 1];
        float acc = 0.f;
#pragma unroll
        for (int a = 0; a <= O; ++a) {
            acc += DS[comp][a];
            Pq[a] = (a < O || mv[comp]) ? (double)acc * facq[comp] : 0.0;
        }
        auto factor = [&](int b, int e) {
            return (double)(S0[d1][b] * (S0[d2][e] + 0.5f * DS[d2][e]) +
                            DS[d1][b] * (0.5f * S0[d2][e] + (1.0f / 3.0f) * DS[d2][e]));
        };
        auto pattern = [&](int a, double F) {
            return (unsigned long long)__double_as_longlong(fma(Pq[a], F, ROUND_MAGIC));
        };
        if (comp < 2) {
            const int t = 1 - comp;  // the transverse axis that is not z
#pragma unroll
            for (int b = 0; b < O + 2; ++b) {
                if (b == O + 1 && !mv[t]) continue;
                unsigned long long sum[O + 1];
#pragma unroll
                for (int z = 0; z < O + 2; ++z) {
                    if (z == O + 1 && !any_z) continue;
                    const double F = comp == 0 ? factor(b, z) : factor(z, b);
#pragma unroll
                    for (int a = 0; a <= O; ++a) sum[a] = z == 0 ? pattern(a, F) : sum[a] + pattern(a, F);
                }
#pragma unroll
                for (int a = 0; a <= O; ++a) {
                    if (a == O && !mv[comp]) continue;
                    atomicAdd(Jc + b * cst[t] + a * cst[comp], sum[a]);
                }
            }
        } else {
#pragma unroll
            for (int b = 0; b < O + 2; ++b) {
                if (b == O + 1 && !mv[0]) continue;
#pragma unroll
                for (int e = 0; e < O + 2; ++e) {
                    if (e == O + 1 && !mv[1]) continue;
                    const double F = factor(b, e);
                    unsigned long long sum = pattern(0, F);
#pragma unroll
                    for (int a = 1; a <= O; ++a) {
                        if (a == O && !any_z) continue;
                        sum += pattern(a, F);
                    }
                    atomicAdd(Jc + b * cst[0] + e * cst[1], sum);
                }
            }
        }
    }
}

// One tile of one run: the whole particle step of the tile's particles of species slots s0 to s1
// (the body shared by the single-run kernel and the batched kernel, so both do identical
// arithmetic).
// Each wavefront takes 128 consecutive slots at a time, lane l the slots l and 64 + l.  In
// the chunks of pairs of the tile order both are a particle of the same cell, whose current
// windows start at the same node unless one of the particles crossed a face the storage did
// not expect; such pairs deposit together with one atomic per node for both.  Where some
// lane's pair does not share a window, that lane's second particle deposits alone in a second
// pass; where no lane's does (the single particles after the chunks), each particle deposits
// alone.  Flat (8x8x1) and runtime-shaped tiles and small boxes take one particle per lane and slot
// (64 consecutive slots per wavefront).
template <int O, class TL, int BS>
__device__ __forceinline__ void gpd32_tile(const Gpd32Args& A, int64_t tile, int s0, int s1, unsigned char* lds_raw) {
    const TL L(A);
    const uint32_t tile32 = (uint32_t)tile, row = tile32 / (uint32_t)A.nt[0];  // tiles are numbered in 32 bits
    const int ti = (int)(tile32 - row * (uint32_t)A.nt[0]);
    const int tk = (int)(row / (uint32_t)A.nt[1]);
    const int tj = (int)(row - (uint32_t)tk * (uint32_t)A.nt[1]);
    const int org[3] = {ti * L.tx, tj * L.ty, tk * L.tz};
    const int n0 = A.n[0], n1 = A.n[1], n2 = A.n[2];
    const double qs = fixed_scale(A.scale);

    // fields first: the gather's LDS reads then use small immediate offsets
    float* fld = (float*)lds_raw;  // 6 * fvol
    unsigned long long* cur = (unsigned long long*)(lds_raw + ((6 * L.fvol * sizeof(float) + 15) & ~(size_t)15));

    double* facq = (double*)(cur + 3 * L.cvol);
    int32_t* slots = (int32_t*)(facq + 4);  // destination-cell counters
    const int nslots = L.dex * L.dey * L.dez;
    // Mesh offsets of the tile's nodes along each axis, counted from the lower end of the halo (the
    // same for the fields, the current and the destination cells): for the compile-time shapes a
    // table, one wrap per node of an axis instead of one per node in each of the three loops below
    // (with a wrap and a division chain per node and component these loops took a tenth of the
    // kernel's instructions at 32 particles per cell: 690 us against 636 for 128x32x32, two
    // species; 40 against 32 for 16^3, quadratic, in 256 threads; 11.60 ms against 11.21 for 128^3, 64 per cell).
    // A runtime shape has no room for it in LDS where its tile was chosen to fill that.
    int32_t* ox = slots + nslots;
    if constexpr (TL::fixed_shape) {
        for (int q = threadIdx.x; q < L.cex + L.cey + L.cez; q += BS) {
            const int y = q - L.cex, z = y - L.cey;
            ox[q] = y < 0   ? wrap_near(org[0] - L.clox + q, n0)
                    : z < 0 ? n0 * wrap_near(org[1] - L.cloy + y, n1)
                            : n0 * n1 * wrap_near(org[2] - L.cloz + z, n2);
        }
        __syncthreads();
    }
    auto mesh = [&](int a, int b, int c) {
        if constexpr (TL::fixed_shape)
            return ox[a] + ox[L.cex + b] + ox[L.cex + L.cey + c];
        else
            return wrap_near(org[0] - L.clox + a, n0) +
                   n0 * (wrap_near(org[1] - L.cloy + b, n1) + n1 * wrap_near(org[2] - L.cloz + c, n2));
    };

    // 1. stage fields, a thread per node and STAGE_NODES nodes' loads in flight before it waits for
    // the first; clear the current block and the counters
    const int fnodes = L.fex * L.fey * L.fez;
    for (int q0 = threadIdx.x; q0 < fnodes; q0 += STAGE_NODES * BS) {
        double v[STAGE_NODES][6];
        int dst[STAGE_NODES];  // LDS entry, or -1 (past the end)
#pragma unroll
        for (int k = 0; k < STAGE_NODES; ++k) {
            // every lane loads (past the end: the first node, which it doesn't write), so that no
            // load waits at a branch
            const int q = q0 + k * BS;
            const int qc = q < fnodes ? q : 0;
            const int row = qc / L.fex, a = qc - row * L.fex, c = row / L.fey, bb = row - c * L.fey;
            dst[k] = q < fnodes ? a + L.frow * bb + L.fplane * c : -1;
            const int g = mesh(a, bb, c);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                v[k][d] = gl(A.E)[d * A.nc + g];
                v[k][3 + d] = gl(A.B)[d * A.nc + g];
            }
        }
#pragma unroll
        for (int k = 0; k < STAGE_NODES; ++k)
            if (dst[k] >= 0) {
#pragma unroll
                for (int comp = 0; comp < 6; ++comp) fld[comp * L.fvol + dst[k]] = (float)v[k][comp];
            }
    }
    for (int q = threadIdx.x; q < 3 * L.cvol; q += BS) cur[q] = 0ull;
    for (int q = threadIdx.x; q < nslots; q += BS) slots[q] = 0;
    __syncthreads();

    TileCtx C;
    for (int d = 0; d < 3; ++d) C.org[d] = org[d];
    C.nxy = (uint32_t)n0 * (uint32_t)n1;
    C.base_cell = (uint32_t)org[0] + (uint32_t)n0 * (uint32_t)org[1] + C.nxy * (uint32_t)org[2];
    C.fld = fld;
    C.cur = cur;
    C.slots = slots;
    C.facq = facq;

    int bad_all = 0;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    for (int s = s0; s < s1; ++s) {
        const Sp32& S = A.sp[s];
        const int32_t start = gl(S.start)[tile];
        const int32_t end = gl(S.start)[tile + 1];
        if (threadIdx.x < 4) facq[threadIdx.x] = (threadIdx.x < 3 ? S.fac[threadIdx.x] : S.qw) * qs;
        __syncthreads();
        if constexpr (!TL::pairs) {
            for (int32_t q = start + threadIdx.x; q < end; q += BS) {
                Win<O> W;
                step_particle<O, TL>(A, S, L, C, q, W, bad_all);
                if (!W.dep) continue;
                if constexpr (TL::flat)
                    deposit_flat<O, TL>(L, cur, W, C.facq);
                else
                    deposit_cc<O, TL, false>(L, cur, W, C.facq, W, C.facq, 0.0f);
            }
        } else {
            for (int32_t b = start + 128 * wave; b < end; b += BS * 2) {
                Win<O> W1, W2;
                const int32_t q1 = b + lane, q2 = b + 64 + lane;
                W1.dep = W2.dep = false;
                // a second particle that deposits nothing still enters the paired deposit with
                // zero prefix sums: its window state must then be finite
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    W2.f[d] = W2.x1[d] = 0.5f;
                    W2.loc[d] = 0;
                }
                if (q1 < end) step_particle<O, TL>(A, S, L, C, q1, W1, bad_all);
                if (q2 < end) step_particle<O, TL>(A, S, L, C, q2, W2, bad_all);
                const bool both = W1.dep && W2.dep;
                const bool same = both && window_start<O, TL>(L, W1, 0) == window_start<O, TL>(L, W2, 0) &&
                                  window_start<O, TL>(L, W1, 1) == window_start<O, TL>(L, W2, 1) &&
                                  window_start<O, TL>(L, W1, 2) == window_start<O, TL>(L, W2, 2);
                if (__any(same)) {
                    // the first particle of every lane (or its second, if only that one deposits),
                    // together with the second where the windows coincide
                    if (!W1.dep && W2.dep) {
                        W1 = W2;
                        W2.dep = false;
                    }
                    if (W1.dep)
                        deposit_cc<O, TL, true>(L, cur, W1, C.facq, W2, C.facq, same ? 1.0f : 0.0f);
                    if (both && !same) deposit_cc<O, TL, false>(L, cur, W2, C.facq, W2, C.facq, 0.0f);
                } else {
                    if (W1.dep) deposit_cc<O, TL, false>(L, cur, W1, C.facq, W1, C.facq, 0.0f);
                    if (W2.dep) deposit_cc<O, TL, false>(L, cur, W2, C.facq, W2, C.facq, 0.0f);
                }
            }
        }
        // reserve the tile's range in each destination cell's count; the sort adds its start to
        // the particles' ranks
        __syncthreads();
        for (int q = threadIdx.x; q < nslots; q += BS) {
            const int c = slots[q];
            slots[q] = 0;
            int first = 0;
            if (c != 0) {
                const int row = q / L.dex, x = q - row * L.dex, z = row / L.dey, y = row - z * L.dey;
                first = atomicAdd(gl(S.cnt) + mesh(x, y, z), c);
            }
            gl(S.base)[tile * nslots + q] = first;
        }
        __syncthreads();
    }
    if (bad_all) atomic_or_flag(gl(A.flags), bad_all);

    // 3. flush the current block (integer adds commute: the sum is order-independent)
    const int cnodes = L.cex * L.cey * L.cez;
    for (int q = threadIdx.x; q < cnodes; q += BS) {
        const int row = q / L.cex, a = q - row * L.cex, c = row / L.cey, bb = row - c * L.cey;
        const int l = a + L.crow * bb + L.cplane * c, g = mesh(a, bb, c);
        unsigned long long raw[3];
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) raw[comp] = cur[comp * L.cvol + l];
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            const long long v = fixed_sum(raw[comp]);
            if (v != 0) atomicAdd(gl(A.Jq) + comp * A.nc + g, (unsigned long long)v);
        }
    }
}

// Wavefronts a SIMD: three with pairs (168 registers; 128 spill, 128^3 11.3 -> 13.5 ms), five in flat
// tiles (96, ten of them spilled; 106 and four take 1 % longer).
template <int O, class TL, int BS>
__global__ void __launch_bounds__(BS, TL::pairs ? 3 : TL::flat ? 5 : 1) k_gpd32(Gpd32Args A) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // XCD-aware tile order: consecutive workgroups go round-robin over the 8 XCDs, so give
    // each XCD a contiguous run of tiles (neighbouring tiles share halos in that XCD's L2).
    const int64_t b = blockIdx.x;
    const int64_t tile = (b & 7) * (int64_t)A.per_xcd + (b >> 3);
    if (tile >= A.ntiles) return;
    // a workgroup per tile and species, or per tile (the current's integer sum is the same)
    const int s0 = gridDim.y > 1 ? (int)blockIdx.y : 0, s1 = gridDim.y > 1 ? s0 + 1 : A.nsp;
    gpd32_tile<O, TL, BS>(A, tile, s0, s1, lds_raw);
}

// Batched: block b of the launch belongs to run r with prefix[r] <= b (prefix = running block counts).
template <int O, class TL>
__global__ void __launch_bounds__(GPD32_BS, TL::pairs ? 3 : 1) k_gpd32_batch(const Gpd32Args* __restrict__ table,
                                                          const int64_t* __restrict__ prefix, int nruns) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, nruns, b);
    if (r < 0) return;
    // as in a single run, an XCD takes a contiguous eighth of the run's tiles (prefix counts whole
    // eights, so the XCD is the same b & 7)
    const int64_t lb = b - prefix[r], tile = (lb & 7) * (int64_t)table[r].per_xcd + (lb >> 3);
    if (tile >= table[r].ntiles) return;
    gpd32_tile<O, TL, GPD32_BS>(table[r], tile, 0, table[r].nsp, lds_raw);
}

// Fixed-point current of a run to FP64, clearing the accumulator for the next step (runs without
// the line solve, whose kernel does both as it reads the current).
struct FixedDesc {
    FixedScale scale;
    unsigned long long* Jq;  // accumulator, 3 * nc
    double* J;
    int64_t n3;
};

__device__ __forceinline__ void fixed_body(const FixedDesc& D, int64_t q, double inv) {
    if (q >= D.n3) return;
    gl(D.J)[q] = (double)(long long)gl(D.Jq)[q] * inv;
    gl(D.Jq)[q] = 0ull;
}

__global__ void __launch_bounds__(256) k_fixed(FixedDesc D) {
    const double inv = 1.0 / fixed_scale(D.scale);  // exact: a power of two
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < D.n3; q += (int64_t)gridDim.x * blockDim.x)
        fixed_body(D, q, inv);
}

__global__ void __launch_bounds__(256) k_fixed_batch(const FixedDesc* __restrict__ T, const int64_t* __restrict__ prefix,
                                                     int n) {
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, n, b);
    if (r < 0) return;
    fixed_body(T[r], (b - prefix[r]) * blockDim.x + threadIdx.x, 1.0 / fixed_scale(T[r].scale));
}

enum TileKind { TILE_444 = 0, TILE_881_FLAT = 1, TILE_RT = 2 };

static int tile_kind(const pp_run* r) {
    const int* t = r->g.t;
    const int* n = r->p.n;
    if (t[0] == 4 && t[1] == 4 && t[2] == 4 && n[0] > 1 && n[1] > 1 && n[2] > 1) return TILE_444;
    if (t[0] == 8 && t[1] == 8 && t[2] == 1 && n[0] > 1 && n[1] > 1 && n[2] == 1) return TILE_881_FLAT;
    return TILE_RT;
}

static void lds_extents(const pp_run* r, int fe[3], int ce[3]) {
    for (int d = 0; d < 3; ++d) {
        const bool single = r->p.n[d] == 1;
        fe[d] = single ? 1 : r->g.t[d] + FLD_LO + fld_hi(r->p.shape_order);
        ce[d] = single ? 1 : r->g.t[d] + cur_lo(r->p.shape_order) + cur_hi(r->p.shape_order);
    }
}

size_t gpd32_lds_bytes(const pp_run* r) {
    int fe[3], ce[3];
    lds_extents(r, fe, ce);
    const size_t fv = tile_kind(r) == TILE_444 ? (size_t)fld_plane_444(r->p.shape_order) * fe[2]
                                                : (size_t)fe[0] * fe[1] * fe[2];
    const int kind = tile_kind(r);
    const size_t cv = kind == TILE_444       ? (size_t)cur_plane_444(r->p.shape_order) * ce[2]
                      : kind == TILE_881_FLAT ? (size_t)cur_row_881 * ce[1]
                                              : (size_t)ce[0] * ce[1] * ce[2];
    const size_t slots = r->g.dest_slots();
    return ((6 * fv * sizeof(float) + 15) & ~(size_t)15) + 3 * cv * sizeof(unsigned long long) + 4 * sizeof(double) +
           (slots + (kind == TILE_RT ? 0 : ce[0] + ce[1] + ce[2])) * sizeof(int32_t);
}

// Host part of the fixed-point exponent: e0 = 50 - ceil(log2(max |fac|)), every contribution
// being at most |fac| = |q w d / dt| in magnitude (|prefix of DS| <= 1 and 0 <= F <= 1).
int gpd32_scale_e0(const pp_run* r) {
    double fmax = 0.0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        const Species& S = r->sp[s];
        if (!S.active) continue;
        for (int d = 0; d < 3; ++d) {
            const double f = fabs(S.q * S.w * r->p.d[d] / r->dt_drift);
            fmax = f > fmax ? f : fmax;
        }
    }
    if (!(fmax > 0.0)) return 0;
    // on a single-cell axis the O+2 window nodes of a particle all land on one LDS node, so a
    // node can receive up to O+2 contributions of one particle per such axis
    int collapsed = 0;
    for (int d = 0; d < 3; ++d) collapsed += r->p.n[d] == 1 ? 1 : 0;
    const int per_axis = (int)ceil(log2((double)(r->p.shape_order + 2)));
    return 50 - (int)ceil(log2(fmax)) - collapsed * per_axis;
}

// Kernel arguments of one run (also the batched table entries).
void gpd32_fill_args(const pp_run* r, Gpd32Args* Ap) {
    Gpd32Args& A = *Ap;
    for (int d = 0; d < 3; ++d) {
        A.n[d] = r->p.n[d];
        A.t[d] = r->g.t[d];
        A.nt[d] = r->g.nt[d];
        A.inv_d[d] = (float)(1.0 / r->p.d[d]);
    }
    A.ntiles = r->g.ntiles;
    A.nc = r->g.ncell;
    A.dt = (float)r->dt_drift;
    A.dtk = (float)r->dt_kick;
    A.pred = (float)r->drift_ratio;
    A.ic = (float)(1.0 / r->p.c);
    A.pusher = r->p.pusher;
    A.nsp = 0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        const Species& S = r->sp[s];
        if (!S.active) continue;
        Sp32& D = A.sp[A.nsp++];
        D.start = S.offsets;
        D.cnt = S.cell_cnt;
        D.rank = S.rank;
        D.base = S.rank_base;
        D.perm = S.pending ? S.perm : nullptr;
        D.cell = S.cur.cell;
        D.cell_o = S.pending ? S.cur.cell_alt : S.cur.cell;
        D.id = S.pending ? S.cur.id : nullptr;
        D.id_o = S.pending ? S.cur.id_alt : nullptr;
        for (int d = 0; d < 3; ++d) {
            D.pos[d] = (const float*)S.cur.pos[d];
            D.u[d] = (const float*)S.cur.u[d];
            D.pos_o[d] = (float*)(S.pending ? S.cur.pos_alt[d] : S.cur.pos[d]);
            D.u_o[d] = (float*)(S.pending ? S.cur.u_alt[d] : S.cur.u[d]);
            D.fac[d] = -S.q * S.w * r->p.d[d] / r->dt_drift;
        }
        D.h = (float)(S.q * r->dt_kick / S.m);
        D.krad = (float)(r->p.rad_tau * S.q * S.q / S.m);
        D.qw = S.q * S.w;
    }
    A.E = r->mesh.E;
    A.B = r->mesh.B;
    A.Jq = (unsigned long long*)r->Jq;
    A.scale = gpd32_scale(r);
    A.flags = r->flags;
    A.per_xcd = (int)((r->g.ntiles + 7) / 8);
    A.direct = r->p.current_scheme == PP_CURRENT_DIRECT ? 1 : 0;
}

FixedScale gpd32_scale(const pp_run* r) { return FixedScale{r->tile_max, gpd32_scale_e0(r)}; }

void gpd32_fixed_desc(const pp_run* r, FixedDesc* D) {
    D->scale = gpd32_scale(r);
    D->Jq = (unsigned long long*)r->Jq;
    D->J = uses_line_solve(r) ? r->J2 : r->mesh.J;
    D->n3 = 3 * r->g.ncell;
}

// blocks of the batched conversion (none where the line solve reads the fixed-point current)
int64_t gpd32_fixed_blocks(const pp_run* r) { return line_reads_fixed(r) ? 0 : (3 * r->g.ncell + 255) / 256; }

int64_t gpd32_blocks(const pp_run* r) { return 8 * ((r->g.ntiles + 7) / 8); }
size_t gpd32_args_size() { return sizeof(Gpd32Args); }
size_t gpd32_fixed_desc_size() { return sizeof(FixedDesc); }
bool gpd32_batchable(const pp_run* r) { return tile_kind(r) == TILE_444; }

static unsigned fixed_grid(int64_t n3) {
    int64_t g = (n3 + 255) / 256;
    if (g > 16384) g = 16384;
    return (unsigned)(g < 1 ? 1 : g);
}

// A workgroup takes one species up to 4096 tiles, which are few rounds of the 768 workgroups that are
// resident at once (three a CU): the last round is shorter.  Two species, cubic, all species of a
// tile in a workgroup -> one each: 900 tiles 255 -> 216 us, 64x32x32 (1024) at 16 per cell 287 -> 254,
// 56x48x40 (1680) 411 -> 387, 64x64x48 (3072) 648 -> 638; 80x80x64 (6400) 1276 -> 1267, and in 128^3
// (32768) staging the fields twice costs more, 11.15 -> 11.28 ms.
// A box of fewer workgroups than that leaves wavefronts' places idle, and its time is the chain one
// wavefront goes through: staging, its particles, flushing.  Larger workgroups that give a lane one
// particle at a time (no pairs, 100 registers) shorten each part of it, with twice the atomics, which
// the idle LDS has room for: 1024 threads up to a workgroup a CU, 512 up to two.  Two species,
// time of pairs in 256 threads -> this: 16^3, 8 per cell, quadratic 33 -> 22.5 us, cubic 46 -> 32;
// 16^3, 32 per cell 109 -> 72 (512 threads: 74); 24^3 (432 workgroups), 32 per cell 136 -> 129;
// 28^3 (686) would take 201 us in 512 threads against 181, which keeps it with the pairs.
template <int O>
static void launch_tiles32(int kind, const Gpd32Args& A, size_t lds, hipStream_t st) {
    const int64_t wgs = A.ntiles * A.nsp;
    const dim3 grid((unsigned)(8 * (int64_t)A.per_xcd), A.ntiles <= 4096 && A.nsp > 0 ? (unsigned)A.nsp : 1u);
    if (kind == TILE_444 && wgs <= 256)
        hipLaunchKernelGGL((k_gpd32<O, Tile444<O, false>, 1024>), grid, dim3(1024), lds, st, A);
    else if (kind == TILE_444 && wgs <= 512)
        hipLaunchKernelGGL((k_gpd32<O, Tile444<O, false>, 512>), grid, dim3(512), lds, st, A);
    else if (kind == TILE_444)
        hipLaunchKernelGGL((k_gpd32<O, Tile444<O, true>, GPD32_BS>), grid, dim3(GPD32_BS), lds, st, A);
    else if (kind == TILE_881_FLAT)
        hipLaunchKernelGGL((k_gpd32<O, Tile881<O>, GPD32_BS>), grid, dim3(GPD32_BS), lds, st, A);
    else
        hipLaunchKernelGGL((k_gpd32<O, TileRT<O>, GPD32_BS>), grid, dim3(GPD32_BS), lds, st, A);
}

hipError_t launch_gpd32(pp_run* r) {
    Gpd32Args A;
    gpd32_fill_args(r, &A);
    const size_t lds = gpd32_lds_bytes(r);
    if (r->p.shape_order == 2)
        launch_tiles32<2>(tile_kind(r), A, lds, r->stream);
    else
        launch_tiles32<3>(tile_kind(r), A, lds, r->stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!line_reads_fixed(r)) {
        FixedDesc F;
        gpd32_fixed_desc(r, &F);
        hipLaunchKernelGGL(k_fixed, dim3(fixed_grid(F.n3)), dim3(256), 0, r->stream, F);
    }
    return hipGetLastError();
}

// Batched particle step of n runs that all use 4x4x4 tiles and the same weight order:
// the tiled kernel, and the conversion to FP64 of the runs that need it.
hipError_t launch_gpd32_batch(const void* args_table, const int64_t* tile_prefix, int64_t total_blocks,
                              const void* fixed_table, const int64_t* fixed_prefix, int64_t total_fixed_blocks, int n,
                              int shape_order, size_t lds, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const Gpd32Args* T = (const Gpd32Args*)args_table;
    if (shape_order == 2)
        hipLaunchKernelGGL((k_gpd32_batch<2, Tile444<2, true>>), dim3((unsigned)total_blocks), dim3(GPD32_BS),
                           lds, st, T, tile_prefix, n);
    else
        hipLaunchKernelGGL((k_gpd32_batch<3, Tile444<3, true>>), dim3((unsigned)total_blocks), dim3(GPD32_BS),
                           lds, st, T, tile_prefix, n);
    if (total_fixed_blocks > 0)
        hipLaunchKernelGGL(k_fixed_batch, dim3((unsigned)total_fixed_blocks), dim3(256), 0, st,
                           (const FixedDesc*)fixed_table, fixed_prefix, n);
    return hipGetLastError();
}

}  // namespace pp
