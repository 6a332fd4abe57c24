// C ABI of libpp (include/pp.h): validation, run state, launch sequencing.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>

#include "pp_internal.hpp"

namespace pp {

static std::mutex g_err_mu;
static char g_err[256] = "";

void set_hip_error(hipError_t e, const char* where) {
    std::lock_guard<std::mutex> lk(g_err_mu);
    snprintf(g_err, sizeof(g_err), "%s: %s", where, hipGetErrorString(e));
}

void set_error_text(const char* msg) {
    std::lock_guard<std::mutex> lk(g_err_mu);
    snprintf(g_err, sizeof(g_err), "%s", msg);
}

// defined in the kernel translation units
void field_setup(pp_run* r, double* consts);  // consts: host copy of the run's constants
int line_setup_axis(int order, int N, double* coef_host, int* off);
int64_t scan_tmp_size(int64_t n);
int diag_acc_count();
int64_t diag_buffer_count(int64_t ncell);
size_t gpd32_lds_bytes(const pp_run* r);

static bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

static pp_status validate(const pp_params* p) {
    if (!p) return PP_E_ARG;
    for (int d = 0; d < 3; ++d) {
        if (p->n[d] < 1 || p->n[d] > (1 << 20)) return PP_E_ARG;
        if (!std::isfinite(p->d[d])) return PP_E_NONFINITE;
        if (!(p->d[d] > 0.0)) return PP_E_ARG;
    }
    const int64_t nc = (int64_t)p->n[0] * p->n[1] * p->n[2];
    if (nc > ((int64_t)1 << 30)) return PP_E_CAPACITY;
    if (!std::isfinite(p->dt) || !std::isfinite(p->c) || !std::isfinite(p->eps0) || !std::isfinite(p->alpha) ||
        !std::isfinite(p->relax_tol) || !std::isfinite(p->rho_background) || !std::isfinite(p->rad_tau))
        return PP_E_NONFINITE;
    if (p->rad_tau < 0.0) return PP_E_ARG;
    if (p->current_scheme != PP_CURRENT_CC && p->current_scheme != PP_CURRENT_DIRECT) return PP_E_ARG;
    if (p->gauss_filter_passes < 0 || p->gauss_filter_passes > PP_MAX_GAUSS_PASSES) return PP_E_ARG;
    if (p->time_order != 2 && p->time_order != 4) return PP_E_ARG;
    if (p->gauss_filter_every < 0 || p->gauss_filter_every > (1 << 20)) return PP_E_ARG;
    if (p->gauss_filter_every > 1 && p->time_order != 2) return PP_E_ARG;
    if (!finite_pos(p->dt) || !finite_pos(p->c) || !finite_pos(p->eps0)) return PP_E_ARG;
    if (p->shape_order != 2 && p->shape_order != 3) return PP_E_ARG;
    if (p->field_order != 2 && p->field_order != 4 && p->field_order != 6) return PP_E_ARG;
    if (!(p->alpha >= 0.5 && p->alpha < 1.0)) return PP_E_ARG;
    if (p->pusher != PP_PUSH_VAY && p->pusher != PP_PUSH_BORIS) return PP_E_ARG;
    if (p->precision != PP_PREC_FP64 && p->precision != PP_PREC_FP32_SPLIT) return PP_E_ARG;
    if (!(p->relax_tol > 0.0 && p->relax_tol < 1.0) || p->relax_max_iter < 1) return PP_E_ARG;
    double dmin = p->d[0];
    for (int d = 1; d < 3; ++d) dmin = p->d[d] < dmin ? p->d[d] : dmin;
    if (!(p->c * p->dt < dmin)) return PP_E_CFL;
    if (p->time_order == 4 && !(FR_THETA * p->c * p->dt < dmin)) return PP_E_CFL;  // the longest drift
    return PP_OK;
}

// Tile shape: powers of two with product TILE_CELLS where the box allows, as close to a cube
// as the box allows (the LDS halo per cell is smallest for a cube): double the shortest tile
// side that is still below the box side.  Boxes at least 4 cells on every side get 4x4x4
// tiles, flat boxes 8x8x1.
static void choose_tiles(const int n[3], int t[3]) {
    t[0] = t[1] = t[2] = 1;
    while (t[0] * t[1] * t[2] < TILE_CELLS) {
        int best = -1;
        for (int d = 0; d < 3; ++d)
            if (t[d] < n[d] && (best < 0 || t[d] < t[best])) best = d;
        if (best < 0) break;
        t[best] *= 2;
    }
}

// The arrays of a run, or of a species, as parts of one device allocation (every hipMalloc and
// hipFree costs tens of microseconds, and a served request creates a run).  The same list gives
// the size alone.
struct Arena {
    static constexpr int MAX = 24;
    void** ptr[MAX];
    size_t off[MAX];
    int count = 0;
    size_t size = 0;

    template <typename T>
    void add(T** p, size_t n) {
        ptr[count] = (void**)p;
        off[count++] = size;
        size += ((n > 0 ? n : 1) * sizeof(T) + 255) & ~(size_t)255;
    }
    bool allocate(void** base) {
        *base = nullptr;
        if (!ok(hipMalloc(base, size), "hipMalloc")) {
            *base = nullptr;
            return false;
        }
        for (int i = 0; i < count; ++i) *ptr[i] = (char*)*base + off[i];
        return true;
    }
};

// values of the run's constants: relaxation weights of each drift, line-solve taps of each axis
static size_t omega_count(const pp_params* p) { return (size_t)p->relax_max_iter + 2; }

static void run_arrays(const pp_params* p, const Geom& g, pp_run* r, Arena& A) {
    const size_t nc = (size_t)g.ncell, n3 = 3 * nc;
    A.add(&r->J2, n3);
    A.add(&r->Bn, n3);
    A.add(&r->Bw, n3);
    A.add(&r->R, n3);
    A.add(&r->rho, nc);
    A.add(&r->rho_prev, nc);
    A.add(&r->sort_cursor, (size_t)g.nbins);
    A.add(&r->scan_tmp, (size_t)scan_tmp_size(g.nbins + 1));
    A.add(&r->dacc, (size_t)diag_buffer_count(g.ncell));
    A.add(&r->consts, 3 * omega_count(p) + 3 * 127);
    // cleared at the start, together: the flag word, a counter, the largest tiles, the fixed-point current
    A.add(&r->flags, 1);
    A.add(&r->tile_count, 1);
    A.add(&r->tile_max, 2 * PP_MAX_SPECIES);
    A.add(&r->Jq, p->precision == PP_PREC_FP32_SPLIT ? n3 : 0);
}

static void species_arrays(const pp_params* p, const Geom& g, int64_t n, Species& S, Arena& A) {
    const bool split = p->precision == PP_PREC_FP32_SPLIT;
    const size_t nt = (size_t)g.ntiles, nb = (size_t)g.nbins;
    A.add(&S.offsets, nb + 1);
    A.add(&S.offsets_next, (split ? nt : nb) + 1);
    A.add(&S.cell_cnt, split ? (size_t)g.ncell : 2 * nb);
    A.add(&S.rank, (size_t)n);
    A.add(&S.perm, (size_t)n);
    if (split) {
        A.add(&S.rounds, nt * SORT_RCAP);
        A.add(&S.rank_base, nt * (size_t)g.dest_slots());
    } else {
        A.add(&S.bin_pre, nb);
        A.add(&S.tile_tot, nt + 1);
    }
}

static void release(pp_run* r) {
    if (r->arena) (void)hipFree(r->arena);
    for (Species& S : r->sp)
        if (S.arena) (void)hipFree(S.arena);
    if (r->ev0) (void)hipEventDestroy(r->ev0);
    if (r->ev1) (void)hipEventDestroy(r->ev1);
}

static pp_status flush_timing(pp_run* r) {
    if (!r->timing || !r->t_pending) return PP_OK;
    if (!ok(hipEventSynchronize(r->ev1), "hipEventSynchronize")) return PP_E_HIP;
    float ms = 0.f;
    if (!ok(hipEventElapsedTime(&ms, r->ev0, r->ev1), "hipEventElapsedTime")) return PP_E_HIP;
    r->t_ms += ms;
    r->t_launches += 1;
    r->t_pending = false;
    return PP_OK;
}

}  // namespace pp

using namespace pp;

extern "C" {

const char* pp_status_str(pp_status st) {
    switch (st) {
    case PP_OK: return "ok";
    case PP_E_ARG: return "invalid argument";
    case PP_E_CFL: return "c*dt must be below the smallest cell size";
    case PP_E_NONFINITE: return "non-finite parameter";
    case PP_E_NOCONV: return "field relaxation did not converge";
    case PP_E_CAPACITY: return "size limit exceeded";
    case PP_E_HIP: return "HIP runtime error";
    case PP_E_STATE: return "call order violated";
    default: return "unknown status";
    }
}

const char* pp_last_hip_error(void) { return g_err; }

// Device bytes pp_create and pp_init_species allocate for a run at most (the caller-owned mesh
// and particle arrays not included): the arrays without particles, the rank and permutation of
// every species' particles and, in the split form, as much again for the largest species (room that
// the first sort no longer takes, in an upper bound that budgets are set by).  Per tile of 64 cells and
// split species 2304 bytes are the sort's round table and, for 4x4x4 tiles, 2048 the ranks that the
// tile's particles start from in each cell around it: each species has its own, so that one launch sorts
// them all, and with few particles per cell they are most of a run's memory (256^3, eight species of one
// particle per cell: 13.8 GB, of which 9.1; 64x32x32, two of 32: 69 MB, 8.9).
static size_t internal_bytes(const pp_params* p, const Geom& g, int64_t nmax, int nsp) {
    pp_run r;
    Arena A, B;
    run_arrays(p, g, &r, A);
    species_arrays(p, g, 0, r.sp[0], B);
    const size_t pair = 2 * (size_t)nmax * sizeof(int32_t);
    return A.size + (size_t)nsp * (B.size + pair) + (p->precision == PP_PREC_FP32_SPLIT ? pair : 0);
}

static void make_geom_host(const pp_params* p, Geom& g) {
    for (int d = 0; d < 3; ++d) g.n[d] = p->n[d];
    choose_tiles(g.n, g.t);
    for (int d = 0; d < 3; ++d) g.nt[d] = (g.n[d] + g.t[d] - 1) / g.t[d];
    g.ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    g.ntiles = (int64_t)g.nt[0] * g.nt[1] * g.nt[2];
    g.nbins = g.ntiles * TILE_CELLS;
}

pp_status pp_workspace_size(const pp_params* params, int64_t max_particles, int32_t nspecies, size_t* bytes) {
    if (!bytes) return PP_E_ARG;
    *bytes = 0;
    pp_status st = validate(params);
    if (st != PP_OK) return st;
    if (max_particles < 0 || nspecies < 0 || nspecies > PP_MAX_SPECIES) return PP_E_ARG;
    if (max_particles >= INT32_MAX) return PP_E_CAPACITY;
    Geom g;
    make_geom_host(params, g);
    if (g.nbins + 1 > INT32_MAX) return PP_E_CAPACITY;
    *bytes = internal_bytes(params, g, max_particles, nspecies);
    return PP_OK;
}

pp_status pp_create(const pp_params* params, const pp_mesh* mesh, void* hip_stream, pp_run** out) {
    if (!out) return PP_E_ARG;
    *out = nullptr;
    pp_status st = validate(params);
    if (st != PP_OK) return st;
    if (!mesh || !mesh->E || !mesh->B || !mesh->J) return PP_E_ARG;
    pp_run* r = new (std::nothrow) pp_run();
    if (!r) return PP_E_CAPACITY;
    r->p = *params;
    r->mesh = *mesh;
    r->stream = (hipStream_t)hip_stream;
    Geom& g = r->g;
    make_geom_host(params, g);
    if (g.nbins + 1 > INT32_MAX) {
        delete r;
        return PP_E_CAPACITY;
    }
    const bool split = params->precision == PP_PREC_FP32_SPLIT;
    if (split) {
        int dev = 0, lds = 0;
        if (!ok(hipGetDevice(&dev), "hipGetDevice") ||
            !ok(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev), "hipDeviceGetAttribute")) {
            delete r;
            return PP_E_HIP;
        }
        if (gpd32_lds_bytes(r) > (size_t)lds) {
            delete r;
            return PP_E_CAPACITY;
        }
    }
    Arena A;
    run_arrays(params, g, r, A);
    r->nrs = params->time_order == 4 ? 3 : 1;
    // the constants are worked out on the host and copied once
    const size_t no = omega_count(params), nconst = 3 * no + 3 * 127;
    double* host = new (std::nothrow) double[nconst]();
    if (!host) {
        delete r;
        return PP_E_CAPACITY;
    }
    bool okk = A.allocate(&r->arena);
    if (!split) r->Jq = nullptr;
    for (int k = 0; k < r->nrs; ++k) r->rs[k].omega = r->consts + k * no;
    if (okk && params->field_order > 2)
        for (int d = 0; d < 3; ++d) {
            LineStencil& L = r->line[d];
            const size_t at = 3 * no + (size_t)d * 127;
            L.coef = r->consts + at;
            int same = -1;  // an axis of the same length before: the same taps
            for (int e = 0; e < d; ++e)
                if (g.n[e] == g.n[d]) same = e;
            if (same >= 0) {
                L.len = r->line[same].len;
                L.off = r->line[same].off;
                std::memcpy(host + at, host + 3 * no + (size_t)same * 127, 127 * sizeof(double));
            } else {
                L.len = line_setup_axis(params->field_order, g.n[d], host + at, &L.off);
                okk = okk && L.len > 0;
            }
        }
    if (okk) field_setup(r, host);
    okk = okk && ok(hipMemcpy(r->consts, host, nconst * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
    delete[] host;
    if (okk) {  // flags .. the end of the arena, all-zero bits
        const size_t bytes = (size_t)((char*)r->arena + A.size - (char*)r->flags);
        okk = ok(launch_fill((double*)r->flags, (int64_t)(bytes / sizeof(double)), 0.0, r->stream), "fill");
    }
    if (!okk) {
        release(r);
        delete r;
        return PP_E_HIP;
    }
    *out = r;
    return PP_OK;
}

pp_status pp_init_species(pp_run* r, int32_t s, double q, double m, double w, const pp_particles* parts) {
    if (!r || !parts || s < 0 || s >= PP_MAX_SPECIES) return PP_E_ARG;
    if (!std::isfinite(q) || !std::isfinite(m) || !std::isfinite(w)) return PP_E_NONFINITE;
    if (!(m > 0.0) || w < 0.0) return PP_E_ARG;
    if (parts->n < 0 || parts->n >= INT32_MAX) return PP_E_CAPACITY;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    if (parts->n > 0) {
        for (int d = 0; d < 3; ++d)
            if (!parts->pos[d] || !parts->u[d] || !parts->pos_alt[d] || !parts->u_alt[d]) return PP_E_ARG;
        if (split && (!parts->cell || !parts->cell_alt)) return PP_E_ARG;
        if (parts->id && !parts->id_alt) return PP_E_ARG;
    }
    Species& S = r->sp[s];
    if (!S.arena || S.arena_n < parts->n) {
        if (S.arena) (void)hipFree(S.arena);
        S.active = false;  // until the new arrays are there
        Arena A;
        species_arrays(&r->p, r->g, parts->n, S, A);
        if (!A.allocate(&S.arena)) return PP_E_HIP;
        S.arena_n = parts->n;
    }
    if (!ok(launch_fill_i32(S.cell_cnt, split ? r->g.ncell : 2 * r->g.nbins, 0, r->stream), "fill")) return PP_E_HIP;
    S.pending = false;
    S.active = true;
    S.q = q;
    S.m = m;
    S.w = w;
    S.n = parts->n;
    S.cur = *parts;
    if (!split) {
        S.cur.cell = nullptr;
        S.cur.cell_alt = nullptr;
    }
    if (!parts->id) S.cur.id_alt = nullptr;
    S.sorted = false;
    S.ranked = false;
    S.binned = false;
    S.handed_out = false;
    // initial sort: the split form needs it before its first push
    hipError_t e = launch_sort(r, s);
    if (!ok(e, "sort")) return PP_E_HIP;
    return PP_OK;
}

pp_status pp_gather_push_deposit(pp_run* r) {
    if (!r) return PP_E_ARG;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    for (int s = 0; s < PP_MAX_SPECIES; ++s)
        if (split && r->sp[s].active && !r->sp[s].sorted) return PP_E_STATE;
    if (flush_timing(r) != PP_OK) return PP_E_HIP;
    double* target = uses_line_solve(r) ? r->J2 : r->mesh.J;  // FP64 form
    hipError_t e = hipSuccess;
    if (!split) {
        e = launch_fill(target, 3 * r->g.ncell, 0.0, r->stream);
        if (!ok(e, "fill")) return PP_E_HIP;
    }
    if (r->timing && !ok(hipEventRecord(r->ev0, r->stream), "hipEventRecord")) return PP_E_HIP;
    if (split) {
        e = launch_gpd32(r);
        if (!ok(e, "gather_push_deposit")) return PP_E_HIP;
        for (int s = 0; s < PP_MAX_SPECIES; ++s) {  // the kernel wrote the pending order
            Species& S = r->sp[s];
            if (!S.active) continue;
            S.moved = S.pending;
            if (!S.pending) continue;
            swap_buffers(S.cur);
            S.pending = false;
        }
    } else {
        unsigned done = 0;
        e = launch_gpd64_tiles(r, target, &done);
        if (!ok(e, "gather_push_deposit")) return PP_E_HIP;
        for (int s = 0; s < PP_MAX_SPECIES; ++s) {
            if (!r->sp[s].active) continue;
            Species& S = r->sp[s];
            S.binned = false;  // the particles move: their bins are those of the last sort
            const bool by_tiles = (done & (1u << s)) != 0;
            if (by_tiles) {
                S.moved = S.pending;
                if (S.pending) swap_buffers(S.cur);  // the kernel wrote the pending order
                S.pending = false;
                S.ranked = true;
                S.handed_out = false;
                continue;
            }
            if (!ok(materialize(r, s), "materialize")) return PP_E_HIP;
            if (!ok(drop_ranks(r, s), "fill")) return PP_E_HIP;  // of an earlier push that no sort has followed
            e = launch_gpd64(r, s, target);
            if (!ok(e, "gather_push_deposit")) return PP_E_HIP;
        }
    }
    if (r->timing) {
        if (!ok(hipEventRecord(r->ev1, r->stream), "hipEventRecord")) return PP_E_HIP;
        r->t_pending = true;
    }
    for (int s = 0; s < PP_MAX_SPECIES; ++s)
        if (split && r->sp[s].active) {
            r->sp[s].sorted = false;
            r->sp[s].ranked = true;  // the kernel counted the new cells for the next sort
        }
    if (uses_line_solve(r)) {
        e = launch_line_solve(r);
        if (!ok(e, "line_solve")) return PP_E_HIP;
    }
    r->step += 1;
    return PP_OK;
}

pp_status pp_field_step(pp_run* r) {
    if (!r) return PP_E_ARG;
    hipError_t e = launch_field_step(r);
    if (!ok(e, "field_step")) return PP_E_HIP;
    const int every = r->p.gauss_filter_every;
    if (r->p.gauss_filter_passes > 0 && (every <= 1 || r->step % every == 0)) {
        e = launch_gauss_filter(r);
        if (!ok(e, "gauss_filter")) return PP_E_HIP;
    }
    // the step is done either way; relax_max_iter sweeps could not reach relax_tol
    return r->jac_converged ? PP_OK : PP_E_NOCONV;
}

pp_status pp_step(pp_run* r) {
    if (!r) return PP_E_ARG;
    if (r->p.time_order != 4) {
        pp_status st = pp_gather_push_deposit(r);
        if (st == PP_OK) st = pp_sort_particles(r, -1);
        if (st == PP_OK) st = pp_field_step(r);
        return st;
    }
    pp_status st = PP_OK;
    bool noconv = false;  // a substep's relaxation capped: the step still completes
    for (int k = 0; k < 3 && st == PP_OK; ++k) {
        use_relax_set(r, k < 2 ? 1 : 2);  // sets 1 and 2 hold the drifts (1-theta)/2 dt and theta dt
        r->dt_kick = FR_KICK[k] * r->p.dt;
        r->drift_ratio = FR_DRIFT[(k + 1) % 3] / FR_DRIFT[k];
        st = pp_gather_push_deposit(r);
        if (st == PP_OK) st = pp_sort_particles(r, -1);
        if (st == PP_OK) st = pp_field_step(r);
        if (st == PP_E_NOCONV) {
            noconv = true;
            st = PP_OK;
        }
    }
    use_relax_set(r, 0);
    r->dt_kick = r->p.dt;
    r->drift_ratio = 1.0;
    r->step -= 2;             // one step, three particle substeps
    r->rho_prev_step = -1;    // J is the last substep's: no continuity check across the step
    return st == PP_OK && noconv ? PP_E_NOCONV : st;
}

pp_status pp_sort_particles(pp_run* r, int32_t s) {
    if (!r || s < -1 || s >= PP_MAX_SPECIES) return PP_E_ARG;
    if (s >= 0 && !r->sp[s].active) return PP_E_STATE;
    return ok(launch_sort(r, s), "sort") ? PP_OK : PP_E_HIP;
}

pp_status pp_diagnostics(pp_run* r, uint32_t what, pp_diag* out) {
    if (!r || !out) return PP_E_ARG;
    double host[64];
    const int na = diag_acc_count();
    hipError_t e = launch_diag(r, what, host);
    if (!ok(e, "diagnostics")) return PP_E_HIP;
    std::memset(out, 0, sizeof(*out));
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        out->kinetic[s] = host[s];
        for (int d = 0; d < 3; ++d) out->momentum[s][d] = host[PP_MAX_SPECIES + 3 * s + d];
    }
    const int base = 4 * PP_MAX_SPECIES;
    out->field_E = host[base + 0];
    out->field_B = host[base + 1];
    out->field_Ex = host[base + 2];
    out->gauss_max = host[base + 3];
    const bool have_prev = host[na + 1] != 0.0;
    out->cc_max = have_prev ? host[base + 4] : NAN;
    out->divB_max = host[base + 5];
    const bool have_relax = host[na + 2] != 0.0;
    out->relax_resid_meas = have_relax ? (host[base + 7] > 0.0 ? host[base + 6] / host[base + 7] : host[base + 6]) : NAN;
    double rref = 0.0;
    const double V = 1.0;
    (void)V;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        const Species& S = r->sp[s];
        if (!S.active) continue;
        // mean number density n_s = w N_s / N_cells
        double ns = S.w * (double)S.n / (double)r->g.ncell;
        double v = std::fabs(S.q) * ns;
        if (v > rref) rref = v;
    }
    out->rho_ref = rref;
    out->relax_resid = r->jac_bound;
    out->relax_iters = r->jac_sweeps;
    out->flags = (int32_t)host[na];
    out->step = r->step;
    return PP_OK;
}

pp_status pp_get_particles(pp_run* r, int32_t s, pp_particles* out) {
    if (!r || !out || s < 0 || s >= PP_MAX_SPECIES) return PP_E_ARG;
    if (!r->sp[s].active) return PP_E_STATE;
    if (!ok(materialize(r, s), "materialize")) return PP_E_HIP;  // the buffers in sort order
    // the caller may write the positions it is handed: the next sort looks at them again
    if (r->p.precision == PP_PREC_FP64 && !ok(drop_ranks(r, s), "fill")) return PP_E_HIP;
    r->sp[s].handed_out = true;
    *out = r->sp[s].cur;
    return PP_OK;
}

pp_status pp_timing_enable(pp_run* r, int32_t enable) {
    if (!r) return PP_E_ARG;
    if (flush_timing(r) != PP_OK) return PP_E_HIP;
    if (enable && !r->ev0 && !ok(hipEventCreate(&r->ev0), "hipEventCreate")) return PP_E_HIP;
    if (enable && !r->ev1 && !ok(hipEventCreate(&r->ev1), "hipEventCreate")) return PP_E_HIP;
    r->timing = enable != 0;
    return PP_OK;
}

pp_status pp_timing_read(pp_run* r, double* ms_total, int64_t* launches) {
    if (!r || !ms_total || !launches) return PP_E_ARG;
    if (flush_timing(r) != PP_OK) return PP_E_HIP;
    *ms_total = r->t_ms;
    *launches = r->t_launches;
    r->t_ms = 0.0;
    r->t_launches = 0;
    return PP_OK;
}

pp_status pp_destroy(pp_run* r) {
    if (!r) return PP_E_ARG;
    if (r->stream) (void)hipStreamSynchronize(r->stream);
    else (void)hipDeviceSynchronize();
    release(r);
    delete r;
    return PP_OK;
}

}  // extern "C"
