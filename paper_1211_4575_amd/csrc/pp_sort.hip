// Per-cell particle sort (Sec. III: between the particle and field updates the particle
// arrays are sorted by cell for cache locality).
//
// FP64 form: particles in cell order, the cells tile by tile (order inside a cell unspecified).
// After a push by tiles the particle kernel has counted and ranked the particles of every new
// cell (ranked sort, as for the split form) or, of those far from their tile, named the cell;
// otherwise a counting sort by tile-major cell key
// (histogram -> exclusive scan -> scatter with atomic cursors).
//
// Split form: particles are laid out tile by tile (64 cells).  Every particle has a rank r
// inside its cell; a tile's particles are laid out in pairs of ranks (see pair_table below):
// pair round R holds, for every cell with at least 2R + 2 particles, its particles of ranks
// 2R and 2R + 1, and the pairs, numbered round by round with cells ascending, come in chunks
// of 64 -- 128 slots, the first particles of the chunk's pairs, then their second particles
// in the same order -- so that a wavefront taking 128 slots holds in lanes l and 64 + l two
// particles of one cell, and in a full round its 64 lanes hold the tile's 64 cells in order.
// The pairs past the last whole chunk and the last particle of a cell with an odd count
// follow singly, rank by rank, cells ascending; ranks of SORT_RCAP and beyond come last.
// After a push the particle kernel has already counted the particles of every new cell and
// ranked each particle inside it, so the sort is a per-tile round table, a scan over tiles
// and the destination slot of every particle, kept as a permutation (ranked sort): the next
// particle kernel moves the particles while it updates them, and reading them (or any other
// use of the order) applies the permutation first; batched runs do the same, with every
// phase one launch over all members.  The first sort of a
// species (arbitrary order) buckets by tile -- a count per tile, a scan, and a scatter whose
// positions come from block-aggregated atomics -- and then rebuilds the tile order tile by
// tile.
#include <type_traits>

#include "pp_device.hpp"
#include "pp_internal.hpp"

namespace pp {

struct KeyGeom {
    int n[3];
    int t[3];
    int nt[3];
};

__device__ __forceinline__ int32_t tile_key(const KeyGeom& G, int i, int j, int k) {
    const int ti = i / G.t[0], tj = j / G.t[1], tk = k / G.t[2];
    const int li = i - ti * G.t[0], lj = j - tj * G.t[1], lk = k - tk * G.t[2];
    const int tile = ti + G.nt[0] * (tj + G.nt[1] * tk);
    return tile * TILE_CELLS + li + G.t[0] * (lj + G.t[1] * lk);
}

// key of an FP64 particle: nearest cell centre
__device__ __forceinline__ int32_t key_f64(const KeyGeom& G, double x, double y, double z) {
    return tile_key(G, nearest_cell(x, G.n[0]), nearest_cell(y, G.n[1]), nearest_cell(z, G.n[2]));
}

__device__ __forceinline__ int32_t key_cell(const KeyGeom& G, int32_t cell) {
    // an index outside the box (not produced by the push) is binned with cell 0; the
    // particle kernel flags it when it finds the particle outside its tile
    if (cell < 0 || cell >= G.n[0] * G.n[1] * G.n[2]) cell = 0;
    const int i = cell % G.n[0];
    const int r = cell / G.n[0];
    const int j = r % G.n[1];
    const int k = r / G.n[1];
    return tile_key(G, i, j, k);
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        p[q] = v;
}

// and one entry elsewhere (nullptr: none)
__global__ void k_copy_i32(int32_t* dst, const int32_t* src, int64_t n, int32_t* one, int32_t value) {
    if (one && blockIdx.x == 0 && threadIdx.x == 0) *one = value;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        dst[q] = src[q];
}

__global__ void __launch_bounds__(256) k_hist_f64(KeyGeom G, const double* __restrict__ x, const double* __restrict__ y,
                                                  const double* __restrict__ z, int64_t n, int32_t* count) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    atomicAdd(count + key_f64(G, x[p], y[p], z[p]), 1);
}

// Block-level aggregation for the bucketing sort: a block of 256 threads handles 1024
// consecutive particles; each wavefront groups its lanes by destination tile (ballot loop),
// the group leader reserves slots in a small LDS table keyed by tile, and after a barrier
// one global atomic per distinct tile of the block reserves the block's run in that tile.
// When a block's particles come from one or two source tiles, its destinations are a few
// tiles of their neighbourhood; in arbitrary order (a fresh load) nearly every particle of a
// block has its own tile, the table fills at once and the probe limit sends the rest straight
// to the global counters.
constexpr int AGG_SLOTS = 128;
constexpr int AGG_PROBES = 8;
constexpr int AGG_PER_THREAD = 4;
constexpr int AGG_BLOCK = 256 * AGG_PER_THREAD;

// LDS slot of a key (open addressing, at most AGG_PROBES probes); -1 when none is free
__device__ __forceinline__ int agg_slot(int32_t* keys, int32_t key) {
    const unsigned h = ((unsigned)key * 2654435761u) >> 25;  // 7 bits
    for (int probe = 0; probe < AGG_PROBES; ++probe) {
        const int sl = (int)((h + (unsigned)probe) & (AGG_SLOTS - 1));
        const int32_t prev = atomicCAS(&keys[sl], -1, key);
        if (prev == -1 || prev == key) return sl;
    }
    return -1;
}

__device__ __forceinline__ void tile_count_block(const KeyGeom& G, const int32_t* __restrict__ cell, int64_t n,
                                                 int32_t* __restrict__ count, int64_t blk) {
    __shared__ int32_t keys[AGG_SLOTS];
    __shared__ int32_t cnt[AGG_SLOTS];
    for (int i = threadIdx.x; i < AGG_SLOTS; i += 256) {
        keys[i] = -1;
        cnt[i] = 0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t base = blk * AGG_BLOCK;
    for (int k = 0; k < AGG_PER_THREAD; ++k) {
        const int64_t p = base + k * 256 + threadIdx.x;
        const bool active = p < n;
        const int32_t tile = active ? key_cell(G, cell[p]) / TILE_CELLS : 0;
        uint64_t todo = __ballot(active);
        while (todo) {
            const int leader = __ffsll((unsigned long long)todo) - 1;
            const int32_t lk = __shfl(tile, leader, 64);
            const uint64_t grp = __ballot(active && tile == lk) & todo;
            if (lane == leader) {
                const int sl = agg_slot(keys, lk);
                if (sl >= 0)
                    atomicAdd(&cnt[sl], (int32_t)__popcll(grp));
                else
                    atomicAdd(count + lk, (int32_t)__popcll(grp));
            }
            todo &= ~grp;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < AGG_SLOTS; i += 256)
        if (keys[i] >= 0 && cnt[i] > 0) atomicAdd(count + keys[i], cnt[i]);
}

__global__ void __launch_bounds__(256) k_tile_count(KeyGeom G, const int32_t* __restrict__ cell, int64_t n,
                                                    int32_t* __restrict__ count) {
    tile_count_block(G, cell, n, count, blockIdx.x);
}

template <typename T>
struct ScatterArgs {
    KeyGeom G;
    int64_t n;
    const int32_t* cell;
    const T* pos[3];
    const T* u[3];
    const int64_t* id;
    int32_t* cell_o;
    T* pos_o[3];
    T* u_o[3];
    int64_t* id_o;
    int32_t* cursor;  // FP64 form: cell-bin starts (consumed); split form: tile starts (consumed)
};

template <typename T>
__global__ void __launch_bounds__(256) k_scatter(ScatterArgs<T> A) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= A.n) return;
    const int32_t key = key_f64(A.G, (double)A.pos[0][p], (double)A.pos[1][p], (double)A.pos[2][p]);
    const int32_t dst = atomicAdd(A.cursor + key, 1);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        A.pos_o[d][dst] = A.pos[d][p];
        A.u_o[d][dst] = A.u[d][p];
    }
    if (A.id) A.id_o[dst] = A.id[p];
}

// split form: bucket by tile with block-level aggregation (see k_tile_count); a wavefront's
// particles bound for one tile get consecutive slots in their source order
template <typename T>
__device__ __forceinline__ void scatter_tiles_block(const ScatterArgs<T>& A, int64_t blk) {
    __shared__ int32_t keys[AGG_SLOTS];
    __shared__ int32_t cnt[AGG_SLOTS];
    __shared__ int32_t gbase[AGG_SLOTS];
    for (int i = threadIdx.x; i < AGG_SLOTS; i += 256) {
        keys[i] = -1;
        cnt[i] = 0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t base = blk * AGG_BLOCK;
    int my_slot[AGG_PER_THREAD];
    int32_t my_off[AGG_PER_THREAD];
#pragma unroll
    for (int k = 0; k < AGG_PER_THREAD; ++k) {
        const int64_t p = base + k * 256 + threadIdx.x;
        const bool active = p < A.n;
        const int32_t tile = active ? key_cell(A.G, A.cell[p]) / TILE_CELLS : 0;
        my_slot[k] = -2;
        my_off[k] = 0;
        uint64_t todo = __ballot(active);
        while (todo) {
            const int leader = __ffsll((unsigned long long)todo) - 1;
            const int32_t lk = __shfl(tile, leader, 64);
            const uint64_t grp = __ballot(active && tile == lk) & todo;
            int sl = 0;
            int32_t off = 0;
            if (lane == leader) {
                sl = agg_slot(keys, lk);
                if (sl >= 0)
                    off = atomicAdd(&cnt[sl], (int32_t)__popcll(grp));
                else
                    off = atomicAdd(A.cursor + lk, (int32_t)__popcll(grp));  // table full: direct
            }
            sl = __shfl(sl, leader, 64);
            off = __shfl(off, leader, 64);
            if ((grp >> lane) & 1ull) {
                my_slot[k] = sl;
                my_off[k] = off + (int32_t)__popcll(grp & ((1ull << lane) - 1ull));
            }
            todo &= ~grp;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < AGG_SLOTS; i += 256)
        if (keys[i] >= 0) gbase[i] = atomicAdd(A.cursor + keys[i], cnt[i]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < AGG_PER_THREAD; ++k) {
        const int64_t p = base + k * 256 + threadIdx.x;
        if (p >= A.n || my_slot[k] == -2) continue;
        const int32_t dst = my_slot[k] >= 0 ? gbase[my_slot[k]] + my_off[k] : my_off[k];
        A.cell_o[dst] = A.cell[p];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            A.pos_o[d][dst] = A.pos[d][p];
            A.u_o[d][dst] = A.u[d][p];
        }
        if (A.id) A.id_o[dst] = A.id[p];
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_scatter_tiles(ScatterArgs<T> A) {
    scatter_tiles_block(A, blockIdx.x);
}

// largest tile population (the fixed-point current's scale depends on it)
__global__ void __launch_bounds__(256) k_tile_max(const int32_t* __restrict__ start, int64_t ntiles, int32_t* out) {
    int m = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < ntiles; t += (int64_t)gridDim.x * blockDim.x) {
        const int c = start[t + 1] - start[t];
        m = c > m ? c : m;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int other = __shfl_xor(m, o, 64);
        m = other > m ? other : m;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(out, m);
}

// The round table of one tile, built by one wavefront with lane = local cell, k = the
// particles the lane's cell holds in the table (min(count, SORT_RCAP)), rmax = the largest k:
// entry r (r < rmax) goes to put(r, entry), called by lane r - base in the pass over ranks
// base .. base + 63.  nchunk = whole chunks of 64 pairs, intable = particles in the table.
// Bound by its instructions, some fifty a round: the rounds that all cells take part in are written
// without counting (128^3 at 32 per cell and species 101 -> 75 us, 512x256 at 64 22 -> 16).
template <class Put>
__device__ __forceinline__ void pair_table(int k, int rmax, Put put, int32_t& nchunk, int32_t& intable) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = lane == 0 ? 0ull : ((1ull << lane) - 1ull);
    int pairs = k >> 1, least = k;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        pairs += __shfl_xor(pairs, o, 64);
        const int other = __shfl_xor(least, o, 64);
        least = other < least ? other : least;
    }
    nchunk = pairs >> 6;
    // the rounds that every cell has a pair for are whole chunks: nothing to count in them
    const int full = __builtin_amdgcn_readfirstlane(least) & ~1;
    int32_t pb = 32 * full, sb = 0;  // pairs of the rounds before, single particles of the ranks before
    for (int base = 0; base < rmax; base += 64) {
        const int nr = rmax - base < 64 ? rmax - base : 64;
        const int first = full > base ? (full - base < nr ? full - base : nr) : 0;
        RoundEntry mine{0ull, 0ull, 0, 0};
        if (lane < first) mine = RoundEntry{~0ull, 0ull, 32 * ((base + lane) & ~1), 0};
        // the two ranks 2R, 2R + 1 of a pair round share its pair mask (base is even)
        for (int rr = first; rr < nr; rr += 2) {
            const int r = base + rr;
            const uint64_t pm = __ballot(k >= r + 2);  // cells with a pair of ranks r, r + 1
            const int32_t g = pb + (int32_t)__popcll(pm & below);
            const bool chunked = ((pm >> lane) & 1ull) && g < (nchunk << 6);
            const uint64_t sm0 = __ballot(k > r && !chunked);
            const uint64_t sm1 = __ballot(k > r + 1 && !chunked);
            const int32_t sb1 = sb + (int32_t)__popcll(sm0);
            if (lane == rr || lane == rr + 1) {
                mine.pmask = pm;
                mine.smask = lane == rr ? sm0 : sm1;
                mine.pbefore = pb;
                mine.sbefore = lane == rr ? sb : sb1;
            }
            // a last rank without its partner (nr odd) counts only its own single particles
            sb = rr + 1 < nr ? sb1 + (int32_t)__popcll(sm1) : sb1;
            pb += (int32_t)__popcll(pm);
        }
        if (lane < nr) put(base + lane, mine);
    }
    intable = (nchunk << 7) + sb;
}

// Slot inside its tile of the rank-r particle (r < SORT_RCAP) of local cell lc.
__device__ __forceinline__ int32_t pair_slot(const RoundEntry& e, int32_t nchunk, int r, int lc) {
    const uint64_t below = lc == 0 ? 0ull : ((1ull << lc) - 1ull);
    if ((e.pmask >> lc) & 1ull) {
        const int32_t g = e.pbefore + (int32_t)__popcll(e.pmask & below);
        if (g < (nchunk << 6)) return ((g >> 6) << 7) + ((r & 1) << 6) + (g & 63);
    }
    return (nchunk << 7) + e.sbefore + (int32_t)__popcll(e.smask & below);
}

// Rebuild of one tile in the tile order (one workgroup per tile): ranks inside cells from LDS
// atomics, the round table from ballots over the 64 cells, then a gather copy so the
// writes are coalesced (the reads stay inside the tile's segment).
constexpr int REORDER_RMAX = 1024;

template <typename T>
struct ReorderArgs {
    KeyGeom G;
    int64_t ntiles;
    const int32_t* start;
    const int32_t* cell;
    const T* pos[3];
    const T* u[3];
    const int64_t* id;
    int32_t* cell_o;
    T* pos_o[3];
    T* u_o[3];
    int64_t* id_o;
    int32_t* rank;  // scratch, one per particle
    int32_t* perm;  // scratch, one per particle
};

template <typename T>
__device__ __forceinline__ void tile_reorder_tile(const ReorderArgs<T>& A, int64_t tile) {
    __shared__ int32_t cnt[TILE_CELLS];
    __shared__ RoundEntry tab[SORT_RCAP];
    __shared__ int32_t nch, intab;
    __shared__ int32_t ovf;
    if (tile >= A.ntiles) return;
    const int32_t s = A.start[tile], e = A.start[tile + 1];
    if (threadIdx.x < TILE_CELLS) cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) ovf = 0;
    __syncthreads();
    for (int32_t i = s + threadIdx.x; i < e; i += 256) {
        const int32_t lc = key_cell(A.G, A.cell[i]) % TILE_CELLS;
        int32_t r = atomicAdd(&cnt[lc], 1);
        r = r < REORDER_RMAX ? r : REORDER_RMAX;
        A.rank[i] = (lc << 24) | r;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const int k = cnt[lane] < SORT_RCAP ? cnt[lane] : SORT_RCAP;
        int mx = k;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const int other = __shfl_xor(mx, o, 64);
            mx = other > mx ? other : mx;
        }
        int32_t nc, it;
        pair_table(k, mx, [&](int r, const RoundEntry& en) { tab[r] = en; }, nc, it);
        if (lane == 0) {
            nch = nc;
            intab = it;
        }
    }
    __syncthreads();
    for (int32_t i = s + threadIdx.x; i < e; i += 256) {
        const int32_t rk = A.rank[i];
        const int lc = rk >> 24;
        const int r = rk & 0xFFFFFF;
        const int32_t pos = r < SORT_RCAP ? pair_slot(tab[r], nch, r, lc) : intab + atomicAdd(&ovf, 1);
        A.perm[s + pos] = i;
    }
    __threadfence_block();
    __syncthreads();
    for (int32_t j = s + threadIdx.x; j < e; j += 256) {
        const int32_t i = A.perm[j];
        A.cell_o[j] = A.cell[i];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            A.pos_o[d][j] = A.pos[d][i];
            A.u_o[d][j] = A.u[d][i];
        }
        if (A.id) A.id_o[j] = A.id[i];
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_tile_reorder(ReorderArgs<T> A) {
    tile_reorder_tile(A, blockIdx.x);
}

// ---- ranked sort (after a push) ---------------------------------------------------------
// The particle kernel left, for each species, the number of particles of each cell at the new
// positions (cnt), and a rank word per particle:
//   slot << 20 | r   the r-th of its tile's particles bound for destination cell `slot` of the
//                    tile's neighbourhood; base[tile][slot] + r is its rank in that cell,
//   bit 31 | rank    bound further away (flagged states) or past r's range: its rank itself,
//   -1               left out (found outside its tile).
// The ranks of a cell are 0 .. cnt - 1, each once.  Where a particle of rank r in local cell lc
// goes inside its tile is in the tile's round table (pair_slot).  Ranks of SORT_RCAP and beyond
// go to an overflow tail of the tile (order there unspecified).
//
// Three launches over every species (four past SORT_SCAN_ONE tiles): the round tables, a scan of the
// tile totals (which also finds the largest tile; an atomic maximum per tile on one address had cost
// 20 us for 2048 tiles) and the permutation.  In small boxes their latency counts, in large ones the
// permutation's bytes: a rank word read and an entry written per particle, the entries of
// particles that change tile one by one into partial lines.  us per step, before (five to seven
// launches a species, cell and completed rank read back, a cleared permutation) and now: 2 x
// 4.2e6 particles in 128x32x32, 170 and 55; 2 x 6.7e7 in 128^3, 1120 and 700; 2 x 3.3e4 in 16^3,
// 46 and 15.

struct RankedArgs {
    Geom G;
    int tsh[3];             // log2 of the tile's sides
    int32_t* cnt;           // per cell (read and cleared by the table kernel)
    RoundEntry* rounds;     // ntiles * SORT_RCAP
    int32_t* tot;           // ntiles + 1: tile totals, scanned into the next tile starts
    int32_t* rtot;          // ntiles: particles in the table's rounds
    int32_t* nchunk;        // ntiles: whole chunks of 64 pairs
    int32_t* ovf;           // ntiles: overflow cursors
    int32_t* tile_max;      // largest tile population; PP_MAX_SPECIES entries on, that of the order before
    const int32_t* start;   // current tile starts (source order)
    const int32_t* rank;    // n rank words
    const int32_t* base;    // ntiles * slots
    int32_t* perm;          // n: perm[slot] = particle
    int64_t n;
    const int32_t* cell;
    // FP64 form: cnt by bin (64 per tile), start and next_bins bin starts, pre the starts of a
    // tile's cells inside it; no round table, rank base or overflow
    int32_t* pre;
    int32_t* next_bins;
};

// FP64 form, one wavefront per tile: the cells' starts inside the tile and its total
__device__ __forceinline__ void bin_prefix_tile(const RankedArgs& A, int64_t t) {
    const int lane = threadIdx.x & 63;
    if (t >= A.G.ntiles) return;
    const int32_t ranked = gl(A.cnt)[t * TILE_CELLS + lane], named = gl(A.cnt)[A.G.nbins + t * TILE_CELLS + lane];
    const int32_t c = (ranked < F64_RANKS ? ranked : F64_RANKS) + named;
    gl(A.cnt)[t * TILE_CELLS + lane] = 0;
    int32_t incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    gl(A.pre)[t * TILE_CELLS + lane] = incl - c;
    if (lane == 63) gl(A.tot)[t] = incl;
}

// one wavefront per tile: lane = local cell
__device__ __forceinline__ void round_table_tile(const RankedArgs& A, int64_t t) {
    const int lane = threadIdx.x & 63;
    const Geom& G = A.G;
    if (t >= G.ntiles) return;
    const int ti = (int)(t % G.nt[0]), tj = (int)((t / G.nt[0]) % G.nt[1]), tk = (int)(t / ((int64_t)G.nt[0] * G.nt[1]));
    const int li = lane & (G.t[0] - 1), lj = (lane >> A.tsh[0]) & (G.t[1] - 1), lk = lane >> (A.tsh[0] + A.tsh[1]);
    const int i = ti * G.t[0] + li, j = tj * G.t[1] + lj, k = tk * G.t[2] + lk;
    int c = 0;
    if (lk < G.t[2] && i < G.n[0] && j < G.n[1] && k < G.n[2]) {
        const int64_t g = (int64_t)i + (int64_t)G.n[0] * (j + (int64_t)G.n[1] * k);
        c = gl(A.cnt)[g];
        gl(A.cnt)[g] = 0;
    }
    int tot = c, mx = c;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        tot += __shfl_xor(tot, o, 64);
        const int other = __shfl_xor(mx, o, 64);
        mx = other > mx ? other : mx;
    }
    const int rmax = mx < SORT_RCAP ? mx : SORT_RCAP;
    const int kc = c < SORT_RCAP ? c : SORT_RCAP;
    int32_t nchunk, intable;
    pair_table(kc, rmax, [&](int r, const RoundEntry& e) { gl(A.rounds)[t * SORT_RCAP + r] = e; }, nchunk, intable);
    if (lane == 0) {
        gl(A.tot)[t] = tot;
        gl(A.rtot)[t] = intable;
        gl(A.nchunk)[t] = nchunk;
        gl(A.ovf)[t] = 0;
    }
}

// Exclusive scan of data[0..n), from carry on, in place by one workgroup of SCAN1_BS threads: four
// entries a thread at a time, the next ones in flight meanwhile.  Returns the total (carry included)
// and the largest entry (to every thread).
constexpr int SCAN1_BS = 1024;

__device__ __forceinline__ void scan_workgroup(int32_t* data, int64_t n, int32_t carry, int32_t& total, int32_t& largest) {
    __shared__ int32_t wsum[2][SCAN1_BS / 64];
    __shared__ int32_t wmax[SCAN1_BS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t mx = 0;
    int32_t v[4], nx[4];
    auto load = [&](int64_t base, int32_t* x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t q = base + 4 * (int64_t)threadIdx.x + e;
            x[e] = q < n ? data[q] : 0;
        }
    };
    load(0, v);
    int buf = 0;
    for (int64_t base = 0; base < n; base += 4 * SCAN1_BS, buf ^= 1) {
        load(base + 4 * SCAN1_BS, nx);
        const int32_t sum = v[0] + v[1] + v[2] + v[3];
        int32_t incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = v[e] > mx ? v[e] : mx;
        if (lane == 63) wsum[buf][wave] = incl;
        __syncthreads();  // two buffers: the next round writes the other one
        int32_t before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < SCAN1_BS / 64; ++w) {
            const int32_t s = wsum[buf][w];
            before += w < wave ? s : 0;
            all += s;
        }
        int32_t run = carry + before + incl - sum;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t q = base + 4 * (int64_t)threadIdx.x + e;
            if (q < n) data[q] = run;
            run += v[e];
            v[e] = nx[e];
        }
        carry += all;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int32_t y = __shfl_xor(mx, o, 64);
        mx = y > mx ? y : mx;
    }
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    for (int w = 0; w < SCAN1_BS / 64; ++w) mx = wmax[w] > mx ? wmax[w] : mx;
    total = carry;
    largest = mx;
}

// What follows from the scan as a whole: the last tile start and the largest tile population.  The
// ranks fill every slot below the total; the slots past it (particles left out) hold no particle.
__device__ __forceinline__ void scan_results(const RankedArgs& A, int32_t total, int32_t largest) {
    if (threadIdx.x == 0) {
        gl(A.tot)[A.G.ntiles] = total;
        // the ranges the particles still lie in until they are moved, and the new ones
        gl(A.tile_max)[PP_MAX_SPECIES] = *gl(A.tile_max);
        *gl(A.tile_max) = largest;
    }
    for (int64_t q = total + (int64_t)threadIdx.x; q < A.n; q += SCAN1_BS) gl(A.perm)[q] = -1;
}

// Next tile starts by one workgroup.
__device__ __forceinline__ void ranked_scan(const RankedArgs& A) {
    int32_t total, largest;
    scan_workgroup(gl(A.tot), A.G.ntiles, 0, total, largest);
    scan_results(A, total, largest);
}

// The same by a workgroup per chunk, in two launches: the chunks' sums and largest entries (nchunks of
// each in sums), then every chunk from the sum of those before it.  11 us with the launch between them
// at any size, against 4.8 of one workgroup for 4096 tiles, 11.2 for 16384, 19.8 for 32768 (128^3) and 155
// for 262144 (256^3).
constexpr int SORT_CHUNK = 4 * SCAN1_BS;
constexpr int64_t SORT_SCAN_ONE = 16384;  // most tiles that one workgroup scans

// sum and largest over a workgroup, to every thread
__device__ __forceinline__ void reduce_workgroup(int32_t& before, int32_t& all, int32_t& largest) {
    __shared__ int32_t sh[3][SCAN1_BS / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        before += __shfl_xor(before, o, 64);
        all += __shfl_xor(all, o, 64);
        const int32_t y = __shfl_xor(largest, o, 64);
        largest = y > largest ? y : largest;
    }
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = before;
        sh[1][threadIdx.x >> 6] = all;
        sh[2][threadIdx.x >> 6] = largest;
    }
    __syncthreads();
    before = all = largest = 0;
#pragma unroll
    for (int w = 0; w < SCAN1_BS / 64; ++w) {
        before += sh[0][w];
        all += sh[1][w];
        largest = sh[2][w] > largest ? sh[2][w] : largest;
    }
}

__device__ __forceinline__ void chunk_sum(const RankedArgs& A, int32_t* sums, int nchunks) {
    int32_t before = 0, all = 0, largest = 0;
    const int64_t base = (int64_t)blockIdx.x * SORT_CHUNK + threadIdx.x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t q = base + e * SCAN1_BS;
        const int32_t v = q < A.G.ntiles ? gl(A.tot)[q] : 0;
        all += v;
        largest = v > largest ? v : largest;
    }
    reduce_workgroup(before, all, largest);
    if (threadIdx.x == 0) {
        sums[blockIdx.x] = all;
        sums[nchunks + blockIdx.x] = largest;
    }
}

__device__ __forceinline__ void chunk_scan(const RankedArgs& A, const int32_t* sums, int nchunks) {
    int32_t before = 0, all = 0, largest = 0;
    for (int c = threadIdx.x; c < nchunks; c += SCAN1_BS) {
        const int32_t v = sums[c], m = sums[nchunks + c];
        before += c < (int)blockIdx.x ? v : 0;
        all += v;
        largest = m > largest ? m : largest;
    }
    reduce_workgroup(before, all, largest);
    const int64_t base = (int64_t)blockIdx.x * SORT_CHUNK, left = A.G.ntiles - base;
    int32_t end, mx;
    scan_workgroup(gl(A.tot) + base, left < SORT_CHUNK ? left : SORT_CHUNK, before, end, mx);
    if (blockIdx.x == 0) scan_results(A, all, largest);
}

// What a particle bound for one destination cell needs: the cell's tile and place in it, the
// tile's next range, whole chunks and table total, and the rank the source tile starts from.
struct DestCell {
    int32_t tile_lc;  // tile << 6 | local cell
    int32_t d0, nd;
    int32_t nchunk;
    int32_t base;
};

__device__ __forceinline__ DestCell dest_cell(const RankedArgs& A, int gx, int gy, int gz, int32_t base) {
    const Geom& G = A.G;
    const int tx = gx >> A.tsh[0], ty = gy >> A.tsh[1], tz = gz >> A.tsh[2];
    const int32_t t = tx + G.nt[0] * (ty + G.nt[1] * tz);
    const int lc = (gx & (G.t[0] - 1)) + ((gy & (G.t[1] - 1)) << A.tsh[0]) + ((gz & (G.t[2] - 1)) << (A.tsh[0] + A.tsh[1]));
    DestCell c;
    c.tile_lc = (t << 6) | lc;
    c.d0 = gl(A.tot)[t];
    c.nd = gl(A.tot)[t + 1] - c.d0;
    c.nchunk = gl(A.nchunk)[t];
    c.base = base;
    return c;
}

// perm[slot] = particle for the particles of source tile T (one workgroup per tile).  The tile's
// destination cells -- a few hundred, against thousands of particles -- are looked up once, in
// LDS; a particle then takes one load of its rank word and one of its round-table entry.  Most
// particles stay in the tile: their entries are collected in an LDS image of T's next range and
// written out in order (entries that particles from neighbouring tiles fill are written by those
// tiles' workgroups, directly); the rest, and every entry of a range larger than the image, are
// written directly.  Each thread issues the loads of PERM_PER particles before it uses any.
// Ranks past the round table take slots at the end of their tile with one atomic per wavefront
// and tile, lanes in lane order (bunched plasmas put hundreds of particles in one cell).
// Bound by the latency of its loads, so by the workgroups a CU holds: seven, at 19 KB with the
// image in 16 bits (a particle's place in its tile) and 20 bytes a cell; four waves of 70 registers
// each, no fewer (64 spill).  The first rank words are loaded before the cells are looked up, the
// next ones a block ahead.  128^3, 2 x 6.7e7: 716 us with 29 KB and the loads in turn, 582 now;
// 128x32x32, 2 x 4.2e6: 48 and 39; eight serving runs: 109 and 82.
constexpr int PERM_PER = 4;
constexpr int PERM_BLOCK = 256 * PERM_PER;
constexpr int PERM_IMG = 4608, IMG_NONE = 0xFFFF;

__device__ __forceinline__ void ranked_perm_tile(const RankedArgs& A, int64_t T, int32_t* lds) {
    const Geom& G = A.G;
    if (T >= G.ntiles) return;
    const int32_t ss = gl(A.start)[T], se = gl(A.start)[T + 1];
    const int32_t d0 = gl(A.tot)[T], nd = gl(A.tot)[T + 1] - d0;
    const bool staged = nd <= PERM_IMG && se - ss < IMG_NONE;
    uint16_t* img = (uint16_t*)lds;  // particle - ss, IMG_NONE: not one of this tile's
    DestCell* dest = (DestCell*)(lds + PERM_IMG / 2);
    if (staged)
        for (int32_t q = threadIdx.x; q < nd; q += blockDim.x) img[q] = IMG_NONE;
    // the first rank words are on their way while the cells are looked up
    int32_t wn[PERM_PER];
    auto load_ranks = [&](int64_t b) {
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            const int64_t p = b + threadIdx.x + k * 256;
            wn[k] = p < se ? gl(A.rank)[p] : -1;
        }
    };
    load_ranks(ss);
    const int e0 = G.dest_ext(0), e1 = G.dest_ext(1), slots = e0 * e1 * G.dest_ext(2);
    const uint32_t row = (uint32_t)T / (uint32_t)G.nt[0], layer = row / (uint32_t)G.nt[1];  // numbered in 32 bits
    const int ox = (int)((uint32_t)T - row * (uint32_t)G.nt[0]) * G.t[0],
              oy = (int)(row - layer * (uint32_t)G.nt[1]) * G.t[1], oz = (int)layer * G.t[2];
    const bool eight = e0 == 8 && e1 == 8;  // 4x4x4 tiles: no divisions
    if (se > ss)
        for (int q = threadIdx.x; q < slots; q += blockDim.x) {
            const int z = eight ? q >> 6 : q / (e0 * e1), r = q - z * e0 * e1;
            const int y = eight ? r >> 3 : r / e0, x = r - y * e0;
            dest[q] = dest_cell(A, e0 == 1 ? 0 : wrap_near(ox + x - DEST_HALO, G.n[0]),
                                e1 == 1 ? 0 : wrap_near(oy + y - DEST_HALO, G.n[1]),
                                G.n[2] == 1 ? 0 : wrap_near(oz + z - DEST_HALO, G.n[2]), gl(A.base)[T * slots + q]);
        }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int64_t b = ss; b < se; b += PERM_BLOCK) {
        int32_t w[PERM_PER], r[PERM_PER];
        DestCell c[PERM_PER];
        RoundEntry e[PERM_PER];
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) w[k] = wn[k];
        load_ranks(b + PERM_BLOCK);
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            c[k] = dest[w[k] >= 0 ? w[k] >> 20 : 0];
            r[k] = w[k] >= 0 ? c[k].base + (w[k] & 0xFFFFF) : -1;
            if (w[k] < -1) {  // its rank itself, in a cell that may lie anywhere
                const int32_t g = gl(A.cell)[b + threadIdx.x + k * 256];
                const bool in = g >= 0 && g < G.ncell;
                const int gx = in ? g % G.n[0] : 0, gr = in ? g / G.n[0] : 0;
                c[k] = dest_cell(A, gx, gr % G.n[1], gr / G.n[1], 0);
                r[k] = w[k] & 0x7FFFFFFF;
            }
        }
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k)
            e[k] = gl(A.rounds)[(int64_t)(c[k].tile_lc >> 6) * SORT_RCAP + (r[k] >= 0 && r[k] < SORT_RCAP ? r[k] : 0)];
        int32_t pos[PERM_PER];
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            // computed for every particle and selected (no branch the table reads could sink into)
            const bool in_table = r[k] >= 0 && r[k] < SORT_RCAP;
            const int32_t ps = pair_slot(e[k], c[k].nchunk, in_table ? r[k] : 0, c[k].tile_lc & 63);
            pos[k] = in_table ? ps : 0;
        }
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            const bool over = r[k] >= SORT_RCAP;
            const int32_t t = c[k].tile_lc >> 6;
            uint64_t todo = __ballot(over);
            while (todo) {
                const int leader = __ffsll((unsigned long long)todo) - 1;
                const int32_t lt = __shfl(t, leader, 64);
                const uint64_t grp = __ballot(over && t == lt) & todo;
                int32_t first = 0;
                if (lane == leader) first = gl(A.rtot)[lt] + atomicAdd(gl(A.ovf) + lt, (int32_t)__popcll(grp));
                first = __shfl(first, leader, 64);
                if (over && t == lt) pos[k] += first + (int32_t)__popcll(grp & ((1ull << lane) - 1ull));
                todo &= ~grp;
            }
        }
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            if (r[k] < 0 || pos[k] >= c[k].nd) continue;
            const int32_t p = (int32_t)(b + threadIdx.x + k * 256);
            if (staged && (c[k].tile_lc >> 6) == (int32_t)T)
                img[pos[k]] = (uint16_t)(p - ss);
            else
                gl(A.perm)[c[k].d0 + pos[k]] = p;
        }
    }
    __syncthreads();
    if (staged)
        for (int32_t q = threadIdx.x; q < nd; q += blockDim.x) {
            const int32_t v = img[q];
            if (v != IMG_NONE) gl(A.perm)[d0 + q] = ss + v;
        }
}

// FP64 form: first slot of a bin, bin of a cell, cell of a destination window's entry along an axis, slot
// of a particle that only names its bin (see bin_perm_tile)
__device__ __forceinline__ int32_t bin_first(const RankedArgs& A, int32_t bin) {
    return gl(A.tot)[bin / TILE_CELLS] + gl(A.pre)[bin];
}

__device__ __forceinline__ int32_t bin_of_cell(const RankedArgs& A, int gx, int gy, int gz) {
    const Geom& G = A.G;
    const int32_t t = (gx >> A.tsh[0]) + G.nt[0] * ((gy >> A.tsh[1]) + G.nt[1] * (gz >> A.tsh[2]));
    return t * TILE_CELLS + (gx & (G.t[0] - 1)) + ((gy & (G.t[1] - 1)) << A.tsh[0]) +
           ((gz & (G.t[2] - 1)) << (A.tsh[0] + A.tsh[1]));
}

__device__ __forceinline__ int window_node(int org, int x, int n) { return n == 1 ? 0 : wrap_near(org + x - DEST_HALO, n); }

__device__ __forceinline__ int32_t named_slot(const RankedArgs& A, int32_t bin) {
    const int32_t end = bin % TILE_CELLS == TILE_CELLS - 1 ? gl(A.tot)[bin / TILE_CELLS + 1] : bin_first(A, bin + 1);
    return end - atomicSub(gl(A.cnt) + A.G.nbins + bin, 1);
}

// FP64 form: perm[slot] = particle for the particles of source tile T, and T's next bin starts.  A
// rank word holds the destination cell and the rank in it (slot << 20 | rank), so a particle's slot is
// one LDS lookup away, or the cell's bin alone (bit 31 | bin: far from its tile, or past F64_RANKS in
// the cell); those fill the cell's range from its end, counting their number down to zero.  Positions
// are not looked at: the slots are a permutation whatever has become of them since the push.
__device__ __forceinline__ void bin_perm_tile(const RankedArgs& A, int64_t T, int32_t* lds) {
    const Geom& G = A.G;
    if (T >= G.ntiles) return;
    const int32_t ss = gl(A.start)[T * TILE_CELLS], se = gl(A.start)[(T + 1) * TILE_CELLS];
    const int32_t d0 = gl(A.tot)[T], nd = gl(A.tot)[T + 1] - d0;
    const bool staged = nd <= PERM_IMG && se - ss < IMG_NONE;
    uint16_t* img = (uint16_t*)lds;
    int32_t* first = lds + PERM_IMG / 2;  // first slot of each destination cell
    if (threadIdx.x < TILE_CELLS) {
        gl(A.next_bins)[T * TILE_CELLS + threadIdx.x] = d0 + gl(A.pre)[T * TILE_CELLS + threadIdx.x];
        if (T == G.ntiles - 1 && threadIdx.x == 0) gl(A.next_bins)[G.nbins] = gl(A.tot)[G.ntiles];
    }
    if (staged)
        for (int32_t q = threadIdx.x; q < nd; q += blockDim.x) img[q] = IMG_NONE;
    const int e0 = G.dest_ext(0), e1 = G.dest_ext(1), slots = e0 * e1 * G.dest_ext(2);
    const int ox = (int)(T % G.nt[0]) * G.t[0], oy = (int)((T / G.nt[0]) % G.nt[1]) * G.t[1],
              oz = (int)(T / ((int64_t)G.nt[0] * G.nt[1])) * G.t[2];
    if (se > ss)
        for (int q = threadIdx.x; q < slots; q += blockDim.x) {
            const int z = q / (e0 * e1), r = q - z * e0 * e1, y = r / e0, x = r - y * e0;
            first[q] = bin_first(A, bin_of_cell(A, window_node(ox, x, G.n[0]), window_node(oy, y, G.n[1]),
                                                window_node(oz, z, G.n[2])));
        }
    __syncthreads();
    for (int64_t b = ss; b < se; b += PERM_BLOCK) {
        int32_t w[PERM_PER];
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            const int64_t p = b + threadIdx.x + k * 256;
            w[k] = p < se ? gl(A.rank)[p] : 0;
        }
#pragma unroll
        for (int k = 0; k < PERM_PER; ++k) {
            const int64_t p = b + threadIdx.x + k * 256;
            if (p >= se) continue;
            int32_t q;
            if (w[k] >= 0) {
                q = first[w[k] >> 20] + (w[k] & 0xFFFFF);
            } else {
                q = named_slot(A, w[k] & 0x7FFFFFFF);
            }
            if (staged && q >= d0 && q < d0 + nd)
                img[q - d0] = (uint16_t)(p - ss);
            else
                gl(A.perm)[q] = (int32_t)p;
        }
    }
    __syncthreads();
    if (staged)
        for (int32_t q = threadIdx.x; q < nd; q += blockDim.x) {
            const int32_t v = img[q];
            if (v != IMG_NONE) gl(A.perm)[d0 + q] = ss + v;
        }
}

// The same for four tiles of a sparse box, a wavefront each: the few particles of a tile look their cells
// up one by one.  Tiles of more than SPARSE_MAX particles are left to the whole workgroup.
constexpr int SPARSE_MAX = 128;

__device__ __forceinline__ void bin_perm_sparse(const RankedArgs& A, int64_t blk, int32_t* lds) {
    const Geom& G = A.G;
    const int64_t T = 4 * blk + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (T < G.ntiles) {
        const int32_t ss = gl(A.start)[T * TILE_CELLS], se = gl(A.start)[(T + 1) * TILE_CELLS];
        gl(A.next_bins)[T * TILE_CELLS + lane] = gl(A.tot)[T] + gl(A.pre)[T * TILE_CELLS + lane];
        if (T == G.ntiles - 1 && lane == 0) gl(A.next_bins)[G.nbins] = gl(A.tot)[G.ntiles];
        const uint32_t row = (uint32_t)T / (uint32_t)G.nt[0], layer = row / (uint32_t)G.nt[1];
        const int ox = (int)((uint32_t)T - row * (uint32_t)G.nt[0]) * G.t[0],
                  oy = (int)(row - layer * (uint32_t)G.nt[1]) * G.t[1], oz = (int)layer * G.t[2];
        const int e0 = G.dest_ext(0), e1 = G.dest_ext(1);
        if (se - ss <= SPARSE_MAX)
            for (int32_t p = ss + lane; p < se; p += 64) {
                const int32_t w = gl(A.rank)[p];
                if (w < 0) {
                    gl(A.perm)[named_slot(A, w & 0x7FFFFFFF)] = p;
                    continue;
                }
                const int sl = w >> 20, z = sl / (e0 * e1), r = sl - z * e0 * e1, y = r / e0, x = r - y * e0;
                gl(A.perm)[bin_first(A, bin_of_cell(A, window_node(ox, x, G.n[0]), window_node(oy, y, G.n[1]),
                                                    window_node(oz, z, G.n[2]))) +
                           (w & 0xFFFFF)] = p;
            }
    }
    for (int k = 0; k < 4; ++k) {
        const int64_t H = 4 * blk + k;
        if (H >= G.ntiles || gl(A.start)[(H + 1) * TILE_CELLS] - gl(A.start)[H * TILE_CELLS] <= SPARSE_MAX) continue;
        __syncthreads();
        bin_perm_tile(A, H, lds);
    }
}

size_t sort_perm_lds(const pp_run* r) {
    return PERM_IMG * sizeof(uint16_t) + (size_t)r->g.dest_slots() * sizeof(DestCell);
}

// ---- exclusive scan of int32, in place ------------------------------------------------
constexpr int SCAN_BS = 256, SCAN_PER = 8, SCAN_CHUNK = SCAN_BS * SCAN_PER;
constexpr int64_t SCAN_ONE_MAX = 32768;  // longest scan that one workgroup does

__global__ void __launch_bounds__(SCAN_BS) k_scan_chunks(int32_t* data, int64_t n, int32_t* sums) {
    __shared__ int32_t sh[2][SCAN_BS];
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_PER;
    int32_t v[SCAN_PER];
    int32_t tot = 0;
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
        int64_t q = base + e;
        v[e] = q < n ? data[q] : 0;
        tot += v[e];
    }
    int cur = 0;
    sh[0][threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < SCAN_BS; off <<= 1) {
        int32_t x = sh[cur][threadIdx.x];
        if ((int)threadIdx.x >= off) x += sh[cur][threadIdx.x - off];
        sh[cur ^ 1][threadIdx.x] = x;
        cur ^= 1;
        __syncthreads();
    }
    int32_t incl = sh[cur][threadIdx.x];
    int32_t run = incl - tot;  // exclusive prefix of this thread
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
        int64_t q = base + e;
        if (q < n) data[q] = run;
        run += v[e];
    }
    if (threadIdx.x == SCAN_BS - 1) sums[blockIdx.x] = incl;
}

__global__ void __launch_bounds__(SCAN_BS) k_scan_add(int32_t* data, int64_t n, const int32_t* sums) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK;
    const int32_t add = sums[blockIdx.x];
    for (int e = threadIdx.x; e < SCAN_CHUNK; e += SCAN_BS) {
        int64_t q = base + e;
        if (q < n) data[q] += add;
    }
}

__global__ void __launch_bounds__(SCAN1_BS) k_scan_one(int32_t* data, int64_t n) {
    int32_t total, largest;
    scan_workgroup(data, n, 0, total, largest);
}

int64_t scan_tmp_size(int64_t n) {
    int64_t tot = 0;
    while (n > 1) {
        n = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
        tot += n + 1;
    }
    return tot + 16;
}

static void scan_inplace(int32_t* data, int64_t n, int32_t* tmp, hipStream_t st) {
    if (n <= SCAN_ONE_MAX) {  // one launch instead of three
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(SCAN1_BS), 0, st, data, n);
        return;
    }
    const int64_t nb = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    hipLaunchKernelGGL(k_scan_chunks, dim3((unsigned)nb), dim3(SCAN_BS), 0, st, data, n, tmp);
    if (nb > 1) {
        scan_inplace(tmp, nb, tmp + nb + 1, st);
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(SCAN_BS), 0, st, data, n, (const int32_t*)tmp);
    }
}


static unsigned grid_for(int64_t n, int bs, int64_t cap = 65535) {
    int64_t g = (n + bs - 1) / bs;
    if (g > cap) g = cap;
    return (unsigned)(g < 1 ? 1 : g);
}

static KeyGeom key_geom(const pp_run* r) {
    KeyGeom G;
    for (int d = 0; d < 3; ++d) {
        G.n[d] = r->g.n[d];
        G.t[d] = r->g.t[d];
        G.nt[d] = r->g.nt[d];
    }
    return G;
}

// ---- launches of the ranked sort: all species of a run, or of all runs of a batch ----------
enum SortPhase { SP_TABLES = 0, SP_SCAN = 1, SP_PERM = 2 };

enum SortForm { SF_SPLIT = 0, SF_FP64 = 1, SF_FP64_SPARSE = 2 };

template <int PHASE, int FORM>
__device__ __forceinline__ void sort_phase(const RankedArgs& A, int64_t blk, int32_t* lds) {
    if constexpr (PHASE == SP_TABLES) {
        const int64_t t = blk * 4 + (threadIdx.x >> 6);
        if constexpr (FORM == SF_SPLIT)
            round_table_tile(A, t);
        else
            bin_prefix_tile(A, t);
    } else if constexpr (PHASE == SP_SCAN) {
        ranked_scan(A);
    } else if constexpr (FORM == SF_SPLIT) {
        ranked_perm_tile(A, blk, lds);
    } else if constexpr (FORM == SF_FP64) {
        bin_perm_tile(A, blk, lds);
    } else {
        bin_perm_sparse(A, blk, lds);
    }
}

constexpr int sort_threads(int phase) { return phase == SP_SCAN ? SCAN1_BS : 256; }

struct SortArgs {
    RankedArgs sp[PP_MAX_SPECIES];
};

template <int PHASE, int FORM>
__global__ void __launch_bounds__(sort_threads(PHASE)) k_sort(SortArgs S) {
    extern __shared__ int32_t lds_sort[];
    sort_phase<PHASE, FORM>(S.sp[blockIdx.y], blockIdx.x, lds_sort);
}

template <bool SCAN>
__global__ void __launch_bounds__(SCAN1_BS) k_sort_chunks(SortArgs S, int32_t* tmp, int nchunks) {
    int32_t* sums = tmp + 2 * (int64_t)nchunks * blockIdx.y;
    if constexpr (SCAN)
        chunk_scan(S.sp[blockIdx.y], sums, nchunks);
    else
        chunk_sum(S.sp[blockIdx.y], sums, nchunks);
}

template <int PHASE>
__global__ void __launch_bounds__(sort_threads(PHASE)) k_sort_batch(const RankedArgs* __restrict__ T,
                                                                    const int64_t* __restrict__ prefix, int nseg) {
    extern __shared__ int32_t lds_sort[];
    const int64_t b = blockIdx.x;
    const int r = find_segment(prefix, nseg, b);
    if (r < 0) return;
    sort_phase<PHASE, SF_SPLIT>(T[r], b - prefix[r], lds_sort);
}

void sort_desc(const pp_run* r, int s, RankedArgs* A) {
    const Species& S = r->sp[s];
    const int64_t nt = r->g.ntiles;
    A->G = r->g;
    for (int d = 0; d < 3; ++d) {
        A->tsh[d] = 0;
        while ((1 << A->tsh[d]) < r->g.t[d]) ++A->tsh[d];
    }
    A->cnt = S.cell_cnt;
    A->rounds = S.rounds;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    A->tot = split ? S.offsets_next : S.tile_tot;
    A->rtot = r->sort_cursor + 3 * nt * s;  // 64 entries per tile, 3 used by each of 8 species
    A->ovf = A->rtot + nt;
    A->nchunk = A->rtot + 2 * nt;
    A->tile_max = r->tile_max + s;
    A->start = S.offsets;
    A->rank = S.rank;
    A->base = S.rank_base;
    A->perm = S.perm;
    A->n = S.n;
    A->cell = S.cur.cell;
    A->pre = S.bin_pre;
    A->next_bins = S.offsets_next;
}

size_t sort_desc_size() { return sizeof(RankedArgs); }

// Blocks each phase needs for one descriptor.
void sort_desc_blocks(const pp_run* r, int s, int64_t blocks[SORT_BATCH_PHASES]) {
    const int64_t nt = r->g.ntiles;
    blocks[SP_TABLES] = (nt + 3) / 4;
    blocks[SP_SCAN] = 1;
    blocks[SP_PERM] = r->sp[s].n > 0 ? nt : 0;
}

// prefixes: one array of nseg + 1 block prefixes (device) per phase, totals: blocks per phase
hipError_t launch_sort_batch(const void* table, const int64_t* const prefixes[SORT_BATCH_PHASES],
                             const int64_t totals[SORT_BATCH_PHASES], int nseg, size_t perm_lds, hipStream_t st) {
    if (nseg == 0) return hipSuccess;
    const RankedArgs* T = (const RankedArgs*)table;
    hipLaunchKernelGGL(k_sort_batch<SP_TABLES>, dim3((unsigned)totals[SP_TABLES]), dim3(sort_threads(SP_TABLES)), 0, st, T,
                       prefixes[SP_TABLES], nseg);
    hipLaunchKernelGGL(k_sort_batch<SP_SCAN>, dim3((unsigned)totals[SP_SCAN]), dim3(sort_threads(SP_SCAN)), 0, st, T,
                       prefixes[SP_SCAN], nseg);
    if (totals[SP_PERM] > 0)
        hipLaunchKernelGGL(k_sort_batch<SP_PERM>, dim3((unsigned)totals[SP_PERM]), dim3(sort_threads(SP_PERM)), perm_lds,
                           st, T, prefixes[SP_PERM], nseg);
    return hipGetLastError();
}

void swap_buffers(pp_particles& c) {
    int32_t* tc = c.cell;
    c.cell = c.cell_alt;
    c.cell_alt = tc;
    int64_t* ti = c.id;
    c.id = c.id_alt;
    c.id_alt = ti;
    for (int d = 0; d < 3; ++d) {
        void* tp = c.pos[d];
        c.pos[d] = c.pos_alt[d];
        c.pos_alt[d] = tp;
        void* tu = c.u[d];
        c.u[d] = c.u_alt[d];
        c.u_alt[d] = tu;
    }
}

// Host bookkeeping once a ranked sort is enqueued: the new tile starts become current and the
// particles stay where they are until the next particle kernel (or materialize) moves them.
void sort_enqueued(pp_run* r, int s) {
    Species& S = r->sp[s];
    int32_t* t = S.offsets;
    S.offsets = S.offsets_next;
    S.offsets_next = t;
    S.ranked = false;
    S.sorted = true;
    S.binned = r->p.precision == PP_PREC_FP64;
    S.pending = S.n > 0;
}

// out[q] = in[perm[q]] for every attribute (the move a pending permutation stands for)
template <typename T>
struct ApplyArgs {
    int64_t n;
    const int32_t* perm;
    const int32_t* cell;
    const T* pos[3];
    const T* u[3];
    const int64_t* id;
    int32_t* cell_o;
    T* pos_o[3];
    T* u_o[3];
    int64_t* id_o;
};

// Each thread moves APPLY_PER particles, their loads in flight together.  The old places of a
// tile's slots lie close together: neighbouring blocks run on one XCD, so that their lines are
// fetched into one L2.  6.7e7 tagged particles: 2.19 ms (2.53 with one a thread on any XCD).
constexpr int APPLY_PER = 4, APPLY_BLOCK = 256 * APPLY_PER;

template <typename T>
__global__ void __launch_bounds__(256) k_apply_perm(ApplyArgs<T> A) {
    const int64_t b = xcd_block(blockIdx.x, (A.n + APPLY_BLOCK - 1) / APPLY_BLOCK);
    if (b < 0) return;
    int64_t q[APPLY_PER];
    int32_t p[APPLY_PER];
    bool live[APPLY_PER];
#pragma unroll
    for (int k = 0; k < APPLY_PER; ++k) {
        q[k] = b * APPLY_BLOCK + k * 256 + threadIdx.x;
        p[k] = q[k] < A.n ? A.perm[q[k]] : -1;
    }
#pragma unroll
    for (int k = 0; k < APPLY_PER; ++k) {
        live[k] = p[k] >= 0;
        p[k] = live[k] ? p[k] : 0;
    }
    auto move = [&](const auto* in, auto* out) {
        std::remove_const_t<std::remove_reference_t<decltype(*in)>> v[APPLY_PER];
#pragma unroll
        for (int k = 0; k < APPLY_PER; ++k) v[k] = in[p[k]];
#pragma unroll
        for (int k = 0; k < APPLY_PER; ++k)
            if (live[k]) out[q[k]] = v[k];
    };
    if (A.cell) move(A.cell, A.cell_o);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        move(A.pos[d], A.pos_o[d]);
        move(A.u[d], A.u_o[d]);
    }
    if (A.id) move(A.id, A.id_o);
}

template <typename T>
static void apply_perm(pp_run* r, const Species& S) {
    ApplyArgs<T> A;
    A.n = S.n;
    A.perm = S.perm;
    A.cell = S.cur.cell;
    A.cell_o = S.cur.cell_alt;
    A.id = S.cur.id;
    A.id_o = S.cur.id ? S.cur.id_alt : nullptr;
    for (int d = 0; d < 3; ++d) {
        A.pos[d] = (const T*)S.cur.pos[d];
        A.u[d] = (const T*)S.cur.u[d];
        A.pos_o[d] = (T*)S.cur.pos_alt[d];
        A.u_o[d] = (T*)S.cur.u_alt[d];
    }
    hipLaunchKernelGGL(k_apply_perm<T>, dim3(xcd_grid((S.n + APPLY_BLOCK - 1) / APPLY_BLOCK)), dim3(256), 0, r->stream, A);
}

hipError_t materialize(pp_run* r, int s) {
    for (int k = 0; k < PP_MAX_SPECIES; ++k) {
        if (s >= 0 && k != s) continue;
        Species& S = r->sp[k];
        if (!S.active || !S.pending) continue;
        if (S.n > 0) {
            if (r->p.precision == PP_PREC_FP32_SPLIT)
                apply_perm<float>(r, S);
            else
                apply_perm<double>(r, S);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            swap_buffers(S.cur);
        }
        S.pending = false;
    }
    return hipSuccess;
}

template <int FORM>
static void launch_ranked(pp_run* r, const SortArgs& A, unsigned ns, bool any, size_t perm_lds) {
    constexpr int TABLES = FORM == SF_SPLIT ? SF_SPLIT : SF_FP64;
    const int64_t nt = r->g.ntiles;
    hipLaunchKernelGGL((k_sort<SP_TABLES, TABLES>), dim3((unsigned)((nt + 3) / 4), ns), dim3(sort_threads(SP_TABLES)), 0,
                       r->stream, A);
    if (nt <= SORT_SCAN_ONE) {
        hipLaunchKernelGGL((k_sort<SP_SCAN, TABLES>), dim3(1, ns), dim3(sort_threads(SP_SCAN)), 0, r->stream, A);
    } else {  // scan_tmp has room for a chunk sum and a maximum of eight species many times over
        const int nchunks = (int)((nt + SORT_CHUNK - 1) / SORT_CHUNK);
        const dim3 grid((unsigned)nchunks, ns);
        hipLaunchKernelGGL((k_sort_chunks<false>), grid, dim3(SCAN1_BS), 0, r->stream, A, r->scan_tmp, nchunks);
        hipLaunchKernelGGL((k_sort_chunks<true>), grid, dim3(SCAN1_BS), 0, r->stream, A, r->scan_tmp, nchunks);
    }
    if (any)
        hipLaunchKernelGGL((k_sort<SP_PERM, FORM>), dim3((unsigned)(FORM == SF_FP64_SPARSE ? (nt + 3) / 4 : nt), ns), dim3(sort_threads(SP_PERM)), perm_lds,
                           r->stream, A);
}

static bool capturing(hipStream_t st) {
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    return st && hipStreamIsCapturing(st, &c) == hipSuccess && c == hipStreamCaptureStatusActive;
}

// The ranked sort of the species in mask, together.
static hipError_t sort_ranked(pp_run* r, unsigned mask) {
    SortArgs A;
    unsigned ns = 0;
    bool any = false;
    int64_t np = 0;
    for (int s = 0; s < PP_MAX_SPECIES; ++s) {
        if (!(mask & (1u << s))) continue;
        sort_desc(r, s, &A.sp[ns++]);
        np += r->sp[s].n;
        any = any || r->sp[s].n > 0;
    }
    if (ns == 0) return hipSuccess;
    if (r->p.precision == PP_PREC_FP32_SPLIT) {
        launch_ranked<SF_SPLIT>(r, A, ns, any, sort_perm_lds(r));
    } else {
        const size_t lds = PERM_IMG * sizeof(uint16_t) + (size_t)r->g.dest_slots() * sizeof(int32_t);
        if (sparse_box(r->g.ntiles, np, (int)ns))
            launch_ranked<SF_FP64_SPARSE>(r, A, ns, any, lds);
        else
            launch_ranked<SF_FP64>(r, A, ns, any, lds);
    }
    hipError_t e = hipGetLastError();
    bool in_place = false;
    for (int s = 0; s < PP_MAX_SPECIES; ++s)
        if (mask & (1u << s)) {
            sort_enqueued(r, s);
            in_place = in_place || !r->sp[s].moved;
        }
    // Captured steps are replayed on the buffers they were captured with, so an even number of them
    // has to end as it began.  With every push writing the order pending before it, it does; where the
    // push before this sort found none (the first after pp_init_species or pp_get_particles), it does
    // if the order is applied at once, as in the buffers' first sort.
    if (e != hipSuccess || !in_place || !capturing(r->stream)) return e;
    for (int s = 0; s < PP_MAX_SPECIES && e == hipSuccess; ++s)
        if ((mask & (1u << s)) && !r->sp[s].moved) e = materialize(r, s);
    return e;
}

template <typename T>
static hipError_t sort_species(pp_run* r, int s) {
    Species& S = r->sp[s];
    const KeyGeom G = key_geom(r);
    const int64_t nbins = r->g.nbins;
    const int64_t ntiles = r->g.ntiles;
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    const int bs = 256;
    const int64_t nkeys = split ? ntiles : nbins;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(nkeys + 1, bs)), dim3(bs), 0, r->stream, S.offsets, nkeys + 1, 0);
    if (S.n > 0) {
        const unsigned pg = (unsigned)((S.n + bs - 1) / bs);
        if (split)
            hipLaunchKernelGGL(k_tile_count, dim3((unsigned)((S.n + AGG_BLOCK - 1) / AGG_BLOCK)), dim3(256), 0,
                               r->stream, G, (const int32_t*)S.cur.cell, S.n, S.offsets);
        else
            hipLaunchKernelGGL(k_hist_f64, dim3(pg), dim3(bs), 0, r->stream, G, (const double*)S.cur.pos[0],
                               (const double*)S.cur.pos[1], (const double*)S.cur.pos[2], S.n, S.offsets);
    }
    scan_inplace(S.offsets, nkeys + 1, r->scan_tmp, r->stream);
    if (split) {
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(1), 0, r->stream, r->tile_max + s, (int64_t)1, 0);
        hipLaunchKernelGGL(k_tile_max, dim3(grid_for(ntiles, bs, 1024)), dim3(bs), 0, r->stream,
                           (const int32_t*)S.offsets, ntiles, r->tile_max + s);
    }
    if (S.n > 0) {
        // FP64 form: an upper bound of the largest tile will do (the push looks for heavy tiles itself)
        hipLaunchKernelGGL(k_copy_i32, dim3(grid_for(nkeys, bs)), dim3(bs), 0, r->stream, r->sort_cursor,
                           (const int32_t*)S.offsets, nkeys, split ? nullptr : r->tile_max + s, (int32_t)S.n);
        ScatterArgs<T> A;
        A.G = G;
        A.n = S.n;
        A.cell = S.cur.cell;
        A.id = S.cur.id;
        A.cell_o = S.cur.cell_alt;
        A.id_o = S.cur.id ? S.cur.id_alt : nullptr;
        for (int d = 0; d < 3; ++d) {
            A.pos[d] = (const T*)S.cur.pos[d];
            A.u[d] = (const T*)S.cur.u[d];
            A.pos_o[d] = (T*)S.cur.pos_alt[d];
            A.u_o[d] = (T*)S.cur.u_alt[d];
        }
        A.cursor = r->sort_cursor;
        if (split)
            hipLaunchKernelGGL(k_scatter_tiles<T>, dim3((unsigned)((S.n + AGG_BLOCK - 1) / AGG_BLOCK)), dim3(256), 0,
                               r->stream, A);
        else
            hipLaunchKernelGGL(k_scatter<T>, dim3((unsigned)((S.n + bs - 1) / bs)), dim3(bs), 0, r->stream, A);
        swap_buffers(S.cur);
        if (split) {
            ReorderArgs<T> B;
            B.G = G;
            B.ntiles = ntiles;
            B.start = S.offsets;
            B.cell = S.cur.cell;
            B.id = S.cur.id;
            B.cell_o = S.cur.cell_alt;
            B.id_o = S.cur.id ? S.cur.id_alt : nullptr;
            for (int d = 0; d < 3; ++d) {
                B.pos[d] = (const T*)S.cur.pos[d];
                B.u[d] = (const T*)S.cur.u[d];
                B.pos_o[d] = (T*)S.cur.pos_alt[d];
                B.u_o[d] = (T*)S.cur.u_alt[d];
            }
            B.rank = S.rank;  // free here: no push since the last sort, no order pending
            B.perm = S.perm;
            hipLaunchKernelGGL(k_tile_reorder<T>, dim3((unsigned)ntiles), dim3(256), 0, r->stream, B);
            swap_buffers(S.cur);
        }
    }
    S.sorted = true;
    S.ranked = false;
    S.binned = !split;
    S.handed_out = false;
    return hipGetLastError();
}

hipError_t launch_sort(pp_run* r, int s) {
    const bool split = r->p.precision == PP_PREC_FP32_SPLIT;
    hipError_t e = materialize(r, s);  // a sort of a sort: apply the pending order first
    if (e != hipSuccess) return e;
    unsigned ranked = 0;
    for (int k = 0; k < PP_MAX_SPECIES; ++k) {
        if ((s >= 0 && k != s) || !r->sp[k].active) continue;
        if (r->sp[k].ranked) {
            ranked |= 1u << k;
            continue;
        }
        e = split ? sort_species<float>(r, k) : sort_species<double>(r, k);
        if (e != hipSuccess) return e;
    }
    return sort_ranked(r, ranked);
}

hipError_t drop_ranks(pp_run* r, int s) {
    Species& S = r->sp[s];
    if (!S.ranked) return hipSuccess;
    S.ranked = false;
    return launch_fill_i32(S.cell_cnt, 2 * r->g.nbins, 0, r->stream);
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace pp
