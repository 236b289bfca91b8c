// Host side of libtpkmc: the C ABI, argument checking, device scratch, the
// precision-independent kernels (clear, prefix sum, per-instance reduction)
// and the step pipeline, plain or captured as a HIP graph.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "tpkmc_internal.h"

#pragma clang fp contract(off)

using namespace tpkmc;

namespace {

constexpr int kScanItems = 8;                       // per thread
constexpr int kScanBlock = 256;
constexpr int kScanTile = kScanItems * kScanBlock;  // per work-group
constexpr int kPhases = 8;
// Default work-group order of the search: chunks of 16 work-groups dealt
// round-robin over the XCDs (StepArgs::order; see the autotuner).
constexpr int kDefaultSearchOrder = 16;

enum Phase { PH_CLEAR = 0, PH_KEY, PH_SCAN, PH_SCATTER, PH_SEARCH, PH_MOVE, PH_FINAL };

// ---------------------------------------------------------------- kernels
// What a step clears before it starts.
struct ClearArgs {
    int32_t* start;
    int64_t ncell;
    unsigned long long *macc, *mexp;  // exact o-bin sums and their exponents, or null
    int64_t nwords, nexp;
    unsigned long long* pair_count;
    uint32_t* ties;
    double* shift;             // velocity shifts to clear, or null
    int64_t nshift;
    uint32_t* status;          // status word to clear, or null
};

__device__ __forceinline__ void clear_all(const ClearArgs& c, int64_t t0, int64_t stride) {
    for (int64_t t = t0; t < c.ncell; t += stride) c.start[t] = 0;
    if (c.macc) {
        for (int64_t t = t0; t < c.nwords; t += stride) c.macc[t] = 0ull;
        for (int64_t t = t0; t < c.nexp; t += stride) c.mexp[t] = 0ull;
    }
    if (c.shift)
        for (int64_t t = t0; t < c.nshift; t += stride) c.shift[t] = 0.0;
    if (t0 == 0) {
        *c.pair_count = 0ull;
        *c.ties = 0u;
        if (c.status) *c.status = 0u;
    }
}

__global__ void __launch_bounds__(256) k_clear(ClearArgs c) {
    clear_all(c, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// The same for a step of one instance, which also writes its tables: the
// instance descriptor comes as a kernel argument and the block and chunk
// tables follow from it, so that no host staging or copy is needed.
template <typename real>
__global__ void __launch_bounds__(256) k_begin(Inst<real> one, Inst<real>* inst, Blk* blk, Chunk* chunks, ClearArgs c) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t0 == 0) *inst = one;
    for (int64_t t = t0; t < one.nblk; t += stride) blk[t] = Blk{0, (int32_t)(one.off + t * kBlock)};
    for (int64_t t = t0; t < one.nchunk; t += stride)
        chunks[t] = Chunk{(int32_t)(t * kChunk), (int32_t)min<int64_t>(kChunk, one.nblk - t * kChunk)};
    clear_all(c, t0, stride);
}

// Exclusive prefix sum of n int32 in place: per-tile totals, then per-tile
// scans that add the totals of the tiles before (read again by every tile, at
// most kScanTop of them; for more a single work-group scans the totals in
// between).  One tile takes the scan alone.  The launches are what a small
// state's scan costs: 10 us with all three, 3 us with one.
constexpr int64_t kScanTop = 2048;

__global__ void __launch_bounds__(kScanBlock) k_scan_reduce(const int32_t* d, int64_t n, int32_t* tile_sum) {
    __shared__ int32_t lds[kScanBlock / 64];
    const int64_t b0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (b0 + k < n) s += d[b0 + k];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int w = 0; w < kScanBlock / 64; ++w) t += lds[w];
        tile_sum[blockIdx.x] = t;
    }
}

// Exclusive scan across one work-group of `v`; returns the prefix, and the
// total in *total.
__device__ __forceinline__ int32_t block_exscan(int32_t v, int32_t* lds, int32_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(inc, o);
        if (lane >= o) inc += u;
    }
    __syncthreads();
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    int32_t woff = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        if (k < w) woff += lds[k];
        tot += lds[k];
    }
    *total = tot;
    return woff + inc - v;
}

__global__ void __launch_bounds__(1024) k_scan_top(int32_t* tile_sum, int64_t ntiles) {
    __shared__ int32_t lds[16];
    int32_t carry = 0;
    for (int64_t c0 = 0; c0 < ntiles; c0 += blockDim.x) {
        const int64_t t = c0 + threadIdx.x;
        const int32_t v = t < ntiles ? tile_sum[t] : 0;
        int32_t total;
        const int32_t ex = block_exscan(v, lds, &total);
        if (t < ntiles) tile_sum[t] = carry + ex;
        carry += total;
        __syncthreads();
    }
}

// tile_off: the tiles' offsets (scanned = true) or totals; null for one tile.
__global__ void __launch_bounds__(kScanBlock) k_scan_apply(int32_t* d, int64_t n, const int32_t* tile_off,
                                                           bool scanned) {
    __shared__ int32_t lds[kScanBlock / 64];
    const int64_t b0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems];
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = b0 + k < n ? d[b0 + k] : 0;
        s += v[k];
    }
    int32_t before = 0;
    if (tile_off) {
        if (scanned) {
            before = tile_off[blockIdx.x];
        } else {
            int32_t part = 0;
            for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanBlock) part += tile_off[t];
            block_exscan(part, lds, &before);
        }
    }
    int32_t total;
    int32_t run = before + block_exscan(s, lds, &total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (b0 + k < n) d[b0 + k] = run;
        run += v[k];
    }
}

// Neumaier (compensated) accumulation.
struct NSum {
    double s = 0.0, c = 0.0;
    __device__ void add(double v) {
        const double t = s + v;
        if (fabs(s) >= fabs(v)) c += (s - t) + v;
        else c += (v - t) + s;
        s = t;
    }
    __device__ double value() const { return s + c; }
};

// Per-instance reduction of the work-group partials, in a fixed order:
// first each chunk of <= kChunk work-groups, then each instance's chunks.
// Sixteen threads per slot (work-groups of 256 threads): thread t of slot k
// folds rows t, t + 16, t + 32, ... (Neumaier sums for the FP slots, max for
// max|v|^2, plain sums for the integer-valued counts), then a butterfly over
// the sixteen lanes combines their partials with a commutative step, so all
// sixteen end with the same total.
constexpr int kSlotLanes = 256 / kGPart;
// Instances of at most this many chunks are folded by the last launch alone
// (k_finalize), which saves one: 5 us against 9 for one chunk, but 27 against
// 13 for four.
constexpr int kDirectChunks = 1;
static_assert(kSlotLanes * kGPart == 256 && (kSlotLanes & (kSlotLanes - 1)) == 0, "slot lanes");

__device__ __forceinline__ void reduce_slots(const double* rows, int nrows, double* out) {
    const int k = threadIdx.x / kSlotLanes, t = threadIdx.x % kSlotLanes;
    double s = 0.0, c = 0.0;
    if (k == GP_VMAX2) {
        for (int r = t; r < nrows; r += kSlotLanes) s = fmax(s, rows[(int64_t)r * kGPart + k]);
        for (int o = 1; o < kSlotLanes; o <<= 1) s = fmax(s, __shfl_xor(s, o));
    } else if (k < GP_ALIVE) {
        NSum a;
        for (int r = t; r < nrows; r += kSlotLanes) a.add(rows[(int64_t)r * kGPart + k]);
        s = a.s;
        c = a.c;
        for (int o = 1; o < kSlotLanes; o <<= 1) {
            const double s2 = __shfl_xor(s, o), c2 = __shfl_xor(c, o);
            const double sum = s + s2;
            const double err = fabs(s) >= fabs(s2) ? (s - sum) + s2 : (s2 - sum) + s;
            c = (c + c2) + err;
            s = sum;
        }
    } else {
        for (int r = t; r < nrows; r += kSlotLanes) s += rows[(int64_t)r * kGPart + k];
        for (int o = 1; o < kSlotLanes; o <<= 1) s += __shfl_xor(s, o);
    }
    if (t == 0) out[k] = s + c;
}

__global__ void __launch_bounds__(256) k_reduce_chunks(const Chunk* chunks, const double* gpart, double* cpart) {
    __shared__ double rows[kChunk * kGPart];
    const Chunk c = chunks[blockIdx.x];
    for (int t = threadIdx.x; t < c.count * kGPart; t += blockDim.x)
        rows[t] = gpart[(int64_t)c.first * kGPart + t];
    __syncthreads();
    reduce_slots(rows, c.count, cpart + (int64_t)blockIdx.x * kGPart);
}

// Counters and globals of one instance, from its chunks' partials (cpart) or,
// with gpart given, from the work-groups' own, at most one chunk of them,
// folded as k_reduce_chunks does.
constexpr int kMomentRows = 256;  // o-bins per work-group of the moments
template <typename real>
__device__ void finalize_one(Inst<real>& I, int k0, const double* cpart, const double* gpart, uint64_t* counters,
                             double* globals, uint32_t* status, const unsigned long long* pair_count,
                             int64_t pair_cap, int advance_step, double* rows) {
    __shared__ double tot[kGPart];
    // Partials of this instance, staged in LDS kChunk rows at a time (folded
    // in order, so the result does not depend on the launch shape).
    double acc = 0.0;
    NSum ns;
    const int nrows = gpart ? I.nblk : I.nchunk;
    const double* src = gpart ? gpart + (int64_t)I.blk0 * kGPart : cpart + (int64_t)I.chunk0 * kGPart;
    for (int c0 = 0; c0 < nrows; c0 += kChunk) {
        const int nr = min(kChunk, nrows - c0);
        __syncthreads();
        for (int t = threadIdx.x; t < nr * kGPart; t += blockDim.x) rows[t] = src[(int64_t)c0 * kGPart + t];
        __syncthreads();
        reduce_slots(rows, nr, tot);  // (folding the one partial of a chunk again would leave it as it is)
        __syncthreads();
        if (threadIdx.x < kGPart) {
            const int k = threadIdx.x;
            if (k == GP_VMAX2) acc = fmax(acc, tot[k]);
            else if (k < GP_ALIVE) ns.add(tot[k]);
            else acc += tot[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < kGPart) tot[threadIdx.x] = threadIdx.x < GP_ALIVE && threadIdx.x != GP_VMAX2 ? ns.value() : acc;
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (counters) {
        uint64_t* c = counters + 8 * k0;
        c[TPKMC_CNT_ALIVE] = (uint64_t)tot[GP_ALIVE];
        c[TPKMC_CNT_PAIRS] = (uint64_t)tot[GP_PAIRS];
        c[TPKMC_CNT_TESTS] = (uint64_t)tot[GP_TESTS2] / 2u;
        c[TPKMC_CNT_CAND] = (uint64_t)tot[GP_CAND];
        c[TPKMC_CNT_FAST] = (uint64_t)tot[GP_FAST];
        c[TPKMC_CNT_NONFINITE] = (uint64_t)tot[GP_NONFINITE];
        c[TPKMC_CNT_ABSORBED] = (uint64_t)tot[GP_ABSORBED];
        c[TPKMC_CNT_HAVE_BEST] = (uint64_t)tot[GP_HAVEBEST];
    }
    if (globals) {
        double* g = globals + 8 * k0;
        g[0] = tot[GP_PX];
        g[1] = tot[GP_PY];
        g[2] = tot[GP_PZ];
        g[3] = tot[GP_EKIN];
        g[4] = tot[GP_VMAX2];
        g[5] = tot[GP_VIR];
        g[6] = tot[GP_MASS];
        g[7] = I.dt_d;
    }
    uint32_t st = 0;
    if (tot[GP_NONFINITE] > 0.0) st |= TPKMC_STATUS_NONFINITE;
    if (tot[GP_FAST] > 0.0) st |= TPKMC_STATUS_FAST;
    if (k0 == 0 && (int64_t)*pair_count > pair_cap) st |= TPKMC_STATUS_PAIR_OVERFLOW;
    if (st) atomicOr(status, st);
    if (advance_step) I.step_lo += 1u;
}

// Exact shifted o-bin sums -> the moments of the output: momentum and central
// second moments; the bin mean becomes the shift of the next step, so the
// sums stay small next time.  Each integer sum is rounded once to double (a
// function of the exact sum only) and scaled by its power-of-two quantum.
// Each work-group (256 threads) stages its 256 o-bins' output rows through
// LDS, so the stores are coalesced; every output value is written.
template <typename real>
__device__ void moments_final(const Inst<real>& I, int block, const ObAcc* macc, const char* mexp, int stride,
                              double* moments, double* shift, double* rows) {
    constexpr int kRows = kMomentRows;
    const int64_t nb = (int64_t)I.no[0] * I.no[1] * I.no[2];
    const int64_t b0 = (int64_t)block * kRows;
    if (b0 >= nb) return;  // whole work-group
    const int nloc = (int)min<int64_t>(kRows, nb - b0);
    if ((int)threadIdx.x < nloc) {
        const int64_t ob = I.obin_off + b0 + threadIdx.x;
        const ObAcc& A = macc[ob];
        const ObExp& X = *reinterpret_cast<const ObExp*>(mexp + ob * stride);
        double* M = rows + threadIdx.x * TPKMC_MOMENT_STRIDE;
        double* S = shift + ob * 3;
        const unsigned long long cnt = X.nc & 0xffffffffull, coll = X.nc >> 32;
        for (int k = 0; k < TPKMC_MOMENT_STRIDE; ++k) M[k] = 0.0;
        if (cnt > 0) {
            // Quanta 2^(E-50+h) of the four kinds (as in the moment pass); each
            // integer sum is rounded once to double, then scaled exactly.
            const int h = acc_headroom(cnt);
            double inv[4];
            for (int k = 0; k < 4; ++k) {
                const int e = X.e[k] > 0 ? X.e[k] - kExpBias : 0;
                inv[k] = ldexp(1.0, max(e, -969) - 50 + h);
            }
            double v[kAccVals];
            for (int k = 0; k < kAccVals; ++k) v[k] = (double)A.sum[k] * inv[acc_kind(k)];
            // Without per-particle masses the moment pass leaves the mass sum out.
            const double mass = (I.flags & kHasMass) ? v[9] : (double)cnt * I.mass_d;
            M[0] = (double)cnt;
            for (int ax = 0; ax < 3; ++ax) {
                const double s1 = v[ax], s2 = v[3 + ax];
                const double mean_off = s1 / mass;
                M[1 + ax] = s1 + mass * S[ax];
                M[4 + ax] = fmax(s2 - s1 * mean_off, 0.0);
                M[7 + ax] = v[6 + ax];
                S[ax] = S[ax] + mean_off;
            }
            M[10] = (double)coll;
            M[11] = mass;
        }
    }
    __syncthreads();
    double* M0 = moments + (I.obin_off + b0) * TPKMC_MOMENT_STRIDE;
    for (int t = threadIdx.x; t < nloc * TPKMC_MOMENT_STRIDE; t += kRows) M0[t] = rows[t];
}

// The step's last launch: work-group 0 of each instance (blockIdx.y) writes
// its counters and globals, the others its o-bins' moments.
template <typename real>
__global__ void __launch_bounds__(256) k_finalize(Inst<real>* inst, const double* cpart, const double* gpart,
                                                 uint64_t* counters, double* globals, uint32_t* status,
                                                 const unsigned long long* pair_count, int64_t pair_cap,
                                                 int advance_step, const ObAcc* macc, const char* mexp, int stride,
                                                 double* moments, double* shift) {
    __shared__ double rows[kChunk * kGPart];
    static_assert(kChunk * kGPart >= kMomentRows * TPKMC_MOMENT_STRIDE, "rows hold either");
    Inst<real>& I = inst[blockIdx.y];
    if (blockIdx.x == 0)
        finalize_one(I, (int)blockIdx.y, cpart, gpart, counters, globals, status, pair_count, pair_cap, advance_step,
                     rows);
    else
        moments_final(I, (int)blockIdx.x - 1, macc, mexp, stride, moments, shift, rows);
}

}  // namespace

// ---------------------------------------------------------------- handle
// Device scratch of one step: owned by a handle (tpkmc_create), or carved
// out of the static scratch array by the allocation-free entry point.
struct Buffers {
    int32_t *rank, *start, *tiles, *src, *best, *perm;
    void *rec, *rec2, *rmass, *inst;
    Blk* blk;
    Chunk* chunks;
    unsigned long long* bkey;
    double *gpart, *cpart, *shift;
    ObAcc* macc;      // exact o-bin sums, 128 B per o-bin
    char* mexp;       // their exponents and counts; null: within the sums
    void* vir;        // colliders' virial terms, 3 reals per particle
    uint8_t* coll;    // collided flags, 1 B per particle
    unsigned long long* pair_count;
    uint32_t* ties;
    uint32_t* status;
    unsigned long long* mix;  // counters of tpkmc_search_mix (handles only)
};

struct ProfRec {
    int phase;
    hipEvent_t a, b;
};

struct tpkmc_handle {
    int device = 0, precision = TPKMC_FP64;
    int64_t max_n = 0, max_cells = 0, max_obins = 0, max_blk = 0;
    int32_t max_inst = 0;
    int64_t max_chunks = 0;
    Buffers b{};  // device scratch, allocated once in tpkmc_create
    hipStream_t last_stream = nullptr;
    hipStream_t own_stream = nullptr;
    int search_block = kWave;
    int search_group = 2;
    int search_order = kDefaultSearchOrder;  // work-group order of the search (StepArgs::order)
    bool shape_chosen = false;  // set by tpkmc_set_search or tpkmc_autotune
    // c-bins chosen by tpkmc_autotune per batch position, each applied while
    // the instance at that position keeps the grid and parameters it was
    // tuned on (the key); capacity of the c-bin counts array.
    struct Cells {
        tpkmc_grid g;
        double sigma, dt;
        uint32_t flags;
        int32_t n[3];   // c-bins of the slow particles (the configured ones: no split)
        double vc;      // speed bound of the slow particles
    };
    std::vector<Cells> cells;
    int64_t cell_cap = 0;
    bool profiling = false;
    std::vector<ProfRec> prof;
    std::vector<hipEvent_t> pool;
    size_t pool_used = 0;
    double prof_ms[kPhases] = {};
    int64_t prof_n[kPhases] = {};
    hipGraphExec_t gexec = nullptr;
    // Pinned staging ring for the instance and block tables: a slot is
    // rewritten only after the copy that last read it has run.
    static constexpr int kRing = 8;
    char* stage[kRing] = {};
    hipEvent_t stage_ev[kRing] = {};
    bool stage_used[kRing] = {};
    size_t stage_bytes = 0;
    int stage_next = 0;
};

namespace {

// Host view of one validated call.
// Target size of one band plane of records (see row_of).
constexpr double kBandBytes = 1 << 20;

int64_t scan_tiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

// Sort cells that a handle's scratch holds for `cbins` c-bins and n
// particles: sub-grids keep kSortCellMin particles a cell.
int64_t sort_cells(int64_t cbins, int64_t n) { return cbins + n / 8; }

struct Plan {
    int n_inst = 0;
    int64_t ncell_tot = 0, nob_tot = 0, max_nob = 0;
    int nblk = 0;
    bool adaptive = false;    // some instance takes the adaptive time step
    bool any_search = false;  // some instance takes partners by closest approach
    bool split = false;       // some instance has c-bins split by speed
    bool subgrid = false;     // some instance's c-bins are cut into sort cells
    bool any_staged = false, any_tiles = false;  // which searches the instances take
    bool caller_order = false;  // some instance keeps the caller's order
    bool any_random = false;  // some instance takes random partners
    int nchunk = 0, max_chunks = 0;
    std::vector<Blk> blk;      // empty for one instance (see make_plan)
    std::vector<Chunk> chunks;
    std::vector<char> inst_bytes;
};

bool bad_ptr(const void* p) { return p == nullptr; }

bool bad_state(const tpkmc_particles* s) {
    return s->n > 0 && (bad_ptr(s->x) || bad_ptr(s->y) || bad_ptr(s->z) || bad_ptr(s->vx) || bad_ptr(s->vy) ||
                        bad_ptr(s->vz) || bad_ptr(s->id));
}

// Tile search or lane walk (FP32: staged, FP64: a record a lane).  Instances that
// can be cut into sort cells (`cut`) take tiles, unless two periodic axes are
// thinner than a pair's reach (a tube of 1e6 as thin as a c-bin is long at 30 per
// c-bin, FP32: 141 us staged, 292 in tiles), and FP32 below kTileDensity particles
// per c-bin is staged (4M tube at 2.9: 0.42 ms staged, 0.58 in tiles).  The rest
// goes by the cost of both in microseconds per 1e6 records, as fitted to the
// search of 2.1e3 uniform states (3e4 to 1e6 particles at 0.3 to 100 per c-bin;
// boxes, planes, tubes of 1 to 4 c-bins across along x and y, slabs of 1 to 8
// c-bins along x; D of 0.1 to 2 widths).
//  - A tile is up to 64 records of one row of c-bins, so a wave's records make
//    1 + 63 / (records of a row) tiles, each with a set-up and blocks of 64
//    partners from its rows, 64 records and two c-bins long.  Along a periodic
//    axis of up to three c-bins it visits the images one by one, those out of
//    reach (D and a c-bin's move) of its cells left out.
//  - A lane tests its half neighbourhood pair by pair; the staged walk also
//    goes tile by tile through the rows.
// A small call takes what one wave needs: the tiles and the FP64 lanes are split
// over waves then (these by rows: a tube of 2261 at 133 per c-bin is one row, 146
// us against 21 in tiles), the staged walk is not.  A batch is settled as a whole, see
// Routes.  Shocks gather the particles: a record has kClump times the mean number
// of neighbours here.  (With one, a uniform gas of one c-bin along a periodic z at
// 10 to 24 per c-bin would be staged, 95 to 150 us instead of 180 to 220, and an
// ensemble with Noh implosions of such densities took 70 ms a pass instead of 48.)
// Measured, lanes against tiles: FP64 boxes at 0.3, 1 and 3 per c-bin 92, 138
// and 248 against 529, 241 and 231 us, tube along y at 3 and 20 56 and 157 against
// 1033 and 260; FP32 tube as thin as a c-bin is long at 16 per c-bin 60 against
// 300 us, box at 9, 14 and 20 per c-bin 201, 271 and 354 against 171, 194 and 209,
// 3e5 in a tube of 3 by 3 c-bins at 100 per c-bin 974 against 292 (FP64 1411
// against 377).
constexpr double kTileDensity = 8.0;
constexpr double kClump = 3.0;

// Of an instance's search by tiles and by lanes: microseconds per 1e6 records,
// and of the wave that takes longest.
struct SearchCost {
    double tile, tile_wave, lane, lane_wave;
    bool open, tiles;  // both are open to it; tiles are the cheaper for a state of its kind
};

template <typename real>
SearchCost search_cost(const Inst<real>& d, const tpkmc_grid& g, double n, double dens, double D, bool planar,
                       const double* cell, bool cut) {
    constexpr bool fp64 = std::is_same<real, double>::value;
    SearchCost c{};
    if (!fp64 && dens < kTileDensity) return c;
    double w = 0.0, rows = 1.0, visits = 1.0;  // narrowest c-bin; rows of a neighbourhood; with images
    for (int a = 0; a < (planar ? 2 : 3); ++a) {
        const double wa = (g.hi[a] - g.lo[a]) / d.nl[a];
        w = w > 0.0 ? std::min(w, wa) : wa;
    }
    int thin = 0;
    for (int a = 0; a < 3; ++a) {
        const double wa = (g.hi[a] - g.lo[a]) / d.nl[a];
        if (a > 0) rows *= std::min(3, d.nl[a]);
        if (g.bc[a] != TPKMC_BC_PERIODIC || d.nl[a] > 3 || (planar && a == 2)) continue;
        // Its c-bins and their images, but for those out of a tile's reach.
        const double v = std::min(3.0 * d.nl[a], 1.5 + (2.0 * (D + w) + cell[a]) / wa);
        if (v >= 2.4 * d.nl[a]) ++thin;
        visits *= v / d.nl[a];
    }
    visits *= rows;
    const double row = std::max(dens * d.nl[0], 1e-3), groups = std::min(64.0, 1.0 + 63.0 / row);
    const double clump = thin < 2 ? kClump : 1.0;  // nine images: the tiles gain nothing from a crowd
    const double span = 64.0 + 2.0 * clump * dens, near = clump * std::min(row, 3.0 * dens);
    const double blocks = 0.5 + 0.5 * visits * std::min(row < 3.0 * dens ? clump * row : row, span) / 64.0;
    const double tests = 0.5 * rows * near, m = n * 1e-6;
    c.tile = fp64 ? 88.0 + groups * (14.0 + 24.0 * blocks) : 63.0 + groups * (18.0 + 16.0 * blocks);
    c.lane = fp64 ? 38.0 + 5.8 * rows + 3.7 * tests : 21.0 + 6.7 * groups * rows + 1.1 * tests;
    c.tile_wave = 18.0 + 8.0 * groups + 0.06 * c.tile;
    c.lane_wave = fp64 ? std::max(8.0 + 0.07 * c.lane, 12.0 + 0.5 * near) : 0.5 * c.lane;
    c.open = !(cut && thin < 2);
    c.tiles = !c.open || !(std::max(m * c.lane, c.lane_wave) < std::max(m * c.tile, c.tile_wave));
    return c;
}

// The instances of a batch that would do better by lanes share one launch of
// them, after that of the tiles; where they are few it takes as long as one of
// its waves.  So those whose lanes cost more than `cap` go to the tiles, with
// the cap (a power of two) that makes both launches together the shortest, if
// their lanes take less than kBatchGain of what they add to the tiles (the costs
// are rough).  Three steps of an ensemble of nine whose one dense thin tube (76479
// particles at 4025 per c-bin) took the lanes alone: 9.57 ms, by tiles 8.9; of 64
// with nine such tubes, 15.4 ms a step, 16.2 by tiles.  At 0.75 these go to the
// tiles, at 0.88 an ensemble of 14 takes 11.4 ms instead of 8.7.  A million in equal
// tubes of 30 to 4000 per c-bin that particles cross in one to three steps: 0.02
// to 4 ms by lanes, 0.24 to 60 by tiles.
constexpr double kBatchGain = 0.8;
struct Routes {
    static constexpr int kBins = 24;
    struct Sum {
        double all = 0.0, wave = 0.0;
        void add(const Sum& o) { all += o.all; wave = std::max(wave, o.wave); }
        double us() const { return std::max(all, wave); }
    };
    Sum tiles, lane[kBins], tile[kBins];  // to the tiles in any case; by lanes, by log2 of their cost
    bool any = false;
    void add(const SearchCost& c, int64_t count, int64_t n_all) {
        if (!c.open && !c.tiles) return;
        const double m = (double)count * 1e-6;
        // Tiles of a large call are not split over waves.
        const Sum t{m * c.tile, std::max(c.tile_wave, c.tile * std::min(0.3, 1.1e-6 * (double)n_all))};
        if (c.tiles) return tiles.add(t);
        const int b = std::min(std::max(std::ilogb(c.lane), 0), kBins - 1);
        tile[b].add(t);
        lane[b].add({m * c.lane, 0.6 * c.lane_wave});
        any = true;
    }
    // Both launches, the bins below b by lanes.
    double us(int b) const {
        Sum t = tiles, l;
        for (int k = 0; k < kBins; ++k) k < b ? l.add(lane[k]) : t.add(tile[k]);
        return t.us() + l.us();
    }
    double cap() const {
        const double rest = tiles.us();
        double best = rest + kBatchGain * (us(0) - rest), at = 1.0;
        for (int b = kBins; b > 0; --b) {
            if (us(b) < best) {
                best = us(b);
                at = b == kBins ? HUGE_VAL : std::ldexp(1.0, b);
            }
        }
        return at;
    }
};

// Sub-grids: c-bins of at least kSubgridDensity particles are halved along
// their widest axis, again and again, while a part keeps kSortCellMin
// particles and its width 0.7 D.  A tile then is compact, and the parts of
// the neighbourhood out of its reach are skipped: the FP64 Sod tube of 4e5
// particles on 100 c-bins 7.9 ms whole, 0.12 in sort cells.  Sparser c-bins
// leave nothing to skip (a tile holds several of them).
constexpr double kSubgridDensity = 24.0;
constexpr double kSortCellMin = 8.0;  // sort_cells() counts on it
constexpr double kSortCellD = 0.7;

template <typename real>
void choose_sort_cells(Inst<real>& d, const tpkmc_grid& g, int64_t count, int64_t n_all, int64_t Cs, double D,
                       bool planar, bool subgrid, uint32_t flags, Routes* routes, double cap) {
    const int naxes = planar ? 2 : 3;
    const double dens = (double)count / (double)Cs;
    // Scale of the tile search's positions: the widest c-bin (half the box on
    // an axis of one; a planar gas has no extent along z).
    double wide = 0.0, w[3];
    for (int a = 0; a < 3; ++a) {
        w[a] = (g.hi[a] - g.lo[a]) / d.nl[a];
        if (a < naxes) wide = std::max(wide, d.nl[a] > 1 ? w[a] : 0.5 * w[a]);
    }
    d.tile_s = (float)(1.0 / wide);
    bool cut = false;
    int32_t kl[3] = {};
    for (double part = dens; dens >= kSubgridDensity && part >= 2.0 * kSortCellMin; part *= 0.5) {
        int a = -1;  // the widest axis that can be halved
        for (int b = 0; b < naxes; ++b)
            if (0.5 * w[b] >= kSortCellD * D && ((int64_t)d.nl[b] << kl[b]) * 2 <= 1 << 24 && (a < 0 || w[b] > w[a]))
                a = b;
        if (a < 0) break;
        kl[a] += 1;
        w[a] *= 0.5;
        cut = true;
    }
    if (!(flags & TPKMC_PAIR_RANDOM)) {
        const SearchCost c = search_cost(d, g, (double)n_all, dens, D, planar, w, cut);
        if (c.tiles || (c.open && c.lane >= cap)) d.flags |= kTiles;
        if (routes) routes->add(c, count, n_all);
    }
    if (subgrid && cut && (d.flags & kTiles)) {
        d.flags |= kSubgrid;
        for (int a = 0; a < 3; ++a) {
            d.kl[a] = kl[a];
            d.n[a] = d.nl[a] << kl[a];
            d.inv_w[a] = (real)((double)d.n[a] / (g.hi[a] - g.lo[a]));
        }
    }
    // Partners of a tile in their places lie at most two c-bins beyond its
    // cells, or two boxes where a periodic axis is visited image by image.
    double x = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double L = g.hi[a] - g.lo[a];
        d.w_sort[a] = (real)(L / d.n[a]);
        if (a >= naxes) continue;
        const bool few = g.bc[a] == TPKMC_BC_PERIODIC && d.nl[a] <= 3;
        x = std::max(x, (few ? 2.0 * L : 0.5 * L / d.n[a] + 2.0 * L / d.nl[a]) / wide);
    }
    d.tile_x = (float)(1.01 * x + 0.01);
    d.tile_dx = (float)(0.505 * ((g.hi[0] - g.lo[0]) / d.n[0]) / wide);
}

// Validates one instance and fills its device descriptor, except the
// offsets into the c-bin, o-bin, block and chunk tables, which the caller
// sets.  C and B: its c-bins and o-bins (d.C: its sort cells).  nref (split
// c-bins): the slow particles' c-bins per axis, vc their speed bound.
// subgrid: the c-bins may be cut into sort cells.  routes, cap: see Routes.
template <typename real>
int fill_inst(const tpkmc_particles* s, const tpkmc_instance& q, Inst<real>& d, int64_t& C, int64_t& B,
              const int32_t* nref = nullptr, double vc = 0.0, bool subgrid = true, Routes* routes = nullptr,
              double cap = HUGE_VAL) {
    const tpkmc_grid& g = q.grid;
    const tpkmc_params& p = q.params;
    if (q.offset < 0 || q.count < 0 || q.offset + q.count > s->n) return TPKMC_EINVAL;
    if (!(std::isfinite(p.sigma) && p.sigma >= 0.0)) return TPKMC_EINVAL;
    if (!(std::isfinite(p.mass) && p.mass > 0.0)) return TPKMC_EINVAL;
    if (!(std::isfinite(p.dt) && p.dt > 0.0)) return TPKMC_EINVAL;
    if (p.instance >= (1u << 24)) return TPKMC_EINVAL;
    if (p.flags & ~(uint32_t)(TPKMC_EMIT_PAIRS | TPKMC_ALLOW_REORDER | TPKMC_ADAPTIVE_DT | TPKMC_PLANAR |
                              TPKMC_RANK_TIME | TPKMC_PAIR_RANDOM))
        return TPKMC_EINVAL;
    if ((p.flags & TPKMC_RANK_TIME) && (p.flags & TPKMC_PAIR_RANDOM)) return TPKMC_EINVAL;
    const bool planar = (p.flags & TPKMC_PLANAR) != 0;
    if (planar && g.ncell[2] != 1) return TPKMC_EINVAL;
    std::memset(&d, 0, sizeof(d));
    C = 1;
    B = 1;
    int64_t Cc = 1;
    double dx = 0.0, wd[3];
    for (int a = 0; a < 3; ++a) {
        if (g.ncell[a] < 1 || g.nobin[a] < 1) return TPKMC_EINVAL;
        if (g.ncell[a] > (1 << 24) || g.nobin[a] > (1 << 24)) return TPKMC_EINVAL;
        if (!(std::isfinite(g.lo[a]) && std::isfinite(g.hi[a]) && g.hi[a] > g.lo[a])) return TPKMC_EINVAL;
        if (g.bc[a] < TPKMC_BC_REFLECT || g.bc[a] > TPKMC_BC_ABSORB) return TPKMC_EINVAL;
        if (g.bc[a] == TPKMC_BC_ABSORB && s->alive == nullptr) return TPKMC_EINVAL;
        if (nref && (nref[a] < g.ncell[a] || nref[a] > (1 << 24))) return TPKMC_EINVAL;
        C *= nref ? nref[a] : g.ncell[a];
        Cc *= g.ncell[a];
        B *= g.nobin[a];
        // Derived grid quantities, in double, in the order of the reference.
        // With split c-bins the slow particles are binned on nc c-bins; the
        // fast ones, the time step and the fast-particle check keep the
        // configured ones.
        const double L = g.hi[a] - g.lo[a];
        const int32_t nc = nref ? nref[a] : g.ncell[a];
        d.n[a] = d.nl[a] = nc;
        d.ncfg[a] = g.ncell[a];
        d.inv_wc[a] = (real)((double)g.ncell[a] / L);
        d.no[a] = g.nobin[a];
        d.bc[a] = g.bc[a];
        d.lo[a] = (real)g.lo[a];
        d.hi[a] = (real)g.hi[a];
        d.L[a] = (real)L;
        d.w[a] = (real)(L / (double)g.ncell[a]);
        wd[a] = L / (double)g.ncell[a];
        if (g.ncell[a] > 1 && (dx == 0.0 || L / (double)g.ncell[a] < dx)) dx = L / (double)g.ncell[a];
        d.inv_w[a] = d.inv_wl[a] = (real)((double)nc / L);
        d.inv_wo[a] = (real)((double)g.nobin[a] / L);
    }
    const bool split = nref && (nref[0] != g.ncell[0] || nref[1] != g.ncell[1] || nref[2] != g.ncell[2]);
    const int64_t Cs = C;  // the c-bins that are searched
    if (split) C = Cs + Cc;
    if (C + 1 > (int64_t)1 << 30 || B > (int64_t)1 << 30) return TPKMC_EINVAL;
    const double Dp = 0.5 * p.sigma;
    const double D = planar ? Dp : std::sqrt(p.sigma / M_PI);
    choose_sort_cells(d, g, q.count, s->n, Cs, D, planar, subgrid, p.flags, routes, cap);
    const int64_t Cf = (int64_t)d.n[0] * d.n[1] * d.n[2];
    const int64_t Csort = split ? Cf + Cc : Cf;
    d.off = q.offset;
    d.cnt = q.count;
    d.C = (int32_t)Csort;
    d.Cf = (int32_t)Cf;
    d.seed_lo = (uint32_t)p.seed;
    d.seed_hi = (uint32_t)(p.seed >> 32);
    d.step_lo = (uint32_t)p.step;
    d.instance = p.instance;
    d.flags |= p.flags | (s->mass ? kHasMass : 0u);
    if (split) {
        d.flags |= kSplit;
        d.vc2 = (real)(vc * vc);
    }
    d.dt = (real)p.dt;
    // Largest accepted d_min^2: sigma = pi D^2 in space, sigma = 2 D in
    // the plane (same expressions as the reference).
    d.D2 = planar ? (real)(Dp * Dp) : (real)(p.sigma / M_PI);
    d.mass = (real)p.mass;
    d.mass_d = p.mass;
    d.dt_d = p.dt;
    d.dt_cap = p.dt;
    d.dx_d = dx;
    // Random partners: the cross section and the c-bin volume (an area
    // in the plane), in the reference's order.
    d.sigma_d = p.sigma;
    d.cellvol_d = planar ? wd[0] * wd[1] : (wd[0] * wd[1]) * wd[2];
    // Band height of the c-bin order: the largest power of two of rows
    // whose band plane (rows x n_x c-bins of records) stays within
    // kBandBytes, so that one XCD's L2 holds the plane its neighbourhood
    // walk reads twice.  Planar and one-row grids keep a single band.
    d.band_log2 = 30;
    if (d.n[2] > 1 && d.n[1] > 1 && q.count > 0) {
        const double row_bytes = (double)d.n[0] * ((double)q.count / (double)Cf) * 8.0 * sizeof(real);
        int h = 0;
        while (h < 30 && (double)(2 << h) * row_bytes <= (double)kBandBytes) ++h;
        if ((1 << h) < d.n[1]) d.band_log2 = h;
    }
    return TPKMC_OK;
}

// Flags that decide the choice of c-bins (with the grid, sigma and dt).
constexpr uint32_t kCellKey = TPKMC_ADAPTIVE_DT | TPKMC_PLANAR | TPKMC_RANK_TIME | TPKMC_PAIR_RANDOM;

// The c-bins autotune chose for batch position k, if the instance there
// keeps the grid and parameters it was tuned on.
const tpkmc_handle::Cells* tuned_cells(const tpkmc_handle* h, int k, const tpkmc_instance& q) {
    if (k >= (int)h->cells.size()) return nullptr;
    const tpkmc_handle::Cells& c = h->cells[k];
    if (std::memcmp(&c.g, &q.grid, sizeof(tpkmc_grid)) != 0 || c.sigma != q.params.sigma ||
        c.dt != q.params.dt || c.flags != (q.params.flags & kCellKey))
        return nullptr;
    return &c;
}

template <typename real>
int make_plan(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, Plan& P,
              bool configured = false, bool tables = true, double cap = HUGE_VAL) {
    if (!s || !in || n_inst < 1) return TPKMC_EINVAL;
    if (n_inst > h->max_inst) return TPKMC_ECAPACITY;
    if (s->n < 0) return TPKMC_EINVAL;
    if (s->n > h->max_n) return TPKMC_ECAPACITY;
    if (bad_state(s)) return TPKMC_EINVAL;
    std::vector<std::pair<int64_t, int64_t>> spans;
    P.inst_bytes.resize(sizeof(Inst<real>) * n_inst);
    Inst<real>* const I = reinterpret_cast<Inst<real>*>(P.inst_bytes.data());
    P.blk.clear();
    P.chunks.clear();
    P.n_inst = n_inst;
    P.adaptive = false;
    P.any_search = false;
    P.split = P.subgrid = P.any_staged = P.any_tiles = P.caller_order = false;
    P.any_random = false;
    P.ncell_tot = 0;
    P.nob_tot = 0;
    P.max_nob = 0;
    P.nblk = P.nchunk = P.max_chunks = 0;
    int64_t before = 0, cbins = 0;  // particles of the instances before; c-bins
    Routes routes;
    const bool settle = n_inst > 1 && cap == HUGE_VAL;
    for (int k = 0; k < n_inst; ++k) {
        const tpkmc_instance& q = in[k];
        Inst<real>& d = I[k];
        int64_t C, B;
        const tpkmc_handle::Cells* tc = configured ? nullptr : tuned_cells(h, k, q);
        const int rc = fill_inst<real>(s, q, d, C, B, tc ? tc->n : nullptr, tc ? tc->vc : 0.0, true,
                                       settle ? &routes : nullptr, cap);
        if (rc) return rc;
        if (d.flags & kSplit) P.split = true;
        if (d.flags & kSubgrid) P.subgrid = true;
        if (!(d.flags & (kTiles | TPKMC_PAIR_RANDOM))) P.any_staged = true;
        if (d.flags & kTiles) P.any_tiles = true;
        if (!(q.params.flags & TPKMC_ALLOW_REORDER)) P.caller_order = true;
        spans.push_back({q.offset, q.count});
        if (q.params.flags & TPKMC_PAIR_RANDOM) P.any_random = true;
        else P.any_search = true;
        if (q.params.flags & TPKMC_ADAPTIVE_DT) P.adaptive = true;
        d.cell_off = P.ncell_tot;
        d.obin_off = P.nob_tot;
        d.base = q.offset - before;
        before += q.count;
        P.ncell_tot += (int64_t)d.C + 1;
        cbins += C + 1;
        P.nob_tot += B;
        P.max_nob = std::max(P.max_nob, B);
        d.blk0 = (int32_t)P.nblk;
        d.nblk = (int32_t)((q.count + kBlock - 1) / kBlock);
        d.chunk0 = P.nchunk;
        d.nchunk = (d.nblk + kChunk - 1) / kChunk;
        P.nblk += d.nblk;
        P.nchunk += d.nchunk;
        P.max_chunks = std::max(P.max_chunks, d.nchunk);
        if (!tables) continue;
        for (int64_t o = 0; o < q.count; o += kBlock) P.blk.push_back({k, (int32_t)(q.offset + o)});
        for (int32_t b = 0; b < d.nblk; b += kChunk)
            P.chunks.push_back({d.blk0 + b, std::min<int32_t>(kChunk, d.nblk - b)});
    }
    if (routes.any && (cap = routes.cap()) < HUGE_VAL)
        return make_plan<real>(h, s, in, n_inst, P, configured, tables, cap);
    std::sort(spans.begin(), spans.end());
    for (size_t k = 1; k < spans.size(); ++k)
        if (spans[k - 1].first + spans[k - 1].second > spans[k].first) return TPKMC_EINVAL;
    if (cbins > h->cell_cap) return TPKMC_ECAPACITY;
    if (P.nob_tot > h->max_obins) return TPKMC_ECAPACITY;
    if (P.nblk > h->max_blk) return TPKMC_ECAPACITY;
    if (P.nchunk > h->max_chunks) return TPKMC_ECAPACITY;
    return TPKMC_OK;
}

int check_outputs(const tpkmc_outputs* o) {
    if (!o) return TPKMC_OK;
    if (o->pairs && o->pair_cap < 0) return TPKMC_EINVAL;
    return TPKMC_OK;
}

hipEvent_t pool_event(tpkmc_handle* h) {
    if (h->pool_used == h->pool.size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        h->pool.push_back(e);
    }
    return h->pool[h->pool_used++];
}

struct PhaseScope {
    tpkmc_handle* h;
    int phase;
    hipStream_t s;
    hipEvent_t b = nullptr;
    PhaseScope(tpkmc_handle* h_, int ph, hipStream_t s_, bool on) : h(h_), phase(ph), s(s_) {
        if (!on) { h = nullptr; return; }
        hipEvent_t a = pool_event(h);
        b = pool_event(h);
        if (!a || !b) { h = nullptr; return; }
        hipEventRecord(a, s);
        h->prof.push_back({phase, a, b});
    }
    ~PhaseScope() {
        if (h) hipEventRecord(b, s);
    }
};

template <typename real>
StepArgs<real> make_args(const Buffers& B, const tpkmc_particles* s, const tpkmc_outputs* o, int nblk, int64_t nob) {
    StepArgs<real> a{};
    a.x = (real*)s->x; a.y = (real*)s->y; a.z = (real*)s->z;
    a.vx = (real*)s->vx; a.vy = (real*)s->vy; a.vz = (real*)s->vz;
    a.id = s->id;
    a.alive = s->alive;
    a.inst = (const Inst<real>*)B.inst;
    a.blk = B.blk;
    a.nblk = nblk;
    a.rank = B.rank;
    a.start = B.start;
    a.rec = (real*)B.rec;
    a.rec2 = (real*)B.rec2;
    a.mass = (real*)s->mass;
    a.rmass = (real*)B.rmass;
    a.src = B.src;
    a.best = B.best;
    a.perm = B.perm;
    a.bkey = B.bkey;
    a.gpart = B.gpart;
    a.shift = B.shift;
    a.macc = (o && o->moments) ? B.macc : nullptr;
    a.mexp = B.mexp ? B.mexp : (char*)&B.macc->shared;
    a.exp_stride = B.mexp ? exp_stride(nob) : (int)sizeof(ObAcc);
    a.vir = (real*)B.vir;
    a.coll = B.coll;
    a.pairs = o ? o->pairs : nullptr;
    a.pair_cap = (o && o->pairs) ? o->pair_cap : 0;
    a.pair_count = B.pair_count;
    a.ties = B.ties;
    a.mix = B.mix;
    a.moments = o ? o->moments : nullptr;
    return a;
}


void enqueue_scan(const Buffers& B, int64_t n, hipStream_t s) {
    const int64_t tiles = scan_tiles(n);
    const bool top = tiles > kScanTop;
    if (tiles > 1) hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)tiles), dim3(kScanBlock), 0, s, B.start, n, B.tiles);
    if (top) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, B.tiles, tiles);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)tiles), dim3(kScanBlock), 0, s, B.start, n,
                       tiles > 1 ? B.tiles : nullptr, top);
}

// Shape of one launch sequence: what enqueue_step needs of a Plan.
struct Shape {
    int n_inst, nblk, nchunk, max_chunks;  // max_chunks: of one instance
    int64_t ncell_tot, nob_tot, max_nob;
    bool prep, any_search, any_random, split;  // prep: some instance needs the prep kernel
    bool any_staged, any_tiles;
    bool caller_order;  // some instance keeps the caller's order
};

Shape shape_of(const Plan& P) {
    return Shape{P.n_inst, P.nblk, P.nchunk, P.max_chunks, P.ncell_tot, P.nob_tot, P.max_nob,
                 P.adaptive || P.subgrid, P.any_search, P.any_random, P.split, P.any_staged, P.any_tiles,
                 P.caller_order};
}

ClearArgs clear_args(const Buffers& B, const Shape& P, bool mom, bool fresh) {
    ClearArgs c{};
    c.start = B.start;
    c.ncell = P.ncell_tot + 1;
    c.macc = mom ? (unsigned long long*)B.macc : nullptr;
    c.nwords = P.nob_tot * (int64_t)(sizeof(ObAcc) / 8);
    c.mexp = (unsigned long long*)B.mexp;
    c.nexp = B.mexp ? exp_bytes(P.nob_tot) / 8 : 0;
    c.pair_count = B.pair_count;
    c.ties = B.ties;
    if (fresh) {
        c.shift = B.shift;
        c.nshift = 3 * std::max<int64_t>(P.nob_tot, 1);
        c.status = B.status;
    }
    return c;
}

// A step of one instance writes its tables on the device; fresh: its scratch
// keeps an earlier call's contents, so shifts and status word are cleared too.
template <typename real>
struct One {
    Inst<real> inst;
    bool fresh;
};

// Everything of one step.  `one`: of one instance, whose tables it writes
// (null: they are on the device).  `h` only records phase timings (null:
// none).
template <typename real>
void enqueue_step(tpkmc_handle* h, const Buffers& B, const StepArgs<real>& a, const tpkmc_outputs* o,
                  const Shape& P, int search_block, int search_group, hipStream_t s, bool prof,
                  int advance_step, const One<real>* one) {
    const bool mom = o && o->moments;
    {
        PhaseScope ps(h, PH_CLEAR, s, prof);
        const ClearArgs c = clear_args(B, P, mom, one && one->fresh);
        const int64_t work = std::max<int64_t>(std::max<int64_t>(c.ncell, c.nwords), one ? P.nblk : 0);
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, 4096));
        if (one)
            hipLaunchKernelGGL(k_begin<real>, dim3(grid), dim3(256), 0, s, one->inst, (Inst<real>*)B.inst, B.blk,
                               B.chunks, c);
        else
            hipLaunchKernelGGL(k_clear, dim3(grid), dim3(256), 0, s, c);
    }
    if (P.nblk > 0) {
        PhaseScope ps(h, PH_KEY, s, prof);
        launch_key<real>(a, s);
        if (P.prep) launch_prep<real>((Inst<real>*)B.inst, B.gpart, P.n_inst, P.max_chunks * kChunk, s);
    }
    {
        PhaseScope ps(h, PH_SCAN, s, prof);
        enqueue_scan(B, P.ncell_tot + 1, s);
    }
    if (P.nblk > 0) {
        {
            PhaseScope ps(h, PH_SCATTER, s, prof);
            launch_scatter<real>(a, s);
        }
        {
            PhaseScope ps(h, PH_SEARCH, s, prof);
            if (P.any_staged) launch_search<real>(a, search_block, search_group, s);
            if (P.any_tiles) launch_search_tiles<real>(a, s);
            if (P.split) launch_search_fast<real>(a, P.n_inst, s);
            if (P.any_search) launch_search_ties<real>(a, s);
            if (P.any_random) launch_random_pairs<real>(a, s);
        }
        {
            PhaseScope ps(h, PH_MOVE, s, prof);
            launch_move<real>(a, s);
            launch_moments<real>(a, P.caller_order, s);
        }
    }
    {
        PhaseScope ps(h, PH_FINAL, s, prof);
        const bool direct = P.max_chunks <= kDirectChunks;
        if (P.nchunk > 0 && !direct)
            hipLaunchKernelGGL(k_reduce_chunks, dim3((unsigned)P.nchunk), dim3(256), 0, s,
                               (const Chunk*)B.chunks, (const double*)B.gpart, B.cpart);
        const unsigned gx = 1 + (mom ? (unsigned)((P.max_nob + kMomentRows - 1) / kMomentRows) : 0u);
        hipLaunchKernelGGL(k_finalize<real>, dim3(gx, P.n_inst), dim3(256), 0, s, (Inst<real>*)B.inst,
                           (const double*)B.cpart, direct ? (const double*)B.gpart : (const double*)nullptr,
                           o ? o->counters : nullptr, o ? o->globals : nullptr, B.status, B.pair_count, a.pair_cap,
                           advance_step, (const ObAcc*)B.macc, (const char*)a.mexp, a.exp_stride,
                           mom ? o->moments : nullptr, B.shift);
    }
}

int upload(tpkmc_handle* h, const Plan& P, hipStream_t s) {
    const size_t ib = P.inst_bytes.size(), bb = sizeof(Blk) * P.blk.size(), cb = sizeof(Chunk) * P.chunks.size();
    if (ib + bb + cb > h->stage_bytes) return TPKMC_ECAPACITY;
    const int k = h->stage_next;
    h->stage_next = (k + 1) % tpkmc_handle::kRing;
    if (h->stage_used[k] && hipEventSynchronize(h->stage_ev[k]) != hipSuccess) return TPKMC_EHIP;
    std::memcpy(h->stage[k], P.inst_bytes.data(), ib);
    if (bb) std::memcpy(h->stage[k] + ib, P.blk.data(), bb);
    if (cb) std::memcpy(h->stage[k] + ib + bb, P.chunks.data(), cb);
    if (hipMemcpyAsync(h->b.inst, h->stage[k], ib, hipMemcpyHostToDevice, s) != hipSuccess) return TPKMC_EHIP;
    if (bb && hipMemcpyAsync(h->b.blk, h->stage[k] + ib, bb, hipMemcpyHostToDevice, s) != hipSuccess)
        return TPKMC_EHIP;
    if (cb && hipMemcpyAsync(h->b.chunks, h->stage[k] + ib + bb, cb, hipMemcpyHostToDevice, s) != hipSuccess)
        return TPKMC_EHIP;
    if (hipEventRecord(h->stage_ev[k], s) != hipSuccess) return TPKMC_EHIP;
    h->stage_used[k] = true;
    return TPKMC_OK;
}

template <typename real>
int step_impl(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst,
              const tpkmc_outputs* o, hipStream_t st) {
    // One instance: its tables are written by the step's first launch.
    const bool single = n_inst == 1;
    Plan P;
    int rc = make_plan<real>(h, s, in, n_inst, P, false, !single);
    if (rc) return rc;
    if ((rc = check_outputs(o))) return rc;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    One<real> one{};
    if (single) std::memcpy(&one.inst, P.inst_bytes.data(), sizeof(one.inst));
    else if ((rc = upload(h, P, st))) return rc;
    StepArgs<real> a = make_args<real>(h->b, s, o, P.nblk, P.nob_tot);
    a.order = h->search_order;
    enqueue_step<real>(h, h->b, a, o, shape_of(P), h->search_block, h->search_group, st, h->profiling, 0,
                       single ? &one : nullptr);
    h->last_stream = st;
    return hipGetLastError() == hipSuccess ? TPKMC_OK : TPKMC_EHIP;
}

template <typename real>
int tune_impl(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, hipStream_t st);

template <typename real>
int run_impl(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, int nsteps,
             const tpkmc_outputs* o, hipStream_t caller) {
    if (nsteps < 0) return TPKMC_EINVAL;
    Plan P;
    int rc = make_plan<real>(h, s, in, n_inst, P, true);  // validation before anything runs
    if (rc) return rc;
    if ((rc = check_outputs(o))) return rc;
    if (nsteps == 0) return TPKMC_OK;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    // Graphs are captured on a non-default stream; order it after the caller.
    hipStream_t st = caller ? caller : h->own_stream;
    hipEvent_t ev = nullptr;
    if (!caller) {
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return TPKMC_EHIP;
        hipEventRecord(ev, nullptr);
        hipStreamWaitEvent(st, ev, 0);
    }
    // First use without a chosen launch shape: tune it on this batch (the
    // state is not modified; every shape gives the same results).
    if (!h->shape_chosen && (rc = tune_impl<real>(h, s, in, n_inst, st))) return rc;
    if ((rc = make_plan<real>(h, s, in, n_inst, P))) return rc;  // with the tuned c-bins
    if ((rc = upload(h, P, st))) return rc;
    StepArgs<real> a = make_args<real>(h->b, s, o, P.nblk, P.nob_tot);
    a.order = h->search_order;
    if (h->gexec) {
        hipStreamSynchronize(h->last_stream ? h->last_stream : st);
        hipGraphExecDestroy(h->gexec);
        h->gexec = nullptr;
    }
    hipGraph_t graph = nullptr;
    if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) return TPKMC_EHIP;
    enqueue_step<real>(nullptr, h->b, a, o, shape_of(P), h->search_block, h->search_group, st, false, 1,
                       (const One<real>*)nullptr);
    if (hipStreamEndCapture(st, &graph) != hipSuccess || !graph) return TPKMC_EHIP;
    if (hipGraphInstantiate(&h->gexec, graph, nullptr, nullptr, 0) != hipSuccess) {
        hipGraphDestroy(graph);
        return TPKMC_EHIP;
    }
    hipGraphDestroy(graph);
    for (int k = 0; k < nsteps; ++k)
        if (hipGraphLaunch(h->gexec, st) != hipSuccess) return TPKMC_EHIP;
    if (!caller) {
        hipEventRecord(ev, st);
        hipStreamWaitEvent(nullptr, ev, 0);
        hipEventDestroy(ev);
    }
    h->last_stream = st;
    return hipGetLastError() == hipSuccess ? TPKMC_OK : TPKMC_EHIP;
}

template <typename T>
int dalloc(T** p, int64_t count) {
    *p = nullptr;
    if (count <= 0) count = 1;
    return hipMalloc((void**)p, sizeof(T) * (size_t)count) == hipSuccess ? 0 : -1;
}

// Scratch that a step is faster with but does without: null where it would take
// more than an eighth of the memory that is free, so that a state that just
// fits the card beside the rest of its scratch still does.
void alloc_extra(void** p, int64_t bytes) {
    size_t room = 0, total = 0;
    *p = nullptr;
    if (hipMemGetInfo(&room, &total) != hipSuccess || bytes <= 0 || (size_t)bytes > room / 8 ||
        hipMalloc(p, (size_t)bytes) != hipSuccess) {
        *p = nullptr;
        hipGetLastError();
    }
}

// Grows the c-bin counts array (and its scan tiles) to hold `need` c-bins.
int grow_cells(tpkmc_handle* h, int64_t need) {
    if (need <= h->cell_cap) return TPKMC_OK;
    if (need >= ((int64_t)1 << 30)) return TPKMC_ECAPACITY;
    if (hipDeviceSynchronize() != hipSuccess) return TPKMC_EHIP;
    if (h->gexec) {
        hipGraphExecDestroy(h->gexec);
        h->gexec = nullptr;
    }
    hipFree(h->b.start);
    hipFree(h->b.tiles);
    h->b.start = nullptr;
    h->b.tiles = nullptr;
    const int64_t cells = sort_cells(need, h->max_n);
    if (dalloc(&h->b.start, cells + 1) || dalloc(&h->b.tiles, scan_tiles(cells + 1) + 1)) {
        h->cell_cap = 0;
        return TPKMC_ENOMEM;
    }
    h->cell_cap = need;
    return TPKMC_OK;
}

// Split c-bins (range S10 of the partner search).  Two particles of speed at
// most v_c that meet the criteria of Sec. 2.4 within the step start at most
// D + 2 v_c dt apart, so the slow particles (|v| <= v_c) can be binned on
// c-bins down to that width without losing a pair, and every pair of them
// that meets the criteria lies in neighbouring configured c-bins too.  The
// fast particles keep the configured c-bins and neighbourhood (the search's
// fast particle pass), so the step's results are the configured grid's
// whatever the speeds do later; only the search's work changes.  The bound
// is v_c = 2 v_rms over the instance's live particles, set for the gas as it
// will be once thermalised: an isolated gas keeps its root-mean-square speed
// (its energy is conserved) while its largest speed grows with the tail of
// the distribution, and a Maxwellian has 0.7% of its particles above 2 v_rms
// in three dimensions (1.8% in two), few enough that the finer c-bins of
// the rest more than pay for their searches.  Where the particles above
// 2 v_rms hold more than half of the kinetic energy (a Maxwellian: 3.5% in
// three dimensions, 9% in two, 26% in one), the gas is far from thermal (a
// point blast): collisions share that energy out and lift many more
// particles above 2 v_rms later in the run.  There the bound is 6 v_rms,
// above which at most 1/36 of the particles can ever be, as long as the
// energy is conserved (Markov's inequality on |v|^2; the 16M Sedov blast:
// 3.11 ms/step, against 3.17 with sqrt(20) v_rms and 3.35 unsplit).  Per
// instance (not with random partners,
// whose draw depends on the c-bin) and per axis, the slow particles' c-bins
// are the largest count whose width keeps a factor 1 + 1/64 over that reach
// (the rounding of the binning and of the pair test), used when it is at
// least 1.25 times the configured count (3 or more on periodic axes, never
// on a planar z), with at most one c-bin per two particles.
constexpr double kSpeedBound = 2.0;      // thermal gases
constexpr double kSpeedBoundHot = 6.0;   // far from thermal
constexpr double kReachMargin = 1.0 + 1.0 / 64.0;
constexpr double kMinRefine = 1.25;
constexpr double kHotEnergy = 0.5;
template <typename real>
int choose_cells(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, hipStream_t st) {
    h->cells.clear();
    Plan P;
    int rc = make_plan<real>(h, s, in, n_inst, P, true);
    if (rc) return rc;
    std::vector<Inst<real>> I(n_inst);
    std::memcpy(I.data(), P.inst_bytes.data(), P.inst_bytes.size());
    std::vector<double> v2sum(n_inst, 0.0), nlive(n_inst, 0.0), hot(n_inst, 0.0);
    if (P.nblk > 0) {
        // Two passes: the root-mean-square speeds, then the energy held above
        // each instance's bound.
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 1) {
                for (int k = 0; k < n_inst; ++k) {
                    const double vc = nlive[k] > 0.0 ? kSpeedBound * sqrt(v2sum[k] / nlive[k]) : 0.0;
                    I[k].vc2 = (real)(vc * vc);
                }
                std::memcpy(P.inst_bytes.data(), I.data(), P.inst_bytes.size());
            }
            if ((rc = upload(h, P, st))) return rc;
            tpkmc_outputs none{};
            StepArgs<real> a = make_args<real>(h->b, s, &none, P.nblk, P.nob_tot);
            launch_speed_stats<real>(a, st);
            std::vector<double> gp((size_t)P.nblk * kGPart);
            if (hipMemcpyAsync(gp.data(), h->b.gpart, sizeof(double) * gp.size(), hipMemcpyDeviceToHost, st) !=
                    hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess)
                return TPKMC_EHIP;
            // Summed in block order, so the same state always gives the same c-bins.
            for (int b = 0; b < P.nblk; ++b) {
                const int k = P.blk[b].inst;
                if (pass == 0) {
                    v2sum[k] += gp[(size_t)b * kGPart + GP_PX];
                    nlive[k] += gp[(size_t)b * kGPart + GP_PY];
                } else {
                    hot[k] += gp[(size_t)b * kGPart + GP_PZ];
                }
            }
        }
    }
    int64_t total = 0;
    for (int k = 0; k < n_inst; ++k) {
        const tpkmc_instance& q = in[k];
        tpkmc_handle::Cells c{q.grid, q.params.sigma, q.params.dt, q.params.flags & kCellKey,
                              {q.grid.ncell[0], q.grid.ncell[1], q.grid.ncell[2]}, 0.0};
        const bool thermal = !(hot[k] > kHotEnergy * v2sum[k]);
        const double vc = nlive[k] > 0.0 ? (thermal ? kSpeedBound : kSpeedBoundHot) * sqrt(v2sum[k] / nlive[k]) : 0.0;
        const double reach = sqrt((double)I[k].D2) + 2.0 * vc * q.params.dt;
        const bool planar = (q.params.flags & TPKMC_PLANAR) != 0;
        int64_t cfg = 1;
        for (int a = 0; a < 3; ++a) cfg *= q.grid.ncell[a];
        if (!(q.params.flags & TPKMC_PAIR_RANDOM) && q.count > 0 && reach > 0.0 && std::isfinite(reach)) {
            const int64_t cap = std::max<int64_t>(cfg, q.count / 2);
            int32_t lo[3];
            for (int a = 0; a < 3; ++a) {
                lo[a] = (int32_t)std::ceil(kMinRefine * q.grid.ncell[a]);
                if (q.grid.bc[a] == TPKMC_BC_PERIODIC) lo[a] = std::max(lo[a], 3);
                if (planar && a == 2) continue;
                const double L = q.grid.hi[a] - q.grid.lo[a];
                const double nmax = std::floor(L / (kReachMargin * reach));
                if (nmax < (double)lo[a] || nmax > (double)(1 << 24)) continue;
                c.n[a] = (int32_t)nmax;
            }
            // At most `cap` c-bins: shrink the most refined axis first.
            for (;;) {
                int64_t prod = (int64_t)c.n[0] * c.n[1] * c.n[2];
                if (prod <= cap) break;
                int a = -1;
                double best = 1.0;
                for (int b = 0; b < 3; ++b) {
                    const double f = (double)c.n[b] / q.grid.ncell[b];
                    if (f > best) { best = f; a = b; }
                }
                if (a < 0) break;
                const int32_t m = (int32_t)std::floor(c.n[a] * 0.9);
                c.n[a] = m >= lo[a] ? m : q.grid.ncell[a];
            }
        }
        const int64_t nslow = (int64_t)c.n[0] * c.n[1] * c.n[2];
        if (nslow != cfg) c.vc = vc;
        total += (nslow != cfg ? nslow + cfg : cfg) + 1;
        h->cells.push_back(c);
    }
    if (total > h->cell_cap && (rc = grow_cells(h, total))) {
        h->cells.clear();
        return rc;
    }
    return TPKMC_OK;
}

template <typename real>
int tune_impl(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, hipStream_t st) {
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    int rc = choose_cells<real>(h, s, in, n_inst, st);
    if (rc) return rc;
    Plan P;
    rc = make_plan<real>(h, s, in, n_inst, P);
    if (rc) return rc;
    if (P.nblk == 0) return TPKMC_OK;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    if ((rc = upload(h, P, st))) return rc;
    tpkmc_outputs none{};
    StepArgs<real> a = make_args<real>(h->b, s, &none, P.nblk, P.nob_tot);
    a.order = 0;  // shapes are timed with contiguous ranges per XCD
    // Bin once (clear, key, prefix, scatter); then time only the search.
    hipLaunchKernelGGL(k_clear, dim3(1024), dim3(256), 0, st, clear_args(h->b, shape_of(P), false, false));
    launch_key<real>(a, st);
    if (P.adaptive || P.subgrid)
        launch_prep<real>((Inst<real>*)h->b.inst, h->b.gpart, P.n_inst, P.max_chunks * kChunk, st);
    enqueue_scan(h->b, P.ncell_tot + 1, st);
    launch_scatter<real>(a, st);
    hipEvent_t e0, e1;
    hipEventCreate(&e0);
    hipEventCreate(&e1);
    // Results-neutral launch shapes: records per lane (1, 2, 4) and lanes per
    // work-group (64, 128, 256).  The default shape (2 records per lane, 64
    // lanes, the fastest on sparse bins) is timed first and is replaced only
    // by a shape at least 5% faster, so that near-ties do not flip the choice
    // from run to run (on the 16M Sedov blast 128 lanes time up to 4% faster
    // on the initial state and 4% slower later in the run).
    float best_ms = 1e30f;
    int best_block = kWave, best_group = 2;
    std::vector<std::pair<int, int>> shapes = {{2, kWave}};
    for (int grp : {1, 2, 4})
        for (int bs : {256, 128, 64})
            if (bs <= kBlock / grp && !(grp == 2 && bs == kWave)) shapes.push_back({grp, bs});
    // Warm the caches and clocks first: the first shape timed would
    // otherwise look slower than it is.
    auto search = [&](int bs, int grp) {
        if (P.any_staged) launch_search<real>(a, bs, grp, st);
        if (P.any_tiles) launch_search_tiles<real>(a, st);
    };
    // The tile search and the FP64 lanes have one shape.
    if (!P.any_staged || std::is_same<real, double>::value) shapes.resize(1);
    for (int r = 0; r < 4; ++r) search(kWave, 2);
    for (const auto& sh : shapes) {
        const int grp = sh.first, bs = sh.second;
        search(bs, grp);  // warm-up
        hipEventRecord(e0, st);
        for (int r = 0; r < 3; ++r) search(bs, grp);
        hipEventRecord(e1, st);
        if (hipEventSynchronize(e1) != hipSuccess) { rc = TPKMC_EHIP; break; }
        float ms = 0.f;
        hipEventElapsedTime(&ms, e0, e1);
        if (ms < 0.95f * best_ms) { best_ms = ms; best_block = bs; best_group = grp; }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc) return rc;
    // Work-group order of the search (results-neutral): chunks of 16
    // work-groups dealt round-robin over the XCDs (the default), contiguous
    // ranges per XCD, or chunks of 1 or 128; another order is kept only when
    // at least 5% faster, timed in the chosen shape.  The default balances
    // the XCDs by construction: where the work concentrates as a run goes on
    // (the shocked core of an implosion, the shell of a blast), contiguous
    // ranges leave it to one or two XCDs, which the initial state does not
    // show (on the Noh 8M implosion 9.7 against 6.8 ms per step).  The tile
    // search's work grows with the density, so it is not given contiguous
    // ranges at all: the same implosion's uniform start runs 5% faster on
    // them, steps 40 to 280 at 1.95 to 3.9 ms, in chunks of 16 at 1.75 to 2.4.
    int best_order = kDefaultSearchOrder;
    if (!rc) {
        hipEvent_t f0, f1;
        hipEventCreate(&f0);
        hipEventCreate(&f1);
        float base_ms = 1e30f;
        for (int order : {kDefaultSearchOrder, 0, 1, 128}) {
            if (order == 0 && P.any_tiles) continue;
            a.order = order;
            search(best_block, best_group);  // warm-up
            hipEventRecord(f0, st);
            for (int r = 0; r < 3; ++r) search(best_block, best_group);
            hipEventRecord(f1, st);
            if (hipEventSynchronize(f1) != hipSuccess) { rc = TPKMC_EHIP; break; }
            float ms = 0.f;
            hipEventElapsedTime(&ms, f0, f1);
            if (order == kDefaultSearchOrder) base_ms = best_ms = ms;
            else if (ms < 0.95f * best_ms && ms < 0.95f * base_ms) { best_ms = ms; best_order = order; }
        }
        hipEventDestroy(f0);
        hipEventDestroy(f1);
        a.order = 0;
    }
    h->search_block = best_block;
    h->search_group = best_group;
    h->search_order = best_order;
    h->shape_chosen = true;
    h->last_stream = st;
    return hipGetLastError() == hipSuccess ? TPKMC_OK : TPKMC_EHIP;
}

// The search's arithmetic mix on a state: bins it (clear, key, prefix,
// scatter) and runs the counting build of the search, which leaves the state
// and the step's outputs untouched.
template <typename real>
int mix_impl(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* in, int n_inst, uint64_t* counts,
             hipStream_t st) {
    if (!counts) return TPKMC_EINVAL;
    Plan P;
    int rc = make_plan<real>(h, s, in, n_inst, P);
    if (rc) return rc;
    counts[0] = counts[1] = counts[2] = 0;
    if (P.nblk == 0) return TPKMC_OK;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    if ((rc = upload(h, P, st))) return rc;
    tpkmc_outputs none{};
    StepArgs<real> a = make_args<real>(h->b, s, &none, P.nblk, P.nob_tot);
    a.order = h->search_order;
    hipLaunchKernelGGL(k_clear, dim3(1024), dim3(256), 0, st, clear_args(h->b, shape_of(P), false, false));
    launch_key<real>(a, st);
    if (P.adaptive || P.subgrid)
        launch_prep<real>((Inst<real>*)h->b.inst, h->b.gpart, P.n_inst, P.max_chunks * kChunk, st);
    enqueue_scan(h->b, P.ncell_tot + 1, st);
    launch_scatter<real>(a, st);
    if (hipMemsetAsync(h->b.mix, 0, 3 * sizeof(unsigned long long), st) != hipSuccess) return TPKMC_EHIP;
    launch_search_mix<real>(a, P.n_inst, P.split, st);
    if (hipMemcpyAsync(counts, h->b.mix, 3 * sizeof(uint64_t), hipMemcpyDeviceToHost, st) != hipSuccess)
        return TPKMC_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) return TPKMC_EHIP;
    h->last_stream = st;
    return hipGetLastError() == hipSuccess ? TPKMC_OK : TPKMC_EHIP;
}


void free_all(tpkmc_handle* h) {
    for (int k = 0; k < tpkmc_handle::kRing; ++k) {
        if (h->stage[k]) hipHostFree(h->stage[k]);
        if (h->stage_ev[k]) hipEventDestroy(h->stage_ev[k]);
    }
    hipFree(h->b.rank); hipFree(h->b.start); hipFree(h->b.tiles);
    hipFree(h->b.src); hipFree(h->b.best); hipFree(h->b.perm); hipFree(h->b.rec); hipFree(h->b.rec2); hipFree(h->b.rmass); hipFree(h->b.inst);
    hipFree(h->b.blk); hipFree(h->b.chunks); hipFree(h->b.bkey); hipFree(h->b.cpart); hipFree(h->b.gpart); hipFree(h->b.shift); hipFree(h->b.macc); hipFree(h->b.mexp); hipFree(h->b.vir); hipFree(h->b.coll); hipFree(h->b.pair_count); hipFree(h->b.status); hipFree(h->b.mix);
}

// ---------------------------------------------------------------- static scratch
// Scratch of the allocation-free entry point: one array per GPU, held until
// the process ends.  Host code never uses the name `scratch` as an address
// (on the host it is only a stand-in); it uses the device address that
// hipGetSymbolAddress returns, looked up once per device with that device
// current and kept in scratch_ptr.
static __device__ __align__(256) unsigned char scratch[TPKMC_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
unsigned char* scratch_ptr[kMaxDevices] = {};

int scratch_of(int device, unsigned char** out) {
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return TPKMC_EHIP;
        scratch_ptr[device] = (unsigned char*)p;
    }
    *out = scratch_ptr[device];
    return TPKMC_OK;
}

// Carves the buffers of one instance out of the region starting at `base`
// (256-byte aligned pieces) and returns the bytes they span; with base 0 it
// only measures.
template <typename real>
size_t carve(uintptr_t base, int64_t n, int64_t ncell_tot, int64_t nob, int nblk, int nchunk, bool masses,
             bool second, bool apart, Buffers& B) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> void* {
        const uintptr_t p = base + off;
        off += (std::max<size_t>(bytes, 1) + 255) & ~(size_t)255;
        return (void*)p;
    };
    const size_t nn = (size_t)std::max<int64_t>(n, 1);
    B.rank = (int32_t*)take(4 * nn);
    B.src = (int32_t*)take(4 * nn);
    // Random partners alone; in FP64 they share the keys' place (see rp_best).
    const bool fp32 = std::is_same<real, float>::value;
    B.best = fp32 ? (int32_t*)take(4 * nn) : nullptr;
    B.perm = fp32 ? (int32_t*)take(4 * nn) : nullptr;
    B.rec = take(8 * sizeof(real) * nn);
    B.rec2 = second ? take(8 * sizeof(real) * nn) : nullptr;
    B.rmass = masses ? take(sizeof(real) * nn) : nullptr;
    B.bkey = (unsigned long long*)take(8 * nn);
    B.start = (int32_t*)take(4 * (size_t)(ncell_tot + 1));
    B.tiles = (int32_t*)take(4 * (size_t)(scan_tiles(ncell_tot + 1) + 1));
    B.inst = take(sizeof(Inst<real>));
    B.blk = (Blk*)take(sizeof(Blk) * (size_t)nblk);
    B.gpart = (double*)take(sizeof(double) * kGPart * (size_t)nblk);
    B.chunks = (Chunk*)take(sizeof(Chunk) * (size_t)nchunk);
    B.cpart = (double*)take(sizeof(double) * kGPart * (size_t)nchunk);
    B.shift = (double*)take(sizeof(double) * 3 * (size_t)std::max<int64_t>(nob, 1));
    B.macc = (ObAcc*)take(sizeof(ObAcc) * (size_t)std::max<int64_t>(nob, 1));
    B.mexp = apart ? (char*)take((size_t)exp_bytes(nob)) : nullptr;
    B.vir = take(3 * sizeof(real) * nn);
    B.coll = (uint8_t*)take(nn);
    B.pair_count = (unsigned long long*)take(2 * sizeof(unsigned long long));
    B.ties = (uint32_t*)(B.pair_count + 1);
    B.status = (uint32_t*)take(sizeof(uint32_t));
    return off;
}

template <typename real>
int step_noalloc_impl(int device, const tpkmc_grid* g, const tpkmc_params* p, const tpkmc_particles* s,
                      const tpkmc_outputs* o, hipStream_t st) {
    if (!g || !p || !s || s->n < 0 || bad_state(s)) return TPKMC_EINVAL;
    int rc = check_outputs(o);
    if (rc) return rc;
    tpkmc_instance q;
    q.offset = 0;
    q.count = s->n;
    q.grid = *g;
    q.params = *p;
    Inst<real> d;
    int64_t C = 0, B = 0;
    if ((rc = fill_inst<real>(s, q, d, C, B))) return rc;
    // Records are addressed with 32-bit byte offsets in the FP32 search.
    if (s->n >= ((int64_t)1 << 27)) return TPKMC_ECAPACITY;
    const int nblk = (int)((s->n + kBlock - 1) / kBlock);
    const int nchunk = (nblk + kChunk - 1) / kChunk;
    int64_t ncell_tot = (int64_t)d.C + 1;
    d.cell_off = 0;
    d.obin_off = 0;
    d.blk0 = 0;
    d.nblk = nblk;
    d.chunk0 = 0;
    d.nchunk = nchunk;
    Buffers Bf{};
    auto fits = [&](bool second, bool apart) {
        return carve<real>(0, s->n, ncell_tot, B, nblk, nchunk, s->mass != nullptr, second, apart, Bf) <=
               TPKMC_NOALLOC_SCRATCH_BYTES;
    };
    if ((d.flags & kSubgrid) && !fits(false, false)) {
        // The sub-grid is an extra: without it where the scratch is short.
        if ((rc = fill_inst<real>(s, q, d, C, B, nullptr, 0.0, false))) return rc;
        ncell_tot = (int64_t)d.C + 1;
        d.blk0 = 0;
        d.nblk = nblk;
        d.chunk0 = 0;
        d.nchunk = nchunk;
    }
    if (!fits(false, false)) return TPKMC_ECAPACITY;
    // So are the second records, which only a state in the caller's order takes,
    // and the o-bins' exponents apart from their sums.
    const bool caller_order = !(p->flags & TPKMC_ALLOW_REORDER);
    const bool second = caller_order && fits(true, false), apart = fits(second, true);
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess) return TPKMC_EHIP;
    if (device < 0 || device >= ndev || device >= kMaxDevices) return TPKMC_EINVAL;
    if (hipSetDevice(device) != hipSuccess) return TPKMC_EHIP;
    unsigned char* base = nullptr;
    if ((rc = scratch_of(device, &base))) return rc;
    carve<real>((uintptr_t)base, s->n, ncell_tot, B, nblk, nchunk, s->mass != nullptr, second, apart, Bf);
    const bool random = (p->flags & TPKMC_PAIR_RANDOM) != 0;
    Shape P{};
    P.n_inst = 1;
    P.nblk = nblk;
    P.nchunk = nchunk;
    P.max_chunks = nchunk;
    P.ncell_tot = ncell_tot;
    P.nob_tot = B;
    P.max_nob = B;
    P.prep = (p->flags & TPKMC_ADAPTIVE_DT) != 0 || (d.flags & kSubgrid) != 0;
    P.any_staged = !random && !(d.flags & kTiles);
    P.any_tiles = !random && (d.flags & kTiles);
    P.caller_order = caller_order;
    P.any_search = !random;
    P.any_random = random;
    P.split = false;
    StepArgs<real> a = make_args<real>(Bf, s, o, nblk, B);
    const One<real> one{d, true};
    enqueue_step<real>(nullptr, Bf, a, o, P, kWave, 2, st, false, 0, &one);
    return hipGetLastError() == hipSuccess ? TPKMC_OK : TPKMC_EHIP;
}

}  // namespace

// ---------------------------------------------------------------- C ABI
extern "C" {

int tpkmc_version(void) { return TPKMC_ABI_VERSION; }

const char* tpkmc_strerror(int code) {
    switch (code) {
        case TPKMC_OK: return "success";
        case TPKMC_EINVAL: return "invalid argument";
        case TPKMC_ENOMEM: return "device allocation failed";
        case TPKMC_EHIP: return "HIP runtime error";
        case TPKMC_ECAPACITY: return "input exceeds the capacity of the handle or of the static scratch";
        case TPKMC_EUNSUPPORTED: return "unsupported";
        default: return "unknown error code";
    }
}

int tpkmc_create(const tpkmc_config* cfg, tpkmc_handle** out) {
    if (!out) return TPKMC_EINVAL;
    *out = nullptr;
    // Records are addressed with 32-bit byte offsets in the FP32 search.
    const int64_t max_n = cfg && cfg->precision == TPKMC_FP32 ? ((int64_t)1 << 27) : ((int64_t)1 << 31);
    if (!cfg || cfg->max_particles < 0 || cfg->max_particles >= max_n || cfg->max_cells < 1 ||
        cfg->max_cells >= ((int64_t)1 << 30) || cfg->max_obins < 0 || cfg->max_obins >= ((int64_t)1 << 30) ||
        cfg->max_instances < 1 || cfg->flags != 0 ||
        (cfg->precision != TPKMC_FP64 && cfg->precision != TPKMC_FP32))
        return TPKMC_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || cfg->device < 0 || cfg->device >= ndev) return TPKMC_EINVAL;
    if (hipSetDevice(cfg->device) != hipSuccess) return TPKMC_EHIP;
    tpkmc_handle* h = new (std::nothrow) tpkmc_handle();
    if (!h) return TPKMC_ENOMEM;
    h->device = cfg->device;
    h->precision = cfg->precision;
    h->max_n = cfg->max_particles;
    h->max_cells = cfg->max_cells;
    h->cell_cap = cfg->max_cells;
    h->max_obins = cfg->max_obins;
    h->max_inst = cfg->max_instances;
    h->max_blk = cfg->max_particles / kBlock + cfg->max_instances + 1;
    h->max_chunks = h->max_blk / kChunk + cfg->max_instances + 1;
    const size_t rs = cfg->precision == TPKMC_FP64 ? sizeof(double) : sizeof(float);
    const size_t inst_sz = cfg->precision == TPKMC_FP64 ? sizeof(Inst<double>) : sizeof(Inst<float>);
    const int64_t cells = sort_cells(cfg->max_cells, cfg->max_particles);
    int bad = 0;
    bad |= dalloc(&h->b.rank, h->max_n);
    bad |= dalloc(&h->b.start, cells + 1);
    bad |= dalloc(&h->b.tiles, scan_tiles(cells + 1) + 1);
    bad |= dalloc(&h->b.src, h->max_n);
    if (cfg->precision == TPKMC_FP32) bad |= dalloc(&h->b.best, h->max_n) | dalloc(&h->b.perm, h->max_n);
    bad |= hipMalloc(&h->b.rec, rs * 8 * (size_t)std::max<int64_t>(h->max_n, 1)) != hipSuccess;
    bad |= hipMalloc(&h->b.rmass, rs * (size_t)std::max<int64_t>(h->max_n, 1)) != hipSuccess;
    bad |= hipMalloc(&h->b.inst, inst_sz * (size_t)h->max_inst) != hipSuccess;
    bad |= dalloc(&h->b.blk, h->max_blk);
    bad |= dalloc(&h->b.gpart, h->max_blk * kGPart);
    bad |= dalloc(&h->b.chunks, h->max_chunks);
    bad |= dalloc(&h->b.cpart, h->max_chunks * kGPart);
    bad |= dalloc(&h->b.bkey, h->max_n);
    bad |= dalloc(&h->b.shift, 3 * std::max<int64_t>(h->max_obins, 1));
    bad |= dalloc(&h->b.macc, std::max<int64_t>(h->max_obins, 1));
    bad |= hipMalloc(&h->b.vir, rs * 3 * (size_t)std::max<int64_t>(h->max_n, 1)) != hipSuccess;
    bad |= dalloc(&h->b.coll, (std::max<int64_t>(h->max_n, 1) + 3) & ~(int64_t)3);  // whole words (see Key)
    bad |= dalloc(&h->b.pair_count, 2);
    bad |= dalloc(&h->b.mix, 3);
    bad |= dalloc(&h->b.status, 1);
    h->stage_bytes = inst_sz * (size_t)h->max_inst + sizeof(Blk) * (size_t)h->max_blk +
                     sizeof(Chunk) * (size_t)h->max_chunks;
    for (int k = 0; k < tpkmc_handle::kRing && !bad; ++k) {
        bad |= hipHostMalloc((void**)&h->stage[k], h->stage_bytes, hipHostMallocDefault) != hipSuccess;
        bad |= hipEventCreateWithFlags(&h->stage_ev[k], hipEventDisableTiming) != hipSuccess;
    }
    if (!bad) {
        bad |= hipMemset(h->b.shift, 0, sizeof(double) * 3 * (size_t)std::max<int64_t>(h->max_obins, 1)) != hipSuccess;
        bad |= hipMemset(h->b.status, 0, sizeof(uint32_t)) != hipSuccess;
        bad |= hipMemset(h->b.gpart, 0, sizeof(double) * kGPart * (size_t)h->max_blk) != hipSuccess;
        bad |= hipStreamCreateWithFlags(&h->own_stream, hipStreamNonBlocking) != hipSuccess;
        bad |= hipDeviceSynchronize() != hipSuccess;
    }
    if (!bad) {
        h->b.ties = (uint32_t*)(h->b.pair_count + 1);
        alloc_extra((void**)&h->b.mexp,
                    std::max(exp_bytes(h->max_obins), exp_bytes(std::min(h->max_obins, kSpreadObins))));
        alloc_extra(&h->b.rec2, (int64_t)rs * 8 * std::max<int64_t>(h->max_n, 1));
    }
    if (bad) {
        free_all(h);
        if (h->own_stream) hipStreamDestroy(h->own_stream);
        delete h;
        hipGetLastError();
        return TPKMC_ENOMEM;
    }
    *out = h;
    return TPKMC_OK;
}

int tpkmc_destroy(tpkmc_handle* h) {
    if (!h) return TPKMC_OK;
    hipSetDevice(h->device);
    hipDeviceSynchronize();
    if (h->gexec) hipGraphExecDestroy(h->gexec);
    for (hipEvent_t e : h->pool) hipEventDestroy(e);
    free_all(h);
    if (h->own_stream) hipStreamDestroy(h->own_stream);
    delete h;
    return TPKMC_OK;
}

int tpkmc_step(tpkmc_handle* h, const tpkmc_grid* g, const tpkmc_params* p, const tpkmc_particles* s,
               const tpkmc_outputs* o, void* stream) {
    if (!h || !g || !p || !s) return TPKMC_EINVAL;
    tpkmc_instance one;
    one.offset = 0;
    one.count = s->n;
    one.grid = *g;
    one.params = *p;
    return tpkmc_step_batched(h, s, &one, 1, o, stream);
}

int tpkmc_step_noalloc(int32_t precision, int32_t device, const tpkmc_grid* g, const tpkmc_params* p,
                       const tpkmc_particles* s, const tpkmc_outputs* o, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (precision == TPKMC_FP64) return step_noalloc_impl<double>(device, g, p, s, o, st);
    if (precision == TPKMC_FP32) return step_noalloc_impl<float>(device, g, p, s, o, st);
    return TPKMC_EINVAL;
}

int tpkmc_step_batched(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* inst, int32_t n_inst,
                       const tpkmc_outputs* o, void* stream) {
    if (!h) return TPKMC_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    return h->precision == TPKMC_FP64 ? step_impl<double>(h, s, inst, n_inst, o, st)
                                      : step_impl<float>(h, s, inst, n_inst, o, st);
}

int tpkmc_run(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* inst, int32_t n_inst,
              int32_t nsteps, const tpkmc_outputs* o, void* stream) {
    if (!h) return TPKMC_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    return h->precision == TPKMC_FP64 ? run_impl<double>(h, s, inst, n_inst, nsteps, o, st)
                                      : run_impl<float>(h, s, inst, n_inst, nsteps, o, st);
}

int tpkmc_autotune(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* inst, int32_t n_inst,
                   void* stream) {
    if (!h) return TPKMC_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    return h->precision == TPKMC_FP64 ? tune_impl<double>(h, s, inst, n_inst, st)
                                      : tune_impl<float>(h, s, inst, n_inst, st);
}

int tpkmc_search_order(tpkmc_handle* h, int32_t* order) {
    if (!h || !order) return TPKMC_EINVAL;
    *order = h->search_order;
    return TPKMC_OK;
}

int tpkmc_set_search_order(tpkmc_handle* h, int32_t order) {
    if (!h || order < 0 || order > 4096) return TPKMC_EINVAL;
    h->search_order = order;
    return TPKMC_OK;
}

int tpkmc_tuned_cells(tpkmc_handle* h, int32_t k, int32_t ncell[3]) {
    if (!h || !ncell || k < 0 || k >= (int32_t)h->cells.size()) return TPKMC_EINVAL;
    for (int a = 0; a < 3; ++a) ncell[a] = h->cells[k].n[a];
    return TPKMC_OK;
}

int tpkmc_tuned_speed(tpkmc_handle* h, int32_t k, double* speed) {
    if (!h || !speed || k < 0 || k >= (int32_t)h->cells.size()) return TPKMC_EINVAL;
    *speed = h->cells[k].vc;
    return TPKMC_OK;
}

int tpkmc_search_mix(tpkmc_handle* h, const tpkmc_particles* s, const tpkmc_instance* inst, int32_t n_inst,
                     uint64_t* counts, void* stream) {
    if (!h) return TPKMC_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    return h->precision == TPKMC_FP64 ? mix_impl<double>(h, s, inst, n_inst, counts, st)
                                      : mix_impl<float>(h, s, inst, n_inst, counts, st);
}

int tpkmc_set_search(tpkmc_handle* h, int32_t group, int32_t block) {
    if (!h) return TPKMC_EINVAL;
    if (block != 64 && block != 128 && block != 256) return TPKMC_EINVAL;
    if (group != 1 && group != 2 && group != 4) return TPKMC_EINVAL;
    if (block > kBlock / group) return TPKMC_EINVAL;
    h->search_group = group;
    h->search_block = block;
    h->search_order = kDefaultSearchOrder;
    h->shape_chosen = true;
    return TPKMC_OK;
}

int tpkmc_get_search(tpkmc_handle* h, int32_t* group, int32_t* block) {
    if (!h || !group || !block) return TPKMC_EINVAL;
    *group = h->search_group;
    *block = h->search_block;
    return TPKMC_OK;
}

int tpkmc_status(tpkmc_handle* h, int32_t* device_status) {
    if (!h || !device_status) return TPKMC_EINVAL;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    if (hipStreamSynchronize(h->last_stream) != hipSuccess) return TPKMC_EHIP;
    uint32_t v = 0;
    if (hipMemcpy(&v, h->b.status, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) return TPKMC_EHIP;
    if (hipMemset(h->b.status, 0, sizeof(v)) != hipSuccess) return TPKMC_EHIP;
    *device_status = (int32_t)v;
    return TPKMC_OK;
}

int tpkmc_profile_enable(tpkmc_handle* h, int32_t on) {
    if (!h) return TPKMC_EINVAL;
    h->profiling = on != 0;
    return TPKMC_OK;
}

int tpkmc_profile_read(tpkmc_handle* h, double* ms, int64_t* launches, int32_t n) {
    if (!h || n < 0 || (n > 0 && (!ms || !launches))) return TPKMC_EINVAL;
    if (hipSetDevice(h->device) != hipSuccess) return TPKMC_EHIP;
    if (!h->prof.empty()) {
        if (hipEventSynchronize(h->prof.back().b) != hipSuccess) return TPKMC_EHIP;
        for (const ProfRec& r : h->prof) {
            float t = 0.f;
            if (hipEventElapsedTime(&t, r.a, r.b) == hipSuccess && r.phase >= 0 && r.phase < kPhases) {
                h->prof_ms[r.phase] += t;
                h->prof_n[r.phase] += 1;
            }
        }
        h->prof.clear();
        h->pool_used = 0;
    }
    for (int k = 0; k < n; ++k) {
        ms[k] = k < kPhases ? h->prof_ms[k] : 0.0;
        launches[k] = k < kPhases ? h->prof_n[k] : 0;
    }
    for (int k = 0; k < kPhases; ++k) { h->prof_ms[k] = 0.0; h->prof_n[k] = 0; }
    return TPKMC_OK;
}

}  // extern "C"
