// Internal declarations shared by the HIP translation units of libtpkmc.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tpkmc.h"

namespace tpkmc {

// Particles per work-group in every per-particle kernel; a work-group never
// spans two instances (see the block table below).
constexpr int kBlock = 256;
constexpr int kWave = 64;

// Slots of the per-work-group partial results (doubles), reduced per
// instance by the finalize kernel.
enum GPart {
    GP_PX = 0, GP_PY, GP_PZ, GP_EKIN, GP_VMAX2, GP_VIR, GP_MASS,
    GP_ALIVE, GP_PAIRS, GP_ABSORBED, GP_TESTS2, GP_CAND, GP_HAVEBEST,
    GP_FAST, GP_NONFINITE, GP_VMAX0, kGPart
};

// Exact o-bin sums, in two passes over the particles.  The move records,
// per o-bin, the exponent E per kind of term of a power of two above every
// term (|x| < 2^E, an integer maximum, so the order does not matter) and the
// counts of particles and colliders.  The moment pass then rounds each term
// once to an integer q, a multiple of 2^(E-50+h) (|q| <= 2^(50-h)), where
// the headroom h = max(0, ceil(log2 n) - 12) grows with the o-bin's n
// particles (none up to 4096): the n integers of a value sum to less than
// 2^62 in magnitude, so every partial and the total fit one int64, and
// integer sums do not depend on the order of the terms.  Kinds: 0 m (v -
// shift) per axis, 1 m (v - shift)^2 per axis, 2 virial terms, 3 mass.  Per
// o-bin: values 0..2 momentum, 3..5 spread, 6..8 virial, 9 mass
// (per-particle masses only); the particle count in the low 32 bits of nc
// and the collider count in its high 32 bits (at most 2^32 - 1 particles
// per o-bin); the four exponents (biased by kExpBias; 0: no nonzero term).
constexpr int kAccVals = 10;
constexpr int kExpBias = 1100;
// The moment pass reads the exponents and counts for every particle while it
// adds to the sums, and a line that atomics go to is slow to read: with both in
// one line of 128 B the pass took 153 us instead of 75 on the 4M tube, 363
// instead of 290 on the 16M blast.  So the exponents lie apart, a line each up
// to kSpreadObins o-bins (packed, the move's atomics on few o-bins meet in the
// same lines: 4M tube 156 us instead of 117), packed above (16M blast, 262144
// o-bins: 5 us less in the moment pass, 7 in the last kernel).  In boxes of 1e6
// and 4e6 at 512 to 32768 o-bins both cost the same within 3%, so the line may
// lie anywhere there.  Where the scratch is short they share the sums' line.
struct ObExp {
    unsigned long long nc;
    int32_t e[4];
    unsigned long long pad;
};
struct ObAcc {
    long long sum[kAccVals];
    unsigned long long pad[2];
    ObExp shared;
};
static_assert(sizeof(ObAcc) == 128 && sizeof(ObExp) == 32, "a line an o-bin");
constexpr int64_t kSpreadObins = 4096;
inline int exp_stride(int64_t nob) { return nob <= kSpreadObins ? (int)sizeof(ObAcc) : (int)sizeof(ObExp); }
inline int64_t exp_bytes(int64_t nob) { return nob * exp_stride(nob); }
__host__ __device__ inline int acc_headroom(unsigned long long n) {
    const int c = n <= 1 ? 0 : 64 - __builtin_clzll(n - 1);  // ceil(log2 n)
    return c > 12 ? c - 12 : 0;
}
__host__ __device__ constexpr int acc_kind(int k) { return k < 3 ? 0 : k < 6 ? 1 : k < 9 ? 2 : 3; }

// Instance descriptor on the device.  Derived grid quantities are computed
// on the host in double, exactly like the CPU oracle, then cast to `real`.
template <typename real>
struct Inst {
    int64_t off, cnt;         // particle slice [off, off + cnt)
    int64_t cell_off;         // first global c-bin; C bins + 1 sentinel bin
    int64_t obin_off;         // first global o-bin
    int32_t C;                // c-bins of this instance
    int32_t n[3], bc[3];      // c-bins and boundary per axis
    int32_t no[3];            // o-bins per axis
    int32_t blk0, nblk;       // range in the block table
    int32_t chunk0, nchunk;   // range in the chunk table (partials reduction)
    uint32_t seed_lo, seed_hi, step_lo, instance;
    uint32_t flags;           // TPKMC_EMIT_PAIRS | TPKMC_ALLOW_REORDER
    int32_t band_log2;        // y-band height 2^band_log2 of the c-bin order
    real lo[3], hi[3], L[3], inv_w[3], inv_wo[3], w[3];
    real dt, D2, mass;
    double mass_d, dt_d;      // dt_d: this step's time step (set on the device with ADAPTIVE_DT)
    double dt_cap, dx_d;      // caller's dt; smallest c-bin width over axes with > 1 c-bin (0: none)
    double sigma_d, cellvol_d; // cross section; c-bin volume (area in the plane), for random partners
    // Adaptive time step: running maximum of |v|^2 (bit pattern of a
    // non-negative double) and the count of prep work-groups done; the last
    // one to finish resets both.
    unsigned long long run_v2;
    uint32_t prep_done;
    // Split c-bins (kSplit): a particle is slow when its |v|^2 <= vc2; slow
    // particles are binned on the n[] c-bins (the first Cf of the C), the
    // others on the configured ncfg[] c-bins after them, numbered
    // x + ncfg[0] * (y + ncfg[1] * z).  inv_wc: configured c-bins per unit
    // length.
    int32_t ncfg[3];
    int32_t Cf;
    uint32_t run_out;         // prep's running maximum: how far one lies outside a periodic axis (see k_key)
    real vc2;
    real inv_wc[3];
    // Tile search: 1 / the length its positions are scaled by (the widest
    // c-bin).
    float tile_s;
    // In that unit, the largest coordinate of a tile's partners relative to
    // it, for a tile of one sort cell, and more per further cell along x.
    float tile_x, tile_dx;
    // Sub-grids (kSubgrid): nl[] c-bins per axis (the refined ones of split
    // c-bins), each cut into 2^kl[] sort cells, n[a] = nl[a] 2^kl[a]; inv_wl:
    // c-bins per unit length.  Without, kl is 0 and n, nl are the same.  vreach: the
    // largest speed among the records sorted on them, with the reach of those
    // outside the box in it (see k_prep).
    int32_t nl[3], kl[3];
    real inv_wl[3];
    real w_sort[3];           // width of a sort cell
    real vreach;
    int64_t base;             // record index of the instance's first: base + start[]
};
// The allocation-free step's scratch gives either of them 512 B.
static_assert(sizeof(Inst<double>) <= 512, "one descriptor is 512 B");

// Bit of Inst::flags set by the host (outside the public flag bits): the
// c-bins are split by speed (slow particles on refined c-bins, see Inst).
constexpr uint32_t kSplit = 1u << 30;

// Bits of Inst::flags set by the host: partners from the tile search (else from
// the lane walks, unless random); the c-bins are cut into sort cells (see Inst).
constexpr uint32_t kTiles = 1u << 29;
constexpr uint32_t kSubgrid = 1u << 28;

// Bit of Inst::flags, set by the host (outside the public flag bits): the
// particles carry their own masses.
constexpr uint32_t kHasMass = 1u << 31;

// Block table entry: instance index and first particle of the work-group.
struct Blk {
    int32_t inst;
    int32_t first;
};

// Chunk of at most kChunk consecutive block-table entries of one instance,
// the unit of the first level of the per-instance reduction.
constexpr int kChunk = 256;
struct Chunk {
    int32_t first;
    int32_t count;
};

// Arguments of one step, shared by all kernels of a precision.
template <typename real>
struct StepArgs {
    // caller state (structure of arrays)
    real *x, *y, *z, *vx, *vy, *vz;
    uint32_t* id;
    uint8_t* alive;
    // scratch
    const Inst<real>* inst;
    const Blk* blk;
    int32_t nblk;
    int32_t* rank;            // rank inside its c-bin
    int32_t* start;           // counts, then exclusive prefix (ncells + 1)
    real* rec;                // c-bin ordered records, 8 reals per particle
    real* mass;               // caller's per-particle masses, or null
    real* rmass;              // masses in record order (with mass only)
    real* rec2;               // records after the move, for a state in the caller's order; or null (no room)
    int32_t* src;             // caller's order only: caller index -> record (without rec2: record -> caller index)
    int32_t *best, *perm;     // random partners in FP32: rank in the c-bin; c-bin-local order -> record (see rp_best)
    unsigned long long* bkey; // record -> (ranking value bits, partner record) of its closest candidate
    uint32_t* ties;           // nonzero: some FP64 record is marked in coll (see Key)
    double* gpart;            // [nblk][kGPart]
    double* shift;            // per-o-bin velocity shift (3 per o-bin)
    int32_t order;            // search work-group order: 0 contiguous per XCD, S > 0 chunks of S round-robin
    ObAcc* macc;              // per-o-bin exact sums, or null (no moments)
    char* mexp;               // their exponents and counts, exp_stride bytes apart
    int exp_stride;
    real* vir;                // virial terms of each collider (3 per particle; record index, or caller index without rec2)
    uint8_t* coll;            // 1 if the particle collided this step (indexed as vir); FP64, until the move: marks
                              // of keys that met an equal one (record index, see Key)
    unsigned long long* mix;  // search mix counters (tests, s0 < 0, s0 < 0 < s1), or null
    // outputs
    uint32_t* pairs;
    int64_t pair_cap;
    unsigned long long* pair_count;
    double* moments;
};

// Launchers implemented per precision (tpkmc_f32.hip / tpkmc_f64.hip).
template <typename real> void launch_key(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_scatter(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_prep(Inst<real>* inst, const double* gpart, int n_inst, int max_nblk,
                                         hipStream_t s);
template <typename real> void launch_search(const StepArgs<real>& a, int block, int group, hipStream_t s);
template <typename real> void launch_search_tiles(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_search_ties(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_search_mix(const StepArgs<real>& a, int n_inst, bool split, hipStream_t s);
template <typename real> void launch_search_fast(const StepArgs<real>& a, int n_inst, hipStream_t s);
template <typename real> void launch_move(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_moments(const StepArgs<real>& a, bool caller_order, hipStream_t s);
template <typename real> void launch_random_pairs(const StepArgs<real>& a, hipStream_t s);
template <typename real> void launch_speed_stats(const StepArgs<real>& a, hipStream_t s);

}  // namespace tpkmc
