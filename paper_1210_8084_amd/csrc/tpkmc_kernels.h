// Device kernels of the collision step, templated on the precision of the
// particle state (float or double).  Included by tpkmc_f32.hip and
// tpkmc_f64.hip; the FP64 unit is compiled without FMA contraction so that
// every expression below rounds exactly like the plain C reference.
//
// Work layout.  Every per-particle kernel runs over a block table: each
// work-group owns kBlock consecutive particles of ONE instance, so a batch of
// independent instances is one launch and per-work-group partial sums belong
// to one instance.  Particles are bucketed by c-bin with a counting sort
// (key -> prefix -> scatter) into 8-real records; because the c-bin index is
// x-fastest, the three c-bins of one x-row of a neighbourhood are contiguous
// records, so the 27-cell neighbourhood is at most 9 (18 with a periodic
// x-seam) contiguous record ranges.
#pragma once

#include <type_traits>

#include "tpkmc_internal.h"

namespace tpkmc {

// ---------------------------------------------------------------- records
// Record layout: x y z id | vx vy vz flags (8 reals).  flags bit 0 = alive;
// after the move (StepArgs::rec2) one of the three words below.
constexpr uint32_t kRecDead = 0u, kRecAlive = 1u, kRecAbsorbed = 2u;
template <typename real> struct Rec;

template <> struct Rec<float> {
    // Position and velocity of record i through a 32-bit byte offset (the
    // host keeps 32 * records below 2^32).
    static __device__ __forceinline__ void load6(const float* r, uint32_t i, float& x, float& y, float& z,
                                                 float& vx, float& vy, float& vz) {
        const char* b = reinterpret_cast<const char*>(r) + i * 32u;
        const float4 a = *reinterpret_cast<const float4*>(b);
        const float4 c = *reinterpret_cast<const float4*>(b + 16);
        x = a.x; y = a.y; z = a.z; vx = c.x; vy = c.y; vz = c.z;
    }
    static __device__ __forceinline__ float from_u32(uint32_t v) { return __uint_as_float(v); }
    static __device__ __forceinline__ uint32_t to_u32(float v) { return __float_as_uint(v); }
    static __device__ __forceinline__ void store(float* r, int64_t i, float x, float y, float z, uint32_t id,
                                                 float vx, float vy, float vz, uint32_t fl) {
        float4* p = reinterpret_cast<float4*>(r + 8 * i);
        p[0] = make_float4(x, y, z, from_u32(id));
        p[1] = make_float4(vx, vy, vz, from_u32(fl));
    }
    static __device__ __forceinline__ void load(const float* r, int64_t i, float& x, float& y, float& z,
                                                uint32_t& id, float& vx, float& vy, float& vz, uint32_t& fl) {
        const float4* p = reinterpret_cast<const float4*>(r + 8 * i);
        float4 a = p[0], b = p[1];
        x = a.x; y = a.y; z = a.z; id = to_u32(a.w);
        vx = b.x; vy = b.y; vz = b.z; fl = to_u32(b.w);
    }
};

template <> struct Rec<double> {
    static __device__ __forceinline__ double from_u32(uint32_t v) { return __longlong_as_double((long long)v); }
    static __device__ __forceinline__ uint32_t to_u32(double v) { return (uint32_t)__double_as_longlong(v); }
    static __device__ __forceinline__ void store(double* r, int64_t i, double x, double y, double z, uint32_t id,
                                                 double vx, double vy, double vz, uint32_t fl) {
        double2* p = reinterpret_cast<double2*>(r + 8 * i);
        p[0] = make_double2(x, y);
        p[1] = make_double2(z, from_u32(id));
        p[2] = make_double2(vx, vy);
        p[3] = make_double2(vz, from_u32(fl));
    }
    static __device__ __forceinline__ void load(const double* r, int64_t i, double& x, double& y, double& z,
                                                uint32_t& id, double& vx, double& vy, double& vz, uint32_t& fl) {
        const double2* p = reinterpret_cast<const double2*>(r + 8 * i);
        double2 a = p[0], b = p[1], c = p[2], d = p[3];
        x = a.x; y = a.y; z = b.x; id = to_u32(b.y);
        vx = c.x; vy = c.y; vz = d.x; fl = to_u32(d.y);
    }
};

// Position and velocity of record i.
__device__ __forceinline__ void load_pv(const float* r, int32_t i, float& x, float& y, float& z, float& vx, float& vy,
                                        float& vz) {
    Rec<float>::load6(r, (uint32_t)i, x, y, z, vx, vy, vz);
}
__device__ __forceinline__ void load_pv(const double* r, int32_t i, double& x, double& y, double& z, double& vx,
                                        double& vy, double& vz) {
    uint32_t id, fl;
    Rec<double>::load(r, i, x, y, z, id, vx, vy, vz, fl);
}

// A record as it was loaded, in whole vectors: a value carried round a loop
// in them is not copied (and so waited for) before it is used.
template <typename real> struct RawRec;

template <> struct RawRec<float> {
    typedef float vec __attribute__((ext_vector_type(4)));
    vec a, b;
    __device__ __forceinline__ void load(const float* r, int32_t i) {
        const char* p = reinterpret_cast<const char*>(r) + (uint32_t)i * 32u;
        a = *reinterpret_cast<const vec*>(p);
        b = *reinterpret_cast<const vec*>(p + 16);
    }
    __device__ __forceinline__ void get(float p[3], float v[3]) {
        asm volatile("" : "+v"(a), "+v"(b));  // keeps the vectors whole
        p[0] = a.x; p[1] = a.y; p[2] = a.z;
        v[0] = b.x; v[1] = b.y; v[2] = b.z;
    }
};

template <> struct RawRec<double> {
    typedef double vec __attribute__((ext_vector_type(2)));
    vec a, b, c, d;
    __device__ __forceinline__ void load(const double* r, int32_t i) {
        const vec* p = reinterpret_cast<const vec*>(r + 8 * (int64_t)i);
        a = p[0]; b = p[1]; c = p[2]; d = p[3];
    }
    __device__ __forceinline__ void get(double p[3], double v[3]) {
        asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
        p[0] = a.x; p[1] = a.y; p[2] = b.x;
        v[0] = c.x; v[1] = c.y; v[2] = d.x;
    }
};

// ---------------------------------------------------------------- helpers
// Bin along one axis: floor((x - lo) * n / L) clamped into [0, n - 1].
template <typename real>
__device__ __forceinline__ int axis_bin(real x, real lo, real inv_w, int n) {
    real t = (x - lo) * inv_w;
    if (!(t >= real(0))) return 0;
    if (t >= real(n)) return n - 1;
    return (int)t;
}

// Sort cell of a coordinate along axis ax: its c-bin (refined for the slow
// particles of split c-bins), cut into 2^kl equal parts where the instance has
// sub-grids.  The c-bin is axis_bin's own, so a sub-grid never moves a
// particle to another c-bin.  Every operation rounds (no contraction), so
// that the kernels that work it out agree to the last bit.
template <typename real>
__device__ __forceinline__ int sort_bin(const Inst<real>& I, int ax, real x) {
#pragma clang fp contract(off)
    const int c = axis_bin(x, I.lo[ax], I.inv_wl[ax], I.nl[ax]);
    const int k = 1 << I.kl[ax];
    if (k == 1) return c;
    const real f = ((x - I.lo[ax]) * I.inv_wl[ax] - (real)c) * (real)k;
    return c * k + (f >= real(1) ? min((int)fmin(f, (real)k), k - 1) : 0);
}

// Row (y, z) of c-bins as its index in the c-bin order, in units of rows
// (the c-bin index is x + n_x * row).  The order is band-major: the y axis is
// cut into bands of 2^band_log2 rows, and within a band the rows run z-major.
// A sweep over consecutive c-bins (one XCD's share of the work-groups) thus
// stays inside one band while it walks through the planes.  The records of the
// next plane, which the neighbourhood walk reads again one plane later, are
// then a band plane away instead of a whole plane.  With one band this is the
// plain y + n_y z.
template <typename real>
__device__ __forceinline__ int row_of(const Inst<real>& I, int y, int z) {
    const int h = I.band_log2;
    const int y0 = (y >> h) << h;                 // first row of y's band
    const int rows = min(1 << h, I.n[1] - y0);    // rows in that band
    return y0 * I.n[2] + (y - y0) + rows * z;
}

template <typename real>
__device__ __forceinline__ bool finite3(real a, real b, real c) {
    return isfinite(a) && isfinite(b) && isfinite(c);
}

__device__ __forceinline__ uint64_t lanes_le(int lane) {
    return lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
}

// Cross-lane moves of a double through the VALU's data-parallel primitives
// (DPP) instead of the LDS permute unit; every lane of the wave must be
// active.  Quad permutations: lane q of each group of four reads lane P[q]
// of its group, encoded P[0] | P[1] << 2 | P[2] << 4 | P[3] << 6.  Row
// shifts (0x100 + n): lane r of each row of 16 lanes reads lane r + n of
// the row (lanes past the row's end read nothing defined and must not use
// the value).  Row rotations (0x120 + n) rotate each row by n.
constexpr int kQuadXor1 = 1 | 0 << 2 | 3 << 4 | 2 << 6;
constexpr int kQuadXor2 = 2 | 3 << 2 | 0 << 4 | 1 << 6;
constexpr int kRowShl1 = 0x101;
constexpr int kRowShl2 = 0x102;
constexpr int kRowShl4 = 0x104;
constexpr int kRowShl8 = 0x108;
constexpr int kRowRor4 = 0x124;
constexpr int kRowRor8 = 0x128;

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum (or maximum) of a double over the 64 lanes, in a fixed order: pairs,
// quads and rows through DPP, then the four row totals.  Every lane must be
// active; the result is returned in every lane.
template <bool MAX>
__device__ __forceinline__ double wave_reduce(double v) {
    auto op = [](double x, double y) { return MAX ? fmax(x, y) : x + y; };
    v = op(v, dpp_move<kQuadXor1>(v));
    v = op(v, dpp_move<kQuadXor2>(v));
    v = op(v, dpp_move<kRowRor4>(v));
    v = op(v, dpp_move<kRowRor8>(v));
    return op(op(lane_value(v, 0), lane_value(v, 16)), op(lane_value(v, 32), lane_value(v, 48)));
}

template <int CTRL>
__device__ __forceinline__ float dpp_movef(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum (or maximum) of a float over the 64 lanes, as wave_reduce.
template <bool MAX>
__device__ __forceinline__ float wave_reducef(float v) {
    auto op = [](float x, float y) { return MAX ? fmaxf(x, y) : x + y; };
    v = op(v, dpp_movef<kQuadXor1>(v));
    v = op(v, dpp_movef<kQuadXor2>(v));
    v = op(v, dpp_movef<kRowRor4>(v));
    v = op(v, dpp_movef<kRowRor8>(v));
    auto at = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    return op(op(at(0), at(16)), op(at(32), at(48)));
}

// Sum of a double over the work-group (blockDim.x <= 1024), result in all threads.
__device__ __forceinline__ double block_sum(double v, double* lds) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int k = 0; k < nw; ++k) t += lds[k];
    return t;
}

// Work-groups are dispatched round-robin over the 8 XCDs; remap so that each
// XCD (own L2) receives a contiguous range of the table, where neighbouring
// work-groups share neighbour c-bins.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int nx = 8;
    const int xcd = bid % nx, local = bid / nx;
    const int per = nb / nx, rem = nb % nx;
    return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// The other order: chunks of S consecutive work-groups dealt round-robin over
// the XCDs (S = 1 keeps the dispatch order).  Contiguous ranges keep what
// neighbouring work-groups share in one L2, but when the work per
// work-group varies along the table (a batch of instances of different
// densities) they leave some XCDs with much more work than others; chunks
// trade some of that locality for balance.  Full rounds of 8 S work-groups
// are permuted; the last, partial round keeps the dispatch order.
__device__ __forceinline__ int xcd_chunk_remap(int bid, int nb, int S) {
    const int round = 8 * S;
    const int r = bid / round, m = bid - r * round;
    if ((r + 1) * round > nb) return bid;
    return r * round + (m & 7) * S + (m >> 3);
}

// ---------------------------------------------------------------- Philox
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
        const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Isotropic unit vector of the pair (idA < idB) from a point (x1, x2) drawn
// uniformly in the unit disk by rejection, two 53-bit uniforms per Philox
// draw (at most 255 draws: the counter ending in 255 is kept for the random
// partners' draws); computed in double in both precisions.  In space: Marsaglia's map
// (2 x1 q, 2 x2 q, 1 - 2 s), q = sqrt(1 - s).  In the plane: the doubled
// angle ((x1^2 - x2^2) / s, 2 x1 x2 / s, 0), which needs s > 0.
__device__ __forceinline__ void pair_direction(uint32_t k0, uint32_t k1, uint32_t step, uint32_t instance,
                                               uint32_t idA, uint32_t idB, bool planar, double n[3]) {
    for (uint32_t attempt = 0; attempt < 255u; ++attempt) {
        uint32_t c[4] = {step, idA, idB, (instance << 8) | attempt};
        philox4x32_10(c, k0, k1);
        const double u1 = ((double)(c[0] >> 5) * 67108864.0 + (double)(c[1] >> 6)) * (1.0 / 9007199254740992.0);
        const double u2 = ((double)(c[2] >> 5) * 67108864.0 + (double)(c[3] >> 6)) * (1.0 / 9007199254740992.0);
        const double x1 = 2.0 * u1 - 1.0;
        const double x2 = 2.0 * u2 - 1.0;
        const double s = x1 * x1 + x2 * x2;
        if (planar) {
            if (s < 1.0 && s > 0.0) {
                n[0] = (x1 * x1 - x2 * x2) / s;
                n[1] = (2.0 * x1 * x2) / s;
                n[2] = 0.0;
                return;
            }
        } else if (s < 1.0) {
            const double q = sqrt(1.0 - s);
            n[0] = (2.0 * x1) * q;
            n[1] = (2.0 * x2) * q;
            n[2] = 1.0 - 2.0 * s;
            return;
        }
    }
    n[0] = planar ? 1.0 : 0.0; n[1] = 0.0; n[2] = planar ? 0.0 : 1.0;
}

// |v|^2 in double, summed in axis order with every product rounded (the
// order the time-step rule and the global maximum are defined in).
__device__ __forceinline__ double speed2(double vx, double vy, double vz) {
#pragma clang fp contract(off)
    return (vx * vx + vy * vy) + vz * vz;
}

// ---------------------------------------------------------------- 1. key
// |v|^2 in the state's precision with fixed fused operations, so that the key
// and scatter kernels class a particle as slow or fast alike.
template <typename real>
__device__ __forceinline__ real speed2_r(real vx, real vy, real vz) {
    return fma(vz, vz, fma(vy, vy, vx * vx));
}

// c-bin key of caller-order particle p: its c-bin, or the instance's trailing
// bin for a dead or non-finite particle.  With split c-bins a fast particle
// (|v|^2 above the instance's bound) takes its configured c-bin, numbered
// after the slow particles' refined ones.  The key and scatter kernels both
// evaluate it on the same loaded values, so the key is never stored.
template <typename real>
__device__ __forceinline__ int cbin_key(const StepArgs<real>& a, const Inst<real>& I, int64_t p, real x, real y,
                                        real z, real vx, real vy, real vz, bool alive, bool& fin) {
    fin = finite3(x, y, z) && finite3(vx, vy, vz);
    if (a.mass) {
        const real m = a.mass[p];
        fin = fin && m > real(0) && m < real(INFINITY);
    }
    if (!(alive && fin)) return (int)(I.cell_off + I.C);
    if ((I.flags & kSplit) && !(speed2_r(vx, vy, vz) <= I.vc2)) {
        const int cx = axis_bin(x, I.lo[0], I.inv_wc[0], I.ncfg[0]);
        const int cy = axis_bin(y, I.lo[1], I.inv_wc[1], I.ncfg[1]);
        const int cz = axis_bin(z, I.lo[2], I.inv_wc[2], I.ncfg[2]);
        return (int)I.cell_off + I.Cf + cx + I.ncfg[0] * (cy + I.ncfg[1] * cz);
    }
    return (int)I.cell_off + sort_bin(I, 0, x) + I.n[0] * row_of(I, sort_bin(I, 1, y), sort_bin(I, 2, z));
}

// The key kernel runs one wave per block-table entry, each lane taking
// kKeyRec particles kWave apart, so that every lane has all its loads, and
// then all its atomics, in flight at once.  With dense c-bins (long runs,
// few atomics) the kernel is otherwise bound by the latency of those two
// dependent steps: measured 1.07 -> 0.50 ms on the 4M-particle Sod tube and
// 0.18 -> 0.10 ms on the 8M Noh implosion; the sparse 16M Sedov blast, bound
// by the throughput of its one atomic per c-bin, is unchanged.  The same
// layout made the scatter kernel slower on the Sedov blast (0.226 -> 0.247 ms),
// so that one keeps a particle per lane.
constexpr int kKeyRec = kBlock / kWave;

// c-bin count of every caller-order particle and its rank inside the c-bin.
// Consecutive particles of the same c-bin (the common case for sorted input)
// take one atomic for the whole run, also across the wave's rounds.
template <typename real>
__global__ void __launch_bounds__(kWave) k_key(StepArgs<real> a) {
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    const int lane = threadIdx.x;
    const int64_t end = I.off + I.cnt;
    const bool want_v2 = (I.flags & (TPKMC_ADAPTIVE_DT | kSplit | kSubgrid)) != 0;
    float out = 0.0f;  // how far a particle lies outside the box along a periodic axis, in units of 1 / tile_s
    real x[kKeyRec], y[kKeyRec], z[kKeyRec], vx[kKeyRec], vy[kKeyRec], vz[kKeyRec];
    bool alive[kKeyRec];
#pragma unroll
    for (int r = 0; r < kKeyRec; ++r) {
        const int64_t p = (int64_t)bt.first + r * kWave + lane;
        x[r] = y[r] = z[r] = vx[r] = vy[r] = vz[r] = real(0);
        alive[r] = false;
        if (p < end) {
            alive[r] = a.alive ? a.alive[p] != 0 : true;
            x[r] = a.x[p]; y[r] = a.y[p]; z[r] = a.z[p];
            vx[r] = a.vx[p]; vy[r] = a.vy[p]; vz[r] = a.vz[p];
        }
    }
    // The wave's kKeyRec * 64 particles in caller order, q = r * 64 + lane,
    // fall into runs of one c-bin (in c-bin order after the first step, one
    // run per c-bin and wave); a run may span rounds.  Its first particle
    // takes one atomic for the whole run.
    int key[kKeyRec], base[kKeyRec];
    uint64_t heads[kKeyRec];
    double nonfin = 0.0, v2 = 0.0;
    int carry = -1;  // key of the previous round's last lane (keys are >= 0)
#pragma unroll
    for (int r = 0; r < kKeyRec; ++r) {
        const int64_t p = (int64_t)bt.first + r * kWave + lane;
        const bool in = p < end;
        bool fin = true;
        key[r] = in ? cbin_key(a, I, p, x[r], y[r], z[r], vx[r], vy[r], vz[r], alive[r], fin) : 0;
        if (in && alive[r] && fin) {
            if (want_v2) {
                v2 = fmax(v2, speed2((double)vx[r], (double)vy[r], (double)vz[r]));
                const real q[3] = {x[r], y[r], z[r]};
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    const real d = fmax(I.lo[ax] - q[ax], q[ax] - I.hi[ax]);
                    if (I.bc[ax] == TPKMC_BC_PERIODIC && d > real(0) && !(ax == 2 && (I.flags & TPKMC_PLANAR)))
                        out = d > real(0.2) * I.L[ax] ? INFINITY : fmaxf(out, (float)(d * (real)I.tile_s));
                }
            }
        } else if (in) {
            nonfin += (alive[r] && !fin) ? 1.0 : 0.0;
        }
        int prev = __shfl_up(key[r], 1);
        if (lane == 0) prev = carry;
        heads[r] = __ballot(in && prev != key[r]);
        carry = __builtin_amdgcn_readlane(key[r], kWave - 1);
    }
    const int nvalid = (int)min<int64_t>(end - (int64_t)bt.first, (int64_t)kKeyRec * kWave);
    int hq[kKeyRec];  // linear index of the run head of each of the lane's particles
#pragma unroll
    for (int r = 0; r < kKeyRec; ++r) {
        const int q = r * kWave + lane;
        const uint64_t below = heads[r] & lanes_le(lane);
        int h = below ? r * kWave + 63 - __clzll((long long)below) : 0;
        if (!below)
            for (int rr = r - 1; rr >= 0; --rr)
                if (heads[rr]) { h = rr * kWave + 63 - __clzll((long long)heads[rr]); break; }
        hq[r] = h;
        base[r] = 0;
        if (q < nvalid && h == q) {
            const uint64_t above = heads[r] & ~lanes_le(lane);
            int nq = above ? r * kWave + __ffsll((long long)above) - 1 : nvalid;
            if (!above)
                for (int rr = r + 1; rr < kKeyRec; ++rr)
                    if (heads[rr]) { nq = min(nvalid, rr * kWave + __ffsll((long long)heads[rr]) - 1); break; }
            base[r] = atomicAdd(&a.start[key[r]], nq - q);
        }
    }
#pragma unroll
    for (int r = 0; r < kKeyRec; ++r) {
        const int q = r * kWave + lane;
        const int hr = hq[r] / kWave, hl = hq[r] % kWave;
        int b = 0;
#pragma unroll
        for (int rr = 0; rr <= r; ++rr) {
            const int t = __shfl(base[rr], hl);
            if (rr == hr) b = t;
        }
        if (q < nvalid) a.rank[(int64_t)bt.first + q] = b + (q - hq[r]);
    }
    nonfin = wave_reduce<false>(nonfin);
    v2 = wave_reduce<true>(v2);
    if (__ballot(out > 0.0f)) out = wave_reducef<true>(out);  // wave-uniform
    if (lane == 0) {
        double* gp = a.gpart + (int64_t)blockIdx.x * kGPart;
        gp[GP_NONFINITE] = nonfin;
        gp[GP_VMAX0] = v2;
        gp[GP_PX] = (double)out;  // for k_prep; the move writes its own sum there later
        gp[GP_FAST] = 0.0;  // counted by the scatter kernel, once dt is known
        // The search kernel may accumulate into these with atomics.
        gp[GP_TESTS2] = 0.0;
        gp[GP_CAND] = 0.0;
    }
}

// Neighbour index along one axis (offset d in -1..1): whether it exists and
// is not a repeat of another offset (periodic axes with 1 or 2 bins), and the
// wrapped index.
__device__ __forceinline__ bool axis_nb(int c, int d, int n, bool periodic, int& out) {
    int v = c + d;
    if (periodic) {
        if (n == 1 && d != 0) return false;
        if (n == 2 && d == 1) return false;
        v = v < 0 ? v + n : (v >= n ? v - n : v);
    } else if (v < 0 || v >= n) {
        return false;
    }
    out = v;
    return true;
}

// x-extent of the neighbourhood as at most two contiguous bin ranges; the
// first always contains cx.
__device__ __forceinline__ int x_ranges(int cx, int n, bool periodic, int xa[2], int xb[2]) {
    if (periodic && n > 3 && cx == 0) { xa[0] = 0; xb[0] = 1; xa[1] = n - 1; xb[1] = n - 1; return 2; }
    if (periodic && n > 3 && cx == n - 1) { xa[0] = n - 2; xb[0] = n - 1; xa[1] = 0; xb[1] = 0; return 2; }
    if (periodic && n <= 3) { xa[0] = 0; xb[0] = n - 1; return 1; }
    xa[0] = cx > 0 ? cx - 1 : 0;
    xb[0] = cx < n - 1 ? cx + 1 : n - 1;
    return 1;
}

// The unordered pairs of c-bin c with itself and with its neighbours, each
// pair of c-bins once (the search's TPKMC_CNT_TESTS), from the sort cells'
// prefix.  Where a c-bin spans many rows of sort cells (`shared`), the 64
// lanes of a wave share them (c is then the same in all of them), else each
// lane takes a c-bin of its own.  Returns the lane's (the wave's) count.
template <typename real>
__device__ double cbin_tests(const StepArgs<real>& a, const Inst<real>& I, int c, int lane, bool shared) {
    const int nl[3] = {I.nl[0], I.nl[1], I.nl[2]}, k[3] = {1 << I.kl[0], 1 << I.kl[1], 1 << I.kl[2]};
    const int x = c % nl[0], y = c / nl[0] % nl[1], z = c / nl[0] / nl[1], nf = k[1] * k[2];
    int xa[2], xb[2];
    const int nxr = x_ranges(x, nl[0], I.bc[0] == TPKMC_BC_PERIODIC, xa, xb);
    double own = 0.0, other = 0.0;
    for (int t = shared ? lane : 0; t < 9 * nf; t += shared ? kWave : 1) {
        const int r = t >> (I.kl[1] + I.kl[2]), f = t & (nf - 1);
        int yy, zz;
        if (!axis_nb(z, r / 3 - 1, nl[2], I.bc[2] == TPKMC_BC_PERIODIC, zz)) continue;
        if (!axis_nb(y, r % 3 - 1, nl[1], I.bc[1] == TPKMC_BC_PERIODIC, yy)) continue;
        const int d = (yy + nl[1] * zz) - (y + nl[1] * z);
        if (d < 0) continue;  // counted from there
        const int32_t* row = a.start + I.cell_off +
                             (int64_t)I.n[0] * row_of(I, yy * k[1] + (f & (k[1] - 1)), zz * k[2] + (f >> I.kl[1]));
        auto records = [&](int c0, int c1) { return (double)(row[(int64_t)(c1 + 1) * k[0]] - row[(int64_t)c0 * k[0]]); };
        if (d == 0) own += records(x, x);
        for (int q = 0; q < nxr; ++q) {
            const int a0 = d > 0 ? xa[q] : max(xa[q], x + 1);
            if (a0 <= xb[q]) other += records(a0, xb[q]);
        }
    }
    if (shared) {
        own = wave_reduce<false>(own);
        other = wave_reduce<false>(other);
    }
    return own * (0.5 * (own - 1.0) + other);
}

// ---------------------------------------------------------------- 3. scatter
// Caller-order particle -> its c-bin-ordered record.  The permutation back to
// the caller's order is kept only when the state is written back in that
// order (without TPKMC_ALLOW_REORDER).  The work-groups of a tile search's
// instance also share the count of its pair tests: here other waves hide its
// loads (in the search, with 3 waves a SIMD, it cost 0.03 ms of the FP64
// blast's 0.4).
template <typename real>
__global__ void __launch_bounds__(kBlock) k_scatter(StepArgs<real> a) {
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    const int64_t p = (int64_t)bt.first + threadIdx.x;
    bool fast = false;
    if (p < I.off + I.cnt) {
        const int64_t base = I.base;
        const bool alive = a.alive ? a.alive[p] != 0 : true;
        const real x = a.x[p], y = a.y[p], z = a.z[p], vx = a.vx[p], vy = a.vy[p], vz = a.vz[p];
        bool fin;
        const int k = cbin_key(a, I, p, x, y, z, vx, vy, vz, alive, fin);
        const int64_t dst = base + a.start[k] + a.rank[p];
        const uint32_t fl = alive ? 1u : 0u;
        Rec<real>::store(a.rec, dst, x, y, z, a.id[p], vx, vy, vz, fl);
        if (!(I.flags & TPKMC_ALLOW_REORDER)) {
            if (a.rec2) a.src[p] = (int32_t)dst;
            else a.src[dst] = (int32_t)p;
        }
        // Every record of the instance starts without a partner; which of
        // them this thread clears is free, so the stores are consecutive.
        a.bkey[p] = ~0ull;
        if constexpr (std::is_same<real, double>::value) a.coll[p] = 0;  // marks of k_search_ties
        if (a.mass) a.rmass[dst] = a.mass[p];
        // Diagnostic: a particle faster than one c-bin per step on some axis.
        const real dt = I.dt;
        fast = alive && fin &&
               (fabs(vx) * dt > I.w[0] || fabs(vy) * dt > I.w[1] || fabs(vz) * dt > I.w[2]);
    }
    if (I.flags & kTiles) {
        const int64_t ncb = (int64_t)I.nl[0] * I.nl[1] * I.nl[2];
        // Four rows a c-bin and fewer go lane by lane: 2e6 particles at 32 to
        // 64 per c-bin, two or four rows each, take 32 us so and 41 to 49
        // shared; with eight rows (at 64 to 512) 32 to 65, and 33 shared.
        // (At 1e5 sharing pays from two rows on: 11 us instead of 17.)
        const bool shared = I.kl[1] + I.kl[2] > 2;
        const int lane = threadIdx.x & (kWave - 1);
        const int64_t me = (int64_t)((int)blockIdx.x - I.blk0) * kBlock + threadIdx.x, all = (int64_t)I.nblk * kBlock;
        double tests = 0.0;
        if (shared) {
            for (int64_t c = me / kWave; c < ncb; c += all / kWave) {
                const double t = cbin_tests(a, I, __builtin_amdgcn_readfirstlane((int)c), lane, true);
                tests += lane == 0 ? t : 0.0;
            }
        } else {
            for (int64_t c = me; c < ncb; c += all) tests += cbin_tests(a, I, (int)c, lane, false);
        }
        if (__ballot(tests != 0.0)) {
            tests = wave_reduce<false>(tests);
            if (lane == 0) unsafeAtomicAdd(a.gpart + (int64_t)blockIdx.x * kGPart + GP_TESTS2, 2.0 * tests);
        }
    }
    const uint64_t fm = __ballot(fast);
    if (fm && (threadIdx.x & 63) == __ffsll((long long)fm) - 1)
        atomicAdd(a.gpart + (int64_t)blockIdx.x * kGPart + GP_FAST, (double)__popcll(fm));
}

// ---------------------------------------------------------------- 4. search
// Per-instance constants of the pair test, held in registers.
template <typename real>
struct Geo {
    real L[3], halfL[3], invL[3];
    real dt, D2;
    bool per[3];
    __device__ __forceinline__ explicit Geo(const Inst<real>& I) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            L[a] = I.L[a];
            halfL[a] = real(0.5) * I.L[a];
            invL[a] = real(1) / I.L[a];
            per[a] = I.bc[a] == TPKMC_BC_PERIODIC;
        }
        dt = I.dt;
        D2 = I.D2;
    }
};

// Minimum image on a periodic axis, written as selects (same value as the
// reference's if / else-if).
template <typename real>
__device__ __forceinline__ real min_image(real r, real L, real halfL) {
    const real up = r - L, dn = r + L;
    return r > halfL ? up : (r < -halfL ? dn : r);
}

// The three criteria for the ordered pair (i, j): chi < 0 within the step
// (s0 = r.u < 0 < s1 = r.u + |u|^2 dt), then d_min^2 <= D^2.  Returns d_min^2,
// or -1 when j is not a candidate.  j == i (or an exact twin) has r.u = 0 and
// is rejected by the first criterion.
//
// Most pairs fail, and a branch taken by any lane of a wave costs the whole
// wave, so the rejection is decided without branches and without a division:
// d_min^2 |u|^2 = |r x u|^2, hence d_min^2 <= D^2  <=>  |r x u|^2 <= D^2 |u|^2.
//  - FP32: that form decides; d_min^2 = |r x u|^2 / |u|^2 only for candidates.
//  - FP64: that form, with FMAs and a margin far above the rounding of either
//    form, only discards pairs that are certainly not candidates; the rest go
//    through the reference's own expressions (t_poca = -s0/|u|^2, PoCA
//    separation r + t_poca u), so decisions and d_min^2 are bit-identical.
// Two-stage screening, both stages without divergent branches:
//  stage 1, criterion 1 (s0 < 0 < s1), on every pair;
//  stage 2, |r x u|^2 <= D^2 |u|^2, only when some lane of the wave passed
//  stage 1 (a wave-uniform branch, so cold regions where no pair of the wave
//  meets within the step skip it).
template <typename real> struct Screen {
    real rx, ry, rz, ux, uy, uz, s0, vv;
};

// PM: the periodic axes as a mask known at compile time (bit a for axis a;
// FP32 alone), or -1 to read them from the instance at run time.
template <typename real, int PM> struct PairTest;

template <int PM> struct PairTest<float, PM> {
    static __device__ __forceinline__ bool stage1(const Geo<float>& G, float xi, float yi, float zi, float vxi,
                                                  float vyi, float vzi, float xj, float yj, float zj, float vxj,
                                                  float vyj, float vzj, Screen<float>& S) {
        float rx = xi - xj, ry = yi - yj, rz = zi - zj;
        // Nearest image: r - L rint(r / L) (ties at exactly L/2 keep r).
        if constexpr (PM < 0) {
            if (G.per[0]) rx = fmaf(-G.L[0], rintf(rx * G.invL[0]), rx);
            if (G.per[1]) ry = fmaf(-G.L[1], rintf(ry * G.invL[1]), ry);
            if (G.per[2]) rz = fmaf(-G.L[2], rintf(rz * G.invL[2]), rz);
        } else {
            if constexpr ((PM & 1) != 0) rx = fmaf(-G.L[0], rintf(rx * G.invL[0]), rx);
            if constexpr ((PM & 2) != 0) ry = fmaf(-G.L[1], rintf(ry * G.invL[1]), ry);
            if constexpr ((PM & 4) != 0) rz = fmaf(-G.L[2], rintf(rz * G.invL[2]), rz);
        }
        const float ux = vxi - vxj, uy = vyi - vyj, uz = vzi - vzj;
        const float s0 = fmaf(rz, uz, fmaf(ry, uy, rx * ux));
        const float vv = fmaf(uz, uz, fmaf(uy, uy, ux * ux));
        const float s1 = fmaf(vv, G.dt, s0);
        S.rx = rx; S.ry = ry; S.rz = rz; S.ux = ux; S.uy = uy; S.uz = uz; S.s0 = s0; S.vv = vv;
        return (s0 < 0.0f) & (s1 > 0.0f);
    }
    static __device__ __forceinline__ bool stage2(const Geo<float>& G, const Screen<float>& S) {
        const float cx = fmaf(S.ry, S.uz, -S.rz * S.uy);
        const float cy = fmaf(S.rz, S.ux, -S.rx * S.uz);
        const float cz = fmaf(S.rx, S.uy, -S.ry * S.ux);
        const float c2 = fmaf(cz, cz, fmaf(cy, cy, cx * cx));
        return c2 <= G.D2 * S.vv;
    }
    // d_min^2 of a pair that passed both stages (always a candidate in FP32).
    static __device__ __forceinline__ float finish(const Geo<float>&, const Screen<float>& S) {
        const float cx = fmaf(S.ry, S.uz, -S.rz * S.uy);
        const float cy = fmaf(S.rz, S.ux, -S.rx * S.uz);
        const float cz = fmaf(S.rx, S.uy, -S.ry * S.ux);
        return fmaf(cz, cz, fmaf(cy, cy, cx * cx)) / S.vv;
    }
    // First contact of the effective radii: the earlier root of
    // |u|^2 t^2 + 2 (u.r) t + |r|^2 - D^2 = 0 (a rounding below zero of the
    // discriminant is taken as 0).
    static __device__ __forceinline__ float contact(const Geo<float>& G, const Screen<float>& S) {
        const float rr = fmaf(S.rz, S.rz, fmaf(S.ry, S.ry, S.rx * S.rx));
        float disc = fmaf(S.s0, S.s0, -S.vv * (rr - G.D2));
        disc = disc > 0.0f ? disc : 0.0f;
        return (-S.s0 - sqrtf(disc)) / S.vv;
    }
};

template <> struct PairTest<double, -1> {
    static __device__ __forceinline__ bool stage1(const Geo<double>& G, double xi, double yi, double zi, double vxi,
                                                  double vyi, double vzi, double xj, double yj, double zj, double vxj,
                                                  double vyj, double vzj, Screen<double>& S) {
        double rx = xi - xj, ry = yi - yj, rz = zi - zj;
        if (G.per[0]) rx = min_image(rx, G.L[0], G.halfL[0]);
        if (G.per[1]) ry = min_image(ry, G.L[1], G.halfL[1]);
        if (G.per[2]) rz = min_image(rz, G.L[2], G.halfL[2]);
        const double ux = vxi - vxj, uy = vyi - vyj, uz = vzi - vzj;
        // Exactly the reference's s0 and s1 (no contraction in this unit).
        const double s0 = (rx * ux + ry * uy) + rz * uz;
        const double vv = (ux * ux + uy * uy) + uz * uz;
        const double s1 = s0 + vv * G.dt;
        S.rx = rx; S.ry = ry; S.rz = rz; S.ux = ux; S.uy = uy; S.uz = uz; S.s0 = s0; S.vv = vv;
        return (s0 < 0.0) & (s1 > 0.0);
    }
    // Conservative: |r x u|^2 <= D^2 |u|^2 with a margin far above the
    // rounding of either form, so no pair the reference accepts is lost.
    static __device__ __forceinline__ bool stage2(const Geo<double>& G, const Screen<double>& S) {
        const double cx = fma(S.ry, S.uz, -S.rz * S.uy);
        const double cy = fma(S.rz, S.ux, -S.rx * S.uz);
        const double cz = fma(S.rx, S.uy, -S.ry * S.ux);
        const double c2 = fma(cz, cz, fma(cy, cy, cx * cx));
        const double rr = fma(S.rz, S.rz, fma(S.ry, S.ry, S.rx * S.rx));
        return c2 <= fma(G.D2 * S.vv, 1.0 + 1e-6, 1e-12 * rr * S.vv);
    }
    // The reference's expressions; -1 when the exact d_min^2 exceeds D^2.
    static __device__ __forceinline__ double finish(const Geo<double>& G, const Screen<double>& S) {
        const double tp = -S.s0 / S.vv;
        const double px = S.rx + tp * S.ux, py = S.ry + tp * S.uy, pz = S.rz + tp * S.uz;
        const double d2 = (px * px + py * py) + pz * pz;
        return d2 <= G.D2 ? d2 : -1.0;
    }
    // First contact time, with the reference's expression and order.
    static __device__ __forceinline__ double contact(const Geo<double>& G, const Screen<double>& S) {
        const double rr = (S.rx * S.rx + S.ry * S.ry) + S.rz * S.rz;
        double disc = S.s0 * S.s0 - S.vv * (rr - G.D2);
        if (!(disc > 0.0)) disc = 0.0;
        return (-S.s0 - sqrt(disc)) / S.vv;
    }
};

// Order-preserving map of a float onto uint32 (negative values included).
__device__ __forceinline__ uint32_t sortable(float v) {
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ unsigned long long sortable(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// The search's result per record is one 64-bit key, the ranking value of
// criterion 3 above the partner record, lowered by atomicMin in any order
// (~0: no candidate).  FP32: all 32 bits of the value, partner in the low
// 32; exact ties go to the lower record.  FP64: the top 33 bits of the value
// and 31 bits of partner.  Values that agree in those 33 bits are not told
// apart by the key, so a record that meets two of them while one is its
// lowest is marked, and k_search_ties settles it with the full values and
// the tie rule of the reference (lower id); about one record in 10^6 is.  The
// mark is one of eight bits, taken from the value, so that most records whose
// lowest value was another in the end are left alone.
template <typename real> struct Key;

template <> struct Key<float> {
    static __device__ __forceinline__ unsigned long long make(float v, uint32_t j) {
        return (unsigned long long)sortable(v) << 32 | j;
    }
    static __device__ __forceinline__ int32_t partner(unsigned long long k) { return (int32_t)(uint32_t)k; }
    static __device__ __forceinline__ void tied(const StepArgs<float>&, int64_t, unsigned long long,
                                                unsigned long long) {}
    // old: the key as read earlier (it only falls, so a key found below k
    // need not be touched).
    static __device__ __forceinline__ void lower(const StepArgs<float>& a, int64_t i, unsigned long long k,
                                                 unsigned long long old) {
        if (old > k) atomicMin(a.bkey + i, k);
    }
};

template <> struct Key<double> {
    static constexpr int kPartnerBits = 31;
    static __device__ __forceinline__ unsigned long long make(double v, uint32_t j) {
        return (sortable(v) >> kPartnerBits << kPartnerBits) | j;
    }
    static __device__ __forceinline__ int32_t partner(unsigned long long k) { return (int32_t)(k & 0x7fffffffull); }
    static __device__ __forceinline__ uint32_t mark(unsigned long long k) {
        return 1u << ((uint32_t)(k >> kPartnerBits) * 0x9E3779B1u >> 29);
    }
    static __device__ __forceinline__ void tied(const StepArgs<double>& a, int64_t i, unsigned long long old,
                                                unsigned long long k) {
        if (((old ^ k) >> kPartnerBits) == 0 && old != k) {
            // The byte's word (the array is aligned, and padded to words).
            atomicOr(reinterpret_cast<uint32_t*>(a.coll) + (i >> 2), mark(k) << (8 * (int)(i & 3)));
            *a.ties = 1u;
        }
    }
    static __device__ __forceinline__ void lower(const StepArgs<double>& a, int64_t i, unsigned long long k,
                                                 unsigned long long old) {
        if (old > k) old = atomicMin(a.bkey + i, k);
        tied(a, i, old, k);
    }
};

template <typename real>
__device__ __forceinline__ unsigned long long key_now(const StepArgs<real>& a, int64_t i) {
    return __hip_atomic_load(a.bkey + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Visits the record ranges of the neighbourhood of record i (bin cx, cy, cz).
// HALF: only pairs (i, j) not visited from j's side -- bins of larger index
// and, in i's own bin, records after i -- so every unordered pair is met once.
// COARSE: the fast particles of split c-bins, on the configured c-bins n[]
// (rows y + n_y z after the slow particles' c-bins).
// One of the nine rows (k = 3 (dz + 1) + dy + 1) of that neighbourhood.
template <bool HALF, bool COARSE = false, typename real, typename F>
__device__ __forceinline__ void neighbourhood_row(const int32_t* start, const Inst<real>& I, int64_t base,
                                                  const int n[3], const bool per[3], int cx, int cy, int cz,
                                                  int32_t i, int k, F&& visit) {
    const int64_t cell_off = COARSE ? I.cell_off + I.Cf : I.cell_off;
    int y, z;
    if (!axis_nb(cz, k / 3 - 1, n[2], per[2], z)) return;
    if (!axis_nb(cy, k % 3 - 1, n[1], per[1], y)) return;
    const int own_row = COARSE ? cy + n[1] * cz : row_of(I, cy, cz);
    const int row_idx = COARSE ? y + n[1] * z : row_of(I, y, z);
    if (HALF && row_idx < own_row) return;
    const bool own = row_idx == own_row;
    int xa[2], xb[2];
    const int nxr = x_ranges(cx, n[0], per[0], xa, xb);
    const int64_t row = cell_off + (int64_t)n[0] * row_idx;
    for (int r = 0; r < nxr; ++r) {
        int32_t j0 = (int32_t)(base + start[row + xa[r]]);
        const int32_t j1 = (int32_t)(base + start[row + xb[r] + 1]);
        if (HALF && own) {
            if (r == 0) j0 = i + 1;           // range holding cx: after i
            else if (xa[r] < cx) continue;    // wrapped bins below cx
        }
        visit(j0, j1);
    }
}

template <bool HALF, bool COARSE = false, typename real, typename F>
__device__ __forceinline__ void for_neighbourhood(const int32_t* start, const Inst<real>& I, int64_t base,
                                                  const int n[3], const bool per[3], int cx, int cy, int cz,
                                                  int32_t i, F&& visit) {
    for (int k = 0; k < 9; ++k) neighbourhood_row<HALF, COARSE>(start, I, base, n, per, cx, cy, cz, i, k, visit);
}

// Visits the record ranges of the c-bins neighbouring that of (x, y, z), its
// own included, on the c-bins sort cells are part of.
template <typename real, typename F>
__device__ __forceinline__ void for_logical(const StepArgs<real>& a, const Inst<real>& I, const bool per[3], real x,
                                            real y, real z, F&& visit) {
    const int bx = axis_bin(x, I.lo[0], I.inv_wl[0], I.nl[0]), by = axis_bin(y, I.lo[1], I.inv_wl[1], I.nl[1]),
              bz = axis_bin(z, I.lo[2], I.inv_wl[2], I.nl[2]);
    int xa[2], xb[2];
    const int k[3] = {1 << I.kl[0], 1 << I.kl[1], 1 << I.kl[2]};
    const int nxr = x_ranges(bx, I.nl[0], per[0], xa, xb);
    for (int r = 0; r < 9; ++r) {
        int yy, zz;
        if (!axis_nb(bz, r / 3 - 1, I.nl[2], per[2], zz)) continue;
        if (!axis_nb(by, r % 3 - 1, I.nl[1], per[1], yy)) continue;
        for (int f = 0; f < k[1] * k[2]; ++f) {
            const int64_t row = I.cell_off + (int64_t)I.n[0] * row_of(I, yy * k[1] + (f & (k[1] - 1)),
                                                                      zz * k[2] + (f >> I.kl[1]));
            for (int q = 0; q < nxr; ++q)
                visit((int32_t)(I.base + a.start[row + (int64_t)xa[q] * k[0]]),
                      (int32_t)(I.base + a.start[row + (int64_t)(xb[q] + 1) * k[0]]));
        }
    }
}

// Records per chunk of a wave's staging buffer in LDS (the staged lane mode
// of the FP32 search, search_staged): kStageCap quads (x, y, z, vx), then
// kStageCap pairs (vy, vz) in 16-byte slots, so that one address serves
// both reads (the pair kStageCap slots further on) and the loop reads 24 B
// per neighbour at a 16-byte stride.  Measured on the 16M Sedov search:
// 1.34 ms reading two quads per neighbour, 1.27 with the pairs packed at an
// 8-byte stride (two addresses), 1.24 with quad and pair interleaved in
// 32-byte slots (one address, four times the LDS bank conflicts), 1.23
// with this layout.
constexpr int kStageCap = 128;
constexpr int kStageBytesPerWave = kStageCap * 32;
static_assert(kStageBytesPerWave % 16 == 0, "each wave's buffer starts on a quad");

// Exact test of the pair of records (i, j): whether it is a candidate, and
// its ranking value (criterion 3) if so.  Every search path ends here, so
// the pairs it accepts and their values are the same whichever found them.
template <typename real>
__device__ __forceinline__ bool test_pair(const Geo<real>& G, bool by_time, real xi, real yi, real zi, real vxi,
                                          real vyi, real vzi, real xj, real yj, real zj, real vxj, real vyj, real vzj,
                                          real& value) {
    Screen<real> S;
    if (!PairTest<real, -1>::stage1(G, xi, yi, zi, vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, S)) return false;
    if (!PairTest<real, -1>::stage2(G, S)) return false;
    const real d2 = PairTest<real, -1>::finish(G, S);
    if (!(d2 >= real(0))) return false;
    value = by_time ? PairTest<real, -1>::contact(G, S) : d2;
    return true;
}

// ---------------------------------------------------------------- tile search
// Half search of 64 consecutive records against their neighbourhood, 32 x 32
// pairs at a time on the matrix units.  With u the relative velocity and r
// the relative position of a pair, a candidate meets
//     s0 = r.u < 0,   -(s0 + |u|^2 dt) < 0   (criterion 1), and
//     |r|^2 + r.u dt - D^2 <= 0              (d_min <= D with t_poca < dt:
//         |r|^2 = d_min^2 + |u|^2 t_poca^2, and r.u dt = -|u|^2 t_poca dt),
// the last of them the sphere over the partner's path of the step, widened by
// D; and all three are bilinear in per-record vectors, so one K = 16 product
// each (v_mfma_f32_32x32x16_f16) evaluates them for 1024 pairs.  The vectors
// are rounded to f16 relative to the tile (positions in units of the c-bin
// width, velocities of 1 / kTileKappa widths per step), and each form is
// lowered by a bound of its rounding error that is bilinear too, so a pair
// whose three forms are not all negative is certainly no candidate.  The
// others, about one in a hundred, go through a queue in LDS to the exact test
// in the state's own precision (test_pair), which alone decides: the filter
// never changes a result.
//
// Per pair this takes two vector instructions (an AND of the three signs and
// a shift into a mask) instead of 16 to 30, and no memory access: a lane
// holds a whole record, and v_permlane32_swap turns 64 records' vectors into
// the operands of two 32-record tiles.  Measured against the scan it
// replaced, one lane per record with scalar or gathered loads (search phase):
// FP64 Sod tube of 4e5 particles on 100 c-bins 19.8 -> 0.12 ms, FP64 blast of
// 2e6 on 64^3 1.06 -> 0.39, FP32 Noh implosion of 8e6 2.1 -> 1.35, 64
// instances of 3.4e7 particles in all 16.4 -> 9.8 (5.9 with the third form
// above instead of |r|^2 - |u|^2 dt^2 - D^2), and 2000 particles in FP64
// 0.61 -> 0.03.
//
// Vector of a record (k = 0..15), j's side:
//   x y z | vx vy vz | p_hi p_lo | q_hi q_lo | r_hi r_lo | 1 1 | Xm | V1
// with Xm the largest |coordinate|, V1 the sum of |velocity| components and
// p, q, r the record's own terms of the three forms, each as two f16.  i's
// side holds the factors of the same slots, one vector per form.
//
// Error bounds, e = 2^-11 (f16 rounding), sums over both records:
//   r.u:    at most 2e (Xm_i + Xm_j)(V1_i + V1_j) from the rounded vectors,
//           e Xm V1 from the factor x + 2 v / kappa, the rest (products
//           summed in FP32, the split terms) below 2^-18 of the same product;
//           kTileE2 = 3.5e covers them;
//   |u|^2:  2e V1^2 / kappa and the factor's rounding: kTileE3 = 5e / kappa;
//   |r|^2:  2e 3 (Xm_i + Xm_j)^2: kTileE6 = 6.6e per ordered product, and
//           6e Xm_i Xm_j from the factor 2 x + v / kappa: kTileE18 = 19.2e for
//           both products of two records;
//   r.u dt: as r.u, / kappa;
// plus kTileAbs (1 + Xm + V1) for f16 subnormals (2^-25 each).
constexpr float kTileKappa = 256.0f;
constexpr float kTileHalfUlp = 1.0f / 2048.0f;
constexpr float kTileE2 = 3.5f * kTileHalfUlp;
constexpr float kTileE3 = 5.0f * kTileHalfUlp / kTileKappa;
constexpr float kTileE6 = 6.6f * kTileHalfUlp;
constexpr float kTileE18 = 19.2f * kTileHalfUlp;
constexpr float kTileAbs = 1e-6f;
// A record outside these (or outside the box along a periodic axis) takes
// part with forms that are negative against every partner ("wild").  The
// speed limit goes with the tile's extent, since f16 holds the products: one
// limit of 512 for any tile (two widths a step, summed over the axes) left 1%
// of a gas that moves 0.4 widths a step wild, and the box of 1e6 at 9 a c-bin
// took 503 us (FP32) and 2.1 times its present search (FP64).
constexpr float kTileXMax = 64.0f;
constexpr float kTileVMax = 2048.0f;
constexpr float kTileOwn = 40000.0f;  // a tame record's own terms, without D^2 and the bounds
constexpr float kTileWild = -50000.0f;  // below minus any tame record's own terms
constexpr float kTileNever = 60000.0f;  // above them: lanes without a record

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float acc16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t pack2(_Float16 a, _Float16 b) {
    const half2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint32_t split_f16(float v) {
    const _Float16 hi = (_Float16)v;
    return pack2(hi, (_Float16)(v - (float)hi));
}

// f16 not below v >= 0 (v is at most a few hundred).
__device__ __forceinline__ _Float16 up_f16(float v) { return (_Float16)fmaf(v, 1.0f + 2.0f * kTileHalfUlp, 1e-7f); }

// The rounded vector of one record and its own terms of the three forms.
struct TileRec {
    _Float16 x[3], v[3];
    float xm, v1;
    float p, q, r;
};

// X: position relative to the tile in c-bin widths, xabs: bound of its
// absolute error in units of e; V: velocity relative to the tile's, scaled;
// hd2: half of D^2 in widths^2.  absent: no record here.
__device__ __forceinline__ TileRec tile_rec(const float X[3], const float V[3], float xabs, float hd2, bool wild,
                                            bool absent) {
    TileRec T;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T.x[k] = (_Float16)X[k];
        T.v[k] = (_Float16)V[k];
    }
    T.xm = fmaxf(fmaxf(fabsf(X[0]), fabsf(X[1])), fabsf(X[2])) + xabs;
    T.v1 = fabsf(V[0]) + fabsf(V[1]) + fabsf(V[2]);
    const float x = (float)T.x[0], y = (float)T.x[1], z = (float)T.x[2];
    const float a = (float)T.v[0], b = (float)T.v[1], c = (float)T.v[2];
    const float xv = fmaf(z, c, fmaf(y, b, x * a));
    const float vv = fmaf(c, c, fmaf(b, b, a * a));
    const float xx = fmaf(z, z, fmaf(y, y, x * x));
    const float lin = fmaf(kTileAbs, T.xm + T.v1, kTileAbs);
    const float m = fmaf(kTileE2 * T.xm, T.v1, lin);
    T.p = xv - m;
    T.q = fmaf(-1.0f / kTileKappa, vv, -xv) - fmaf(kTileE3 * T.v1, T.v1, m);
    T.r = fmaf(1.0f / kTileKappa, xv, xx) - hd2 -
          fmaf(kTileE6 * T.xm, T.xm, fmaf(kTileE2 / kTileKappa * T.xm, T.v1, lin));
    if (wild || absent) {
#pragma unroll
        for (int k = 0; k < 3; ++k) T.x[k] = T.v[k] = (_Float16)0.0f;
        T.xm = T.v1 = 0.0f;
        T.p = T.q = T.r = absent ? kTileNever : kTileWild;
    }
    return T;
}

// Operands of two 32-record tiles from the lanes' 16-vectors w (packed in
// pairs): tile 0 holds lanes 0..31's records, tile 1 lanes 32..63's; each
// lane gets the 8 values its half of the wave supplies (k = 0..7 or 8..15).
__device__ __forceinline__ void tile_operands(const uint32_t w[8], half8_t out[2]) {
    uint32_t t0[4], t1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const auto s = __builtin_amdgcn_permlane32_swap(w[k], w[4 + k], false, false);
        t0[k] = s[0];
        t1[k] = s[1];
    }
    out[0] = __builtin_bit_cast(half8_t, *reinterpret_cast<uint4*>(t0));
    out[1] = __builtin_bit_cast(half8_t, *reinterpret_cast<uint4*>(t1));
}

// Each lane's value of lane l & 31 (out[0]) and of lane 32 + (l & 31) (out[1]).
__device__ __forceinline__ void both_halves(int32_t v, int32_t out[2]) {
    const auto s = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    out[0] = (int32_t)s[0];
    out[1] = (int32_t)s[1];
}

// Per-wave LDS of the tile search: pairs that passed the filter (x = i's
// lane | code << 6, y = record j), the records of the i tile and their keys,
// and the records of the j block.
constexpr int kHitQueue = 128;
template <typename real>
struct TileLds {
    uint2 hit[kHitQueue];
    unsigned long long key[kWave];
    real pv[6][kWave];
    uint2 blk[kWave];  // x: record, y: its image (2 bits per axis, shift + 1) | (x c-bin + 2) << 6
};
// Image code of a hit: 2 bits per axis, the box's shift + 1 at which j was
// met, 3 where any will do.
constexpr uint32_t kCodeAny = 3u, kCodeAllAny = 63u;
constexpr uint32_t kCodeHome = 1u | 1u << 2 | 1u << 4;  // no shift

// Periodic axes of so few c-bins that the c-bins do not fix which image of a
// neighbour is the near one: the images are visited one by one ("imaged"),
// and a pair is taken at the one the pair test's minimum-image rule picks.
// With four c-bins only pairs half a box apart, from edge to edge of their
// c-bins, are open; records that close to an edge are wild.
__device__ __forceinline__ int image_of(const Geo<double>& G, int ax, double r) {
    return r > G.halfL[ax] ? 1 : (r < -G.halfL[ax] ? -1 : 0);
}
__device__ __forceinline__ int image_of(const Geo<float>& G, int ax, float r) {
    const float k = rintf(r * G.invL[ax]);
    return k > 0.0f ? 1 : (k < 0.0f ? -1 : 0);
}

// Exact tests of `count` queued pairs, one per lane.  (Loading a batch's
// partners when it leaves the queue and testing it when the next one does
// hides the wait, but its registers spill: 4.96 ms against 4.42 on the planar
// equilibration of 2e7 particles, where every particle has 14 candidates.)
template <typename real>
__device__ __forceinline__ void tile_hits(const StepArgs<real>& a, const Geo<real>& G, bool by_time, int32_t wbase,
                                          TileLds<real>& L, int count, int lane, int32_t& nc) {
    if (lane >= count) return;
    const uint2 e = L.hit[lane];
    const int il = (int)(e.x & 63u);
    const int32_t i = wbase + il, j = (int32_t)e.y;
    real xj, yj, zj, vxj, vyj, vzj;
    load_pv(a.rec, j, xj, yj, zj, vxj, vyj, vzj);
    const unsigned long long kj = key_now(a, j);
    const real xi = L.pv[0][il], yi = L.pv[1][il], zi = L.pv[2][il];
    const uint32_t code = e.x >> 6;
    if (code != kCodeAllAny) {
        const real r[3] = {xi - xj, yi - yj, zi - zj};
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const uint32_t c = (code >> (2 * ax)) & 3u;
            if (c != kCodeAny && image_of(G, ax, r[ax]) != (int)c - 1) return;
        }
    }
    real value;
    if (!test_pair(G, by_time, xi, yi, zi, L.pv[3][il], L.pv[4][il], L.pv[5][il], xj, yj, zj, vxj, vyj, vzj, value))
        return;
    ++nc;
    Key<real>::lower(a, j, Key<real>::make(value, (uint32_t)i), kj);
    const unsigned long long k = Key<real>::make(value, (uint32_t)j);
    const unsigned long long old = atomicMin(&L.key[il], k);
    Key<real>::tied(a, i, old, k);
}

// One periodic or bounded axis of a group's neighbourhood: the sort cells
// [first, first + count) to visit, unwrapped, times `images` images.
struct TileAxis {
    int first, count, images;
};

// c: the group's sort cell (its lowest, chi its highest); m: cells that a
// candidate can be away (sub-grids), at least 1.
template <typename real>
__device__ __forceinline__ TileAxis tile_axis(const Inst<real>& I, int ax, bool periodic, int c, int chi, int m) {
    const int n = I.n[ax], nl = I.nl[ax], kl = I.kl[ax];
    TileAxis A;
    const bool near = 2 * ((int64_t)m + 1) < n;  // the nearest image is known
    A.images = periodic && nl <= 3 && !near ? 3 : 1;
    if (A.images == 3) {
        A.first = 0;
        A.count = n;
        return A;
    }
    int lo = c - m, hi = chi + m;
    if (!periodic || nl > 3) {
        lo = max(lo, ((c >> kl) - 1) << kl);
        hi = min(hi, (((chi >> kl) + 2) << kl) - 1);
    }
    if (!periodic) {
        lo = max(lo, 0);
        hi = min(hi, n - 1);
    }
    A.first = lo;
    A.count = hi - lo + 1;
    return A;
}

// Called by every lane of a wave holding a live slow record: the records
// wbase .. wbase + 63 before `stop`, against part `part` of `parts` of their
// neighbourhood.
template <typename real>
__device__ void search_tiles(const StepArgs<real>& a, const Inst<real>& I, int32_t wbase, int32_t stop, int part,
                             int parts, TileLds<real>& L, double& cand) {
    const Geo<real> G(I);
    const int lane = (int)(threadIdx.x & 63);
    const int n[3] = {I.n[0], I.n[1], I.n[2]};
    const int32_t base = (int32_t)I.base;
    const int64_t cell_off = I.cell_off;
    const bool by_time = (I.flags & TPKMC_RANK_TIME) != 0;
    const bool sub = (I.flags & kSubgrid) != 0;
    const int32_t i = wbase + lane;
    const bool valid = i < stop;
    // In FP32 a group reads the records again from LDS, which leaves the
    // registers to its loops (spilled 26 -> 9; Noh implosion 1.15 -> 1.12 ms,
    // planar gas of 1e5 31 -> 29.6 us); in FP64, which has registers left, that
    // only adds a wait (2M blast 377 -> 390 us).
    constexpr bool kReload = sizeof(real) == 4;
    real p0[3], v0[3];
    load_pv(a.rec, valid ? i : wbase, p0[0], p0[1], p0[2], v0[0], v0[1], v0[2]);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        L.pv[ax][lane] = p0[ax];
        L.pv[3 + ax][lane] = v0[ax];
    }
    L.key[lane] = ~0ull;
    const int c0[3] = {sort_bin(I, 0, p0[0]), sort_bin(I, 1, p0[1]), sort_bin(I, 2, p0[2])};
    const int own_row = row_of(I, c0[1], c0[2]);
    const real sx = (real)I.tile_s;
    // A planar gas has one z: no pair differs along it or is nearest by an image
    // there, and the plane may lie far from the middle of its c-bin, on the
    // scale of c-bins in the plane.  (At the lower wall of a unit box on 223 x
    // 223 c-bins every record was beyond kTileXMax: 1e6 particles at 20 a c-bin
    // took 1.6 ms a step instead of 0.7 in FP64, 1.0 instead of 0.5 in FP32.)
    const bool planar = (I.flags & TPKMC_PLANAR) != 0;
    const real sv = I.dt * sx * (real)kTileKappa;
    // At most 30000: beyond, D spans every tame pair.
    const float hd2 = fminf(0.5001f * (float)(I.D2 * sx * sx), 30000.0f);
    const real lo[3] = {I.lo[0], I.lo[1], I.lo[2]}, hi[3] = {I.hi[0], I.hi[1], I.hi[2]};
    const real iw[3] = {I.inv_w[0], I.inv_w[1], I.inv_w[2]};
    const real ws[3] = {I.w_sort[0], I.w_sort[1], I.w_sort[2]};
    const real iwl[3] = {I.inv_wl[0], I.inv_wl[1], I.inv_wl[2]};
    const int nl0 = I.nl[0];
    // The box along the periodic axes; records outside are wild.
    real box_lo[3], box_hi[3];
    bool four[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        box_lo[ax] = G.per[ax] ? lo[ax] : -real(INFINITY);
        box_hi[ax] = G.per[ax] ? hi[ax] : real(INFINITY);
        four[ax] = G.per[ax] && I.nl[ax] == 4;
    }
    const bool any_four = four[0] || four[1] || four[2];
    auto untame = [&](const real p[3], const float X[3], const float V[3], float xcap, float vcap) {
        const float xm = fmaxf(fmaxf(fabsf(X[0]), fabsf(X[1])), fabsf(X[2]));
        bool t = (xm <= xcap) & (fabsf(V[0]) + fabsf(V[1]) + fabsf(V[2]) <= vcap);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) t &= (p[ax] >= box_lo[ax]) & (p[ax] < box_hi[ax]);
        if (any_four)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const real u = (p[ax] - lo[ax]) * iwl[ax], f = u - floor(u);
                t &= !four[ax] | ((f > real(1e-4)) & (f < real(1.0 - 1e-4)));
            }
        return !t;
    };
    int32_t nc = 0;
    int nq = 0;  // queued hits (wave-uniform)
    const int j_row = 4 * (lane >> 5);  // the lane's first row of a product
    uint64_t pending = __ballot(valid);
    while (pending) {
        // One group of lanes per row of sort cells: consecutive lanes with
        // non-decreasing x cells.
        const int lead = __ffsll((long long)pending) - 1;
        const int R = __builtin_amdgcn_readlane(own_row, lead);
        const bool in = valid && own_row == R;
        const uint64_t gm = __ballot(in);
        pending &= ~gm;
        const int last = 63 - __clzll((long long)gm);
        if (kReload) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        real pi[3], vi[3];
        int ci[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            pi[ax] = kReload ? L.pv[ax][lane] : p0[ax];
            vi[ax] = kReload ? L.pv[3 + ax][lane] : v0[ax];
            ci[ax] = kReload ? sort_bin(I, ax, pi[ax]) : c0[ax];
        }
        const int cx = ci[0], cy = ci[1], cz = ci[2];
        const int gcy = __builtin_amdgcn_readlane(cy, lead), gcz = __builtin_amdgcn_readlane(cz, lead);
        const int cxf = __builtin_amdgcn_readlane(cx, lead), cxl = __builtin_amdgcn_readlane(cx, last);
        const int32_t after = wbase + lead;  // partners come after the first record (half search)
        // Tile origin: the middle of the group's cells; its mean velocity.
        real org[3], Ls[3], vo[3];
        float xabs = 0.0f;  // rounding of a shifted origin, in units of e (unshifted it is i's and j's alike)
        const float inv = 1.0f / (float)__popcll(gm);
        const real mid[3] = {real(0.5) * (real)(cxf + cxl + 1), real(0.5) + (real)gcy, real(0.5) + (real)gcz};
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            org[ax] = (lo[ax] + mid[ax] * ws[ax]) * sx;
            Ls[ax] = G.L[ax] * sx;
            vo[ax] = (real)(wave_reducef<false>(in ? (float)(vi[ax] * sv) : 0.0f) * inv);
            if (G.per[ax])  // elsewhere nothing is shifted
                xabs = fmaxf(xabs, (fabsf((float)org[ax]) + (float)Ls[ax]) * (sizeof(real) == 4 ? 1.0f / 1024.0f : 1e-9f));
        }
        // How far apart a candidate pair of this group can start: with
        // sub-grids from the group's and the instance's largest speeds, so
        // that a pair's own image is always visited.  Without, only images
        // other than the unshifted one are skipped, by a bound for partners
        // up to vcap; faster ones are wild, and wild pairs are taken
        // unshifted.
        real reach = real(INFINITY);
        int m[3] = {1 << 24, 1 << 24, 1 << 24};
        if (sub) {
            // In widths per step, where FP32 has room below and above whatever
            // the units of an FP64 state (infinite or no number: no bound).
            float V[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) V[ax] = (float)(vi[ax] * sv);
            float v = in ? sqrtf(V[0] * V[0] + V[1] * V[1] + V[2] * V[2]) : 0.0f;
            v = v < INFINITY ? v : INFINITY;
            reach = (sqrt(I.D2) + I.vreach * I.dt + (real)(wave_reducef<true>(v) * (1.0f / kTileKappa)) / sx) *
                    real(1.001);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const real c = reach * iw[ax] + real(1e-3) + real(1e-6) * (real)n[ax];
                m[ax] = c < (real)(1 << 24) ? 1 + (int)c : 1 << 24;
            }
        }
        const TileAxis AX = tile_axis(I, 0, G.per[0], cxf, cxl, m[0]);
        const TileAxis AY = tile_axis(I, 1, G.per[1], gcy, gcy, m[1]);
        const TileAxis AZ = tile_axis(I, 2, G.per[2] && !planar, gcz, gcz, m[2]);
        // A shifted origin too coarse for the filter: shifted partners are
        // wild, and where a partner is visited in several places it is so in
        // all of them.  (Taken for unshifted ones too, an FP32 box of 1e6 at
        // 16 a c-bin and a thousand box lengths from the origin took 1.7 ms a
        // step instead of 0.55.)
        const bool coarse = !(xabs <= 16.0f);
        const bool coarse_home = coarse && AX.images * AY.images * AZ.images > 1;
        // The largest coordinate of a partner in its place, and a speed whose
        // own terms beside it, x v + v^2 / kTileKappa, stay below kTileOwn.
        const float xcap = fminf(fmaf(I.tile_dx, (float)(cxl - cxf), I.tile_x), kTileXMax);
        const float vlim = fminf(kTileVMax, kTileOwn * __builtin_amdgcn_rcpf(xcap + kTileVMax / kTileKappa));
        half8_t BP[2], BQ[2], BR[2];
        uint64_t wild_i;
        float vmax;
        {
            float X[3], V[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                X[ax] = (float)fma(pi[ax], sx, -org[ax]);
                V[ax] = (float)fma(vi[ax], sv, -vo[ax]);
            }
            if (planar) X[2] = 0.0f;
            const bool wild = coarse_home || untame(pi, X, V, xcap, vlim);
            wild_i = __ballot(in && wild);
            const TileRec T = tile_rec(X, V, 0.0f, hd2, wild, !in);
            vmax = wave_reducef<true>(T.v1);
            const _Float16 one = (_Float16)1.0f;
            const _Float16 mv = -up_f16(kTileE2 * T.v1), mx = -up_f16(kTileE2 * T.xm);
            const uint32_t wp[8] = {pack2(-T.v[0], -T.v[1]), pack2(-T.v[2], -T.x[0]), pack2(-T.x[1], -T.x[2]),
                                    pack2(one, one), 0u, 0u, split_f16(T.p), pack2(mv, mx)};
            tile_operands(wp, BP);
            constexpr float k2 = 2.0f / kTileKappa;
            const _Float16 f0 = (_Float16)k2 * T.v[0] + T.x[0];
            const _Float16 f1 = (_Float16)k2 * T.v[1] + T.x[1];
            const _Float16 f2 = (_Float16)k2 * T.v[2] + T.x[2];
            const _Float16 mq = -up_f16(fmaf(kTileE2, T.xm, 2.0f * kTileE3 * T.v1));
            const uint32_t wq[8] = {pack2(T.v[0], T.v[1]), pack2(T.v[2], f0), pack2(f1, f2), 0u,
                                    pack2(one, one), 0u, split_f16(T.q), pack2(mv, mq)};
            tile_operands(wq, BQ);
            constexpr float k1 = 1.0f / kTileKappa;
            _Float16 g[3], h[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                // Scaling by powers of two is exact, so each rounds once.
                g[ax] = (_Float16)(-k1) * T.v[ax] - (_Float16)2.0f * T.x[ax];
                h[ax] = (_Float16)(-k1) * T.x[ax];
            }
            const _Float16 mrx = -up_f16(fmaf(kTileE18, T.xm, kTileE2 * k1 * T.v1)), mrv = -up_f16(kTileE2 * k1 * T.xm);
            const uint32_t wr[8] = {pack2(g[0], g[1]), pack2(g[2], h[0]), pack2(h[1], h[2]), 0u, 0u,
                                    pack2(one, one), split_f16(T.r), pack2(mrx, mrv)};
            tile_operands(wr, BR);
        }
        float vcap = vlim;
        real reach_im = reach;
        if (!sub && AX.images * AY.images * AZ.images > 1) {
            vcap = fminf(vlim, 2.0f * vmax + 1e-3f);
            const float uu = (vmax + vcap) * (1.01f / kTileKappa);
            if (!wild_i) reach_im = (real)(1.001f * sqrtf(fmaf(uu, uu, 2.0f * hd2)) / I.tile_s);
        }
        // The group's extent along the imaged axes (elsewhere its cells'),
        // widened by the rounding of the cells, in sort cells.
        real ext_lo[3] = {(real)cxf, (real)gcy, (real)gcz}, ext_hi[3] = {(real)(cxl + 1), (real)(gcy + 1), (real)(gcz + 1)};
        const int images[3] = {AX.images, AY.images, AZ.images};
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            if (images[ax] == 3) {
                const float t = (float)((pi[ax] - lo[ax]) * iw[ax]);
                ext_hi[ax] = (real)wave_reducef<true>(in ? t : -INFINITY);
                ext_lo[ax] = -(real)wave_reducef<true>(in ? -t : -INFINITY);
            }
            const real eps = real(1e-3) + real(1e-6) * (real)n[ax];
            ext_lo[ax] -= eps;
            ext_hi[ax] += eps;
        }
        // Along x: the images of a whole row, or the part of the range inside
        // the box and the parts wrapped at its lower and upper end.
        const int xend = AX.first + AX.count;  // exclusive, unwrapped
        const bool lw = AX.images == 1 && AX.first < 0, rw = AX.images == 1 && xend > n[0];
        const int nx = AX.images == 3 ? 3 : 1 + (lw ? 1 : 0) + (rw ? 1 : 0);
        const int ny = AY.count * AY.images, nz = AZ.count * AZ.images;
        // A periodic x axis of at most three c-bins, all of them neighbours,
        // goes by image; else the c-bins decide, as the tile's x range is
        // wider than a record's own.
        const bool by_image = G.per[0] && nl0 <= 3;
        const uint32_t any_mask = (by_image ? 0u : kCodeAny) | (AY.images == 1 ? kCodeAny << 2 : 0u) |
                                  (AZ.images == 1 ? kCodeAny << 4 : 0u);
        const uint32_t wild_mask =
            sub ? 0u : (kCodeAny << 2) | (kCodeAny << 4) | (AX.images == 3 ? kCodeAny : 0u);
        int32_t bi[2];  // x c-bin + 1 of the lane's record in either i tile
        both_halves(by_image ? 2 : (cx >> I.kl[0]) + 1, bi);
        const int64_t total = (int64_t)nx * ny * nz;
        // Quotients of the small numbers below by their float reciprocals:
        // exact while the dividend is below 2^20.
        const float inx = __builtin_amdgcn_rcpf((float)nx), iny = __builtin_amdgcn_rcpf((float)ny);
        const float iay = __builtin_amdgcn_rcpf((float)AY.count), iaz = __builtin_amdgcn_rcpf((float)AZ.count);
        auto quot = [](uint32_t t, float inv) { return (uint32_t)(((float)t + 0.5f) * inv); };
        for (int64_t t0 = 0; t0 < total; t0 += kWave) {
            // One part of the neighbourhood per lane: a run of records, or
            // none where it is out of reach.
            int32_t u0 = 0, len = 0;
            uint32_t shw = 0;
            if (t0 + lane < total) {
                const uint32_t t = (uint32_t)(t0 + lane);
                const bool small = total < (1 << 20);  // uniform
                const uint32_t tr = small ? quot(t, inx) : t / (uint32_t)nx;
                const uint32_t tz = small ? quot(tr, iny) : tr / (uint32_t)ny;
                const int s = (int)(t - tr * (uint32_t)nx), ty = (int)(tr - tz * (uint32_t)ny);
                const int qy = small ? (int)quot((uint32_t)ty, iay) : ty / AY.count;
                const int qz = small ? (int)quot(tz, iaz) : (int)tz / AZ.count;
                int y = AY.first + ty - qy * AY.count, z = AZ.first + (int)tz - qz * AZ.count;
                int shy = 0, shz = 0, shx = 0;
                if (AY.images == 3) shy = qy - 1;
                else if (y < 0) { y += n[1]; shy = -1; }
                else if (y >= n[1]) { y -= n[1]; shy = 1; }
                if (AZ.images == 3) shz = qz - 1;
                else if (z < 0) { z += n[2]; shz = -1; }
                else if (z >= n[2]) { z -= n[2]; shz = 1; }
                int xa = max(AX.first, 0), xb = min(xend, n[0]) - 1;
                if (AX.images == 3) shx = s - 1;
                else if (s == 1 && lw) { shx = -1; xa = AX.first + n[0]; xb = n[0] - 1; }
                else if (s >= 1) { shx = 1; xa = 0; xb = xend - n[0] - 1; }
                xa = max(xa, 0);
                xb = min(xb, n[0] - 1);
                // Gap between the group and the sort cells c0..c1 (unwrapped).
                auto gap = [&](int ax, int c0, int c1) {
                    const real g = fmax((real)c0 - ext_hi[ax], ext_lo[ax] - (real)(c1 + 1));
                    return g > real(0) ? g * ws[ax] : real(0);
                };
                const real gx = gap(0, xa + shx * n[0], xb + shx * n[0]);
                const real gy = gap(1, y + shy * n[1], y + shy * n[1]), gz = gap(2, z + shz * n[2], z + shz * n[2]);
                const bool shifted = (AX.images == 3 && shx != 0) || (AY.images == 3 && shy != 0) ||
                                     (AZ.images == 3 && shz != 0);
                const real rr = shifted ? reach_im : reach;
                if (!(gx * gx + gy * gy + gz * gz > rr * rr)) {
                    const int64_t row = cell_off + (int64_t)n[0] * row_of(I, y, z);
                    u0 = max(base + a.start[row + xa], after + 1);
                    len = max(base + a.start[row + xb + 1] - u0, 0);
                    shw = (uint32_t)(shx + 1) | (uint32_t)(shy + 1) << 2 | (uint32_t)(shz + 1) << 4;
                }
            }
            int32_t end = len;  // inclusive prefix of the lengths
            for (int o = 1; o < kWave; o <<= 1) {
                const int32_t v = __shfl_up(end, o);
                if (lane >= o) end += v;
            }
            const int32_t njs = __builtin_amdgcn_readlane(end, kWave - 1);
            uint64_t runs = __ballot(len > 0);
            // Blocks of 64 records taken from the runs in order.
            int32_t nj = 0;
            uint32_t ncode = kCodeHome;
            RawRec<real> next;  // the next block's records, on their way
            auto fetch = [&](int32_t b) {
                nj = after;
                while (runs) {
                    const int v = __ffsll((long long)runs) - 1;
                    const int32_t e1 = __builtin_amdgcn_readlane(end, v), l1 = __builtin_amdgcn_readlane(len, v);
                    if (e1 - l1 >= b + kWave) break;
                    const int32_t g = b + lane - (e1 - l1);
                    const bool mine = g >= 0 && g < l1;
                    const int32_t s = __builtin_amdgcn_readlane(u0, v);
                    const uint32_t c1 = (uint32_t)__builtin_amdgcn_readlane((int)shw, v);
                    nj = mine ? s + g : nj;
                    ncode = mine ? c1 : ncode;
                    if (e1 > b + kWave) break;  // goes on in the next block
                    runs &= runs - 1;
                }
                next.load(a.rec, nj);
            };
            const int32_t step = parts * kWave;
            if (part * kWave < njs) fetch(part * kWave);
            for (int32_t b = part * kWave; b < njs; b += step) {
                const int32_t jj = nj;
                const uint32_t code = ncode;
                real pj[3], vj[3];
                next.get(pj, vj);
                if (b + step < njs) fetch(b + step);
                float X[3], V[3];
                const bool home = __ballot(code != kCodeHome) == 0;  // wave-uniform
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) V[ax] = (float)fma(vj[ax], sv, -vo[ax]);
                if (home) {
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) X[ax] = (float)fma(pj[ax], sx, -org[ax]);
                } else {
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax)
                        X[ax] = (float)fma(pj[ax], sx, (real)((int)(code >> (2 * ax) & 3u) - 1) * Ls[ax] - org[ax]);
                }
                if (planar) X[2] = 0.0f;
                const bool absent = b + lane >= njs;
                const bool wild = coarse_home | (coarse & (code != kCodeHome)) | untame(pj, X, V, xcap, vcap);
                const bool shifted = !home && !sub && ((AX.images == 3 && (code & 3u) != 1u) ||
                                                       (AY.images == 3 && (code >> 2 & 3u) != 1u) ||
                                                       (AZ.images == 3 && (code >> 4 & 3u) != 1u));
                const uint64_t wild_j = __ballot(wild && !absent);
                const uint64_t shift_j = __ballot(shifted && !absent);
                const TileRec T =
                    tile_rec(X, V, code != kCodeHome ? xabs : 0.0f, hd2, wild, absent || (wild && shifted));
                const _Float16 one = (_Float16)1.0f;
                const uint32_t w[8] = {pack2(T.x[0], T.x[1]), pack2(T.x[2], T.v[0]), pack2(T.v[1], T.v[2]),
                                       split_f16(T.p), split_f16(T.q), split_f16(T.r), pack2(one, one),
                                       pack2(up_f16(T.xm), up_f16(T.v1))};
                half8_t A[2];
                tile_operands(w, A);
                int bj = 0;
                if (!by_image) bj = axis_bin(pj[0], lo[0], iwl[0], nl0) + ((int)(code & 3u) - 1) * nl0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                L.blk[lane] = make_uint2((uint32_t)jj, code | (uint32_t)(bj + 2) << 6);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (b + 32 * c >= njs) continue;  // wave-uniform
                    uint32_t W = 0;
                    // The later tile's bits end up low: q = 1 first.
#pragma unroll
                    for (int q = 1; q >= 0; --q) {
                        const acc16_t zero = {};
                        const acc16_t P = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[c], BP[q], zero, 0, 0, 0);
                        const acc16_t Qf = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[c], BQ[q], zero, 0, 0, 0);
                        const acc16_t Rf = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[c], BR[q], zero, 0, 0, 0);
#pragma unroll
                        for (int r = 15; r >= 0; --r) {
                            const int s = __float_as_int(P[r]) & __float_as_int(Qf[r]) & __float_as_int(Rf[r]);
                            W = __builtin_amdgcn_alignbit(W, (uint32_t)s, 31);
                        }
                    }
                    // Bit b of W: i tile b >> 4, row b & 15 of the product's
                    // layout.
                    while (__ballot(W != 0)) {
                        const int bit = W ? __ffs((int)W) - 1 : 0;
                        bool take = W != 0;
                        W &= W - 1;
                        const int jl = j_row + 32 * c + (bit & 15) + (bit & 12);
                        const int il = (lane & 31) + 2 * (bit & 16);
                        const uint2 e = L.blk[jl];
                        const uint32_t dx = (e.y >> 6) - (uint32_t)((bit & 16) ? bi[1] : bi[0]);
                        take = take && (int32_t)e.x > wbase + il && dx <= 2u;
                        uint32_t cd = (e.y & 63u) | any_mask;
                        if (wild_i | wild_j) {
                            const bool wi = (wild_i >> il) & 1ull, wj = (wild_j >> jl) & 1ull;
                            take = take && !(wi && ((shift_j >> jl) & 1ull));
                            cd = wi || wj ? cd | wild_mask : cd;
                        }
                        const uint64_t tm = __ballot(take);
                        if (take)
                            L.hit[nq + __popcll(tm & ((1ull << lane) - 1ull))] = make_uint2((uint32_t)il | cd << 6, e.x);
                        nq += __popcll(tm);
                        if (nq >= kWave) {
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                            tile_hits(a, G, by_time, wbase, L, kWave, lane, nc);
                            const bool mv = lane < nq - kWave;
                            uint2 h = make_uint2(0u, 0u);
                            if (mv) h = L.hit[kWave + lane];
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                            if (mv) L.hit[lane] = h;
                            nq -= kWave;
                        }
                    }
                }
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    tile_hits(a, G, by_time, wbase, L, nq, lane, nc);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const unsigned long long k = L.key[lane];
    if (valid && k != ~0ull) Key<real>::lower(a, i, k, key_now(a, i));
    cand = 2.0 * (double)nc;
}

// FP64 half scan of record i, record by record; SPLIT: of the nine rows of its
// neighbourhood those k = part, part + parts, ... alone.  The pairs tested are
// those of the tile search, and so is the combination of the keys.
template <bool SPLIT>
__device__ __forceinline__ void search_lane(const StepArgs<double>& a, const Inst<double>& I, int32_t i, int part,
                                            int parts, double& tests, double& cand) {
    const Geo<double> G(I);
    const int n[3] = {I.n[0], I.n[1], I.n[2]};
    const bool by_time = (I.flags & TPKMC_RANK_TIME) != 0;
    double xi, yi, zi, vxi, vyi, vzi;
    load_pv(a.rec, i, xi, yi, zi, vxi, vyi, vzi);
    const int cx = axis_bin(xi, I.lo[0], I.inv_w[0], n[0]), cy = axis_bin(yi, I.lo[1], I.inv_w[1], n[1]),
              cz = axis_bin(zi, I.lo[2], I.inv_w[2], n[2]);
    int32_t seen = 0, nc = 0;
    unsigned long long mine = ~0ull;
    auto row = [&](int32_t j0, int32_t j1) {
        seen += j1 > j0 ? j1 - j0 : 0;
        for (int32_t j = j0; j < j1; ++j) {
            double xj, yj, zj, vxj, vyj, vzj, value;
            load_pv(a.rec, j, xj, yj, zj, vxj, vyj, vzj);
            if (!test_pair(G, by_time, xi, yi, zi, vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, value)) continue;
            ++nc;
            Key<double>::lower(a, j, Key<double>::make(value, (uint32_t)i), key_now(a, j));
            const unsigned long long key = Key<double>::make(value, (uint32_t)j);
            Key<double>::tied(a, i, mine, key);
            mine = key < mine ? key : mine;
        }
    };
    if constexpr (SPLIT) {
        for (int k = part; k < 9; k += parts)
            neighbourhood_row<true>(a.start, I, I.base, n, G.per, cx, cy, cz, i, k, row);
    } else {
        for_neighbourhood<true>(a.start, I, I.base, n, G.per, cx, cy, cz, i, row);
    }
    if (mine != ~0ull) Key<double>::lower(a, i, mine, key_now(a, i));
    tests = (double)seen;
    cand = 2.0 * (double)nc;
}

// Plain half scan of one record, counting what the pair tests meet (the
// diagnostic mix): the pairs that cbin_tests counts, record by record.
template <typename real>
__device__ void count_mix(const StepArgs<real>& a, const Inst<real>& I, int32_t i, double& tests, uint32_t& n_s0,
                          uint32_t& n_c1) {
    const Geo<real> G(I);
    real xi, yi, zi, vxi, vyi, vzi;
    load_pv(a.rec, i, xi, yi, zi, vxi, vyi, vzi);
    int64_t seen = 0;
    for_logical(a, I, G.per, xi, yi, zi, [&](int32_t j0, int32_t j1) {
        if (j0 <= i) j0 = i + 1;
        seen += j1 > j0 ? j1 - j0 : 0;
        for (int32_t j = j0; j < j1; ++j) {
            real xj, yj, zj, vxj, vyj, vzj;
            load_pv(a.rec, j, xj, yj, zj, vxj, vyj, vzj);
            Screen<real> S;
            const bool p1 = PairTest<real, -1>::stage1(G, xi, yi, zi, vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, S);
            n_s0 += S.s0 < real(0) ? 1u : 0u;
            n_c1 += p1 ? 1u : 0u;
        }
    });
    tests = (double)seen;
}

// Lane mode of the FP32 half scans, staged through LDS.  A wave that owns
// 64 G consecutive records takes them in G passes of 64, one record per lane
// (record wbase + 64 p + lane in pass p), so that its registers are those of
// one record whatever G is; G > 1 saves work-groups.
// In each pass, the lanes whose records share one row walk every neighbour
// row together: the wave copies the union of their ranges in that row, a
// contiguous run of records, into its LDS buffer in chunks of kStageCap, and
// each lane reads its own part of each chunk from there.  A neighbour record
// is then fetched from memory once per wave instead of once per lane whose
// range holds it.  Records whose x-neighbourhood wraps around a periodic
// axis walk their own rows with global loads.  The pairs tested, the
// arithmetic and the combination of the keys are those of the tile search,
// so the results are too.  Called by every lane of a wave holding a live slow
// record; stop ends the slow records.
template <int PM, int G>
__device__ __forceinline__ void search_staged(const StepArgs<float>& a, const Inst<float>& I, int64_t base,
                                              int32_t wbase, int32_t stop, double& tests, double& cand) {
    const Geo<float> G_(I);
    const int n[3] = {I.n[0], I.n[1], I.n[2]};
    extern __shared__ float4 tpkmc_stage[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float4* const sp = tpkmc_stage + wave * (kStageBytesPerWave / 16);
    const int lane = (int)(threadIdx.x & 63);
    const bool by_time = (I.flags & TPKMC_RANK_TIME) != 0;
    int32_t seen = 0, nc = 0;
    for (int p = 0; p < G; ++p) {
        const int32_t i = wbase + p * kWave + lane;
        const bool valid = i < stop;
        if (__ballot(valid) == 0) break;  // uniform: later passes start further on
        float xi, yi, zi, vxi, vyi, vzi;
        Rec<float>::load6(a.rec, (uint32_t)(valid ? i : wbase), xi, yi, zi, vxi, vyi, vzi);
        const int cx = axis_bin(xi, I.lo[0], I.inv_w[0], n[0]);
        const int cy = axis_bin(yi, I.lo[1], I.inv_w[1], n[1]);
        const int cz = axis_bin(zi, I.lo[2], I.inv_w[2], n[2]);
        int xa[2], xb[2];
        const bool joint = valid && x_ranges(cx, n[0], G_.per[0], xa, xb) == 1;
        unsigned long long mine = ~0ull;
        auto screen = [&](int32_t j, float xj, float yj, float zj, float vxj, float vyj, float vzj, bool take) {
            Screen<float> S;
            // Criterion 1 as two votes on the compares themselves, so that
            // the wave's decision stays in scalar masks.
            (void)PairTest<float, PM>::stage1(G_, xi, yi, zi, vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, S);
            const bool a0 = take & (S.s0 < 0.0f);
            const bool a1 = fmaf(S.vv, G_.dt, S.s0) > 0.0f;
            const uint64_t m = __builtin_amdgcn_ballot_w64(a0) & __builtin_amdgcn_ballot_w64(a1);
            const bool p1 = a0 & a1;
            if (m == 0) return;
            if (p1 && PairTest<float, PM>::stage2(G_, S)) {
                const float d2 = PairTest<float, PM>::finish(G_, S);
                if (d2 >= 0.0f) {
                    ++nc;
                    const float key = by_time ? PairTest<float, PM>::contact(G_, S) : d2;
                    const unsigned long long hi = (unsigned long long)sortable(key) << 32;
                    // An empty barrier on j keeps the compiler from carrying
                    // a 64-bit key pointer through the whole loop for this
                    // rare path.
                    int32_t jh = j;
                    asm volatile("" : "+v"(jh));
                    atomicMin(a.bkey + jh, hi | (uint32_t)i);
                    const unsigned long long kk = hi | (uint32_t)j;
                    mine = kk < mine ? kk : mine;
                }
            }
        };
        // Two neighbours j and j + 1 of the staged chunk, one vote: the two
        // tests are independent, so their LDS reads and arithmetic overlap
        // (the loop takes neighbours in pairs; measured on the 16M Sedov
        // search 1.23 -> 1.18 ms, the Noh and Sod searches 2-3% faster).
        auto screen2 = [&](int32_t j, const float4& pa, const float2& va, const float4& pb, const float2& vb) {
            Screen<float> SA, SB;
            (void)PairTest<float, PM>::stage1(G_, xi, yi, zi, vxi, vyi, vzi, pa.x, pa.y, pa.z, pa.w, va.x, va.y, SA);
            (void)PairTest<float, PM>::stage1(G_, xi, yi, zi, vxi, vyi, vzi, pb.x, pb.y, pb.z, pb.w, vb.x, vb.y, SB);
            const bool qa0 = SA.s0 < 0.0f, qa1 = fmaf(SA.vv, G_.dt, SA.s0) > 0.0f;
            const bool qb0 = SB.s0 < 0.0f, qb1 = fmaf(SB.vv, G_.dt, SB.s0) > 0.0f;
            const uint64_t m = (__builtin_amdgcn_ballot_w64(qa0) & __builtin_amdgcn_ballot_w64(qa1)) |
                               (__builtin_amdgcn_ballot_w64(qb0) & __builtin_amdgcn_ballot_w64(qb1));
            const bool pa1 = qa0 & qa1, pb1 = qb0 & qb1;
            if (m == 0) return;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const Screen<float>& S = h ? SB : SA;
                if ((h ? pb1 : pa1) && PairTest<float, PM>::stage2(G_, S)) {
                    const float d2 = PairTest<float, PM>::finish(G_, S);
                    if (d2 >= 0.0f) {
                        ++nc;
                        const float key = by_time ? PairTest<float, PM>::contact(G_, S) : d2;
                        const unsigned long long hk = (unsigned long long)sortable(key) << 32;
                        int32_t jh = j + h;  // see screen
                        asm volatile("" : "+v"(jh));
                        atomicMin(a.bkey + jh, hk | (uint32_t)i);
                        const unsigned long long kk = hk | (uint32_t)(j + h);
                        mine = kk < mine ? kk : mine;
                    }
                }
            }
        };
        // Lanes taking part in the copies: all of the wave's.
        const int own_row_l = row_of(I, cy, cz);
        uint64_t pending = __ballot(joint);
        while (pending) {
            // One group of lanes per row.  Records are in c-bin order, so the
            // group's lanes are consecutive and their x-bins non-decreasing:
            // the first lane holds the union's lower end, the last its upper.
            const int lead = __ffsll((long long)pending) - 1;
            const int R = __builtin_amdgcn_readlane(own_row_l, lead);
            const bool in = joint && own_row_l == R;
            const uint64_t gm = __ballot(in);
            pending &= ~gm;
            const int last = 63 - __clzll((long long)gm);
            const int gcy = __builtin_amdgcn_readlane(cy, lead);
            const int gcz = __builtin_amdgcn_readlane(cz, lead);
            const int ga = __builtin_amdgcn_readlane(xa[0], lead);
            const int gb = __builtin_amdgcn_readlane(xb[0], last);
            const int32_t gi = __builtin_amdgcn_readlane(i, lead);
            for (int rr = 0; rr < 9; ++rr) {
                int y, z;
                if (!axis_nb(gcz, rr / 3 - 1, n[2], G_.per[2], z)) continue;
                if (!axis_nb(gcy, rr % 3 - 1, n[1], G_.per[1], y)) continue;
                const int row_idx = row_of(I, y, z);
                if (row_idx < R) continue;  // half scans: rows of larger index, and own
                const bool own = row_idx == R;
                const int64_t row = I.cell_off + (int64_t)n[0] * row_idx;
                int32_t lo = 0, hi = 0;  // the lane's range in this row
                if (in) {
                    lo = own ? i + 1 : (int32_t)(base + a.start[row + xa[0]]);
                    hi = (int32_t)(base + a.start[row + xb[0] + 1]);
                    seen += hi > lo ? hi - lo : 0;
                }
                const int32_t u0 = own ? gi + 1 : (int32_t)(base + a.start[row + ga]);
                const int32_t u1 = (int32_t)(base + a.start[row + gb + 1]);
                for (int32_t c0 = u0; c0 < u1; c0 += kStageCap) {
                    const int32_t c1 = u1 - c0 < kStageCap ? u1 : c0 + kStageCap;
                    // Copy [c0, c1): each record's position and velocity.
                    // The previous chunk's reads have all returned: their
                    // values were used before its loop ended.
                    const float4* src = reinterpret_cast<const float4*>(a.rec) + 2 * (int64_t)c0;
                    for (int t = lane; t < c1 - c0; t += kWave) {
                        const float4 qa = src[2 * t], qb = src[2 * t + 1];
                        sp[t] = make_float4(qa.x, qa.y, qa.z, qb.x);
                        *reinterpret_cast<float2*>(sp + kStageCap + t) = make_float2(qb.y, qb.z);
                    }
                    // The wave's own writes, complete before any lane reads.
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    const int32_t j0 = lo > c0 ? lo : c0;
                    const int32_t j1 = hi < c1 ? hi : c1;
                    int32_t j = j0;
                    for (; j + 1 < j1; j += 2) {
                        const float4 pa = sp[j - c0], pb = sp[j + 1 - c0];
                        const float2 va = *reinterpret_cast<const float2*>(sp + kStageCap + (j - c0));
                        const float2 vb = *reinterpret_cast<const float2*>(sp + kStageCap + (j + 1 - c0));
                        screen2(j, pa, va, pb, vb);
                    }
                    if (j < j1) {
                        const float4 pj = sp[j - c0];
                        const float2 vj = *reinterpret_cast<const float2*>(sp + kStageCap + (j - c0));
                        screen(j, pj.x, pj.y, pj.z, pj.w, vj.x, vj.y, true);
                    }
                }
            }
        }
        if (valid && !joint) {
            for_neighbourhood<true>(a.start, I, base, n, G_.per, cx, cy, cz, i, [&](int32_t j0, int32_t j1) {
                seen += j1 > j0 ? j1 - j0 : 0;
                for (int32_t j = j0; j < j1; ++j) {
                    float xj, yj, zj, vxj, vyj, vzj;
                    Rec<float>::load6(a.rec, (uint32_t)j, xj, yj, zj, vxj, vyj, vzj);
                    screen(j, xj, yj, zj, vxj, vyj, vzj, true);
                }
            });
        }
        if (valid && mine != ~0ull) atomicMin(a.bkey + i, mine);
    }
    tests = (double)seen;
    cand = 2.0 * (double)nc;
}

// ---------------------------------------------------------------- 4a. fast particles of split c-bins
// With split c-bins the slow particles are binned on refined c-bins, at
// least as wide as the largest distance at which two slow particles can
// meet the criteria of Sec. 2.4 within the step (D + 2 v_c dt, v_c the speed
// bound), so every candidate pair of two slow particles lies in
// neighbouring refined c-bins, and every such pair that meets the criteria
// also lies in neighbouring configured c-bins.  The fast particles keep the
// configured c-bins and the configured 27-bin neighbourhood: their
// candidates are exactly those of the unsplit grid.

__device__ __forceinline__ int floor_div(int64_t a, int64_t b) {  // b > 0
    return (int)(a >= 0 ? a / b : -((-a + b - 1) / b));
}

// Fine (refined) c-bins along one axis that a fast particle at coordinate x,
// in configured c-bin cc, can meet a slow partner in: those that meet its
// configured neighbours' extent (cc - 1 .. cc + 1, wrapped on a periodic
// axis), cut to the fine c-bins within its reach (any pair meeting the
// criteria starts at most D + (|v_i| + v_c) dt apart on every axis), both
// widened by a rounding margin of the binnings (1e-3 + 1e-6 n_f fine
// c-bins, above the few-ulp error of an FP32 bin coordinate).  At most two
// ranges [fa, fb]; 0 when empty.  A record found there is kept only when
// its configured c-bin is a neighbour (checked exactly by the caller).  On
// an axis that is not refined the neighbours' extent is exact.
template <typename real>
__device__ __forceinline__ int fast_span(const Inst<real>& I, int ax, real x, double reach, int cc, bool periodic,
                                         int fa[2], int fb[2]) {
    const int nc = I.ncfg[ax], nf = I.n[ax];
    const double eps = 1e-3 + 1e-6 * (double)nf;
    const bool all = periodic && nc <= 3;  // every configured c-bin is a neighbour
    int lo = 0, hi = nf - 1;
    if (!all) {
        int c0 = cc - 1, c1 = cc + 1;
        if (!periodic) { c0 = c0 < 0 ? 0 : c0; c1 = c1 > nc - 1 ? nc - 1 : c1; }
        lo = c0;
        hi = c1;
        if (nf != nc) {
            const double r = (double)nf / (double)nc;
            lo = (int)floor((double)c0 * r - eps);
            hi = (int)floor((double)(c1 + 1) * r + eps);
        }
    }
    // The reach in fine c-bins (positions far outside the box keep the
    // neighbours' extent; bins of positions outside are clamped, as here).
    const double t = ((double)x - (double)I.lo[ax]) * (double)I.inv_w[ax];
    const double d = reach * (double)I.inv_w[ax];
    if (t > -0.5 * nf && t < 1.5 * nf) {
        int bl = (int)floor(t - d - eps), bh = (int)floor(t + d + eps);
        if (!periodic) {
            bl = bl < 0 ? 0 : (bl > nf - 1 ? nf - 1 : bl);
            bh = bh < 0 ? 0 : (bh > nf - 1 ? nf - 1 : bh);
        }
        if (all) { lo = bl; hi = bh; }
        else { lo = lo > bl ? lo : bl; hi = hi < bh ? hi : bh; }
    }
    if (hi < lo) return 0;
    if (!periodic) {
        fa[0] = lo < 0 ? 0 : lo;
        fb[0] = hi > nf - 1 ? nf - 1 : hi;
        return fb[0] >= fa[0] ? 1 : 0;
    }
    if (hi - lo + 1 >= nf) { fa[0] = 0; fb[0] = nf - 1; return 1; }
    const int k = floor_div(lo, nf);  // shift by whole periods so that 0 <= lo < nf
    lo -= k * nf;
    hi -= k * nf;
    if (hi > nf - 1) { fa[0] = lo; fb[0] = nf - 1; fa[1] = 0; fb[1] = hi - nf; return 2; }
    fa[0] = lo; fb[0] = hi;
    return 1;
}

// Index t of the concatenation of at most two ranges [a[r], b[r]].
__device__ __forceinline__ int span_at(const int a[2], const int b[2], int len0, int t) {
    return t < len0 ? a[0] + t : a[1] + (t - len0);
}

// The configured neighbours of configured c-bin cc along one axis as
// (first, count - 1), wrapped on a periodic axis: bin c is a neighbour when
// (c - first) mod n <= span.  check: whether a slow record the fast
// particle at coordinate x can reach may lie outside them, so that its
// configured c-bin has to be checked.  The neighbours extend at least one
// configured c-bin beyond the particle's own; a record beyond the reach
// cannot meet the criteria, and one within it lies inside the neighbours
// unless the reach (widened by the rounding margin of the binnings) crosses
// a side that has a configured c-bin beyond it.  On an axis that is not
// refined the fine rows hold exactly the neighbours.
template <typename real>
__device__ __forceinline__ void coarse_nb(const Inst<real>& I, int ax, real x, double reach, int cc, bool periodic,
                                          int& first, int& span, bool& check) {
    const int nc = I.ncfg[ax];
    check = false;
    if (periodic && nc <= 3) { first = 0; span = nc - 1; return; }
    if (periodic) { first = cc == 0 ? nc - 1 : cc - 1; span = 2; }
    else {
        first = cc > 0 ? cc - 1 : 0;
        span = (cc < nc - 1 ? cc + 1 : nc - 1) - first;
    }
    if (I.n[ax] == nc) return;
    const double eps = 1e-3 + 1e-6 * (double)nc;  // in configured c-bins
    const double t = ((double)x - (double)I.lo[ax]) * (double)I.inv_wc[ax];
    const double d = reach * (double)I.inv_wc[ax];
    const bool below = periodic || cc >= 2, above = periodic || cc <= nc - 3;
    check = (below && t - d < (double)(cc - 1) + eps) || (above && t + d > (double)(cc + 2) - eps);
}

// Whether a slow record at (x, y, z) lies in a configured c-bin neighbouring
// the fast particle's, on the axes that need the check.
template <typename real>
__device__ __forceinline__ bool coarse_in(const Inst<real>& I, const bool chk[3], const int nc[3], const int first[3],
                                          const int span[3], real x, real y, real z) {
    const real p[3] = {x, y, z};
    bool in = true;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        if (!chk[ax]) continue;
        int u = axis_bin(p[ax], I.lo[ax], I.inv_wc[ax], nc[ax]) - first[ax];
        u += u < 0 ? nc[ax] : 0;
        in = in && u <= span[ax];
    }
    return in;
}

// Reach of a fast particle of speed^2 v2 towards slow partners, with the
// margin of the c-bin refinement for the rounding of the pair test.
template <typename real>
__device__ __forceinline__ double fast_reach(const Inst<real>& I, double v2) {
    return (sqrt((double)I.D2) + (sqrt(v2) + sqrt((double)I.vc2)) * (double)I.dt) * (1.0 + 1.0 / 64.0);
}

// The search of fast record i by a whole wave.  Its rows (the fine rows of
// fast_span and the nine rows of configured c-bins of the fast particles, half
// neighbourhood) are found one per lane, and their records are then taken 64
// at a time from the rows laid end to end, so that a wave loads whole runs of
// records and its lanes stay busy however short the rows are.  Of `parts`
// waves that share a record, this one takes every parts-th 64.  Every
// candidate lowers both keys with atomicMin, in any order.
struct FastRows {
    int32_t end[kWave];  // inclusive prefix of the rows' lengths
    int4 row[kWave];     // place p: record x + p below place z, else y + p
};

template <typename real, bool MIX>
__device__ void fast_record(const StepArgs<real>& a, const Inst<real>& I, int64_t base, int32_t i, int part, int parts,
                            int lane, FastRows& R, uint32_t& seen, uint32_t& cand, uint32_t& n_s0, uint32_t& n_c1) {
    const Geo<real> G_(I);
    const bool by_time = (I.flags & TPKMC_RANK_TIME) != 0;
    const int nf[3] = {I.n[0], I.n[1], I.n[2]};
    const int nc[3] = {I.ncfg[0], I.ncfg[1], I.ncfg[2]};
    real pi[3], vxi, vyi, vzi;
    load_pv(a.rec, i, pi[0], pi[1], pi[2], vxi, vyi, vzi);
    const double reach = fast_reach(I, speed2((double)vxi, (double)vyi, (double)vzi));
    // The three axes' spans, found by a lane each.
    int cc[3], first[3], span[3], n_r[3], fa[3][2], fb[3][2];
    bool chk[3];
    {
        const int ax = min(lane, 2);
        const real p = ax == 0 ? pi[0] : ax == 1 ? pi[1] : pi[2];
        const bool per = ax == 0 ? G_.per[0] : ax == 1 ? G_.per[1] : G_.per[2];
        const int c = axis_bin(p, I.lo[ax], I.inv_wc[ax], I.ncfg[ax]);
        int f, s, a2[2] = {0, 0}, b2[2] = {0, 0};
        bool ck;
        coarse_nb(I, ax, p, reach, c, per, f, s, ck);
        const int r = fast_span(I, ax, p, reach, c, per, a2, b2);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            cc[l] = __builtin_amdgcn_readlane(c, l);
            first[l] = __builtin_amdgcn_readlane(f, l);
            span[l] = __builtin_amdgcn_readlane(s, l);
            chk[l] = __builtin_amdgcn_readlane((int)ck, l) != 0;
            n_r[l] = __builtin_amdgcn_readlane(r, l);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                fa[l][q] = __builtin_amdgcn_readlane(a2[q], l);
                fb[l][q] = __builtin_amdgcn_readlane(b2[q], l);
            }
        }
    }
    const int *xa = fa[0], *xb = fb[0], *ya = fa[1], *yb = fb[1], *za = fa[2], *zb = fb[2];
    const int nxr = n_r[0], nyr = n_r[1], nzr = n_r[2];
    const int ly0 = nyr ? yb[0] - ya[0] + 1 : 0, lz0 = nzr ? zb[0] - za[0] + 1 : 0;
    const int ny = ly0 + (nyr > 1 ? yb[1] - ya[1] + 1 : 0);
    const int nz = lz0 + (nzr > 1 ? zb[1] - za[1] + 1 : 0);
    const int slow = nxr ? ny * nz : 0;
    unsigned long long best = ~0ull;
    for (int r0 = 0; r0 < slow + 9; r0 += kWave) {
        const int t = r0 + lane;
        int32_t j0[2] = {0, 0}, len[2] = {0, 0};
        if (t < slow) {
            const int y = span_at(ya, yb, ly0, t % ny), z = span_at(za, zb, lz0, t / ny);
            const int64_t row = I.cell_off + (int64_t)nf[0] * row_of(I, y, z);
#pragma unroll
            for (int rx = 0; rx < 2; ++rx) {
                if (rx >= nxr) continue;
                j0[rx] = (int32_t)(base + a.start[row + xa[rx]]);
                len[rx] = (int32_t)(base + a.start[row + xb[rx] + 1]) - j0[rx];
            }
        } else if (t < slow + 9) {
            int k = 0;
            neighbourhood_row<true, true>(a.start, I, base, nc, G_.per, cc[0], cc[1], cc[2], i, t - slow,
                                          [&](int32_t u0, int32_t u1) {
                const int32_t l = max(u1 - u0, 0);
                if (k == 0) { j0[0] = u0; len[0] = l; }
                else { j0[1] = u0; len[1] = l; }
                ++k;
            });
        }
        int32_t end = len[0] + len[1];
        for (int o = 1; o < kWave; o <<= 1) {
            const int32_t v = __shfl_up(end, o);
            if (lane >= o) end += v;
        }
        const int32_t total = __builtin_amdgcn_readlane(end, kWave - 1);
        const int32_t second = end - len[1];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        R.end[lane] = end;
        R.row[lane] = make_int4(j0[0] - (second - len[0]), j0[1] - second, second, t);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int32_t p = part * kWave + lane; p < total; p += parts * kWave) {
            int o = 0;  // the row place p lies in: the rows that end at or before it
#pragma unroll
            for (int h = kWave / 2; h; h >>= 1) o += R.end[o + h - 1] <= p ? h : 0;
            const int4 row = R.row[o];
            const int32_t j = p + (p < row.z ? row.x : row.y);
            real xj, yj, zj, vxj, vyj, vzj;
            load_pv(a.rec, j, xj, yj, zj, vxj, vyj, vzj);
            if (row.w < slow && !coarse_in(I, chk, nc, first, span, xj, yj, zj)) continue;
            ++seen;
            if constexpr (MIX) {
                Screen<real> S;
                const bool p1 = PairTest<real, -1>::stage1(G_, pi[0], pi[1], pi[2], vxi, vyi, vzi, xj, yj, zj, vxj,
                                                           vyj, vzj, S);
                n_s0 += S.s0 < real(0) ? 1u : 0u;
                n_c1 += p1 ? 1u : 0u;
            } else {
                real value;
                if (!test_pair(G_, by_time, pi[0], pi[1], pi[2], vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, value))
                    continue;
                cand += 2;  // both orders
                Key<real>::lower(a, j, Key<real>::make(value, (uint32_t)i), key_now(a, j));
                const unsigned long long k = Key<real>::make(value, (uint32_t)j);
                if constexpr (sizeof(real) == 4) best = k < best ? k : best;
                else Key<real>::lower(a, i, k, key_now(a, i));
            }
        }
    }
    if constexpr (!MIX && sizeof(real) == 4)
        if (best != ~0ull) Key<real>::lower(a, i, best, key_now(a, i));
}

template <int G>
__device__ __forceinline__ void search_staged_for_axes(int pm, const StepArgs<float>& a, const Inst<float>& I,
                                                       int64_t base, int32_t wbase, int32_t stop, double& tests,
                                                       double& cand) {
#define TPKMC_STAGED(PMV) search_staged<PMV, G>(a, I, base, wbase, stop, tests, cand)
    // Builds for the periodic masks of the usual boxes (none; z, as in the
    // Noh implosions and the planar gases; y and z, as in the Sod tubes; all
    // three) leave the other axes out of the pair test.
    switch (pm) {
        case 0: TPKMC_STAGED(0); break;
        case 4: TPKMC_STAGED(4); break;
        case 6: TPKMC_STAGED(6); break;
        case 7: TPKMC_STAGED(7); break;
        default: TPKMC_STAGED(-1); break;
    }
#undef TPKMC_STAGED
}

// First and last (exclusive) live slow record of an instance; with split
// c-bins the fast ones after them are searched by k_search_fast.
template <typename real>
__device__ __forceinline__ int64_t slow_stop(const StepArgs<real>& a, const Inst<real>& I, int64_t base) {
    const int64_t end = I.off + I.cnt;
    const int64_t live = base + a.start[I.cell_off + ((I.flags & kSplit) ? I.Cf : I.C)];
    return live < end ? live : end;
}

// Adds a work-group's share of the search's work counters to entry's row.
__device__ __forceinline__ void add_work(double* gpart, int entry, double tests, double cand, double* lds) {
    const double t = block_sum(tests, lds);
    const double c = block_sum(cand, lds);
    if (threadIdx.x == 0 && (t != 0.0 || c != 0.0)) {
        double* gp = gpart + (int64_t)entry * kGPart;
        unsafeAtomicAdd(gp + GP_TESTS2, 2.0 * t);
        unsafeAtomicAdd(gp + GP_CAND, c);
    }
}

// FP32 search of the instances that do not go to the tiles (see search_cost).
// One table entry (kBlock records) is covered by kBlock / G lanes, split into work-groups of
// blockDim.x lanes, with one LDS staging buffer per wave
// (kStageBytesPerWave of dynamic LDS).
// The two-records-per-lane shape (the usual autotuner choice) is held to at
// most 72 VGPRs, 7 waves per SIMD (with a lane mode walking both records at
// once it needed 78, and the seventh wave was worth 3-4% on the search);
// with the staged lane mode, one record per pass, it needs 68.
template <int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 2 ? 7 : 1, 8)))
k_search(StepArgs<float> a) {
    __shared__ double lds[16];
    const int lanes = kBlock / G;
    const int sub = lanes / blockDim.x;
    const int lb = a.order > 0 ? xcd_chunk_remap(blockIdx.x, gridDim.x, a.order) : xcd_remap(blockIdx.x, gridDim.x);
    const int entry = lb / sub;
    const Blk bt = a.blk[entry];
    const Inst<float>& I = a.inst[bt.inst];
    if (I.flags & (TPKMC_PAIR_RANDOM | kTiles)) return;  // partners from k_rp_* or k_search_tiles
    const int64_t i0 = (int64_t)bt.first + ((int64_t)(lb % sub) * blockDim.x + (threadIdx.x & ~63u)) * G;
    const int64_t base = I.base;
    const int64_t stop = slow_stop(a, I, base);
    const int pm = (I.bc[0] == TPKMC_BC_PERIODIC ? 1 : 0) | (I.bc[1] == TPKMC_BC_PERIODIC ? 2 : 0) |
                   (I.bc[2] == TPKMC_BC_PERIODIC ? 4 : 0);
    double tests = 0.0, cand = 0.0;
    if (i0 < stop)  // wave-uniform: every lane of the wave takes part
        search_staged_for_axes<G>(pm, a, I, base, __builtin_amdgcn_readfirstlane((int32_t)i0), (int32_t)stop, tests,
                                  cand);
    add_work(a.gpart, entry, tests, cand, lds);
}

// FP64 search of the instances that do not go to the tiles (see search_cost),
// a record a lane; SPLIT: and a share of its rows (blockIdx.y), for launches too
// small to fill the chip.  What bounds it is the latency of the gathered
// records and of the row bounds: 1e6 particles at 0.3, 1 and 3 a c-bin take 92,
// 138 and 248 us (3D), 36, 42 and 56 as a thin tube along y, against 529, 241
// and 231, and 1982, 1729 and 1033 in tiles, which hold a row's records each.
// (The ordered scans that came before both: 255, 349 and 564; 72, 94 and 135.)
template <typename real, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_search_lanes(StepArgs<real> a) {
    __shared__ double lds[16];
    const int entry =
        a.order > 0 ? xcd_chunk_remap(blockIdx.x, gridDim.x, a.order) : xcd_remap(blockIdx.x, gridDim.x);
    const Blk bt = a.blk[entry];
    const Inst<real>& I = a.inst[bt.inst];
    if (I.flags & (TPKMC_PAIR_RANDOM | kTiles)) return;
    const int64_t i = (int64_t)bt.first + threadIdx.x;
    double tests = 0.0, cand = 0.0;
    if (i < slow_stop(a, I, I.base))
        search_lane<SPLIT>(a, I, (int32_t)i, (int)blockIdx.y, (int)gridDim.y, tests, cand);
    add_work(a.gpart, entry, tests, cand, lds);
}

// The instances of the tile search (see search_cost),
// one wave per 64 records and part of their neighbourhood (blockIdx.y).
template <typename real>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(real) == 4 ? 3 : 2)))
k_search_tiles(StepArgs<real> a) {
    __shared__ double lds[16];
    __shared__ TileLds<real> tl[kBlock / kWave];
    const int entry =
        a.order > 0 ? xcd_chunk_remap(blockIdx.x, gridDim.x, a.order) : xcd_remap(blockIdx.x, gridDim.x);
    const Blk bt = a.blk[entry];
    const Inst<real>& I = a.inst[bt.inst];
    if (!(I.flags & kTiles)) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t i0 = bt.first + wave * kWave;
    const int64_t stop = slow_stop(a, I, I.base);
    double cand = 0.0;
    if (i0 < stop) search_tiles(a, I, i0, (int32_t)stop, (int)blockIdx.y, (int)gridDim.y, tl[wave], cand);
    add_work(a.gpart, entry, 0.0, cand, lds);
}

// Diagnostic: counts of the pair tests (never part of a step).
template <typename real>
__global__ void __launch_bounds__(kBlock) k_search_mix(StepArgs<real> a) {
    __shared__ double lds[16];
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    if (I.flags & TPKMC_PAIR_RANDOM) return;
    const int64_t i = (int64_t)bt.first + threadIdx.x;
    const int64_t base = I.base;
    double tests = 0.0;
    uint32_t n_s0 = 0, n_c1 = 0;
    if (i < slow_stop(a, I, base)) count_mix(a, I, (int32_t)i, tests, n_s0, n_c1);
    const double t0 = block_sum(tests, lds), t1 = block_sum((double)n_s0, lds), t2 = block_sum((double)n_c1, lds);
    if (threadIdx.x == 0) {
        atomicAdd(a.mix + 0, (unsigned long long)t0);
        atomicAdd(a.mix + 1, (unsigned long long)t1);
        atomicAdd(a.mix + 2, (unsigned long long)t2);
    }
}

// The fast records of split c-bins, in a launch of their own after the slow
// ones' search (the keys combine with atomicMin in any order), one wave per
// record.  All instances' records are dealt to the waves in turn, as one list;
// an instance with fewer records than waves has up to kFastParts waves on each.
// It waits for its loads: with a lane per row of a record, each walking its
// row alone, the 4M tube took 0.164 ms, the 64-instance ensemble 4.6 ms late in
// its run; with a wave per record 0.066 and 0.80 ms.
constexpr int kFastParts = 8;
template <typename real, bool MIX = false>
__global__ void __launch_bounds__(256) k_search_fast(StepArgs<real> a, int n_inst) {
    __shared__ double lds[16];
    __shared__ FastRows rows[256 / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int own = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const uint32_t nw = gridDim.x * (256 / kWave), wave = blockIdx.x * (256 / kWave) + own;
    uint32_t turn = wave;  // this wave's first place in the instance's list
    uint32_t n_seen = 0, n_s0 = 0, n_c1 = 0;
    for (int k = 0; k < n_inst; ++k) {
        const Inst<real>& I = a.inst[k];
        if (!(I.flags & kSplit) || (I.flags & TPKMC_PAIR_RANDOM)) continue;
        const int64_t base = I.base;
        const int64_t f0 = base + a.start[I.cell_off + I.Cf];
        const int64_t live_end = base + a.start[I.cell_off + I.C];
        const int64_t f1 = live_end < I.off + I.cnt ? live_end : I.off + I.cnt;
        if (f1 <= f0) continue;
        const uint32_t n = (uint32_t)(f1 - f0), parts = n >= nw ? 1u : min(nw / n, (uint32_t)kFastParts);
        uint32_t seen = 0, cand = 0;
        uint64_t q = turn;
        for (; q < (uint64_t)n * parts; q += nw)
            fast_record<real, MIX>(a, I, base, (int32_t)(f0 + (uint32_t)q / parts), (int)((uint32_t)q % parts),
                                   (int)parts, lane, rows[own], seen, cand, n_s0, n_c1);
        turn = (uint32_t)(q - (uint64_t)n * parts);
        if constexpr (MIX) {
            n_seen += seen;
        } else if (__ballot(seen != 0)) {
            const double t = wave_reduce<false>((double)seen), c = wave_reduce<false>((double)cand);
            if (lane == 0) {
                double* gp = a.gpart + (int64_t)(I.blk0 + (int)(wave % (uint32_t)I.nblk)) * kGPart;
                unsafeAtomicAdd(gp + GP_TESTS2, 2.0 * t);
                unsafeAtomicAdd(gp + GP_CAND, c);
            }
        }
    }
    if constexpr (MIX) {
        const double t0 = block_sum((double)n_seen, lds), t1 = block_sum((double)n_s0, lds);
        const double t2 = block_sum((double)n_c1, lds);
        if (threadIdx.x == 0) {
            if (t0 > 0.0) atomicAdd(a.mix + 0, (unsigned long long)t0);
            if (t1 > 0.0) atomicAdd(a.mix + 1, (unsigned long long)t1);
            if (t2 > 0.0) atomicAdd(a.mix + 2, (unsigned long long)t2);
        }
    }
}

// Lexicographic minimum over the wave of (value, id) with a partner
// (j >= 0), the tie rule of the reference.
__device__ __forceinline__ void wave_best(int32_t& bj, double& bv, uint32_t& bid) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const int32_t oj = __shfl_xor(bj, m);
        const double ov = __shfl_xor(bv, m);
        const uint32_t oi = __shfl_xor(bid, m);
        if (oj >= 0 && (bj < 0 || ov < bv || (ov == bv && oi < bid))) { bj = oj; bv = ov; bid = oi; }
    }
}

// The partner of record i by the full ranking value and, where that is
// equal, the lower id: a whole wave scans every record that may be a
// candidate of i.  Without split c-bins, its neighbourhood; with them, the
// slow records (of the fine rows in reach of a fast i, of the neighbouring
// fine c-bins of a slow i) and the fast records of its configured
// neighbourhood.
inline __device__ void settle_tie(const StepArgs<double>& a, const Inst<double>& I, int64_t base, int32_t i, int lane) {
    const Geo<double> G(I);
    const bool by_time = (I.flags & TPKMC_RANK_TIME) != 0;
    const bool split = (I.flags & kSplit) != 0;
    const int nf[3] = {I.n[0], I.n[1], I.n[2]}, nc[3] = {I.ncfg[0], I.ncfg[1], I.ncfg[2]};
    double xi, yi, zi, vxi, vyi, vzi;
    uint32_t idi, fl;
    Rec<double>::load(a.rec, i, xi, yi, zi, idi, vxi, vyi, vzi, fl);
    const double pi[3] = {xi, yi, zi};
    int32_t bj = -1;
    double bv = 0.0;
    uint32_t bid = 0;
    int first[3] = {0, 0, 0}, span[3] = {0, 0, 0}, cc[3];
    bool chk[3] = {false, false, false};
    auto scan = [&](int32_t j0, int32_t j1, bool check) {
        for (int32_t j = j0 + lane; j < j1; j += kWave) {
            double xj, yj, zj, vxj, vyj, vzj;
            uint32_t idj, flj;
            Rec<double>::load(a.rec, j, xj, yj, zj, idj, vxj, vyj, vzj, flj);
            if (check && !coarse_in(I, chk, nc, first, span, xj, yj, zj)) continue;
            Screen<double> S;
            if (!PairTest<double, -1>::stage1(G, xi, yi, zi, vxi, vyi, vzi, xj, yj, zj, vxj, vyj, vzj, S)) continue;
            if (!PairTest<double, -1>::stage2(G, S)) continue;
            const double d2 = PairTest<double, -1>::finish(G, S);
            if (!(d2 >= 0.0)) continue;
            const double v = by_time ? PairTest<double, -1>::contact(G, S) : d2;
            if (bj < 0 || v < bv || (v == bv && idj < bid)) { bj = j; bv = v; bid = idj; }
        }
    };
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) cc[ax] = axis_bin(pi[ax], I.lo[ax], I.inv_wc[ax], nc[ax]);
    if (split && i >= base + a.start[I.cell_off + I.Cf]) {
        const double reach = fast_reach(I, speed2(vxi, vyi, vzi));
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) coarse_nb(I, ax, pi[ax], reach, cc[ax], G.per[ax], first[ax], span[ax], chk[ax]);
        int xa[2], xb[2], ya[2], yb[2], za[2], zb[2];
        const int nxr = fast_span(I, 0, xi, reach, cc[0], G.per[0], xa, xb);
        const int nyr = fast_span(I, 1, yi, reach, cc[1], G.per[1], ya, yb);
        const int nzr = fast_span(I, 2, zi, reach, cc[2], G.per[2], za, zb);
        const int ly0 = nyr ? yb[0] - ya[0] + 1 : 0, lz0 = nzr ? zb[0] - za[0] + 1 : 0;
        const int ny = ly0 + (nyr > 1 ? yb[1] - ya[1] + 1 : 0), nz = lz0 + (nzr > 1 ? zb[1] - za[1] + 1 : 0);
        for (int t = 0; t < ny * nz; ++t) {
            const int64_t row = I.cell_off + (int64_t)nf[0] * row_of(I, span_at(ya, yb, ly0, t % ny),
                                                                     span_at(za, zb, lz0, t / ny));
            for (int rx = 0; rx < nxr; ++rx)
                scan((int32_t)(base + a.start[row + xa[rx]]), (int32_t)(base + a.start[row + xb[rx] + 1]), true);
        }
    } else {
        for_logical(a, I, G.per, xi, yi, zi, [&](int32_t j0, int32_t j1) { scan(j0, j1, false); });
    }
    if (split)
        for_neighbourhood<false, true>(a.start, I, base, nc, G.per, cc[0], cc[1], cc[2], i,
                                       [&](int32_t j0, int32_t j1) { scan(j0, j1, false); });
    wave_best(bj, bv, bid);
    if (lane == 0 && bj >= 0) a.bkey[i] = (unsigned long long)(uint32_t)bj;
}

// FP64 records whose lowest key met an equal one (see Key): settled one by
// one, by a wave each.  Returns at once where there is none, the usual case.
template <typename real>
__global__ void __launch_bounds__(kBlock) k_search_ties(StepArgs<real> a) {
    if (*a.ties == 0u) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int entry = blockIdx.x; entry < a.nblk; entry += gridDim.x) {
        const Blk bt = a.blk[entry];
        const Inst<real>& I = a.inst[bt.inst];
        if (I.flags & TPKMC_PAIR_RANDOM) continue;
        const int64_t base = I.base;
        const int32_t i0 = bt.first + wave * kWave;
        const int64_t i = (int64_t)i0 + lane;
        uint64_t marked = __ballot(i < I.off + I.cnt && (a.coll[i] & Key<double>::mark(a.bkey[i])) != 0);
        while (marked) {
            const int l = __ffsll((long long)marked) - 1;
            marked &= marked - 1;
            settle_tie(a, I, base, i0 + l, lane);
        }
    }
}

// ---------------------------------------------------------------- 4b. random partners
// Random partners inside each c-bin (TPKMC_PAIR_RANDOM, the usual DSMC rule
// of Sec. 2.3) in place of the search: every live record gets a Philox key,
// the records of a c-bin are ranked by (key, id), and ranks (0, 1), (2, 3),
// ... pair up.  Three passes (launch boundaries order them): the keys; the
// rank of every record among its c-bin's (a loop over the c-bin, O(n_c^2)
// per c-bin like the neighbourhood search) with the c-bin-local order in
// perm; the partners.  The rank goes through `best` (free until the last
// pass writes the FP64 partner there) and the keys through `rank` (free
// after the scatter).

__device__ __forceinline__ uint32_t random_key(const uint32_t k0, const uint32_t k1, uint32_t step,
                                               uint32_t instance, uint32_t id) {
    uint32_t c[4] = {step, id, id, (instance << 8) | 255u};
    philox4x32_10(c, k0, k1);
    return c[0];
}

template <typename real> __device__ __forceinline__ uint32_t record_id(const real* rec, int64_t i);
template <> __device__ __forceinline__ uint32_t record_id<float>(const float* rec, int64_t i) {
    return reinterpret_cast<const uint32_t*>(rec)[8 * i + 3];
}
template <> __device__ __forceinline__ uint32_t record_id<double>(const double* rec, int64_t i) {
    return (uint32_t)reinterpret_cast<const unsigned long long*>(rec)[8 * i + 3];
}

// Rank (FP64: later the partner) and c-bin-local order of an instance's
// records, indexed from its first.  In FP64 they lie in the place of the keys,
// which an instance with random partners does not use.
template <typename real>
__device__ __forceinline__ int32_t* rp_best(const StepArgs<real>& a, const Inst<real>& I) {
    if constexpr (std::is_same<real, double>::value) return reinterpret_cast<int32_t*>(a.bkey + I.off);
    else return a.best + I.off;
}
template <typename real>
__device__ __forceinline__ int32_t* rp_perm(const StepArgs<real>& a, const Inst<real>& I) {
    if constexpr (std::is_same<real, double>::value) return reinterpret_cast<int32_t*>(a.bkey + I.off) + I.cnt;
    else return a.perm + I.off;
}

// Global c-bin of a record, from its position (the key kernel's arithmetic).
template <typename real>
__device__ __forceinline__ int64_t record_cbin(const Inst<real>& I, real x, real y, real z) {
    const int cx = axis_bin(x, I.lo[0], I.inv_w[0], I.n[0]);
    const int cy = axis_bin(y, I.lo[1], I.inv_w[1], I.n[1]);
    const int cz = axis_bin(z, I.lo[2], I.inv_w[2], I.n[2]);
    return I.cell_off + cx + (int64_t)I.n[0] * row_of(I, cy, cz);
}

template <typename real>
__global__ void __launch_bounds__(kBlock) k_rp_key(StepArgs<real> a) {
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    if (!(I.flags & TPKMC_PAIR_RANDOM)) return;
    const int64_t base = I.base;
    const int64_t live_end = base + a.start[I.cell_off + I.C];
    const int64_t i = (int64_t)bt.first + threadIdx.x;
    if (i < live_end && i < I.off + I.cnt)
        reinterpret_cast<uint32_t*>(a.rank)[i] =
            random_key(I.seed_lo, I.seed_hi, I.step_lo, I.instance, record_id<real>(a.rec, i));
}

template <typename real>
__global__ void __launch_bounds__(kBlock) k_rp_rank(StepArgs<real> a) {
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    if (!(I.flags & TPKMC_PAIR_RANDOM)) return;
    const int64_t base = I.base;
    const int64_t live_end = base + a.start[I.cell_off + I.C];
    const int64_t i = (int64_t)bt.first + threadIdx.x;
    if (!(i < live_end && i < I.off + I.cnt)) return;
    real x, y, z, vx, vy, vz;
    uint32_t id, fl;
    Rec<real>::load(a.rec, i, x, y, z, id, vx, vy, vz, fl);
    const int64_t k = record_cbin(I, x, y, z);
    const int64_t lo = base + a.start[k], hi = base + a.start[k + 1];
    const uint32_t* key = reinterpret_cast<const uint32_t*>(a.rank);
    const uint32_t mine = key[i];
    int32_t r = 0;
    for (int64_t j = lo; j < hi; ++j) {
        const uint32_t kj = key[j];
        r += (kj < mine || (kj == mine && record_id<real>(a.rec, j) < id)) ? 1 : 0;
    }
    rp_perm(a, I)[lo - I.off + r] = (int32_t)i;
    rp_best(a, I)[i - I.off] = r;
}

template <typename real>
__global__ void __launch_bounds__(kBlock) k_rp_partner(StepArgs<real> a) {
    __shared__ double lds[16];
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    if (!(I.flags & TPKMC_PAIR_RANDOM)) return;
    const int64_t base = I.base;
    const int64_t live_end = base + a.start[I.cell_off + I.C];
    const int64_t i = (int64_t)bt.first + threadIdx.x;
    double formed = 0.0, paired = 0.0;
    if (i < I.off + I.cnt) {
        int32_t partner = -1;
        if (i < live_end) {
            real x, y, z, vx, vy, vz;
            uint32_t id, fl;
            Rec<real>::load(a.rec, i, x, y, z, id, vx, vy, vz, fl);
            const int64_t k = record_cbin(I, x, y, z);
            const int64_t lo = base + a.start[k], nc = base + a.start[k + 1] - lo;
            const int32_t r = rp_best(a, I)[i - I.off], q = r ^ 1;
            if (q < nc) {
                partner = rp_perm(a, I)[lo - I.off + q];
                paired = 1.0;
                formed = (r & 1) == 0 ? 1.0 : 0.0;
            }
        }
        if constexpr (std::is_same<real, double>::value) rp_best(a, I)[i - I.off] = partner;
        else a.bkey[i] = partner >= 0 ? (unsigned long long)(uint32_t)partner : ~0ull;
    }
    const double f = block_sum(formed, lds);
    const double c = block_sum(paired, lds);
    if (threadIdx.x == 0 && (f != 0.0 || c != 0.0)) {
        double* gp = a.gpart + (int64_t)blockIdx.x * kGPart;
        unsafeAtomicAdd(gp + GP_TESTS2, 2.0 * f);
        unsafeAtomicAdd(gp + GP_CAND, c);
    }
}

// Whether the random pair of record i (position x, y, z) and its partner
// collides: u < (((n_c - 1) sigma) g) dt / V_c in double, with the pair's own
// Philox draw; both records of the pair take the same decision.
template <typename real>
__device__ __forceinline__ bool random_pair_collides(const StepArgs<real>& a, const Inst<real>& I, real x, real y,
                                                     real z, uint32_t idi, real vxi, real vyi, real vzi,
                                                     uint32_t idj, real vxj, real vyj, real vzj) {
#pragma clang fp contract(off)
    const bool iA = idi < idj;
    const double ux = iA ? (double)vxi - (double)vxj : (double)vxj - (double)vxi;
    const double uy = iA ? (double)vyi - (double)vyj : (double)vyj - (double)vyi;
    const double uz = iA ? (double)vzi - (double)vzj : (double)vzj - (double)vzi;
    const double g = sqrt((ux * ux + uy * uy) + uz * uz);
    const int64_t k = record_cbin(I, x, y, z);
    const int64_t nc = (int64_t)a.start[k + 1] - a.start[k];
    const double prob = ((((double)(nc - 1) * I.sigma_d) * g) * I.dt_d) / I.cellvol_d;
    uint32_t c[4] = {I.step_lo, iA ? idi : idj, iA ? idj : idi, (I.instance << 8) | 255u};
    philox4x32_10(c, I.seed_lo, I.seed_hi);
    const double u = ((double)(c[0] >> 5) * 67108864.0 + (double)(c[1] >> 6)) * (1.0 / 9007199254740992.0);
    return u < prob;
}

// ---------------------------------------------------------------- 5. move
// Partner record of record i after the search, or -1 (random partners of an
// FP64 state come as plain indices in `best`).
template <typename real>
__device__ __forceinline__ int32_t partner_of(const StepArgs<real>& a, const Inst<real>& I, int64_t i) {
    if constexpr (std::is_same<real, double>::value)
        if (I.flags & TPKMC_PAIR_RANDOM) return rp_best(a, I)[i - I.off];
    const unsigned long long k = a.bkey[i];
    return k == ~0ull ? -1 : Key<real>::partner(k);
}

// o-bin (with the instance's offset) of a position.
template <typename real>
__device__ __forceinline__ int obin_of(const Inst<real>& I, real x, real y, real z) {
    const int bx = axis_bin(x, I.lo[0], I.inv_wo[0], I.no[0]);
    const int by = axis_bin(y, I.lo[1], I.inv_wo[1], I.no[1]);
    const int bz = axis_bin(z, I.lo[2], I.inv_wo[2], I.no[2]);
    return (int)(I.obin_off + bx + (int64_t)I.no[0] * (by + (int64_t)I.no[1] * bz));
}

// ------------------------------------------------------- exact o-bin sums
// The moment terms of one particle (kinds as in ObAcc), computed the same
// way in both passes: m (v - shift), m (v - shift)^2, the virial terms and
// the mass.
__device__ __forceinline__ void moment_terms(double m, double vx, double vy, double vz, const double* S,
                                             double virx, double viry, double virz, double t[kAccVals]) {
    const double ex = vx - S[0], ey = vy - S[1], ez = vz - S[2];
    t[0] = m * ex; t[1] = m * ey; t[2] = m * ez;
    t[3] = t[0] * ex; t[4] = t[1] * ey; t[5] = t[2] * ez;
    t[6] = virx; t[7] = viry; t[8] = virz;
    t[9] = m;
}

// Biased exponent E + kExpBias of the smallest power of two 2^E > |x| (0 for
// x = 0), from the exponent bits (below the normal doubles one value serves:
// the quantum is the same there, see fixed_scale).
__device__ __forceinline__ int exp_above(double x) {
    const int hi = __double2hiint(x) & 0x7fffffff;
    const int e = max(hi >> 20, 1) + (1 - 1023 + kExpBias);
    return (hi | __double2loint(x)) != 0 ? e : 0;
}

// x rounded to the nearest multiple of 2^(E-50), in units of that quantum;
// scale = 2^(50-E) and |x| < 2^E, so |x scale| < 2^50.  Adding 1.5 2^52
// rounds x scale to an integer (nearest, ties to even; the product is exact)
// and leaves that integer plus 2^51 in the low mantissa bits.
__device__ __forceinline__ long long to_fixed(double x, double scale) {
    constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
    return __double_as_longlong(fma(x, scale, kMagic)) - 0x4338000000000000ll;
}

// 2^(50-h-E) for a biased exponent E and headroom h, kept a normal double.
__device__ __forceinline__ double fixed_scale(int eb, int h) {
    const int e = eb > 0 ? eb - kExpBias : 0;
    return ldexp(1.0, 50 - h - max(e, -969));
}

template <int CTRL>
__device__ __forceinline__ long long dpp_move64(long long v) {
    const uint32_t l0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, false);
    const uint32_t l1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)((unsigned long long)v >> 32), CTRL,
                                                           0xF, 0xF, false);
    return (long long)(((unsigned long long)l1 << 32) | l0);
}

// Adds one work-group (or lane) sum of a value to the global sum of an
// o-bin (one int64; see ObAcc for the bound).
__device__ __forceinline__ void global_acc_add(ObAcc& G, int k, long long v) {
    if (v) atomicAdd((unsigned long long*)&G.sum[k], (unsigned long long)v);
}

// Work-group tables keyed by o-bin (open addressing), flushed to the global
// accumulators once per work-group: exponent maxima in the move, value sums
// in the moment pass.  Probes are limited: where a work-group meets more
// o-bins than the table holds, the rest go to the global accumulators at once
// instead of probing the whole table first (DSMC box of 2e5, 6 particles an
// o-bin: move 25 -> 21 us, moments 34 -> 24; 16M blast: move 476 -> 447).
// The moment pass takes more of them, since a global add there is 8 atomics
// wide (16M blast at 8 probes: 377 us, at 24: 362).
constexpr int kSlots = 64;       // exponent table (the move's 256 records)
constexpr int kMomSlots = 128;   // value table (the moment pass's kMomEntries * 256 records)
constexpr int kTabWords = kAccVals;  // the values' integer sums
struct MomentTable {
    static constexpr int kN = kMomSlots, kProbes = 24;
    int key[kN];
    long long val[kN][kTabWords];
};
struct ExpTable {
    static constexpr int kN = kSlots, kProbes = 8;
    int key[kN];
    int e[kN][4];
    uint32_t n[kN][2];  // particles, colliders
};

template <typename Table>
__device__ __forceinline__ int table_slot(Table& T, int ob) {
    constexpr int N = Table::kN;
    const int h = (int)((ob * 0x9E3779B1u) >> 24);  // 8 bits
// Unrolled, the moment pass took 359 us instead of 303 on the 20M equilibrium.
#pragma unroll 1
    for (int probe = 0; probe < Table::kProbes; ++probe) {
        const int s = (h + probe) & (N - 1);
        const int cur = T.key[s];
        if (cur == ob) return s;
        if (cur == -1) {
            const int prev = atomicCAS(&T.key[s], -1, ob);
            if (prev == -1 || prev == ob) return s;
        }
    }
    return -1;
}

// Runs of one o-bin across the lanes of a wave: whether this lane starts
// one, and lim = the lanes of its run inside its row of 16 lanes, from this
// lane on (for a segmented maximum by DPP row shifts of 1, 2, 4 and 8).
__device__ __forceinline__ int row_lim(int mob, int lane, bool& head) {
    const int prev_mob = __shfl_up(mob, 1);
    head = lane == 0 || prev_mob != mob;
    const uint64_t heads = __ballot(head);
    const uint64_t after = heads & ~lanes_le(lane);
    const int seg1 = after ? __ffsll((long long)after) - 1 : 64;
    const int rl = lane & 15;
    return min(seg1, lane - rl + 16) - lane;
}

__device__ __forceinline__ long long row_sum64(long long v, int lim) {
    long long u = dpp_move64<kRowShl1>(v);
    if (1 < lim) v += u;
    u = dpp_move64<kRowShl2>(v);
    if (2 < lim) v += u;
    u = dpp_move64<kRowShl4>(v);
    if (4 < lim) v += u;
    u = dpp_move64<kRowShl8>(v);
    if (8 < lim) v += u;
    return v;
}

__device__ __forceinline__ uint32_t row_sum32(uint32_t v, int lim) {
    uint32_t u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl1, 0xF, 0xF, false);
    if (1 < lim) v += u;
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl2, 0xF, 0xF, false);
    if (2 < lim) v += u;
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl4, 0xF, 0xF, false);
    if (4 < lim) v += u;
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl8, 0xF, 0xF, false);
    if (8 < lim) v += u;
    return v;
}

// The same for the maxima of two 16-bit numbers at once.
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t max16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a),
                                                                  __builtin_bit_cast(ushort2_t, b)));
}
__device__ __forceinline__ uint32_t row_max16(uint32_t v, int lim) {
    uint32_t u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl1, 0xF, 0xF, false);
    if (1 < lim) v = max16(v, u);
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl2, 0xF, 0xF, false);
    if (2 < lim) v = max16(v, u);
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl4, 0xF, 0xF, false);
    if (4 < lim) v = max16(v, u);
    u = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kRowShl8, 0xF, 0xF, false);
    if (8 < lim) v = max16(v, u);
    return v;
}

// Sums over each row of 16 lanes, in a fixed order; every lane must be
// active.  row_sum4: of four doubles at once, lane l getting the sum of value
// l & 3 (each exchange halves the values a lane still carries, 27
// instructions instead of 92 for four whole reductions).
template <bool MAX>
__device__ __forceinline__ double row_reduce(double v) {
    auto op = [](double x, double y) { return MAX ? fmax(x, y) : x + y; };
    v = op(v, dpp_move<kQuadXor1>(v));
    v = op(v, dpp_move<kQuadXor2>(v));
    v = op(v, dpp_move<kRowRor4>(v));
    return op(v, dpp_move<kRowRor8>(v));
}
__device__ __forceinline__ double row_sum4(double v0, double v1, double v2, double v3, int lane) {
    const bool odd = lane & 1, high = lane & 2;
    const double a = (odd ? v1 : v0) + dpp_move<kQuadXor1>(odd ? v0 : v1);
    const double b = (odd ? v3 : v2) + dpp_move<kQuadXor1>(odd ? v2 : v3);
    double r = (high ? b : a) + dpp_move<kQuadXor2>(high ? a : b);
    r += dpp_move<kRowRor4>(r);
    return r + dpp_move<kRowRor8>(r);
}

template <typename real>
__device__ __forceinline__ ObExp& exp_of(const StepArgs<real>& a, int64_t ob) {
    return *reinterpret_cast<ObExp*>(a.mexp + ob * a.exp_stride);
}

// A lane's run maxima and counts of one o-bin into the work-group table, or
// straight into the global accumulators when the table is full.
template <typename real>
__device__ __forceinline__ void exp_flush(ExpTable& tab, const StepArgs<real>& a, int ob, const int* e, uint32_t cnt,
                                          uint32_t coll) {
    const int slot = table_slot(tab, ob);
    int* d = slot >= 0 ? tab.e[slot] : nullptr;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!e[k]) continue;
        if (d) atomicMax(d + k, e[k]);
        else atomicMax(&exp_of(a, ob).e[k], e[k]);
    }
    if (d) {
        if (cnt) atomicAdd(&tab.n[slot][0], cnt);
        if (coll) atomicAdd(&tab.n[slot][1], coll);
    } else if (cnt) {
        atomicAdd(&exp_of(a, ob).nc, (unsigned long long)cnt | ((unsigned long long)coll << 32));
    }
}

// Unambiguous pairs (each the other's closest candidate) scatter; every
// particle moves and meets the walls; global sums; with moments, the first
// pass of the exact o-bin sums (see ObAcc): the exponent maxima, and each
// particle's collider flag and virial terms for the moment pass.  One record
// per lane.  The new state goes to the caller's arrays (c-bin order kept), to
// records in a second buffer that the moment pass reads and puts back in the
// caller's order, or, where there is no room for that, scattered into the
// caller's arrays.
// On the 16M blast it takes 0.44 ms; without the o-bin part it takes 0.28,
// near what its 85 B a particle need, so the o-bins' exponents are taken from
// the bits of the largest term per kind and their counts by votes.
template <typename real>
__global__ void __launch_bounds__(kBlock) k_move(StepArgs<real> a) {
    __shared__ ExpTable tab;
    // Per row of 16 lanes: momentum, kinetic energy, max |v|^2, virial, mass;
    // per wave: alive, pairs, absorbed, with a partner.
    constexpr int kWaves = kBlock / kWave, kRows16 = kBlock / 16;
    __shared__ double red[kRows16][7];
    __shared__ int votes[kWaves][4];
    // Consecutive work-groups on one XCD: partners' records and keys, a few
    // c-bins away in record order, are then mostly in that XCD's L2.
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const Blk bt = a.blk[lb];
    const Inst<real>& I = a.inst[bt.inst];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int64_t end = I.off + I.cnt;
    const bool reorder = (I.flags & TPKMC_ALLOW_REORDER) != 0;
    const bool has_mass = (I.flags & kHasMass) != 0;
    if (a.macc) {
        for (int t = tid; t < kSlots; t += kBlock) {
            tab.key[t] = -1;
            for (int k = 0; k < 4; ++k) tab.e[t][k] = 0;
            tab.n[t][0] = tab.n[t][1] = 0;
        }
        __syncthreads();
    }
    double gpx = 0, gpy = 0, gpz = 0, gek = 0, gvm = 0, gvir = 0, gm = 0;
    bool counted = false, first_of_pair = false, absorbed = false, has_best = false;
    int mob = -1;                              // o-bin
    uint32_t me01 = 0, me23 = 0;               // exponents per kind, two a word
    bool collider = false;
    const int64_t i = (int64_t)bt.first + tid;
    uint32_t emit_a = 0, emit_b = 0;
    {
        real x = 0, y = 0, z = 0, vx = 0, vy = 0, vz = 0;
        uint32_t idi = 0, fl = 0;
        int32_t j_pre = -1;
        if (i < end) {
            Rec<real>::load(a.rec, i, x, y, z, idi, vx, vy, vz, fl);
            j_pre = partner_of<real>(a, I, i);
        }
        if (i < end) {
            // Where the state, and its collider flag and virial terms, go.
            const bool direct = reorder || !a.rec2;
            const int64_t dst = reorder || a.rec2 ? i : (int64_t)a.src[i];
            const bool alive = (fl & 1u) != 0;
            if (!alive) {
                if (!direct) Rec<real>::store(a.rec2, i, x, y, z, idi, vx, vy, vz, kRecDead);
                if (reorder) {
                    a.x[dst] = x; a.y[dst] = y; a.z[dst] = z;
                    a.vx[dst] = vx; a.vy[dst] = vy; a.vz[dst] = vz;
                    a.id[dst] = idi;
                    if (a.alive) a.alive[dst] = 0;
                    if (has_mass) a.mass[dst] = a.rmass[i];
                }
            } else {
                const real dt = I.dt;
                const real mi = has_mass ? a.rmass[i] : I.mass;
                const int32_t j = j_pre;
                bool mutual = j >= 0 && partner_of<real>(a, I, j) == (int32_t)i;
                has_best = j >= 0;
                real nx = x, ny = y, nz = z, nvx = vx, nvy = vy, nvz = vz;
                double virx = 0, viry = 0, virz = 0;
                const bool random_pairs = (I.flags & TPKMC_PAIR_RANDOM) != 0;
                real xj = 0, yj = 0, zj = 0, vxj = 0, vyj = 0, vzj = 0;
                uint32_t idj = 0, flj = 0;
                if (mutual) {
                    Rec<real>::load(a.rec, j, xj, yj, zj, idj, vxj, vyj, vzj, flj);
                    if (random_pairs)
                        mutual = random_pair_collides(a, I, x, y, z, idi, vx, vy, vz, idj, vxj, vyj, vzj);
                }
                if (mutual) {
                    const bool isA = idi < idj;
                    // Pair quantities with A = lower id, B = higher id.
                    const real xA = isA ? x : xj, yA = isA ? y : yj, zA = isA ? z : zj;
                    const real xB = isA ? xj : x, yB = isA ? yj : y, zB = isA ? zj : z;
                    const real vxA = isA ? vx : vxj, vyA = isA ? vy : vyj, vzA = isA ? vz : vzj;
                    const real vxB = isA ? vxj : vx, vyB = isA ? vyj : vy, vzB = isA ? vzj : vz;
                    real rx = xA - xB, ry = yA - yB, rz = zA - zB;
                    if (I.bc[0] == TPKMC_BC_PERIODIC) rx = min_image(rx, I.L[0], real(0.5) * I.L[0]);
                    if (I.bc[1] == TPKMC_BC_PERIODIC) ry = min_image(ry, I.L[1], real(0.5) * I.L[1]);
                    if (I.bc[2] == TPKMC_BC_PERIODIC) rz = min_image(rz, I.L[2], real(0.5) * I.L[2]);
                    const real ux = vxA - vxB, uy = vyA - vyB, uz = vzA - vzB;
                    const real s0 = (rx * ux + ry * uy) + rz * uz;
                    const real vv = (ux * ux + uy * uy) + uz * uz;
                    // Random partners collide at the start of the step.
                    const real tp = random_pairs ? real(0) : -s0 / vv;
                    double nh[3];
                    pair_direction(I.seed_lo, I.seed_hi, I.step_lo, I.instance, isA ? idi : idj, isA ? idj : idi,
                                   (I.flags & TPKMC_PLANAR) != 0, nh);
                    // Centre-of-mass velocity and relative speed g kept, outgoing
                    // directions opposite along nhat.  Equal masses: the mean
                    // velocity, each moving g/2; masses mA, mB: the
                    // mass-weighted mean, A moving mB g / (mA + mB) and B
                    // mA g / (mA + mB).
                    const real g = sqrt(vv);
                    const real sg = isA ? real(1) : real(-1);
                    if (!has_mass) {
                        const real h = real(0.5) * g;
                        const real cmx = real(0.5) * (vxA + vxB), cmy = real(0.5) * (vyA + vyB),
                                   cmz = real(0.5) * (vzA + vzB);
                        const real hx = h * (real)nh[0], hy = h * (real)nh[1], hz = h * (real)nh[2];
                        nvx = isA ? cmx + hx : cmx - hx;
                        nvy = isA ? cmy + hy : cmy - hy;
                        nvz = isA ? cmz + hz : cmz - hz;
                    } else {
                        const real mj = a.rmass[j];
                        const real mA = isA ? mi : mj, mB = isA ? mj : mi;
                        const real M = mA + mB;
                        const real hA = (mB / M) * g, hB = (mA / M) * g;
                        const real cmx = (mA * vxA + mB * vxB) / M, cmy = (mA * vyA + mB * vyB) / M,
                                   cmz = (mA * vzA + mB * vzB) / M;
                        nvx = isA ? cmx + hA * (real)nh[0] : cmx - hB * (real)nh[0];
                        nvy = isA ? cmy + hA * (real)nh[1] : cmy - hB * (real)nh[1];
                        nvz = isA ? cmz + hA * (real)nh[2] : cmz - hB * (real)nh[2];
                    }
                    // Split move at the point of closest approach.
                    const real rest = dt - tp;
                    nx = (x + vx * tp) + nvx * rest;
                    ny = (y + vy * tp) + nvy * rest;
                    nz = (z + vz * tp) + nvz * rest;
                    // Virial: separation at closest approach (from the partner to
                    // this particle) times this particle's momentum change.
                    const real sx = sg * (rx + tp * ux), sy = sg * (ry + tp * uy), sz = sg * (rz + tp * uz);
                    virx = (double)(real(0.5) * sx * (mi * (nvx - vx)) / dt);
                    viry = (double)(real(0.5) * sy * (mi * (nvy - vy)) / dt);
                    virz = (double)(real(0.5) * sz * (mi * (nvz - vz)) / dt);
                    first_of_pair = isA;
                    emit_a = idi;
                    emit_b = idj;
                } else {
                    nx = x + vx * dt;
                    ny = y + vy * dt;
                    nz = z + vz * dt;
                }
                // Walls, once per axis.
                bool gone = false;
                real* pos[3] = {&nx, &ny, &nz};
                real* vel[3] = {&nvx, &nvy, &nvz};
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    const real lo = I.lo[ax], hi = I.hi[ax], q = *pos[ax];
                    if (I.bc[ax] == TPKMC_BC_REFLECT) {
                        if (q < lo) { *pos[ax] = lo + (lo - q); *vel[ax] = -*vel[ax]; }
                        else if (q > hi) { *pos[ax] = hi - (q - hi); *vel[ax] = -*vel[ax]; }
                    } else if (I.bc[ax] == TPKMC_BC_PERIODIC) {
                        real r = q;
                        if (r < lo) r = r + I.L[ax];
                        if (r >= hi) r = r - I.L[ax];
                        *pos[ax] = r;
                    } else {
                        if (q < lo || q >= hi) gone = true;
                    }
                }
                absorbed = gone;
                if (direct) {
                    a.x[dst] = nx; a.y[dst] = ny; a.z[dst] = nz;
                    a.vx[dst] = nvx; a.vy[dst] = nvy; a.vz[dst] = nvz;
                    if (reorder) a.id[dst] = idi;
                    if (reorder && has_mass) a.mass[dst] = mi;
                    if (a.alive && (reorder || gone)) a.alive[dst] = gone ? 0 : 1;
                } else {
                    Rec<real>::store(a.rec2, i, nx, ny, nz, idi, nvx, nvy, nvz, gone ? kRecAbsorbed : kRecAlive);
                }
                const bool fin = finite3(nx, ny, nz) && finite3(nvx, nvy, nvz) &&
                                 (!has_mass || (mi > real(0) && mi < real(INFINITY)));
                if (!gone && fin) {
                    const double m = has_mass ? (double)mi : I.mass_d;
                    const double dvx = (double)nvx, dvy = (double)nvy, dvz = (double)nvz;
                    const double v2 = (dvx * dvx + dvy * dvy) + dvz * dvz;
                    gpx += m * dvx; gpy += m * dvy; gpz += m * dvz;
                    gek += (0.5 * m) * v2;
                    gvm = v2;
                    gvir = (virx + viry) + virz;
                    gm = m;
                    counted = true;
                    if (a.macc) {
                        mob = obin_of(I, nx, ny, nz);
                        const double* S = a.shift + (int64_t)mob * 3;
                        // The largest term of a kind is that of the largest
                        // offset (rounding keeps the order).
                        const double e = fmax(fmax(fabs(dvx - S[0]), fabs(dvy - S[1])), fabs(dvz - S[2]));
                        const double t0 = m * e, t1 = t0 * e;
                        me01 = (uint32_t)exp_above(t0) | (uint32_t)exp_above(t1) << 16;
                        if (mutual) me23 = (uint32_t)exp_above(fmax(fmax(fabs(virx), fabs(viry)), fabs(virz)));
                        if (has_mass) me23 |= (uint32_t)exp_above(m) << 16;
                        collider = mutual;
                        a.coll[dst] = mutual ? 1 : 0;
                        if (mutual) {
                            a.vir[3 * dst] = (real)virx;
                            a.vir[3 * dst + 1] = (real)viry;
                            a.vir[3 * dst + 2] = (real)virz;
                        }
                    }
                }
            }
        }
        // Pair list: one atomic per wave.
        if (a.pairs) {
            const bool emit = first_of_pair && (I.flags & TPKMC_EMIT_PAIRS) != 0;
            const uint64_t em = __ballot(emit);
            if (em) {
                const int leader = __ffsll((long long)em) - 1;
                unsigned long long pos0 = 0;
                if (lane == leader) pos0 = atomicAdd(a.pair_count, (unsigned long long)__popcll(em));
                pos0 = __shfl(pos0, leader);
                if (emit) {
                    const unsigned long long pos = pos0 + __popcll(em & ((1ull << lane) - 1ull));
                    if ((int64_t)pos < a.pair_cap) {
                        a.pairs[2 * pos] = emit_a;
                        a.pairs[2 * pos + 1] = emit_b;
                    }
                }
            }
        }
    }
    if (a.macc) {
        // Consecutive lanes hold consecutive records, so their o-bins come in
        // runs: within each row of 16 lanes the run's maxima and counts go to
        // its first lane, which alone goes through the work-group's table;
        // then the table goes to the global accumulators.
        bool head;
        const int lim = row_lim(mob, lane, head);
        me01 = row_max16(me01, lim);
        if (__ballot(me23 != 0)) me23 = row_max16(me23, lim);  // wave-uniform
        const uint32_t n = row_sum32(mob >= 0 ? (collider ? 0x10001u : 1u) : 0u, lim);
        if ((head || (lane & 15) == 0) && mob >= 0) {
            const int e[4] = {(int)(me01 & 0xffffu), (int)(me01 >> 16), (int)(me23 & 0xffffu), (int)(me23 >> 16)};
            exp_flush(tab, a, mob, e, n & 0xffffu, n >> 16);
        }
        __syncthreads();
        for (int t = tid; t < kSlots * 5; t += kBlock) {
            const int slot = t / 5, k = t % 5;
            const int ob = tab.key[slot];
            if (ob < 0) continue;
            if (k < 4) {
                if (tab.e[slot][k]) atomicMax(&exp_of(a, ob).e[k], tab.e[slot][k]);
            } else if (tab.n[slot][0]) {
                atomicAdd(&exp_of(a, ob).nc,
                          (unsigned long long)tab.n[slot][0] | ((unsigned long long)tab.n[slot][1] << 32));
            }
        }
    }
    // Global sums: over rows of 16 lanes here, the rows in order below.
    const uint64_t nalive = __ballot(counted), npairs = __ballot(first_of_pair), nabs = __ballot(absorbed),
                   nhave = __ballot(has_best);
    const double s4 = row_sum4(gpx, gpy, gpz, gek, lane);
    const double vm = row_reduce<true>(gvm);
    double vir = 0.0, mass = 0.0;
    if (__ballot(gvir != 0.0)) vir = row_reduce<false>(gvir);  // wave-uniform
    if (has_mass) mass = row_reduce<false>(gm);
    const int row = tid >> 4;
    if ((lane & 15) < 4) red[row][lane & 3] = s4;
    if ((lane & 15) == 0) {
        red[row][4] = vm;
        red[row][5] = vir;
        red[row][6] = mass;
    }
    if (lane == 0) {
        int* w = votes[tid >> 6];
        w[0] = __popcll(nalive);
        w[1] = __popcll(npairs);
        w[2] = __popcll(nabs);
        w[3] = __popcll(nhave);
    }
    __syncthreads();
    double* gp = a.gpart + (int64_t)lb * kGPart;
    if (tid < 7) {
        double v = red[0][tid];
        for (int r = 1; r < kRows16; ++r) v = tid == 4 ? fmax(v, red[r][tid]) : v + red[r][tid];
        if (tid == 6 && !has_mass) {
            int n = 0;
            for (int w = 0; w < kWaves; ++w) n += votes[w][0];
            v = (double)n * I.mass_d;
        }
        gp[GP_PX + tid] = v;  // momentum, kinetic energy, max |v|^2, virial, mass
    } else if (tid >= kWave && tid < kWave + 4) {
        const int k = tid - kWave;
        int n = 0;
        for (int w = 0; w < kWaves; ++w) n += votes[w][k];
        gp[k == 3 ? GP_HAVEBEST : GP_ALIVE + k] = (double)n;  // alive, pairs, absorbed
    }
}

// Second pass of the exact o-bin sums (see ObAcc), over the step's output
// state in record order, one record per lane in the move's blocks: each
// term is rounded to its o-bin's quantum; the integers of the lanes of one
// o-bin run are summed within each row of 16 lanes, then in the
// work-group's table, then into the global accumulators.  The sums are
// integers, so none of these orders is visible.  One record per lane, with
// the block and its instance uniform over the work-group (scalar loads),
// measured fastest on the sparse 16M Sedov blast; several consecutive
// records per lane lose more to their strided loads than they save.
template <typename real>
__device__ __forceinline__ void value_flush(MomentTable& tab, const StepArgs<real>& a, int ob, const long long* q) {
    const int slot = table_slot(tab, ob);
    if (slot >= 0) {
        unsigned long long* T = reinterpret_cast<unsigned long long*>(tab.val[slot]);
#pragma unroll
        for (int k = 0; k < kAccVals; ++k)
            if (q[k]) atomicAdd(T + k, (unsigned long long)q[k]);
    } else {
        ObAcc& G = a.macc[ob];
#pragma unroll
        for (int k = 0; k < kAccVals; ++k) global_acc_add(G, k, q[k]);
    }
}

// Block-table entries per work-group of the moment pass: its table sums the
// records of each o-bin over that many entries before the global atomics
// (measured with 1, 2, 4 and 8: 3.12, 3.05, 3.08 and 3.20 ms/step on the
// 16M Sedov blast, 1.18, 1.16, 1.16 and 1.17 on the Sod 4M tube).
constexpr int kMomEntries = 2;

// RECS: some instance keeps the caller's order by way of the second records.
template <typename real, bool RECS>
__global__ void __launch_bounds__(kBlock) k_moments(StepArgs<real> a) {
    __shared__ MomentTable tab;
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    for (int t = tid; t < kMomSlots; t += kBlock) tab.key[t] = -1;
    for (int t = tid; t < kMomSlots * kTabWords; t += kBlock) (&tab.val[0][0])[t] = 0;
    __syncthreads();
    for (int ent = 0; ent < kMomEntries; ++ent) {
        const int entry = lb * kMomEntries + ent;
        if (entry >= a.nblk) break;  // uniform
        const Blk bt = a.blk[entry];
        const Inst<real>& I = a.inst[bt.inst];
        const int64_t end = I.off + I.cnt;
        const bool reorder = (I.flags & TPKMC_ALLOW_REORDER) != 0;
        const bool has_mass = (I.flags & kHasMass) != 0;
        const int64_t i = (int64_t)bt.first + tid;
        int ob = -1;
        long long q[kAccVals];
#pragma unroll
        for (int k = 0; k < kAccVals; ++k) q[k] = 0;
        bool coll = false;
        if (RECS && !reorder && i < end) {
            // Back to the caller's order: one record, a line or less, gathered
            // per particle, and consecutive stores.
            real x, y, z, vx, vy, vz;
            uint32_t id, fl;
            Rec<real>::load(a.rec2, a.src[i], x, y, z, id, vx, vy, vz, fl);
            if (fl != kRecDead) {
                a.x[i] = x; a.y[i] = y; a.z[i] = z;
                a.vx[i] = vx; a.vy[i] = vy; a.vz[i] = vz;
                if (a.alive && fl == kRecAbsorbed) a.alive[i] = 0;
            }
        }
        if (RECS && !a.macc) continue;  // uniform
        if (i < end) {
            // The same particles as the move's moment terms: alive after the
            // step (not absorbed), finite, with a valid mass.
            const bool direct = reorder || !RECS;
            const int64_t p = reorder || RECS ? i : (int64_t)a.src[i];
            real x, y, z, vx, vy, vz;
            bool alive;
            if (direct) {
                alive = a.alive ? a.alive[p] != 0 : true;
                x = a.x[p]; y = a.y[p]; z = a.z[p]; vx = a.vx[p]; vy = a.vy[p]; vz = a.vz[p];
            } else {
                uint32_t id, fl;
                Rec<real>::load(a.rec2, i, x, y, z, id, vx, vy, vz, fl);
                alive = fl == kRecAlive;
            }
            const real mi = has_mass ? (direct ? a.mass[p] : a.rmass[i]) : I.mass;
            const bool fin = finite3(x, y, z) && finite3(vx, vy, vz) &&
                             (!has_mass || (mi > real(0) && mi < real(INFINITY)));
            if (alive && fin) {
                ob = obin_of(I, x, y, z);
                const bool c = a.coll[p] != 0;
                double vir[3] = {0.0, 0.0, 0.0};
                if (c) {
                    vir[0] = (double)a.vir[3 * p];
                    vir[1] = (double)a.vir[3 * p + 1];
                    vir[2] = (double)a.vir[3 * p + 2];
                }
                const double m = has_mass ? (double)mi : I.mass_d;
                const double* S = a.shift + (int64_t)ob * 3;
                double t[kAccVals];
                moment_terms(m, (double)vx, (double)vy, (double)vz, S, vir[0], vir[1], vir[2], t);
                // The quanta of the o-bin: its exponents and the headroom of its
                // particle count, both from the move.
                const ObExp& G = exp_of(a, ob);
                const int h = acc_headroom(G.nc & 0xffffffffull);
                const double s0 = fixed_scale(G.e[0], h), s1 = fixed_scale(G.e[1], h);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    q[k] = to_fixed(t[k], s0);
                    q[3 + k] = to_fixed(t[3 + k], s1);
                }
                if (c) {
                    const double s2 = fixed_scale(G.e[2], h);
#pragma unroll
                    for (int k = 6; k < 9; ++k) q[k] = to_fixed(t[k], s2);
                }
                if (has_mass) q[9] = to_fixed(t[9], fixed_scale(G.e[3], h));
                coll = c;
            }
        }
        bool head;
        const int lim = row_lim(ob, lane, head);
        const bool anyc = __ballot(coll) != 0;
#pragma unroll
        for (int k = 0; k < kAccVals; ++k) {
            if ((k >= 6 && k <= 8 && !anyc) || (k == 9 && !has_mass)) continue;  // wave-uniform
            q[k] = row_sum64(q[k], lim);
        }
        if ((head || (lane & 15) == 0) && ob >= 0) value_flush(tab, a, ob, q);
    }
    if (RECS && !a.macc) return;
    __syncthreads();
    // The table to the global sums: one thread per (slot, value).
    for (int t = tid; t < kMomSlots * kTabWords; t += kBlock) {
        const int slot = t / kTabWords, wd = t % kTabWords;
        const int o = tab.key[slot];
        if (o >= 0) global_acc_add(a.macc[o], wd, tab.val[slot][wd]);
    }
}

// Per instance, from the work-group maxima of |v|^2 left by the key kernel:
// the step's largest speed (with split c-bins it bounds the fast particles'
// reach in the search); with ADAPTIVE_DT the time step of Sec. 3,
// dt = dx / v_max (dx of the configured c-bins), the caller's dt being the
// cap.  gridDim.x work-groups per instance fold the maxima into a running
// maximum (a single work-group would wait on its loads one after another);
// the last to arrive writes the instance's quantities for the later kernels.
template <typename real>
__global__ void __launch_bounds__(256) k_prep(Inst<real>* inst, const double* gpart) {
    __shared__ double lds[16];
    __shared__ bool last;
    Inst<real>& I = inst[blockIdx.y];
    if (!(I.flags & (TPKMC_ADAPTIVE_DT | kSubgrid))) return;  // whole work-group
    double v = 0.0, out = 0.0;
    const double* g0 = gpart + (int64_t)I.blk0 * kGPart;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < I.nblk; b += gridDim.x * blockDim.x)
    {
        v = fmax(v, g0[(int64_t)b * kGPart + GP_VMAX0]);
        out = fmax(out, g0[(int64_t)b * kGPart + GP_PX]);
    }
    v = wave_reduce<true>(v);
    out = wave_reduce<true>(out);
    if ((threadIdx.x & 63) == 0) {
        lds[threadIdx.x >> 6] = v;
        lds[4 + (threadIdx.x >> 6)] = out;
    }
    __syncthreads();
    v = fmax(fmax(lds[0], lds[1]), fmax(lds[2], lds[3]));
    out = fmax(fmax(lds[4], lds[5]), fmax(lds[6], lds[7]));
    if (threadIdx.x == 0) {
        // Non-negative numbers order like their bit patterns.
        atomicMax(&I.run_v2, (unsigned long long)__double_as_longlong(v));
        atomicMax(&I.run_out, __float_as_uint((float)out));
        __threadfence();
        last = atomicAdd(&I.prep_done, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last || threadIdx.x != 0) return;
    __threadfence();
    const double vmax2 = __longlong_as_double((long long)atomicExch(&I.run_v2, 0ull));
    atomicExch(&I.prep_done, 0u);
    if (I.flags & TPKMC_ADAPTIVE_DT) {
        double dt = I.dt_cap;
        if (I.dx_d > 0.0 && vmax2 > 0.0) {
            const double t = I.dx_d / sqrt(vmax2);
            if (t < dt) dt = t;
        }
        I.dt_d = dt;
        I.dt = (real)dt;
    }
    // Largest speed among the records of the sub-grid, the bound of its
    // reach.  A particle outside the box along a periodic axis lies in the
    // cell at the edge, as far from it as from the box, so the reach of a
    // pair grows by that of both, spread over the step (from a fifth of the
    // box on, no bound: then k_key says infinite).  With no bound for any
    // such particle, the FP32 tube of 4e5 on 100 c-bins took 7.7 ms instead
    // of 0.33 for one that lies on its upper edge.
    const double vr = (I.flags & kSplit) ? (double)I.vc2 : vmax2;
    double reach = sqrt(vr);
    if (const uint32_t stray = atomicExch(&I.run_out, 0u))
        reach += 2.0 * (double)__uint_as_float(stray) / ((double)I.tile_s * I.dt_d);
    I.vreach = (real)(reach * (1.0 + 1e-6));
}

// Tuning statistics of the speeds: per work-group, over the live particles
// with a finite state, the sum of |v|^2, their count, and the sum of |v|^2
// over those with |v|^2 above the instance's vc2 (0 when vc2 is 0), in the
// slots GP_PX, GP_PY and GP_PZ (free until the move writes them).
template <typename real>
__global__ void __launch_bounds__(kBlock) k_speed_stats(StepArgs<real> a) {
    __shared__ double lds[16];
    const Blk bt = a.blk[blockIdx.x];
    const Inst<real>& I = a.inst[bt.inst];
    const int64_t p = (int64_t)bt.first + threadIdx.x;
    double v2 = 0.0, n = 0.0, hot = 0.0;
    if (p < I.off + I.cnt && (a.alive == nullptr || a.alive[p] != 0)) {
        const double vx = (double)a.vx[p], vy = (double)a.vy[p], vz = (double)a.vz[p];
        if (finite3((double)a.x[p], (double)a.y[p], (double)a.z[p]) && finite3(vx, vy, vz)) {
            v2 = speed2(vx, vy, vz);
            n = 1.0;
            hot = I.vc2 > real(0) && v2 > (double)I.vc2 ? v2 : 0.0;
        }
    }
    v2 = block_sum(v2, lds);
    n = block_sum(n, lds);
    hot = block_sum(hot, lds);
    if (threadIdx.x == 0) {
        a.gpart[(int64_t)blockIdx.x * kGPart + GP_PX] = v2;
        a.gpart[(int64_t)blockIdx.x * kGPart + GP_PY] = n;
        a.gpart[(int64_t)blockIdx.x * kGPart + GP_PZ] = hot;
    }
}

// ---------------------------------------------------------------- launchers
template <typename real>
void launch_key(const StepArgs<real>& a, hipStream_t s) {
    hipLaunchKernelGGL(k_key<real>, dim3(a.nblk), dim3(kWave), 0, s, a);
}
template <typename real>
void launch_scatter(const StepArgs<real>& a, hipStream_t s) {
    hipLaunchKernelGGL(k_scatter<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
}
template <typename real>
void launch_prep(Inst<real>* inst, const double* gpart, int n_inst, int max_nblk, hipStream_t s) {
    const int gx = std::max(1, std::min(64, (max_nblk + 1023) / 1024));
    hipLaunchKernelGGL(k_prep<real>, dim3(gx, n_inst), dim3(256), 0, s, inst, gpart);
}
template <typename real>
void launch_speed_stats(const StepArgs<real>& a, hipStream_t s) {
    hipLaunchKernelGGL(k_speed_stats<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
}
// Small launches split each record's neighbourhood over several waves, up to
// kSplitWaves waves in all (4 a work-group).
constexpr int kTileParts = 16, kSplitWaves = 4096;
template <typename real>
void launch_search(const StepArgs<real>& a, int block, int group, hipStream_t s) {
    if constexpr (std::is_same<real, float>::value) {
        const int lanes = kBlock / group;
        const int bs = block < lanes ? block : lanes;
        const unsigned grid = (unsigned)a.nblk * (unsigned)(lanes / bs);
        const size_t lds = (size_t)(bs / kWave) * kStageBytesPerWave;  // staging buffers
        if (group == 4) hipLaunchKernelGGL((k_search<4>), dim3(grid), dim3(bs), lds, s, a);
        else if (group == 2) hipLaunchKernelGGL((k_search<2>), dim3(grid), dim3(bs), lds, s, a);
        else hipLaunchKernelGGL((k_search<1>), dim3(grid), dim3(bs), lds, s, a);
    } else {
        const int parts = std::max(1, std::min(9, kSplitWaves / (4 * a.nblk)));
        if (parts > 1) hipLaunchKernelGGL((k_search_lanes<real, true>), dim3(a.nblk, parts), dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((k_search_lanes<real, false>), dim3(a.nblk), dim3(kBlock), 0, s, a);
    }
}
template <typename real>
void launch_search_tiles(const StepArgs<real>& a, hipStream_t s) {
    const int parts = std::max(1, std::min(kTileParts, kSplitWaves / (4 * a.nblk)));
    hipLaunchKernelGGL(k_search_tiles<real>, dim3(a.nblk, parts), dim3(kBlock), 0, s, a);
}
// Work-groups that settle ties.  Where most records tie to the end (a beam of 2e5
// along x, all at closest approach 0) 64 of them made it a step of 1.31 ms, 512 of
// 0.40, 1024 of 0.33, 2048 of 0.33; where none does, the usual case, all return
// at once alike.  (The ordered scans that settled ties in passing took 0.18.)
constexpr int kTieGroups = 1024;
template <typename real>
void launch_search_ties(const StepArgs<real>& a, hipStream_t s) {
    if constexpr (std::is_same<real, double>::value) {
        const unsigned grid = (unsigned)std::max(1, std::min(kTieGroups, a.nblk));
        hipLaunchKernelGGL(k_search_ties<real>, dim3(grid), dim3(kBlock), 0, s, a);
    }
}
template <typename real>
void launch_search_mix(const StepArgs<real>& a, int n_inst, bool split, hipStream_t s) {
    hipLaunchKernelGGL(k_search_mix<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    if (split) {
        const unsigned fg = (unsigned)std::max(1, std::min(2048, a.nblk));
        hipLaunchKernelGGL((k_search_fast<real, true>), dim3(fg), dim3(256), 0, s, a, n_inst);
    }
}
template <typename real>
void launch_search_fast(const StepArgs<real>& a, int n_inst, hipStream_t s) {
    const unsigned fg = (unsigned)std::max(64, std::min(2048, 4 * a.nblk));
    hipLaunchKernelGGL((k_search_fast<real>), dim3(fg), dim3(256), 0, s, a, n_inst);
}
template <typename real>
void launch_random_pairs(const StepArgs<real>& a, hipStream_t s) {
    hipLaunchKernelGGL(k_rp_key<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rp_rank<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rp_partner<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
}
template <typename real>
void launch_move(const StepArgs<real>& a, hipStream_t s) {
    hipLaunchKernelGGL(k_move<real>, dim3(a.nblk), dim3(kBlock), 0, s, a);
}
template <typename real>
void launch_moments(const StepArgs<real>& a, bool caller_order, hipStream_t s) {
    const unsigned grid = (unsigned)((a.nblk + kMomEntries - 1) / kMomEntries);
    if (caller_order && a.rec2) hipLaunchKernelGGL((k_moments<real, true>), dim3(grid), dim3(kBlock), 0, s, a);
    else if (a.macc) hipLaunchKernelGGL((k_moments<real, false>), dim3(grid), dim3(kBlock), 0, s, a);
}

}  // namespace tpkmc
