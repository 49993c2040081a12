// HIP kernels of the Cherenkov photon-bunch path for gfx950 (CDNA4).
//
// Pipeline of one run (all on the caller's stream, no host synchronisation):
//   init      - zero the control block, validate shower offsets, count tiles
//               (a tile = up to tile_segs consecutive steps of one shower);
//   emit      - persistent: each wavefront claims tiles; per tile it computes
//               the step setups (FP64, one step per lane: photon yield, bunch
//               count, Cherenkov angle, frame) and the azimuths at which each
//               step's light can reach a sphere; a first pass over the bunches of
//               the steps that can (one per lane) takes the azimuth's draw only
//               and queues the bunches in those azimuths; the queue's bunches,
//               64 at a time, get their draws, sub-step emission point, direction
//               on the cone, table lookup, refraction series, ground point and
//               candidate spheres, and every crossing is recorded in a staging
//               area together with its rank among the tile's crossings of the
//               same telescope;
//   finalize  - per-telescope prefix sums over tiles, CSR offsets per
//               (shower, telescope), and a scatter of the staged records to
//               their final slots (ascending step, then bunch).
// Paper mapping: App. A (steps -> photon count -> bunches of ~5 photons, one
// per sub-step -> propagation -> telescope output), App. B (observed
// direction, displacement, travel time), sec. 3.3.2 (uniform fine tables).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>
#include <set>
#include <type_traits>
#include <utility>

#include "ckv_internal.h"

namespace ckv {

// --------------------------------------------------------------------------
// kernel arguments
// --------------------------------------------------------------------------
struct Args {
    const double *x0, *y0, *h0, *u, *v, *w, *len, *t0, *energy;
    const uint8_t* ptype;
    int64_t n;
    const uint32_t* step_id;    // counter word 1 per step, or NULL
    const int64_t* seg_offsets;
    const double* t_ref;
    const uint32_t* shower_ids;
    const int64_t* seg_id_base;
    int32_t n_showers;
    // atmosphere
    int32_t n_nodes;
    double h_obs, step, inv_step, h_top, n_obs;
    const double* node64;
    const float* cell32;
    // node tables (binary-search lookups): n_nodes altitudes then n_nodes-1 inverse
    // widths; NULL for the uniform grid
    const double* hnodes;
    int32_t search_pow2;        // largest power of two below n_nodes - 1
    // longitudinal profile (prof_bins = 0: none)
    const double* depth;        // n_nodes, vertical depth [g/cm^2]
    double* prof_ph;            // n_showers x prof_bins
    int64_t* prof_bu;
    double inv_bin;
    int32_t prof_bins;
    // telescopes and candidate grid
    int32_t n_tel;
    const double* tel;          // X, Y, R, R^2
    double gx0, gy0, inv_cell;
    int32_t nx, ny, level_cells;
    const uint16_t* cell_list;
    const uint2* cell_ent;      // per cell: {offset, count | first sphere << 16}
    // parameters
    double bunch_size, k_ft, inv_l1, dl, w_min;
    int32_t grazing_exact;      // 1: bunches with 0 < w <= w_min take propagate_exact
    double earth_r;             // > 0: spherical shells of this radius (curved variant)
    double r_obs;               // earth_r + h_obs
    uint32_t key0, key1;
    int32_t tile_segs;
    int32_t report_segs;        // tile size of the report and of a cut (a multiple of it)
    // first step of the run (a resume cursor; step 0 of shower 0 without one)
    int64_t cur_step;
    int32_t cur_shower;
    // workspace and output
    int64_t* ctrl;
    int64_t* tiles_before;
    int64_t* blocks_before;
    int64_t* shower_first;      // first step of each shower in this run
    int64_t* tile_run_off;
    int32_t* tile_run_n;
    int32_t* tile_hits;
    int64_t* runs;
    int64_t run_cap;
    int32_t* block_sums;        // telescope-major: block_sums[k * max_row_blocks + b]
    int64_t* block_hits;
    int32_t* shower_tel;
    int32_t* stage_fill;
    StageEntry* stage;
    int64_t stage_blocks;
    int64_t max_tiles;
    int64_t max_row_blocks;
    float* records;
    int64_t* ids;
    int64_t capacity;
    int64_t* tel_offsets;
    ckv_result* result;
    // screening pass of the soft response (kFeatScreen): frozen bunch counts and the
    // list of candidate bunches {ids, capacity, count}
    const int64_t* nb_frozen;
    uint64_t* list_ids;
    int64_t list_cap;
    int64_t* list_count;
    // the soft tile kernels' per-step cull (cull_rmax = 0: off): the largest screening
    // radius; x0 = (psi_max - psi_min) / (1 + psi_min); b0 = x0 times the bound of
    // |1 - T4(x)| / |x| (1/2 for psi non-increasing with altitude, 4/5 otherwise); a
    // bound of (n_e / n_obs)^2
    double cull_rmax, cull_x0, cull_b0, cull_rho2;
    // the bunch kernel's azimuth sectors (light_cone; sec_rmax = 0: off): the largest
    // sphere radius and the largest distance of a centre from the origin; psi's largest
    // slope with altitude (0 where psi is not non-increasing), largest and smallest value
    double sec_rmax, sec_dmax, sec_slope, sec_psi_max, sec_psi_min;
    int32_t sec_falls;          // psi non-increasing with altitude at every node
    // sphere centres near a ground point (ckv_reach; reach_levels 0: none)
    const ReachLevel* reach_lev;
    const uint2* reach_rec;
    const uint2* reach_list;
    int32_t reach_levels;
    int64_t* claims;            // claim counters, kClaimStride apart
    int32_t span_tiles;         // tiles of a unit whose bunches a wave takes together
    int32_t grid_waves;         // waves of the bunch kernel's launch
    int32_t head_units;         // units of 32 steps at its start (0 or grid_waves)
    int32_t static_blocks;      // staging and run blocks dealt to them beforehand
    // smaller tiles only: per kHeavySteps steps, whether a step of theirs may be in a refused
    // tile of the report's size, and per step of those, whether it is (else NULL)
    int32_t* heavy;
    uint8_t* heavy_step;
};

// Memory accesses whose address space is explicit.  Where one access may go to LDS
// or to HBM, a generic pointer makes the compiler use one generic (flat)
// instruction for both, which costs every access, also the LDS ones; reads and
// atomics through these types keep the two kinds apart.
typedef float f32x4 __attribute__((ext_vector_type(4)));
using LdsF64 = __attribute__((address_space(3))) double;
using HbmF64 = __attribute__((address_space(1))) double;
using HbmF32x4 = __attribute__((address_space(1))) f32x4;

// The launch's argument block at the address the kernel passes to a called function:
// wave-uniform and read-only, so the function reads it with scalar loads.
__device__ __forceinline__ const Args& args_from(uint64_t at)
{
    const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
    return *(const Args*)reinterpret_cast<const __attribute__((address_space(4))) Args*>(u);
}

__device__ __forceinline__ const LdsF64* as_lds(const double* p) { return (const LdsF64*)p; }
__device__ __forceinline__ const HbmF64* as_hbm(const double* p) { return (const HbmF64*)p; }
__device__ __forceinline__ const HbmF32x4* as_hbm4(const float* p) { return (const HbmF32x4*)p; }

__device__ __forceinline__ void lds_add(double* p, double v)
{
    __hip_atomic_fetch_add((LdsF64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void hbm_add(double* p, double v)
{
    __hip_atomic_fetch_add((HbmF64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// --------------------------------------------------------------------------
// wave helpers
// --------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Any value, by no instruction, for lanes that never read theirs.  (A variable left
// uninitialised before a branch and read only behind it is carried round its loop by a
// register copy a turn: 33 of the 280 instructions a chunk of 64 bunches took.)
template <typename T>
__device__ __forceinline__ T any_of()
{
    T x;
    asm volatile("" : "=v"(x));
    return x;
}
__device__ __forceinline__ uint32_t any_u32() { return any_of<uint32_t>(); }
__device__ __forceinline__ double any_f64() { return any_of<double>(); }
// bits of m at lanes below this one, and at this lane and below.  The builds of
// ckv_slowpath.hip, which keep loop invariants in registers, keep the lane's masks there
// (grazing 3000 steps 874 us, 930 with the counts below).
#ifdef CKV_SLOWPATH
__device__ __forceinline__ uint64_t lt_mask() { return lane_id() == 0 ? 0ull : (~0ull >> (64 - lane_id())); }
__device__ __forceinline__ int lanes_below(uint64_t m) { return __popcll(m & lt_mask()); }
__device__ __forceinline__ int lanes_upto(uint64_t m) { return __popcll(m & (lt_mask() | (1ull << lane_id()))); }
#else
__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ int lanes_upto(uint64_t m) { return lanes_below(m >> 1) + (int)(m & 1); }
#endif

// x of the lane the DPP control CTRL names as source, in the rows ROWS enables; 0
// where there is no source or the row is masked off
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t dpp_take(int64_t x)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)x >> 32), CTRL, ROWS,
                                                              0xf, false);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Inclusive sum of x over lanes 0..lane by DPP lane moves (no LDS round trips):
// shifts by 1, 2, 4 and 8 inside each row of 16 lanes, then lane 15 of rows 0 and 2
// into rows 1 and 3 (row_bcast:15), then lane 31 into rows 2 and 3 (row_bcast:31).
// Called by the whole wave.
__device__ __forceinline__ int64_t wave_incl_scan(int64_t x)
{
    x += dpp_take<0x111, 0xf>(x);   // row_shr:1
    x += dpp_take<0x112, 0xf>(x);   // row_shr:2
    x += dpp_take<0x114, 0xf>(x);   // row_shr:4
    x += dpp_take<0x118, 0xf>(x);   // row_shr:8
    x += dpp_take<0x142, 0xa>(x);   // row_bcast:15
    x += dpp_take<0x143, 0xc>(x);   // row_bcast:31
    return x;
}

// x of lane 63 (a register read, not an LDS round trip)
__device__ __forceinline__ int64_t wave_last(int64_t x)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, kWave - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), kWave - 1);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Smallest x over the lanes where it is below `none` (at least one lane is):
// take the first such lane's value and repeat while a lane holds a smaller one.
// Passes = distinct values below the result + 1, usually one or two; ballots
// and lane reads only, no LDS round trips.
__device__ __forceinline__ int wave_min_sparse(int x, int none)
{
    uint64_t below = __ballot(x < none);
    int m = none;
    while (below) {
        m = __builtin_amdgcn_readlane(x, __builtin_ctzll(below));
        below = __ballot(x < m);
    }
    return m;
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename T>
__device__ __forceinline__ T uniform(T x)
{
    return __shfl(x, 0);
}

// A value every lane holds alike, made visibly uniform to the compiler (a scalar
// register), so that control flow depending on it stays scalar.
__device__ __forceinline__ int64_t scalar64(int64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Candidate-grid level for a line with observed w^2 = wo2 (>= kLevelW2[0]):
// the deepest level whose w floor the line clears, with a 1e-6 margin that
// covers the rounding of wo2.
constexpr double kLevelW2[kGridLevels] = {
    kGridWLevel[0] * kGridWLevel[0] + 1e-6, kGridWLevel[1] * kGridWLevel[1] + 1e-6,
    kGridWLevel[2] * kGridWLevel[2] + 1e-6};
static_assert(kGridLevels == 3, "grid_level selects among three levels");

__device__ __forceinline__ int grid_level(double wo2)
{
    return wo2 >= kLevelW2[2] ? 2 : (wo2 >= kLevelW2[1] ? 1 : 0);
}

// --------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds, multipliers applied to
// words 0 and 2, key advanced by the Weyl constants between rounds.
// --------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t r[4])
{
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    r[0] = c0; r[1] = c1; r[2] = c2; r[3] = c3;
}

// --------------------------------------------------------------------------
// Step setup, FP64, without FMA contraction: the bunch count must come out of
// exactly these IEEE operations.  App. A: photons per step, split into
// bunches of about bunch_size photons, one per equal sub-step.
// --------------------------------------------------------------------------
struct Setup {
    int status;        // -1: emits light; otherwise CKV_DROP_*
    int64_t nb;
    double photons, cos_t, sin_t, ds, inv_bc;
    double b1x, b1y, b1z, b2x, b2y, b2z;
    double x0, y0, h0, t0, u, v, w;   // the step's inputs as loaded (for its record)
    double len, psi;                  // its length; psi at its midpoint
};

__device__ __forceinline__ double psi_fp64(const Args& a, double h)
{
#pragma clang fp contract(off)
    double hc = h < a.h_obs ? a.h_obs : (h > a.h_top ? a.h_top : h);
    int64_t i;
    double f;
    if (a.hnodes) {
        // node tables: binary search for the bracketing pair, then the fraction
        int lo = 0, hi = a.n_nodes - 1;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.hnodes[mid] <= hc) lo = mid; else hi = mid;
        }
        i = lo;
        f = (hc - a.hnodes[lo]) / (a.hnodes[lo + 1] - a.hnodes[lo]);
    } else {
        double x = (hc - a.h_obs) * a.inv_step;
        i = (int64_t)floor(x);
        if (i > a.n_nodes - 2) i = a.n_nodes - 2;
        f = x - (double)i;
    }
    double lo = a.node64[kNode64 * i], hi = a.node64[kNode64 * (i + 1)];
    return lo + f * (hi - lo);
}

// Curved variant: x, y horizontal at the array origin, z along the origin's
// vertical from sea level, the Earth's centre at (0, 0, -R).  The altitude of a
// point is its distance from the centre minus R, written without the
// cancellation of sqrt(...) - R; no contraction, so drop decisions and table
// cells match the FP64 definition's operations.
__device__ __forceinline__ double curved_altitude(double R, double x, double y, double z)
{
#pragma clang fp contract(off)
    const double q = x * x + y * y;
    const double rz = R + z;
    const double r = sqrt(q + rz * rz);
    return (q + z * (2.0 * R + z)) / (r + R);
}

__device__ __forceinline__ void step_setup(const Args& a, int64_t i, Setup& st)
{
#pragma clang fp contract(off)
    st.nb = 0;
    st.status = -1;
    const double x0 = a.x0[i], y0 = a.y0[i], h0 = a.h0[i];
    const double u = a.u[i], v = a.v[i], w = a.w[i];
    const double L = a.len[i], t0 = a.t0[i], E = a.energy[i];
    const double m = a.ptype[i] == CKV_MUON ? kMassMuon : kMassElectron;
    st.x0 = x0; st.y0 = y0; st.h0 = h0; st.t0 = t0; st.u = u; st.v = v; st.w = w;
    st.len = L;
    // (E c with c = m / 1 GeV in (0, 1) is finite exactly when E is; testing it, with
    // every test evaluated (no short circuit), puts all the step's loads in one round)
    const int n_finite = (int)isfinite(x0) + (int)isfinite(y0) + (int)isfinite(h0) + (int)isfinite(u) +
                         (int)isfinite(v) + (int)isfinite(w) + (int)isfinite(L) + (int)isfinite(t0) +
                         (int)isfinite(E * (m * 1e-3));
    const bool finite = n_finite == 9;
    if (!finite || !(L > 0.0)) { st.status = CKV_DROP_NONFINITE; return; }
    const double r = m / E;
    const double r2 = r * r;                           // 1 - beta^2
    if (!(r2 < 1.0)) { st.status = CKV_DROP_MASS; return; }
    double h_mid;                                      // index at the step midpoint
    if (a.earth_r > 0.0) {
        const double hl = 0.5 * L;
        h_mid = curved_altitude(a.earth_r, x0 + hl * u, y0 + hl * v, h0 - hl * w);
    } else {
        h_mid = h0 - (0.5 * L) * w;
    }
    const double psi = psi_fp64(a, h_mid);
    st.psi = psi;
    const double n2 = 1.0 + psi;
    const double num = psi - n2 * r2;                  // beta^2 n^2 - 1
    if (!(num > 0.0)) { st.status = CKV_DROP_THRESHOLD; return; }
    const double sin2 = num / (n2 * (1.0 - r2));       // sin^2 of the Cherenkov angle
    const double N = (a.k_ft * L) * sin2;              // Frank-Tamm photon count
    const double nbd = ceil(N / a.bunch_size);
    st.nb = (int64_t)nbd;
    st.photons = N / nbd;
    st.cos_t = 1.0 / sqrt((1.0 - r2) * n2);           // 1 / (beta n)
    st.sin_t = sqrt(sin2);
    st.ds = L / nbd;
    st.inv_bc = 1.0 / (sqrt(1.0 - r2) * kSpeedOfLight);
    // orthonormal frame around D = (u, v, -w) (Duff et al., JCGT 2017)
    const double Dx = u, Dy = v, Dz = -w;
    const double sgn = copysign(1.0, Dz);
    const double ia = -1.0 / (sgn + Dz);
    const double ib = Dx * Dy * ia;
    st.b1x = 1.0 + sgn * Dx * Dx * ia;
    st.b1y = sgn * ib;
    st.b1z = -sgn * Dx;
    st.b2x = ib;
    st.b2y = sgn + Dy * Dy * ia;
    st.b2z = -Dy;
}

// --------------------------------------------------------------------------
// sin and cos of 2 pi (r + 1/2) / 2^32 from the integer draw r, in turns.
// Mixed path: the hardware sine and cosine, which take their argument in turns:
// the quadrant from the top two bits, the angle inside it as an FP32 number of
// turns in [0, 1/4) (rounding below 1e-7 rad); errors near 1e-7, i.e. ~2e-9 in
// the photon direction once scaled by sin(theta_c) < 0.03.  The quadrant's
// rotation, (s, c) = (sq, cq), (cq, -sq), (-sq, -cq), (-cq, sq) for q = 0..3, is
// a swap on bit 30 of r and sign flips on bit 31 (sine) and on bit 31 of
// r + 2^30 (cosine).
// --------------------------------------------------------------------------
__device__ __forceinline__ void sincos_turns_hw(uint32_t r, float& s, float& c)
{
    const float t = fmaf((float)(r & 0x3FFFFFFFu), 2.3283064365386963e-10f, 1.16415321826934814e-10f);
    const float sq = __builtin_amdgcn_sinf(t), cq = __builtin_amdgcn_cosf(t);
    const bool swap = (r & 0x40000000u) != 0;
    const uint32_t s0 = __float_as_uint(swap ? cq : sq), c0 = __float_as_uint(swap ? sq : cq);
    s = __uint_as_float(s0 ^ (r & 0x80000000u));
    c = __uint_as_float(c0 ^ ((r + 0x40000000u) & 0x80000000u));
}

// The same in FP64 for the FP64 path: quadrant and half-quadrant fold from the
// integer draw, then Taylor series of sin and cos on |a| <= pi/4 to a^17 and a^16
// (next terms below 1e-17).
__device__ __forceinline__ void sincos_turns64(uint32_t r, double& s, double& c)
{
    const uint32_t q = r >> 30;
    const uint32_t low = r & 0x3FFFFFFFu;
    const bool upper = low >= 0x20000000u;
    const uint32_t m = upper ? (0x3FFFFFFFu - low) : low;
    const double kq = 1.4629180792671596e-09;          // (pi/2) / 2^30
    const double a = fma((double)m, kq, 0.5 * kq);
    const double a2 = a * a;
    double sa = fma(a2, 1.0 / 355687428096000.0, -1.0 / 1307674368000.0);
    sa = fma(a2, sa, 1.0 / 6227020800.0);
    sa = fma(a2, sa, -1.0 / 39916800.0);
    sa = fma(a2, sa, 1.0 / 362880.0);
    sa = fma(a2, sa, -1.0 / 5040.0);
    sa = fma(a2, sa, 1.0 / 120.0);
    sa = fma(a2, sa, -1.0 / 6.0);
    sa = a * fma(a2, sa, 1.0);
    double ca = fma(a2, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);
    ca = fma(a2, ca, 1.0 / 479001600.0);
    ca = fma(a2, ca, -1.0 / 3628800.0);
    ca = fma(a2, ca, 1.0 / 40320.0);
    ca = fma(a2, ca, -1.0 / 720.0);
    ca = fma(a2, ca, 1.0 / 24.0);
    ca = fma(a2, ca, -0.5);
    ca = fma(a2, ca, 1.0);
    const double cq = upper ? sa : ca;
    const double sq = upper ? ca : sa;
    c = (q == 0) ? cq : (q == 1) ? -sq : (q == 2) ? -cq : sq;
    s = (q == 0) ? sq : (q == 1) ? cq : (q == 2) ? -sq : -cq;
}

// 1/x in FP64 from the hardware reciprocal and two Newton steps (to an ulp or so,
// without the correctly rounded division's scaling sequence)
__device__ __forceinline__ double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// --------------------------------------------------------------------------
// Exact propagation of a grazing bunch (0 < w <= w_min), cell by cell in FP64
// from the FP64 node table, where the moment series is not used (sec. 4.3.1 and
// App. C: rare bunches take a slow path).  With Snell's invariant
// p = n_e sin(theta_e), s = n cos(theta) obeys s^2 = n_e^2 w^2 + psi - psi_e,
// linear inside a cell, and a cell of height dz between s_t (top) and s_b
// (bottom) adds 2 p dz / (s_t + s_b) to the horizontal advance and
// (2/3) dz (s_t^2 + s_t s_b + s_b^2) / (s_t + s_b) + 2 p^2 dz / (s_t + s_b)
// to c times the travel time; a downward ray never turns.
__device__ __forceinline__ void propagate_exact(const Args& a, double xe, double ye, double he,
                                             double u, double v, double w, double& xg, double& yg,
                                             double& T, double& ne)
{
    const double* nd = a.node64;
    const double x = (he - a.h_obs) * a.inv_step;
    int c = min((int)x, a.n_nodes - 2);
    const double f = x - (double)c;
    const double psi_e = nd[kNode64 * c] + f * (nd[kNode64 * (c + 1)] - nd[kNode64 * c]);
    const double ne2 = 1.0 + psi_e;
    ne = sqrt(ne2);
    const double sin_e = sqrt(u * u + v * v);
    const double p = ne * sin_e;
    const double s0sq = ne2 * w * w;
    double X = 0.0, cT = 0.0, h_top = he, s_t = sqrt(s0sq);
    for (int i = c; i >= 0; --i) {
        const double h_b = a.h_obs + (double)i * a.step;
        const double dz = h_top - h_b;
        const double s_b = sqrt(s0sq + (nd[kNode64 * i] - psi_e));
        if (dz > 0.0) {
            const double inv = 1.0 / (s_t + s_b);
            X += 2.0 * p * dz * inv;
            cT += (2.0 / 3.0) * dz * (s_t * s_t + s_t * s_b + s_b * s_b) * inv + 2.0 * p * p * dz * inv;
        }
        h_top = h_b;
        s_t = s_b;
    }
    xg = sin_e > 0.0 ? xe + (u / sin_e) * X : xe;
    yg = sin_e > 0.0 ? ye + (v / sin_e) * X : ye;
    T = cT / kSpeedOfLight;
}

// FP64 reciprocal square root: hardware estimate refined by two Newton steps.
__device__ __forceinline__ double rsqrt64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// One Newton step on the hardware estimates (relative errors below 2^-23 for rsq
// and 2^-24 for rcp on this chip): ~1e-14 relative, for the per-cell factors of
// the curved tracer, where such errors stay far below the result's rounding.
__device__ __forceinline__ double rsqrt64_1(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

__device__ __forceinline__ double rcp64_1(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}

// Curved atmosphere: exact propagation through spherical shells (radius R =
// a.earth_r, centre (0, 0, -R)).  n depends on the altitude h = r - R only, so
// the ray stays in the plane of the centre, its emission point and direction,
// and keeps Bouguer's invariant K = n r sin(zeta) (zeta from the local
// vertical).  With s = sqrt(n^2 r^2 - K^2), the polar angle about the centre
// and the optical path down to the observation sphere r_obs are
//   theta = int K / (r s) dr,    c T = int n^2 r / s dr,
// integrated cell by cell (psi linear in h inside a cell).  s^2 is written
// relative to the emission point, s^2 = s_e^2 + (h - h_e)(r + r_e) + psi r^2 -
// psi_e r_e^2 with s_e = n_e r_e cos(zeta_e), which stays accurate for grazing
// rays.  Over a cell s^2 is nearly linear in h, so the substitution
// h = h_b + dh (u^2 - s_b^2) / (s_t^2 - s_b^2), u from s_b to s_t, turns
//   int F / s dh  into  dh / (s_t + s_b) * sum of F u / s at the 2-point
// Gauss-Legendre nodes of [s_b, s_t] (u / s is 1 up to the cell's curvature of
// s^2, ~1e-9, so two nodes reach FP64 rounding).  The ground point is the
// emission point's radial direction turned by theta towards the ray's tangential
// direction, at r_obs; the arrival direction has sin(zeta_g) = K / (n_obs r_obs).
// While n r grows with r (air at the Earth's radius: no ducting) the ray reaches
// the ground iff s^2 > 0 there, and one with cos(zeta_e) <= 0 never comes down.
// The upward and turning decisions use the FP64 definition's operations.
// Returns -1 (reached the ground), CKV_DROP_UPWARD or CKV_DROP_GRAZING.
__device__ __forceinline__ int propagate_curved(const Args& a, double xe, double ye, double ze,
                                                double he, double u, double v, double w,
                                                double& xg, double& yg, double& T, double& uo,
                                                double& vo)
{
    const double R = a.earth_r;
    const double* nd = a.node64;
    double rz, r_e, mu_num, psi_e, ne2, K, s2e, Mre, s2g;
    {
#pragma clang fp contract(off)
        rz = R + ze;
        r_e = sqrt(xe * xe + ye * ye + rz * rz);
        mu_num = w * rz - u * xe - v * ye;          // r_e cos(zeta_e), zeta_e from the downward vertical
        if (!(mu_num > 0.0)) return CKV_DROP_UPWARD;
        psi_e = psi_fp64(a, he);
        ne2 = 1.0 + psi_e;
        const double Lx = -ye * w - rz * v, Ly = rz * u + xe * w, Lz = xe * v - ye * u;
        K = sqrt(ne2) * sqrt(Lx * Lx + Ly * Ly + Lz * Lz);   // n_e |(P_e - C) x D|
        s2e = ne2 * (mu_num * mu_num);
        Mre = psi_e * r_e * r_e;
        s2g = s2e + ((a.h_obs - he) * (a.r_obs + r_e) + nd[0] * a.r_obs * a.r_obs - Mre);
        if (!(s2g > 0.0)) return CKV_DROP_GRAZING;
    }
    const double x = (he - a.h_obs) * a.inv_step;
    const int c = min((int)x, a.n_nodes - 2);
    constexpr double kg = 0.57735026918962576451;   // 1/sqrt(3)
    double theta = 0.0, opt = 0.0;
    double h_t = he, s2t = s2e, s_t = s2e * rsqrt64_1(s2e);
    for (int i = c; i >= 0; --i) {
        const double h_b = a.h_obs + (double)i * a.step;
        const double psi_b = nd[kNode64 * i];
        const double r_b = R + h_b;
        const double s2b = i == 0 ? s2g : s2e + ((h_b - he) * (r_b + r_e) + psi_b * r_b * r_b - Mre);
        const double s_b = s2b * rsqrt64_1(s2b);
        const double dh = h_t - h_b;
        if (dh > 0.0 && s2t != s2b) {    // (a cell of zero s^2 span adds ~dh/s: nothing)
            const double g = (nd[kNode64 * (i + 1)] - psi_b) * a.inv_step;   // dpsi/dh in the cell
            const double inv_ds2 = rcp64_1(s2t - s2b);
            const double inv_rb = rcp64_1(r_b);
            const double mid = 0.5 * (s_t + s_b), half = (0.5 * kg) * (s_t - s_b);
            double a_th = 0.0, a_op = 0.0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double uq = q ? mid + half : mid - half;
                const double xq = dh * ((uq * uq - s2b) * inv_ds2);     // h_q - h_b
                const double psq = fma(g, xq, psi_b);
                const double rq = r_b + xq;
                const double s2q = s2e + ((h_b + xq - he) * (rq + r_e) + psq * rq * rq - Mre);
                const double ratio = uq * rsqrt64_1(s2q);
                const double e = xq * inv_rb;                            // 1/r_q = (1 - e + e^2) / r_b
                a_th += ratio * (inv_rb * fma(e, e - 1.0, 1.0));
                a_op += ((1.0 + psq) * rq) * ratio;
            }
            const double scale = dh * rcp64_1(s_t + s_b);
            theta = fma(scale, K * a_th, theta);
            opt = fma(scale, a_op, opt);
        }
        h_t = h_b;
        s2t = s2b;
        s_t = s_b;
    }
    // ground point and arrival direction in the ray plane
    const double inv_re = rcp64(r_e);
    const double rho0 = xe * inv_re, rho1 = ye * inv_re, rho2 = rz * inv_re;
    const double mu = mu_num * inv_re;
    double t0 = fma(mu, rho0, u), t1 = fma(mu, rho1, v), t2 = fma(mu, rho2, -w);
    const double sz2 = t0 * t0 + t1 * t1 + t2 * t2;
    const double isz = sz2 > 0.0 ? rsqrt64(sz2) : 0.0;
    t0 *= isz; t1 *= isz; t2 *= isz;
    double sth, cth;
    sincos(theta, &sth, &cth);
    const double rg0 = cth * rho0 + sth * t0, rg1 = cth * rho1 + sth * t1;
    const double tg0 = cth * t0 - sth * rho0, tg1 = cth * t1 - sth * rho1;
    const double inv_nr = rcp64(a.n_obs * a.r_obs);
    const double sin_g = K * inv_nr, cos_g = s2g * rsqrt64(s2g) * inv_nr;
    xg = a.r_obs * rg0;
    yg = a.r_obs * rg1;
    uo = sin_g * tg0 - cos_g * rg0;
    vo = sin_g * tg1 - cos_g * rg1;
    T = opt * (1.0 / kSpeedOfLight);
    return -1;
}

// The two slow propagations as called functions: their loops over the cells then keep
// their constants in scalar registers of their own (inline, the bunch kernel's spilled
// ones came back by lane reads in every cell: 24 % more instructions).
// They start on an instruction cache line: elsewhere, where code before them puts their
// loops, the same instructions take up to 8 % longer (1e5 steps at 70 degrees 427-461 us
// by where, 435 on a line).
#define CKV_LINE __attribute__((aligned(64)))
struct SlowRay {
    int status;
    double xg, yg, T, uo, vo;    // uo, vo: curved; flat: uo holds n_e
};

static __device__ __noinline__ CKV_LINE SlowRay propagate_curved_call(uint64_t args_at, double xe, double ye, double ze, double he,
                                                             double u, double v, double w)
{
    SlowRay r;
    r.status = propagate_curved(args_from(args_at), xe, ye, ze, he, u, v, w, r.xg, r.yg, r.T, r.uo, r.vo);
    return r;
}

static __device__ __noinline__ CKV_LINE SlowRay propagate_exact_call(uint64_t args_at, double xe, double ye, double he, double u,
                                                            double v, double w)
{
    SlowRay r;
    r.status = -1;
    r.vo = 0.0;
    propagate_exact(args_from(args_at), xe, ye, he, u, v, w, r.xg, r.yg, r.T, r.uo);
    return r;
}

// Depth bin of an emission altitude h_obs <= h < h_top, given its table cell c
// and fraction f (x = (h - h_obs) / step, c = floor(x), f = x - c): the depth
// table read like the index and binned by floor(X * (1/width)), in FP64
// without contraction, so the bin is the one the FP64 definition gives.
__device__ __forceinline__ int profile_bin(const Args& a, int c, double f)
{
#pragma clang fp contract(off)
    const double X = a.depth[c] + f * (a.depth[c + 1] - a.depth[c]);
    int b = (int)floor(X * a.inv_bin);
    b = max(0, min(b, a.prof_bins - 1));
    return b;
}

template <int PREC>
struct StepEntry;

// mixed: FP64 position/time/direction, FP32 perpendicular cone vectors
template <>
struct alignas(16) StepEntry<1> {
    double x0, y0, h0, t0, u, v, w, cos_t, ds, inv_bc;
    double photons;  // FP64: the longitudinal profile sums it
    float sb1x, sb1y, sb1z, sb2x, sb2y, sb2z;
    int32_t sidx;   // lane of the step in its unit (modulo the tile size: step in the tile)
    uint32_t ctr1;  // counter word 1 of the step's random numbers
};
static_assert(sizeof(StepEntry<1>) == 128, "step entry size");

template <>
struct alignas(16) StepEntry<0> {
    double x0, y0, h0, t0, u, v, w, cos_t, ds, inv_bc;
    double sb1x, sb1y, sb1z, sb2x, sb2y, sb2z, photons;
    int32_t sidx;
    uint32_t ctr1;
};
static_assert(sizeof(StepEntry<0>) == 144, "step entry size");

// per-wave counters kept in LDS (wave-uniform increments by lane 0)
enum WaveCounter { kWcBunches = 0, kWcEmitting, kWcHits, kWcDrop0, kWcCount = kWcDrop0 + CKV_N_DROP };

// Azimuth sectors of a step's light cone: the bunches of a step leave at azimuths
// uniform in [0, 1) turns (the top bits of their second draw); one bit per sector says
// whether its light may reach a sphere.
constexpr int kSectorBits = 8;
constexpr int kSectors = 1 << kSectorBits;
constexpr int kSectorWords = kSectors / 32;

// Per step, what the bunch loop's first pass needs: first bunch in the pass, step in
// the tile, and the product of the second Philox round that depends on the step only.
struct alignas(16) StepPass {
    int32_t boff;
    int32_t sidx;
    uint32_t hi0, lo0;
};

// Crossings a step that a run's first units are given room for in the staging area.
constexpr int kDenseHits = 14;

// Candidate rounds of the sector search that are worth it: for a unit, and for each chunk
// of 64 bunches in it.
constexpr int kSearchFree = 8;
constexpr int kSearchPerChunk = 5;

// Bunches that the first pass let through, waiting for a full chunk of 64.
constexpr int kQueue = 2 * kWave;
constexpr int kPairs = 2 * kWave;      // (step, sphere) pairs of the tile setup, same room

// The largest atmosphere table the library takes, the same whatever a kernel keeps in LDS
// (the bunch kernel leaves the table in global memory, so it needs none of this room): as
// much as 160 KB hold beside the sphere table and one wave's area of 148 (FP64) or 128 bytes
// a step (with the profile or the screening pass, the table's lowest 1536 entries count), or,
// for FP64 runs that ask for 16 waves, those entries beside 16 such areas.
constexpr int kTableLimitEntries = 1536;

__host__ __device__ inline size_t table_bytes(int prec, int n_nodes, bool part)
{
    int n = prec == 0 ? n_nodes : n_nodes - 1;
    if (part && n > kTableLimitEntries) n = kTableLimitEntries;
    return (size_t)n * (prec == 0 ? kNode64 * sizeof(double) : kCell32 * sizeof(float));
}

// Steps with bunches in the pass that a wave keeps records of at a time.
__host__ __device__ constexpr int stash_steps(int tile_segs) { return tile_segs > 32 ? tile_segs : 32; }

__host__ __device__ inline size_t wave_bytes(int prec, int tile_segs, int n_tel, int prof_bins)
{
    size_t b = (size_t)stash_steps(tile_segs) *
               ((prec == 0 ? sizeof(StepEntry<0>) : sizeof(StepEntry<1>)) + sizeof(StepPass));
    b += (size_t)kWave * kSectorWords * sizeof(uint32_t);
    b += (size_t)kQueue * (sizeof(uint32_t) + sizeof(uint8_t));  // queue (tile setup: pairs)
    b += (size_t)kWcCount * sizeof(int64_t);            // counters
    b += ((size_t)n_tel * sizeof(int32_t) + 15) & ~(size_t)15;   // telescope counters
    if (prof_bins) b += 2 * sizeof(int64_t) + (size_t)prof_bins * (sizeof(double) + sizeof(uint32_t));
    return (b + 15) & ~(size_t)15;
}

// one wave's area beside the table in the limit above
constexpr size_t kLimitScreenBytes = 70 * sizeof(int64_t);

__host__ __device__ inline size_t limit_wave_bytes(int prec, int tile_segs, int n_tel, int prof_bins)
{
    size_t b = (size_t)tile_segs * (prec == 0 ? 148 : 128) + 256 + (size_t)kWcCount * sizeof(int64_t);
    b += ((size_t)n_tel * sizeof(int32_t) + 15) & ~(size_t)15;
    b += (size_t)prof_bins * (sizeof(double) + sizeof(uint32_t));
    return (b + 15) & ~(size_t)15;
}

constexpr int kSoftIdBits = 24;                          // bunch index bits of a list id
constexpr unsigned long long kSoftListInvalid = 1ull << 62;   // or-ed into the count

// --------------------------------------------------------------------------
// the bunch kernel
// --------------------------------------------------------------------------
// FEAT bits: kFeatProfile (longitudinal profile), kFeatExact (grazing bunches
// traced exactly); each combination is its own kernel, so runs without them
// carry none of their code or registers.
constexpr int kFeatProfile = 1;
constexpr int kFeatExact = 2;
constexpr int kFeatSearch = 4;   // node tables: binary search per bunch (alone, 32-step tiles)
constexpr int kFeatCurved = 8;   // spherical shells, every bunch traced exactly (alone, 32-step tiles)
// soft-response screening (mixed, alone, 32-step tiles): bunch counts frozen, each
// bunch tested against spheres of the soft cut radius plus a margin, the candidates'
// ids listed; no records
constexpr int kFeatScreen = 32;

__host__ __device__ inline size_t search_bytes(int n_nodes)
{
    return ((size_t)(2 * n_nodes - 1) * sizeof(double) + 15) & ~(size_t)15;
}

// LDS layout of the bunch kernel: the node altitudes of the search variant, the sphere
// table {X, Y, R^2}, then the waves.  The atmosphere table stays in global memory: only
// the bunches that can reach a sphere look it up (1-3 % of them; their cells, 11 KB
// between 2 and 20 km on a 50 m grid, stay in the vector cache).
// sphere table in LDS: {X, Y, R^2} per sphere (at most CKV_MAX_TEL: 24 KB)
__host__ __device__ inline size_t tel_bytes(int n_tel)
{
    return ((size_t)n_tel * 3 * sizeof(double) + 15) & ~(size_t)15;
}

// Workgroup size the variant is compiled for: the exact-path variants (grazing,
// curved) carry FP64 tracing state and get the registers of 8 waves; the others are
// built for 16 waves (128 registers, four waves per SIMD).
constexpr int emit_threads(int prec, int feat)
{
    return (feat & (kFeatExact | kFeatCurved)) != 0 ? 512 : 1024;
}

// Screening cull (soft response, plane-parallel atmosphere, FP64 pass as computed by
// soft_bunch).  A step's bunches leave from E(s) = P0 + s a, s in [0, L], in directions
// p = cos_t a + sin_t e with e a unit vector normal to a.  With T(d) = d_h / w_d
// (horizontal part over downward cosine) a bunch reaches the ground at
// g = E_h + T(p) S, where S = int T4(x) dh over the path, T4 the four-term series of
// (1 + x)^(-1/2) and x = q (psi - psi_e), q = 1 / (n_e w_p)^2 (App. B, the horizontal
// displacement, here as the moment series).  All of E(s) project along a to one point
// G = P0_h + (h0 - h_obs) T(a), so g - G = dh (T(p) - T(a)) - T(p) (dh - S), and:
// |T(p) - T(a)| = sin_t |(e x a)_h| / (w_p w_a), with |(e x a)_h| in [w_a, 1];
// w_p lies in [cos(zeta_a + t), cos(zeta_a - t)]; for x in [0, 1] (psi non-increasing
// with altitude) 0 <= 1 - T4(x) <= x/2, for |x| <= 1/2 |1 - T4(x)| <= 4|x|/5; and
// x <= x0 / w_p^2.  The bunch weights a sphere of radius R centred at c on the ground
// only if its observed line passes within R of c, so only if |g - c| <= R / w_o, with
// w_o^2 >= 1 - rho2 (1 - w_p^2).  Hence a step whose sphere centres all lie outside
// the annulus returned here (centre G, |d^2 - mid| <= half) gives no bunch a soft
// weight.  The bound takes a margin of 0.1 m plus 1e-6 relative for rounding; it is
// not applied (false) where its conditions fail: a direction not unit to 1e-9, w_a
// below 0.05, x0 / w_p^2 above 1/2 or w_o near zero.
__device__ inline bool screen_annulus(const Args& a, double x0, double y0, double h0, double u,
                                      double v, double w, double len, double ct, double st,
                                      double& gx, double& gy, double& mid, double& half)
{
    const double n2 = u * u + v * v + w * w;
    if (!(fabs(n2 - 1.0) <= 1e-9) || !(w >= 0.05)) return false;
    const double sa = sqrt(fmax(0.0, (1.0 - w) * (1.0 + w)));
    const double s_hi = st * (1.0 + 1e-9) + 1e-12, s_lo = fmax(st * (1.0 - 1e-9) - 1e-12, 0.0);
    // w_p of the bunches the FP64 pass keeps (w_p > w_min)
    const double wp_hi = fmin(1.0, w * ct + sa * s_hi + 1e-12);
    const double wp_lo = fmax(w * ct - sa * s_hi - 1e-12, a.w_min);
    if (!(wp_lo > 0.0)) return false;
    const double iw2 = 1.0 / (wp_lo * wp_lo);
    if (!(a.cull_x0 * iw2 <= 0.5)) return false;
    const double B = a.cull_b0 * iw2;                          // bound of |1 - S / dh|
    const double t_max = sqrt((1.0 - wp_lo) * (1.0 + wp_lo)) / wp_lo;   // bound of |T(p)|
    const double dh0 = h0 - a.h_obs;
    const double dh_top = fmax(dh0, 0.0), dh_bot = fmax(dh0 - len * w, 0.0);
    const double f_lo = s_lo / wp_hi - B * t_max;
    const double f_hi = s_hi / (wp_lo * w) + B * t_max;
    const double r_lo = f_lo > 0.0 ? dh_bot * f_lo : 0.0;      // |g - G| in [r_lo, r_hi]
    const double r_hi = dh_top * f_hi;
    const double wo2 = 1.0 - fmin(1.0, a.cull_rho2 * (1.0 - wp_lo) * (1.0 + wp_lo));
    if (!(wo2 > 1e-6)) return false;
    const double reach = a.cull_rmax / sqrt(wo2);
    const double m = 0.1 + 1e-6 * (dh_top + r_hi);
    const double inner = fmax(r_lo - reach - m, 0.0), outer = r_hi + reach + m;
    const double iw = 1.0 / w;
    gx = x0 + dh0 * (u * iw);
    gy = y0 + dh0 * (v * iw);
    mid = 0.5 * (outer * outer + inner * inner);
    half = 0.5 * (outer * outer - inner * inner) * (1.0 + 1e-9) + 1e-6;
    return true;
}

// The sphere test of the cull for a tile of at most 32 steps, step l in lane l: lanes
// l and l + 32 test the lower half [0, nh) and the upper half [n_tel - nh, n_tel) of
// the sphere table (STRIDE doubles per sphere, X and Y first; one sphere twice when
// n_tel is odd), the same count and stride in both, in a uniform loop whose loads do
// not wait on the tests before them.  ok: the lane's step has an annulus (gx, gy, mid,
// half from screen_annulus).  True in lane l < 32 when step l's annulus holds a sphere
// centre.  Called by the whole wave.
template <int STRIDE>
__device__ __forceinline__ bool annulus_holds_centre(const double* tel, int n_tel, int lane, int ok, double gx,
                                                     double gy, double mid, double half)
{
    const int src = lane & (kWave / 2 - 1);
    const int ok_s = __shfl(ok, src);
    gx = __shfl(gx, src);
    gy = __shfl(gy, src);
    mid = __shfl(mid, src);
    half = __shfl(half, src);
    const int nh = (n_tel + 1) >> 1;
    const double* tp = tel + STRIDE * (lane < kWave / 2 ? 0 : n_tel - nh);
    bool reach = false;
#pragma unroll 4
    for (int i = 0; i < nh; ++i) {
        const double dx = tp[STRIDE * i] - gx, dy = tp[STRIDE * i + 1] - gy;
        reach |= fabs(fma(dy, dy, dx * dx) - mid) <= half;
    }
    reach = reach && ok_s;
    const uint64_t rm = __ballot(reach);
    return (((rm >> src) | (rm >> (src + kWave / 2))) & 1ull) != 0;
}

// A wave's area in the bunch kernel's LDS.
template <int PREC, int TS>
struct WaveArea {
    StepEntry<PREC>* stash;    // steps with bunches in the pass, compacted
    StepPass* pass;            // compacted like the stash
    uint32_t* masks;           // kSectorWords per step of the unit
    uint32_t* qk;              // waiting bunches: bunch in its step ...
    uint8_t* qs;               // ... and stash entry; setup: (sphere << 8) | step pairs
    int64_t* wcnt;
    int32_t* tcount;
    int64_t* prof;             // profile: shower of the bins below (-1: none), their bunches
    double* hph;               // photons (FP64) and bunches per depth bin
    uint32_t* hbu;
    __device__ __forceinline__ WaveArea(unsigned char* at, int n_tel, int prof_bins)
    {
        auto take = [&](size_t b) { unsigned char* q = at; at += b; return q; };
        stash = reinterpret_cast<StepEntry<PREC>*>(take(stash_steps(TS) * sizeof(StepEntry<PREC>)));
        pass = reinterpret_cast<StepPass*>(take(stash_steps(TS) * sizeof(StepPass)));
        masks = reinterpret_cast<uint32_t*>(take(kWave * kSectorWords * sizeof(uint32_t)));
        qk = reinterpret_cast<uint32_t*>(take(kQueue * sizeof(uint32_t)));
        qs = take(kQueue);
        wcnt = reinterpret_cast<int64_t*>(take(kWcCount * sizeof(int64_t)));
        tcount = reinterpret_cast<int32_t*>(take(((size_t)n_tel * sizeof(int32_t) + 15) & ~(size_t)15));
        prof = reinterpret_cast<int64_t*>(take(prof_bins ? 2 * sizeof(int64_t) : 0));
        hph = reinterpret_cast<double*>(take(prof_bins * sizeof(double)));
        hbu = reinterpret_cast<uint32_t*>(at);
    }
};
static_assert(kPairs * sizeof(uint32_t) <= kQueue * sizeof(uint32_t), "pairs share the queue's room");

// --------------------------------------------------------------------------
// Which bunches of a step can reach a sphere, from their azimuth alone.
//
// The bunches of a step leave from E(s) = P0 + s a, s in [0, L], in directions
// p = cos_t a + sin_t (cos(phi) b1 + sin(phi) b2).  All of E(s) lie on one line, so a
// point y of a bunch's straight emission line, tau > 0 ahead of E(s), has
//   (y - P0) . a = s + tau cos_t,   (y - P0) normal to a = tau sin_t (cos(phi), sin(phi)):
// its azimuth about the axis is phi wherever on the step the bunch was emitted, and its
// distance from the axis obeys  n(y) - t (y - P0) . a = -t s  with t = tan(theta_c).
// A bunch crosses a sphere (centre c, radius R) only if its observed line has a point
// y' within R of c.  light_cone gives `base`, a bound of the distance from y' to the
// straight emission line of a shifted centre c' (the shift px - x0, py - y0 is applied to
// P0 instead), so some y lies within rho = R + base of c' and
//   - n(c') - t A in [-t L - rho / cos_t, rho / cos_t], A = (c' - P0) . a  (n(y) - t (y .
//     a) changes by at most 1 / cos_t per metre), and
//   - |phi - azimuth of c'| <= asin(rho / n(c')), any phi when rho >= n(c').
// A step's azimuths that no sphere's window covers hold no crossing.
//
// Plane-parallel: the path's ground point is g = E_h + T(p) S, T(p) = p_h / w_p, S = dh
// (1 - beta) with beta in [0, B] for psi non-increasing with altitude, else in [-B, B]:
// S = int T4(x) dh with T4 the four-term series of (1 + x)^(-1/2), x = q (psi - psi_e),
// q = 1 / (n_e w_p)^2; for x in [0, 1/2] 0 <= 1 - T4(x) <= x / 2, for |x| <= 1/2
// |1 - T4(x)| <= 4 |x| / 5; x <= (psi_obs - psi_e) / (n_e w_p)^2 with psi_e taken at the
// step's start from the midpoint's and the table's largest slope.  The straight line's
// ground point is g + beta T(p) dh; with beta0 = B / 2 the centre moves by beta0 T(a) dh0
// and the rest is bounded by (B / 2) t_max dh0 + beta0 (|T(p) - T(a)| dh0 + |T(a)| w L),
// |T(p) - T(a)| <= sin_t / (w_p w).  The observed direction is within |1 - n_e / n_obs|
// (1 + 2 / w_p) of p, over at most R / w_o of the line.
// Spherical shells: the ray bends by at most t_max (n_obs - n_e), t_max the largest
// tangent of the local zenith angle along it (Bouguer: sin grows by r_e / r_obs at most),
// so it leaves the straight line by at most that times the path length; the planar
// array lies up to d^2 / (2 r_obs) above the observation sphere.
// On the 20 degree TeV shower (100 spheres) 19 % of the bunches are in steps with some
// window and 1.7 % lie in one (1.0 % cross), so 81 % of the bunches cost nothing and 98 %
// no propagation: 3083 VALU instructions per 32-step tile against 9570 with every bunch
// propagated; mixed kernel 1150 -> 550 us, FP64 2036 -> 580 us (2e6 steps; with the setup
// and the chunks shared by tiles, below, 1580 instructions, 239 and 247 us); spherical
// shells at 70 degrees, where a propagated bunch walks 250 cells, 3608 -> 360 us (1e5
// steps).  A bitmask of 256 sectors (2.9 m of a 120 m ring) takes any number of windows at
// one LDS read per bunch.
// Margins: 5 cm, 1e-6 of the distance (FP32 window arithmetic) and the mixed path's
// ground-point error, twice the screening pass's bound of it.
// A direction of length other than 1 by rounding, off = ||a|^2 - 1|: the path taken and
// the windows then use a, b1, b2 that differ from the unit step's orthonormal ones by off
// / 2, 1.12 off and 1.12 off (the frame's slope along a is below 2.24), so a bunch's p by
// delta = (0.51 + 1.7 sin_t) off.  Against the unit step's bunch its ground point moves by
// at most 4.1 delta dh / w_p^2 (p_h / w_p by 2, the advance S by 1.25), the test with its
// observed direction allows 2 delta R / w_o^2 more, the windows' coordinates of c' are
// wrong by 1.66 off |c' - P0| and the step's length by off / 2; with shells, where a cell
// takes the tangent from the invariant and the cosine separately, the first is 6 delta
// D / cos^2 of the path length D.  Directions stored in FP32 have off up to 1.2e-7 (2 cm at
// 20 km); refused from 1e-9 on, as they were, a 5e5-step TeV shower with such directions
// has every bunch propagated: 449 us, now 150.
//
// false where the bound does not hold (direction farther from unit, flat rays, psi's range
// too large) or where a bunch of the step might be dropped: the caller then takes every
// bunch, so drops are counted bunch by bunch as ever.
// --------------------------------------------------------------------------
template <bool CURVED, bool SCREEN>
__device__ __forceinline__ bool light_cone(const Args& a, const Setup& st, double& px, double& py, double& base,
                                           double& unit)
{
    const double u = st.u, v = st.v, w = st.w, ct = st.cos_t;
    const double dh0 = st.h0 - a.h_obs;
    px = st.x0;
    py = st.y0;
    base = 0.0;
    const double h2 = fma(u, u, v * v), e = fma(w, w, h2 - 1.0), off = fabs(e);
    unit = fma(e, fma(e, 0.375, -0.5), 1.0);         // 1 / |a|, to off^3
    if (!(off <= (CURVED ? 1e-6 : 1e-4)) || !(w >= 0.05)) return false;
    const double s_hi = st.sin_t * (1.0 + 1e-9) + 1e-12;
    const double sa = sqrt(h2);
    double wp = w * ct - sa * s_hi - 1e-12;          // lower bound of w_p
    // (the FP64 pass behind the screen drops w_p <= w_min itself)
    if (SCREEN) wp = fmax(wp, a.w_min);
    if (!SCREEN && !(wp > a.w_min + 1e-6)) return false;
    wp -= (0.51 + 1.7 * s_hi) * off;                 // and of the unit step's
    if (!(wp >= 0.03)) return false;
    // psi_obs - psi_e, with psi_e at the step's start, its highest point
    const double x_psi = a.sec_falls ? fmax(a.sec_psi_max - st.psi + a.sec_slope * (0.5 * st.len), 0.0)
                                     : a.sec_psi_max - a.sec_psi_min;
    const double iw = rcp64(wp), iw2 = iw * iw;
    double m = 0.05 + dh0 * (1e-6 * iw);
    if (CURVED) {
        if (!a.sec_falls) return false;
        // local zenith angle at both ends: r cos(zeta) from the downward vertical
        const double R = a.earth_r;
        const double rz0 = R + st.h0;
        const double r0 = sqrt(st.x0 * st.x0 + st.y0 * st.y0 + rz0 * rz0);
        const double alt0 = curved_altitude(R, st.x0, st.y0, st.h0);
        const double x1 = st.x0 + st.len * u, y1 = st.y0 + st.len * v, h1 = st.h0 - st.len * w;
        const double alt1 = curved_altitude(R, x1, y1, h1);
        // the smaller cosine
        const double c1 = (w * (R + h1) - u * x1 - v * y1) / (R + alt1) * (1.0 - off);
        if (!(c1 > 0.03) || !(alt0 < a.h_top - 1.0)) return false;
        const double c_lo = c1 * ct - sqrt(fmax(0.0, (1.0 - c1) * (1.0 + c1))) * s_hi - 1e-12;
        if (!(c_lo > 0.03)) return false;
        const double s_max = (r0 / a.r_obs) * sqrt((1.0 - c_lo) * (1.0 + c_lo)) * (1.0 + 1e-9);
        if (!(s_max < 0.9995)) return false;
        const double c_ray = sqrt((1.0 - s_max) * (1.0 + s_max));
        const double bend = (s_max / c_ray) * (0.5 * x_psi) * (1.0 + 1e-6);
        if (!(wp - bend >= 0.03)) return false;
        const double reach = a.sec_rmax / (wp - bend);
        const double d = a.sec_dmax + reach;
        base = bend * (alt0 - a.h_obs) / c_ray + 0.51 * d * d / a.r_obs + reach * bend +
               m + 1e-6 * (alt0 - a.h_obs) / c_ray;
        const double c = fmin(c_ray, wp - bend);
        base += off * rcp64(c * c) * ((8.0 + 12.0 * s_hi) * ((alt0 - a.h_obs) / c_ray) +
                                      (4.0 + 4.0 * s_hi) * a.sec_rmax + 3.0 * base);
        if (!(alt1 - a.h_obs > a.sec_rmax + base + 1.0)) return false;
    } else {
        const double x0 = x_psi / (1.0 + a.sec_psi_min);
        if (!(x0 * iw2 <= 0.5) || !(st.h0 < a.h_top - 1.0)) return false;
        const double B = (a.sec_falls ? 0.5 : 0.8) * x0 * iw2;
        const double t_max = sqrt((1.0 - wp) * (1.0 + wp)) * iw;
        const double iwa = rcp64(w), beta0 = a.sec_falls ? 0.5 * B : 0.0;
        double wo2 = wp * wp;
        if (!a.sec_falls) {
            wo2 = 1.0 - (1.0 + a.sec_psi_max) / (1.0 + a.sec_psi_min) * (1.0 - wp) * (1.0 + wp);
            if (!(wo2 > 1e-3)) return false;
        }
        const double iwo = rcp64(sqrt(wo2));
        m += dh0 * ((1e-6 * st.sin_t + 2e-9) * (iw + iw2) + 4e-6 * a.sec_psi_max * iw * iw2);
        base = (B - beta0) * t_max * dh0 + beta0 * (s_hi * iw * iwa * dh0 + sa * st.len) +
               a.sec_rmax * iwo * (0.51 * x0 * (1.0 + 2.0 * iw)) + m;
        base += off * ((5.0 + 8.0 * s_hi) * (dh0 * iw2 + a.sec_rmax * (iwo * iwo)) + 3.0 * base);
        px = st.x0 - beta0 * dh0 * (u * iwa);
        py = st.y0 - beta0 * dh0 * (v * iwa);
    }
    return dh0 - st.len * w > a.sec_rmax + base + 1.0;
}

// What the windows need of a step (in the stash's room during the setup).
struct ConeStep {
    double px, py;
    float b1x, b1y, b1z, b2x, b2y, b2z;
    float u, v, w, dh0, t, ict, len, base;
};
static_assert(kWave * sizeof(ConeStep) <= stash_steps(32) * (sizeof(StepEntry<1>) + sizeof(StepPass)),
              "cone steps share the room of the stash and the pass");

// Sectors of step c's azimuths whose light may reach sphere (X, Y, R^2), or-ed into its
// mask words.  FP32: its errors are inside light_cone's margin and the 2e-5 turns here.
__device__ __forceinline__ void add_window(const ConeStep& c, double X, double Y, double R2, uint32_t* words)
{
    const float dx = (float)(X - c.px), dy = (float)(Y - c.py), dz = -c.dh0;
    const float v1 = dx * c.b1x + dy * c.b1y + dz * c.b1z;
    const float v2 = dx * c.b2x + dy * c.b2y + dz * c.b2z;
    const float A = dx * c.u + dy * c.v - dz * c.w;
    const float rho = __builtin_amdgcn_sqrtf((float)R2) * 1.00001f + c.base;
    const float s2 = v1 * v1 + v2 * v2;
    const float n = __builtin_amdgcn_sqrtf(s2);
    const float rc = rho * c.ict + 1e-5f * n;
    if (!(n <= c.t * A + rc) || !(n >= c.t * (A - c.len) - rc)) return;
    const float q2 = rho * rho * __builtin_amdgcn_rcpf(s2);
    int pos = 0, left = kSectors;
    if (q2 < 0.64f) {
        // asin(q) <= q / sqrt(1 - q^2)
        const float half = __builtin_amdgcn_sqrtf(q2 * __builtin_amdgcn_rcpf(1.0f - q2)) * 0.15916f + 2e-5f;
        const float mid = atan2f(v2, v1) * 0.15915494f;
        const int lo = (int)floorf((mid - half) * (float)kSectors);
        const int hi = (int)floorf((mid + half) * (float)kSectors);
        pos = lo & (kSectors - 1);
        left = min(hi - lo + 1, kSectors);
    }
    while (left > 0) {
        const int bit = pos & 31, n_bits = min(32 - bit, left);
        atomicOr(&words[pos >> 5], (0xFFFFFFFFu >> (32 - n_bits)) << bit);
        pos = (pos + n_bits) & (kSectors - 1);
        left -= n_bits;
    }
}

// Longitudinal profile: the wave's bins to their shower's row.  Called by the whole wave.
template <typename Area>
__device__ __forceinline__ void flush_profile(const Args& a, const Area& wa, int lane)
{
    const int64_t s = wa.prof[0];
    for (int kk = lane; kk < a.prof_bins; kk += kWave) {
        const uint32_t c = wa.hbu[kk];
        if (c) {
            atomicAdd(&a.prof_ph[s * a.prof_bins + kk], wa.hph[kk]);
            atomicAdd((unsigned long long*)&a.prof_bu[s * a.prof_bins + kk], (unsigned long long)c);
            wa.hph[kk] = 0.0;
            wa.hbu[kk] = 0u;
        }
    }
    wave_lds_sync();
    if (lane == 0) wa.prof[1] = 0;
}

// A step's bunches into the depth bins, one step per lane.  The depth at a bunch's emission
// point is monotonic along the step and sub-step k holds bunch k, so a range of sub-steps
// whose ends lie in one bin (with 1e-6 m to spare, far above the rounding of a bunch's
// altitude) is counted at once; only a bunch whose sub-step holds a bin's edge, or an end
// of the table, takes its random number.  20 g/cm^2 bins hold 95 % of the steps whole.
template <typename Area>
__device__ __forceinline__ void profile_step(const Args& a, const Setup& st, int32_t nb, uint32_t ctr1,
                                             uint32_t shower_id, const Area& wa)
{
    auto depth = [&](double h) {
        const double x = (h - a.h_obs) * a.inv_step;
        const int c = max(0, min((int)x, a.n_nodes - 2));
        const double f = x - (double)c;
        return a.depth[c] + f * (a.depth[c + 1] - a.depth[c]);
    };
    auto bin = [&](double X) { return max(0, min((int)floor(X * a.inv_bin), a.prof_bins - 1)); };
    constexpr double slack = 1e-6;
    constexpr int kOutside = -1, kMixed = -2;
    // bin of all of sub-steps [ka, kb), kOutside (none of them counted) or kMixed
    auto bin_of = [&](int32_t ka, int32_t kb) {
        const double ha = st.h0 - ((double)ka * st.ds) * st.w, hb = st.h0 - ((double)kb * st.ds) * st.w;
        const double up = fmax(ha, hb) + slack, down = fmin(ha, hb) - slack;
        if (up < a.h_obs || down >= a.h_top) return kOutside;
        if (down < a.h_obs || up >= a.h_top) return kMixed;
        const int b = bin(depth(up) * (1.0 - 1e-13));
        return b == bin(depth(down) * (1.0 + 1e-13)) ? b : kMixed;
    };
    auto add = [&](int b, int32_t n) {
        if (b < 0) return;
        atomicAdd(&wa.hph[b], (double)n * st.photons);
        atomicAdd(&wa.hbu[b], (uint32_t)n);
    };
    int32_t k = 0;
    while (k < nb) {
        int b = bin_of(k, nb);
        int32_t end = nb;
        if (b == kMixed) {
            // the longest range from k in one bin: first where a linear depth puts the
            // edge, then by halving
            int32_t lo = k, hi = nb;
            const double Xk = depth(fmax(fmin(st.h0 - ((double)k * st.ds) * st.w, a.h_top), a.h_obs));
            const double Xe = depth(fmax(fmin(st.h0 - ((double)nb * st.ds) * st.w, a.h_top), a.h_obs));
            const double edge = (floor(Xk * a.inv_bin) + (Xe > Xk ? 1.0 : 0.0)) / a.inv_bin;
            const double part = Xe != Xk ? (edge - Xk) / (Xe - Xk) : 0.5;
            int32_t mid = k + (int32_t)(fmin(fmax(part, 0.0), 1.0) * (double)(nb - k));
            for (int probe = 0; hi - lo > 1; ++probe) {
                mid = max(lo + 1, min(mid, hi - 1));
                const int bm = bin_of(k, mid);
                if (bm != kMixed) { lo = mid; b = bm; } else { hi = mid; }
                mid = probe == 0 ? (bm != kMixed ? lo + 1 : hi - 1) : lo + (hi - lo) / 2;
            }
            end = lo;
        }
        if (end > k) add(b, end - k);
        k = end;
        if (k < nb) {
            // bunch k by its own emission point, as the bunch loop computes it
            uint32_t r[4];
            philox4x32_10((uint32_t)k, ctr1, shower_id, 0u, a.key0, a.key1, r);
            const double u0 = fma((double)r[0], 2.3283064365386963e-10, 1.1641532182693481e-10);
            const double s_along = ((double)k + u0) * st.ds;
            double he;
            {
#pragma clang fp contract(off)
                he = st.h0 - s_along * st.w;
            }
            const double xcell = (he - a.h_obs) * a.inv_step;
            const int ci = min((int)xcell, a.n_nodes - 2);
            if (he >= a.h_obs && he < a.h_top) add(profile_bin(a, ci, xcell - (double)ci), 1);
            ++k;
        }
    }
}

// Step setups of a unit, 1 or 64 / TS consecutive tiles (h_all), one step per lane: the
// bunch counts, which steps' light can reach a sphere and at which azimuths, the records
// of the steps that stay and the step-level counters.  With one tile the lanes past its
// steps repeat them and share the search over the spheres.  It covers the unit's tiles
// from h_first on, as many whole ones as the stash has room for; the caller comes back
// for the rest.  Called by the whole wave.
struct TileSetup {
    int32_t excl, incl;      // bunches of the pass before this lane's step, and through it
    int32_t shower;          // of this lane's tile
    bool in_pass;            // this lane's step has bunches in the pass
    bool masked;             // and they are taken by azimuth
    int32_t h_end;           // tiles h_first .. h_end - 1 are covered
};

template <int PREC, int TS, int FEAT>
__device__ __forceinline__ TileSetup tile_setup(const Args& a, int64_t t0, int h_first, int h_all, int lane,
                                                const WaveArea<PREC, TS>& wa,
                                                const double* tel_sh)
{
    constexpr bool SCREEN = (FEAT & kFeatScreen) != 0;
    constexpr bool PROF = (FEAT & kFeatProfile) != 0;
    constexpr bool CURVED = (FEAT & kFeatCurved) != 0;
    using T = typename std::conditional<PREC == 0, double, float>::type;
    using Entry = StepEntry<PREC>;
    // this lane's tile, its shower and its step
    const int l = lane & (TS * h_all - 1), h = l / TS;
    const bool own = lane == l;
    const bool covered = h >= h_first;
    const int64_t t = t0 + (covered ? h : h_first);
    int s = 0;
    for (int hi = a.n_showers; hi - s > 1;) {     // tiles_before[s] <= t < tiles_before[hi]
        const int mid = (s + hi) >> 1;
        if (a.tiles_before[mid] <= t) s = mid; else hi = mid;
    }
    const int64_t seg0 = a.seg_offsets[s], seg1 = a.seg_offsets[s + 1];
    const int64_t g = a.shower_first[s] + (t - a.tiles_before[s]) * (int64_t)TS + (l & (TS - 1));
    const uint32_t shower_id = a.shower_ids ? a.shower_ids[s] : (uint32_t)s;
    int64_t nb = 0;
    int status = -2;   // -2: no step in this lane
    Setup st;
    uint32_t ctr1 = 0;
    int32_t heavy = 0;
    if (covered && g < seg1) {
        if (TS < 32 && a.heavy) heavy = a.heavy[g / kHeavySteps];
        // screening: the frozen count loaded with the step's inputs, not after them
        const int64_t f = SCREEN ? a.nb_frozen[g] : 0;
        ctr1 = a.step_id ? a.step_id[g] : (uint32_t)((a.seg_id_base ? a.seg_id_base[s] : 0) + (g - seg0));
        step_setup(a, g, st);
        status = st.status;
        if (st.status < 0) nb = st.nb;
        if (SCREEN && st.status < 0) {
            // the soft response's sub-steps: the frozen count, light or not at
            // the current atmosphere decided above
            if (f > 0) {
                nb = f;
                st.ds = st.len / (double)f;
            } else {
                nb = 0;
                status = -4;
            }
        }
    }
    const int l_first = l & ~(TS - 1), l_last = l | (TS - 1);
    int64_t tile_nb, unit_nb;
    {
        const int64_t n = own ? nb : 0, c = wave_incl_scan(n);
        unit_nb = scalar64(wave_last(c));
        tile_nb = __shfl(c, l_last) - __shfl(c - n, l_first);
    }
    bool over = tile_nb >= ((int64_t)1 << 30);
    if (TS < 32 && heavy) over = over || a.heavy_step[g] != 0;
    if (over) {
        // bunch offsets inside a tile are 32-bit: refuse such a tile
        nb = 0;
        tile_nb = 0;
        status = status == -1 ? -3 : status;
    }
    const bool emits = status == -1;
    // ---- azimuth sectors: the pairs (step, sphere) that pass the cone test, then their
    // windows, a pair per lane
    bool cone = false, seen = true;
    const bool live = emits && nb > 0;
    if (a.sec_rmax > 0.0) {
        double px = 0.0, py = 0.0, base = 0.0, unit = 0.0;
        if (live) cone = light_cone<CURVED, SCREEN>(a, st, px, py, base, unit);
        const double ict = cone ? rcp64(st.cos_t) : 0.0;
        const double tn = cone ? st.sin_t * ict : 0.0;
        const double dh0 = cone ? st.h0 - a.h_obs : 0.0;
        const double rc = cone ? (a.sec_rmax + base) * ict : -1.0;
        // (the unit direction: n2 below is the difference of two squares near the distance's)
        const double du = cone ? st.u * unit : 0.0, dv = cone ? st.v * unit : 0.0, dw = cone ? st.w * unit : 1.0;
        // candidates: the spheres near the cone's ground ellipse: a centre d from G, the
        // axis's ground point, has n >= d w and A <= dh0 / w + d sin(zeta_a), so passing takes
        // d (w - t sin(zeta_a)) <= t dh0 / w + rc; all spheres beyond the lists
        uint2 near{0u, 0u};
        bool far = true;
        if (cone && a.reach_levels > 0) {
            const double iw = rcp64(dw), s_a = sqrt(du * du + dv * dv);
            const double room = dw - tn * s_a;
            const float r = (float)(fma(tn * dh0, iw, rc) * rcp64(room)) * 1.0001f;
            const int lv = max(0, (int)ceilf(2.0f * __log2f(r * (float)(1.0 / kReachMin)) + 1e-3f));
            far = !(room > 1e-3) || !(r < 1e6f) || lv >= a.reach_levels;
            if (!far) {
                const ReachLevel lev = a.reach_lev[lv];
                const double fx = (fma(dh0 * iw, du, px) - lev.x0) * (double)lev.inv_cell;
                const double fy = (fma(dh0 * iw, dv, py) - lev.y0) * (double)lev.inv_cell;
                // (a ground point outside the grid is farther than the level's radius)
                if (fx >= 0.0 && fy >= 0.0 && fx < (double)lev.nx && fy < (double)lev.ny)
                    near = a.reach_rec[lev.rec + (uint32_t)((int)fx * lev.ny + (int)fy)];
            }
        }
        int n4 = cone ? ((far ? a.n_tel : (int)near.y) + kReachPad - 1) / kReachPad : 0;
        const int groups = kWave / (TS * h_all);
        // A round of 4 candidates a lane costs about a sixth of a chunk of bunches: where the
        // longest list takes more, all bunches are taken (2e5-3e5 TeV steps, 1024 spheres, us
        // searched / taken / as ruled: 60 degrees 190 / 300 / 191, with ten times larger
        // bunches 197 / 152 / 166 and before, all spheres a step, 516 and 730; 75 degrees over
        // 400 spheres 187 / 222 / 170).  A chunk through the shells costs 50 times as much.
        if (!CURVED) {
            const int most = kSearchFree + (int)(min(unit_nb, (int64_t)1 << 20) * kSearchPerChunk / kWave);
            if (__ballot(n4 > most * groups)) {
                cone = false;
                n4 = 0;
            }
        }
        if (__ballot(cone)) {
            for (int q = lane; q < TS * h_all * kSectorWords; q += kWave) wa.masks[q] = 0u;
            ConeStep* cs = reinterpret_cast<ConeStep*>(wa.stash);
            if (cone && own) {
                ConeStep& c = cs[l];
                c.px = px; c.py = py;
                c.b1x = (float)st.b1x; c.b1y = (float)st.b1y; c.b1z = (float)st.b1z;
                c.b2x = (float)st.b2x; c.b2y = (float)st.b2y; c.b2z = (float)st.b2z;
                c.u = (float)st.u; c.v = (float)st.v; c.w = (float)st.w;
                c.dh0 = (float)dh0;
                c.t = (float)tn; c.ict = (float)ict; c.len = (float)st.len; c.base = (float)base * 1.00001f;
            }
            wave_lds_sync();
            uint32_t* pairs = wa.qk;
            const double kA = dh0 * dw, kz = dh0 * dh0;
            const double rl = -(tn * st.len + rc);
            auto passes = [&](int k) {
                const double dx = tel_sh[3 * k] - px, dy = tel_sh[3 * k + 1] - py;
                const double A = fma(dx, du, fma(dy, dv, kA));
                const double n2 = fma(-A, A, fma(dx, dx, fma(dy, dy, kz)));
                const double hi = fma(tn, A, rc), lo = fmax(fma(tn, A, rl), 0.0);
                return fma(-hi, hi, n2) <= 0.0 && fma(-lo, lo, n2) >= 0.0;
            };
            int np = 0;
            auto windows = [&]() {
                wave_lds_sync();
                if (lane < np) {
                    const uint32_t e = pairs[lane];
                    const double* tq = tel_sh + 3 * (e >> 8);
                    add_window(cs[e & 0xFFu], tq[0], tq[1], tq[2], wa.masks + kSectorWords * (e & 0xFFu));
                }
                wave_lds_sync();
                if (np > kWave && lane < np - kWave) pairs[lane] = pairs[kWave + lane];
                np = np > kWave ? np - kWave : 0;
            };
            // candidates 4 at a time: the lane's next list entries, or all spheres in order
            for (int i = lane / (TS * h_all); __ballot(i < n4); i += groups) {
                uint2 four{0xFFFFFFFFu, 0xFFFFFFFFu};
                if (!far && i < n4) four = a.reach_list[near.x / kReachPad + i];
                uint32_t p4 = 0;
#pragma unroll
                for (int q = 0; q < kReachPad; ++q) {
                    int k = (int)(((q < 2 ? four.x : four.y) >> (16 * (q & 1))) & 0xFFFFu);
                    if (far) k = kReachPad * i + q;
                    if (i < n4 && k < a.n_tel && passes(k)) p4 |= 1u << q;
                }
                while (__ballot(p4 != 0u)) {
                    const int q = p4 ? __builtin_ctz(p4) : 0;
                    const int k = far ? kReachPad * i + q
                                      : (int)(((q < 2 ? four.x : four.y) >> (16 * (q & 1))) & 0xFFFFu);
                    const uint64_t m = __ballot(p4 != 0u);
                    if (p4) pairs[np + lanes_below(m)] = ((uint32_t)k << 8) | (uint32_t)l;
                    np += __popcll(m);
                    p4 &= p4 - 1;
                    if (np >= kWave) windows();
                }
            }
            while (np > 0) windows();
            wave_lds_sync();
            if (cone) {
                uint32_t any = 0;
#pragma unroll
                for (int q = 0; q < kSectorWords; ++q) any |= wa.masks[kSectorWords * l + q];
                seen = any != 0u;
            }
            // (the reads above before the stash's writes below)
            wave_lds_sync();
        }
    }
    // ---- the tiles covered now: whole ones, while their steps in the pass fit the stash and
    // their bunches 30 bits (the profile's bins are one shower's)
    bool in_pass = own && live && seen;
    int h_end = h_first;
    {
        const uint64_t stay = __ballot(in_pass);
        int64_t sum = 0;
        int n = 0;
        for (; h_end < h_all; ++h_end) {
            const int l0 = h_end * TS;
            n += __popcll((stay >> l0) & (~0ull >> (64 - TS)));
            sum += scalar64(__shfl(tile_nb, l0));
            if (h_end > h_first && (n > stash_steps(TS) || sum >= ((int64_t)1 << 30))) break;
            if (PROF && __shfl(s, l0) != __shfl(s, h_first * TS)) break;
        }
    }
    const bool now = own && covered && h < h_end;
    in_pass = in_pass && now;
    if (over && now && lane == l_first && a.result) atomicOr(&a.result->error, 2);
    const bool masked = in_pass && cone;
    if (__ballot(masked) != 0ull && in_pass && !cone) {
        // no bound for this step: every azimuth
#pragma unroll
        for (int q = 0; q < kSectorWords; ++q) wa.masks[kSectorWords * lane + q] = 0xFFFFFFFFu;
    }
    const int32_t nbp = in_pass ? (int32_t)nb : 0;
    const int32_t incl = (int32_t)wave_incl_scan((int64_t)nbp);
    const int32_t excl = incl - nbp;      // first bunch of this lane's step
    const uint64_t pass_mask = __ballot(in_pass);
    if (in_pass) {
        const int at = lanes_below(pass_mask);
        Entry& e = wa.stash[at];
        e.ctr1 = ctr1;
        // Philox: the first round's word 0 is the same for all bunches of the step, and
        // with it the second round's product of that word
        const uint32_t w0 = __umulhi(0xCD9E8D57u, shower_id) ^ ctr1 ^ a.key0;
        StepPass sp;
        sp.boff = excl;
        sp.sidx = lane;
        sp.hi0 = __umulhi(0xD2511F53u, w0);
        sp.lo0 = 0xD2511F53u * w0;
        wa.pass[at] = sp;
        e.x0 = st.x0;
        e.y0 = st.y0;
        e.h0 = st.h0;
        e.t0 = st.t0;
        e.u = st.u;
        e.v = st.v;
        e.w = st.w;
        e.cos_t = st.cos_t;
        e.ds = st.ds;
        e.inv_bc = st.inv_bc;
        e.sb1x = (T)(st.sin_t * st.b1x);
        e.sb1y = (T)(st.sin_t * st.b1y);
        e.sb1z = (T)(st.sin_t * st.b1z);
        e.sb2x = (T)(st.sin_t * st.b2x);
        e.sb2y = (T)(st.sin_t * st.b2y);
        e.sb2z = (T)(st.sin_t * st.b2z);
        e.photons = st.photons;
        e.sidx = lane;
    }
    const int64_t total_now = scalar64(wave_last(wave_incl_scan(now ? nb : 0)));
    {
        const int n_emit = __popcll(__ballot(now && emits));
        const int d_mass = __popcll(__ballot(now && status == CKV_DROP_MASS));
        const int d_thr = __popcll(__ballot(now && status == CKV_DROP_THRESHOLD));
        const int d_nf = __popcll(__ballot(now && status == CKV_DROP_NONFINITE));
        if (lane == 0) {
            wa.wcnt[kWcBunches] += total_now;
            wa.wcnt[kWcEmitting] += n_emit;
            wa.wcnt[kWcDrop0 + CKV_DROP_MASS] += d_mass;
            wa.wcnt[kWcDrop0 + CKV_DROP_THRESHOLD] += d_thr;
            wa.wcnt[kWcDrop0 + CKV_DROP_NONFINITE] += d_nf;
        }
    }
    if constexpr (PROF) {
        // the bins hold one shower's bunches, fewer than 2^32 of them
        const int s_now = __builtin_amdgcn_readlane(s, h_first * TS);
        if (wa.prof[0] >= 0 && (wa.prof[0] != s_now || wa.prof[1] + total_now >= ((int64_t)1 << 32)))
            flush_profile(a, wa, lane);
        wave_lds_sync();
        if (lane == 0) {
            wa.prof[0] = s_now;
            wa.prof[1] += total_now;
        }
        if (now && live) profile_step(a, st, (int32_t)nb, ctr1, shower_id, wa);
    }
    return TileSetup{excl, incl, s, in_pass, masked, h_end};
}

// The same with the arguments where the launch put them, the kernel argument segment,
// and the wave's places in LDS as offsets: the bunch loop's copies of them then take no
// registers here, nor these there.
template <int PREC, int TS, int FEAT>
__device__ __forceinline__ TileSetup tile_setup_at(uint64_t args_at, int64_t t0, int h_first, int h_all, int lane,
                                                   uint32_t area_at, uint32_t tel_at)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const Args& a = args_from(args_at);
    const WaveArea<PREC, TS> wa(lds + __builtin_amdgcn_readfirstlane((int)area_at),
                                (FEAT & kFeatScreen) != 0 ? 0 : a.n_tel * a.span_tiles, (FEAT & kFeatProfile) != 0 ? a.prof_bins : 0);
    return tile_setup<PREC, TS, FEAT>(a, scalar64(t0), __builtin_amdgcn_readfirstlane(h_first),
                                      __builtin_amdgcn_readfirstlane(h_all), lane, wa,
                                      reinterpret_cast<const double*>(
                                          lds + __builtin_amdgcn_readfirstlane((int)tel_at)));
}

// As a called function, for the builds that keep loop invariants in registers
// (kFeatExact, kFeatCurved): the step setup's then take no room in the bunch loop.
template <int PREC, int TS, int FEAT>
__device__ __noinline__ CKV_LINE TileSetup tile_setup_call(uint64_t args_at, int64_t t0, int h_first, int h_all, int lane,
                                                  uint32_t area_at, uint32_t tel_at)
{
    return tile_setup_at<PREC, TS, FEAT>(args_at, t0, h_first, h_all, lane, area_at, tel_at);
}

// Screening pass: the n ids of a wave's buffer to the list; one atomic claims exactly
// their slots.  Called by the whole wave.
constexpr int kScreenBuf = 256;

__device__ __forceinline__ void flush_list(const Args& a, const uint64_t* buf, int n, int lane)
{
    if (n == 0) return;
    int64_t base = 0;
    if (lane == 0) base = (int64_t)atomicAdd((unsigned long long*)a.list_count, (unsigned long long)n);
    base = scalar64(base);
    wave_lds_sync();
    for (int q = lane; q < n; q += kWave)
        if (base + q >= 0 && base + q < a.list_cap) a.list_ids[base + q] = buf[q];
    wave_lds_sync();
}

// Tiles are worked on in units that a wave sets up together: 64 steps' worth of tiles, then
// the last two rounds of the grid's waves tile by tile, so that the launch ends evenly.  With
// head (the waves), the first round goes in units of 32 steps and one at the end tile by tile.
struct Units {
    int64_t head, wide;      // units of 32 steps (at least a tile), then units of 64
    int64_t count;
};

__device__ __forceinline__ Units units_of(int64_t n_tiles, int head, int grid_waves, int tile_segs)
{
    // (tiles of a unit are powers of two)
    const int per = 6 - __builtin_ctz(tile_segs), half = max(per - 1, 0);
    int64_t left = max(n_tiles - (head ? 1 : 2) * (int64_t)grid_waves, (int64_t)0);
    const int64_t first = min((int64_t)head, left >> half);
    left -= first << half;
    const int64_t wide = left >> per;
    return Units{first, wide, first + wide + (n_tiles - (first << half) - (wide << per))};
}

template <int PREC, int TS, int FEAT>
__global__ void __launch_bounds__(emit_threads(PREC, FEAT)) emit_kernel(Args a)
{
    constexpr bool PROF = (FEAT & kFeatProfile) != 0;
    constexpr bool EXACT = (FEAT & kFeatExact) != 0;
    constexpr bool SEARCH = (FEAT & kFeatSearch) != 0;
    constexpr bool CURVED = (FEAT & kFeatCurved) != 0;
    constexpr bool SCREEN = (FEAT & kFeatScreen) != 0;
    constexpr bool SLOWPATH = EXACT || CURVED;    // lanes that leave the moment series
    using T = typename std::conditional<PREC == 0, double, float>::type;
    using Entry = StepEntry<PREC>;
    extern __shared__ __align__(16) unsigned char lds[];

    const int lane = lane_id();
    // scalar, so that the wave's LDS addresses take no lane registers (the slow-path builds
    // have those to spare)
    const int wave = SLOWPATH ? (int)threadIdx.x / kWave : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);

    // node tables: altitudes and inverse widths
    double* hn_lds = reinterpret_cast<double*>(lds);
    const size_t srch_bytes = SEARCH ? search_bytes(a.n_nodes) : 0;
    if (SEARCH)
        for (int q = threadIdx.x; q < 2 * a.n_nodes - 1; q += blockDim.x) hn_lds[q] = a.hnodes[q];
    // sphere table {X, Y, R^2} after them
    double* tel_sh = reinterpret_cast<double*>(lds + srch_bytes);
    for (int q = threadIdx.x; q < a.n_tel; q += blockDim.x) {
        tel_sh[3 * q] = a.tel[4 * q];
        tel_sh[3 * q + 1] = a.tel[4 * q + 1];
        tel_sh[3 * q + 2] = a.tel[4 * q + 3];
    }
    const int prof_bins = PROF ? a.prof_bins : 0;
    const int n_count = SCREEN ? 0 : a.n_tel * a.span_tiles;      // crossings counted per tile and sphere
    const size_t wv_bytes = wave_bytes(PREC, TS, n_count, prof_bins);
    const size_t wv_stride = wv_bytes + (SCREEN ? kScreenBuf * sizeof(uint64_t) : 0);
    unsigned char* wbase = lds + srch_bytes + tel_bytes(a.n_tel) + (size_t)wave * wv_stride;
    const WaveArea<PREC, TS> wa(wbase, n_count, prof_bins);
    // screening: ids on their way to the list
    uint64_t* const buf = reinterpret_cast<uint64_t*>(wbase + wv_bytes);
    int buf_n = 0;
    Entry* const stash = wa.stash;
    int64_t* const wcnt = wa.wcnt;
    int32_t* const tcount = wa.tcount;
    for (int k = lane; k < n_count; k += kWave) tcount[k] = 0;
    if (PROF) {
        for (int k = lane; k < prof_bins; k += kWave) { wa.hph[k] = 0.0; wa.hbu[k] = 0u; }
        if (lane < 2) wa.prof[lane] = lane == 0 ? -1 : 0;
    }
    if (lane < kWcCount) wcnt[lane] = 0;
    __syncthreads();

    const T a1 = (T)-0.5, a2 = (T)0.375, a3 = (T)-0.3125, a4 = (T)0.2734375;
    const double inv_c = 1.0 / kSpeedOfLight;
    const float step32 = __builtin_bit_cast(
        float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, (float)a.step)));
    // n - 1 at the observation level, for the observed direction
    const double inv_nobs64 = 1.0 / a.n_obs;
    const float d_obs = (float)(a.n_obs - 1.0);
    const float inv_1pdobs = 1.0f / (1.0f + d_obs);
    // grazing limit of the drop rules, read once (a scalar load in the bunch loop made
    // its wait cover the loop's LDS reads as well).  Screening keeps bunches down to
    // w_min - 1e-6, ten times the mixed direction's error: the FP64 candidate pass
    // applies the exact rule.
    const double w_graze = __builtin_bit_cast(double, scalar64(__builtin_bit_cast(int64_t,
                               SCREEN ? a.w_min - 1e-6 : a.w_min)));

    int64_t blk = -1;          // current staging block; -1: none, -2: staging full
    int blk_fill = 0;
    int64_t lost = INT64_MAX;  // first tile of this wave with a crossing that found no slot
    int64_t rblk = -1;         // current run block; -1: none
    int rfill = 0;
    const int64_t n_tiles = a.ctrl[kNumTiles];

    // Atmosphere at an emission point in cell ci at fraction f (node tables: dcell_
    // above the cell's lower node h_i): psi_e and D_k = int_{h_obs}^{h_e} (psi -
    // psi_e)^k dh, k = 1..5.  Below h_i the node moments are shifted to psi_e,
    // sum_j C(k,j) (-psi_e)^(k-j) P_j(h_i) with P_0(h_i) = h_i - h_obs (Pascal-triangle
    // shift); inside the cell psi is linear from psi_i to psi_e, so the rest is
    // dz (psi_i - psi_e)^k / (k+1).  The bunch loop takes D_1..D_4 for the advance;
    // the arrival time, needed only for a crossing's record, takes D_5 as well.
    struct CellMoments { T psi_e, D1, D2, D3, D4, D5; };
    auto cell_moments = [&](int ci, T f, double dcell_) {
        T psi_i, dpsi, P0, P1, P2, P3, P4, P5;
        if (PREC == 0) {
            const HbmF64* nd = as_hbm(a.node64) + (size_t)kNode64 * ci;
            psi_i = nd[0];
            dpsi = nd[kNode64] - psi_i;
            P0 = SEARCH ? hn_lds[ci] - a.h_obs : (double)ci * a.step;
            P1 = nd[1]; P2 = nd[2]; P3 = nd[3]; P4 = nd[4]; P5 = nd[5];
        } else {
            const HbmF32x4* cg = as_hbm4(a.cell32) + 2 * (size_t)ci;
            const f32x4 c_a = cg[0], c_b = cg[1];
            psi_i = c_a.x; dpsi = c_a.y; P1 = c_a.z; P2 = c_a.w;
            P3 = c_b.x; P4 = c_b.y; P5 = c_b.z;
            P0 = c_b.w;
        }
        CellMoments m;
        m.psi_e = psi_i + f * dpsi;
        const T dz = SEARCH ? (T)dcell_ : f * (PREC == 0 ? (T)a.step : (T)step32);
        const T c1 = -m.psi_e;
        T X0 = P0, X1 = P1, X2 = P2, X3 = P3, X4 = P4, X5 = P5;
        X5 += c1 * X4; X4 += c1 * X3; X3 += c1 * X2; X2 += c1 * X1; X1 += c1 * X0;
        X5 += c1 * X4; X4 += c1 * X3; X3 += c1 * X2; X2 += c1 * X1;
        X5 += c1 * X4; X4 += c1 * X3; X3 += c1 * X2;
        X5 += c1 * X4; X4 += c1 * X3;
        X5 += c1 * X4;
        const T del = -f * dpsi;               // psi_i - psi_e
        const T e1 = dz * del, e2 = e1 * del, e3 = e2 * del, e4 = e3 * del, e5 = e4 * del;
        m.D1 = X1 + e1 * (T)0.5;
        m.D2 = X2 + e2 * (T)(1.0 / 3.0);
        m.D3 = X3 + e3 * (T)0.25;
        m.D4 = X4 + e4 * (T)0.2;
        m.D5 = X5 + e5 * (T)(1.0 / 6.0);
        return m;
    };
    // Index terms at emission (n_e = 1 + delta_e) for a photon of vertical cosine w:
    // n_e, 1/w, n_e / n_obs (the observed direction's scale), q = 1/(n_e w)^2, 1/n_e
    // and n_e^2.
    struct IndexTerms { double ne, inv_w; T ratio, q, inv_ne, ne2; };
    auto index_terms = [&](T psi_e, double pw) {
        IndexTerms x;
        x.ne2 = (T)1 + psi_e;
        if (PREC == 0) {
            x.ne = sqrt(1.0 + (double)psi_e);
            x.ratio = (T)(x.ne * inv_nobs64);
            x.inv_w = rcp64(pw);
            x.inv_ne = (T)rcp64(x.ne);
            x.q = (T)(x.inv_w * x.inv_w) * (x.inv_ne * x.inv_ne);
        } else {
            const float de = (float)psi_e * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_sqrtf(1.0f + (float)psi_e));
            x.ne = 1.0 + (double)de;
            x.ratio = 1.0f + (de - d_obs) * inv_1pdobs;
            // reciprocal of w: the hardware estimate (relative error below 2^-24 on
            // this chip) and one Newton step, 2e-15 relative
            const double r_w = __builtin_amdgcn_rcp(pw);
            x.inv_w = fma(r_w, fma(-pw, r_w, 1.0), r_w);
            x.q = (T)__builtin_amdgcn_rcpf((float)x.ne2 * (float)(pw * pw));
            x.inv_ne = (T)__builtin_amdgcn_rcpf(1.0f + de);
        }
        return x;
    };
    // series part of the horizontal advance, S - dh = sum_{k>=1} a_k q^k D_k
    auto advance_series = [&](const CellMoments& m, T q) {
        return q * (a1 * m.D1 + q * (a2 * m.D2 + q * (a3 * m.D3 + q * a4 * m.D4)));
    };
    // travel time from the emission height dh above the observation level:
    // c * time * w = n_e dh + (1/n_e) [D1 + sum_{k>=1} a_k q^k (n_e^2 D_k + D_{k+1})]
    //              = n_e dh + (1/n_e) [D1 + n_e^2 s_corr + sum_{k>=1} a_k q^k D_{k+1}]
    auto travel_time = [&](const CellMoments& m, const IndexTerms& ix, T s_corr, double dh) {
        const T q = ix.q;
        const T t_corr = m.D1 + ix.ne2 * s_corr +
                         q * (a1 * m.D2 + q * (a2 * m.D3 + q * (a3 * m.D4 + q * a4 * m.D5)));
        const double ctw = fma(ix.ne, dh, (double)(t_corr * ix.inv_ne));
        return ctw * ix.inv_w * inv_c;
    };

    // Units of tiles are dealt in kTileClasses interleaved classes, one per group of
    // workgroups, each with its claim counter on its own cache line: all waves' claims on
    // one address came 13 ns apart, which bounded the kernel once a tile took less (62 500
    // tiles: 0.83 ms).  Each wave's first unit goes by its place in the grid, a workgroup's
    // first wave first.
    const int n_cls = min(kTileClasses, (int)gridDim.x), cls = (int)blockIdx.x % n_cls;
    const int cls_groups = ((int)gridDim.x - cls + n_cls - 1) / n_cls;
    const int cls_waves = cls_groups * (int)(blockDim.x / kWave);
    const Units units = units_of(n_tiles, a.head_units, a.grid_waves, TS);
    int64_t unit = cls + (int64_t)n_cls * scalar64(wave * cls_groups + (int)blockIdx.x / n_cls);
    // a wave with a first unit has a staging and a run block of its own from the start (all
    // waves' first claims would queue at the counters: 50 us of a launch)
    if (unit < a.static_blocks && unit < units.count) blk = rblk = unit;
    while (unit < units.count) {
        int64_t claimed = 0;
        constexpr int kPer = kWave / TS, kHalf = kPer > 1 ? kPer / 2 : 1;
        const int64_t at = unit - units.head;
        const bool wide = at >= 0 && at < units.wide;
        const int64_t t0 = at < 0 ? unit * kHalf
                                  : units.head * kHalf + at + min(at, units.wide) * (kPer - 1);
        const int h_all = wide ? kPer : at < 0 ? kHalf : 1;
        TileSetup ts_;
        ts_.h_end = 0;
        for (int h = 0, h_next; h < h_all; h = h_next) {
        // ---- step setups of the unit.  A call saves 40 registers a lane to scratch, more HBM
        // traffic than all else; inlined, 2e6 steps take 280 against 286 us, FP64 268 against
        // 282 (268 and 264 with the wave index scalar and the lane masks counted).  Where
        // loop invariants are kept in registers the call is the better one.
        if (h >= ts_.h_end) {
            const uint64_t args_at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
            const uint32_t area_at = (uint32_t)(wbase - lds);
            const uint32_t tel_at = (uint32_t)(reinterpret_cast<unsigned char*>(tel_sh) - lds);
            if constexpr (SLOWPATH)
                ts_ = tile_setup_call<PREC, TS, FEAT>(args_at, t0, h, h_all, lane, area_at, tel_at);
            else
                ts_ = tile_setup_at<PREC, TS, FEAT>(args_at, t0, h, h_all, lane, area_at, tel_at);
            ts_.h_end = __builtin_amdgcn_readfirstlane(ts_.h_end);
            wave_lds_sync();
        }
        // ---- a span: tiles of one shower that were set up together, their bunches taken
        // together (a tile's fill 1.3 chunks of the second pass, two tiles' 1.8)
        const int s = __builtin_amdgcn_readlane(ts_.shower, h * TS);
        for (h_next = h + 1; h_next < ts_.h_end && h_next < h + a.span_tiles; ++h_next)
            if (__builtin_amdgcn_readlane(ts_.shower, h_next * TS) != s) break;
        const uint32_t shower_id = a.shower_ids ? a.shower_ids[s] : (uint32_t)s;
        const double t_ref = a.t_ref[s];
        const bool in_pass = ts_.in_pass;
        const int excl = ts_.excl;
        const int c_end = __builtin_amdgcn_readlane(ts_.incl, h_next * TS - 1);
        // every bunch is taken, whatever its azimuth
        const bool direct = __ballot(ts_.masked) == 0ull;

        // ---- bunches of the span, one per lane.  Where azimuths count, a first pass tests
        // each bunch's draw against its step's sectors; those that may reach a sphere wait
        // in the queue until 64 are there, in (step, bunch) order.
        // Where all are taken they go straight to their chunk, past draw test and queue: 5e5
        // TeV steps in mixed precision whose w_min drops every bunch 275 -> 249 us (297 with
        // any_of's copies as well; 271 before there were sectors, the table in LDS).
        int c0 = __builtin_amdgcn_readlane(excl, h * TS), qn = 0;
        // step of bunch c0 + lane: the pass's steps starting at or before c0, plus those
        // starting inside this chunk at or before it (one to three, by lane reads)
        auto step_at = [&]() {
            const int cnt0 = __popcll(__ballot(in_pass && excl <= c0));
            uint64_t starts = 0;
            for (uint64_t in = __ballot(in_pass && excl > c0 && excl < c0 + kWave); in; in &= in - 1)
                starts |= 1ull << (__builtin_amdgcn_readlane(excl, __builtin_ctzll(in)) - c0);
            return cnt0 - 1 + lanes_upto(starts);
        };
        for (;;) {
            // ---- a chunk: bunch k of stash entry si
            bool active;
            int32_t k = any_of<int32_t>();
            int si;
            if (direct) {
                if (c0 >= c_end) break;
                wave_lds_sync();
                active = c0 + lane < c_end;
                si = step_at();
                if (active) k = c0 + lane - wa.pass[si].boff;
                c0 += kWave;
            } else {
                while (qn < kWave && c0 < c_end) {
                    const int sj = step_at();
                    // Philox round keys, advanced on the scalar unit inside the loop
                    const uint32_t opaque = (uint32_t)((uint64_t)(uint32_t)c0 >> 31);   // 0; keeps the schedule in the loop
                    uint32_t kr0 = a.key0 + opaque, kr1 = a.key1 + opaque;
                    bool take = false;
                    int32_t kj = any_of<int32_t>();
                    if (c0 + lane < c_end) {
                        const StepPass sp = wa.pass[sj];
                        kj = c0 + lane - sp.boff;
                        // Philox as far as the second draw: its last two rounds need one
                        // product each
                        const uint64_t f0 = (uint64_t)0xD2511F53u * (uint32_t)kj;
                        const uint32_t f1_lo = 0xCD9E8D57u * shower_id;
                        uint32_t c_0, c_1, c_2, c_3;
                        {
                            const uint64_t p1 = (uint64_t)0xCD9E8D57u * ((uint32_t)(f0 >> 32) ^ kr1);
                            kr0 += 0x9E3779B9u;
                            kr1 += 0xBB67AE85u;
                            c_0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), f1_lo, kr0, 0x96);
                            c_2 = __builtin_amdgcn_bitop3_b32(sp.hi0, (uint32_t)f0, kr1, 0x96);
                            c_1 = (uint32_t)p1;
                            c_3 = sp.lo0;
                        }
#pragma unroll
                        for (int rr = 2; rr < 7; ++rr) {
                            kr0 += 0x9E3779B9u;
                            kr1 += 0xBB67AE85u;
                            const uint64_t p0 = (uint64_t)0xD2511F53u * c_0;
                            const uint64_t p1 = (uint64_t)0xCD9E8D57u * c_2;
                            c_0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c_1, kr0, 0x96);
                            c_2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c_3, kr1, 0x96);
                            c_1 = (uint32_t)p1;
                            c_3 = (uint32_t)p0;
                        }
                        kr0 += 0x9E3779B9u;      // eighth round: words 0 and 3
                        kr1 += 0xBB67AE85u;
                        c_3 = 0xD2511F53u * c_0;
                        c_0 = __builtin_amdgcn_bitop3_b32(__umulhi(0xCD9E8D57u, c_2), c_1, kr0, 0x96);
                        kr1 += 0xBB67AE85u;      // ninth: word 2
                        c_2 = __builtin_amdgcn_bitop3_b32(__umulhi(0xD2511F53u, c_0), c_3, kr1, 0x96);
                        const uint32_t r1 = 0xCD9E8D57u * c_2;     // tenth: word 1
                        const uint32_t w = wa.masks[kSectorWords * sp.sidx + (int)(r1 >> 29)];
                        take = ((w >> ((r1 >> 24) & 31u)) & 1u) != 0;
                    }
                    const uint64_t m = __ballot(take);
                    if (take) {
                        const int at = qn + lanes_below(m);
                        wa.qk[at] = (uint32_t)kj;
                        wa.qs[at] = (uint8_t)sj;
                    }
                    qn += __popcll(m);
                    c0 += kWave;
                }
                if (qn == 0) break;
                wave_lds_sync();
                active = lane < qn;
                k = (int32_t)wa.qk[lane];
                si = wa.qs[lane];
                if (qn > kWave && lane < qn - kWave) {
                    wa.qk[lane] = wa.qk[kWave + lane];
                    wa.qs[lane] = wa.qs[kWave + lane];
                }
                qn = qn > kWave ? qn - kWave : 0;
            }
            const uint32_t opaque = (uint32_t)((uint64_t)(uint32_t)c0 >> 31);   // 0, as above
            uint32_t kr0 = a.key0 + opaque, kr1 = a.key1 + opaque;

            bool alive = false;
            int drop_why = -1;
            // read only in lanes that emit a live bunch: any value elsewhere
            double xg = any_f64(), yg = any_f64(), he = any_f64();
            double uod = any_f64(), vod = any_f64();   // observed direction for the sphere test
            bool screen_all = false;   // screening: listed whatever its sphere tests say
            // fraction and height of the emission point in its cell
            double fcell = any_f64(), dcell = SEARCH ? any_f64() : 0.0;
            int ci = (int)any_u32();
            // what a crossing's record needs beyond the above; the record itself is
            // completed only in chunks that hold a crossing
            double t_rec = any_f64();   // mixed fast path: emission time - t_ref; else the arrival time
            double w_rec = any_f64();   // mixed fast path: w of the photon at emission
            T f_rec = any_of<T>();      // mixed fast path: fraction of the emission point in its cell
            bool fast_rec = false;
            uint32_t r2_rec = any_u32();   // the wavelength's draw
            if (active) {
                const Entry& e = stash[si];
                // Philox4x32-10 with counter (k, step index in shower, shower id, 0)
                uint32_t c_0 = (uint32_t)k, c_2 = shower_id, c_3 = 0u;
                uint32_t c_1 = e.ctr1;
#pragma unroll
                for (int rr = 0; rr < 10; ++rr) {
                    const uint64_t p0 = (uint64_t)0xD2511F53u * c_0;
                    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c_2;
                    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c_1, kr0, 0x96);
                    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c_3, kr1, 0x96);
                    c_1 = (uint32_t)p1;
                    c_3 = (uint32_t)p0;
                    c_0 = n0;
                    c_2 = n2;
                    kr0 += 0x9E3779B9u;
                    kr1 += 0xBB67AE85u;
                }
                const uint32_t r0 = c_0, r1 = c_1, r2 = c_2;
                // emission point, uniform inside sub-step k (FP64)
                const double u0 = fma((double)r0, 2.3283064365386963e-10, 1.1641532182693481e-10);
                const double s_along = ((double)k + u0) * e.ds;
                const double tu = e.u, tv = e.v, tw = e.w;
                double xe, ye, ze;
                {
                    // rounded as the FP64 definition rounds it: the drop tests and the
                    // profile bin take their decisions on this value (and, curved, on
                    // the altitude of (x, y, z))
#pragma clang fp contract(off)
                    he = e.h0 - s_along * tw;
                    if (CURVED) {
                        xe = e.x0 + s_along * tu;
                        ye = e.y0 + s_along * tv;
                    }
                }
                if (!CURVED) {
                    xe = fma(s_along, tu, e.x0);
                    ye = fma(s_along, tv, e.y0);
                }
                ze = he;
                if (CURVED) he = curved_altitude(a.earth_r, xe, ye, ze);
                const double te = fma(s_along, e.inv_bc, e.t0);
                // table cell and fraction of the emission altitude (index and depth)
                if (SEARCH) {
                    // node tables: branch-free binary search in LDS (sec. 3.3.1)
                    int lo = 0;
                    for (int stp = a.search_pow2; stp > 0; stp >>= 1) {
                        const int c = lo + stp;
                        if (c < a.n_nodes - 1 && hn_lds[c] <= he) lo = c;
                    }
                    ci = lo;
                    dcell = he - hn_lds[ci];
                    fcell = dcell * hn_lds[a.n_nodes + ci];
                } else {
                    const double xcell = (he - a.h_obs) * a.inv_step;
                    ci = min((int)xcell, a.n_nodes - 2);
                    fcell = xcell - (double)ci;
                }
                const double ct = e.cos_t;
                // direction on the Cherenkov cone
                double pu, pv, pw;
                if (PREC == 0) {
                    double sp, cp;
                    sincos_turns64(r1, sp, cp);
                    pu = ct * tu + (cp * (double)e.sb1x + sp * (double)e.sb2x);
                    pv = ct * tv + (cp * (double)e.sb1y + sp * (double)e.sb2y);
                    pw = ct * tw - (cp * (double)e.sb1z + sp * (double)e.sb2z);
                } else {
                    float sp, cp;
                    sincos_turns_hw(r1, sp, cp);
                    const float px = fmaf(cp, (float)e.sb1x, sp * (float)e.sb2x);
                    const float py = fmaf(cp, (float)e.sb1y, sp * (float)e.sb2y);
                    const float pz = fmaf(cp, (float)e.sb1z, sp * (float)e.sb2z);
                    pu = fma(ct, tu, (double)px);
                    pv = fma(ct, tv, (double)py);
                    pw = fma(ct, tw, -(double)pz);
                }
                r2_rec = r2;
                // drop rules, in this order: below the observation level, above the top,
                // upward, grazing (selects, no branches)
                const bool d_below = he < a.h_obs, d_above = he >= a.h_top;
                const bool d_up = !CURVED && pw <= 0.0, d_graze = !CURVED && pw <= w_graze;
                const bool kept = !d_below && !d_above && !d_up;
                drop_why = d_below ? CKV_DROP_BELOW_OBS
                           : d_above ? CKV_DROP_ABOVE_TOP
                           : d_up ? CKV_DROP_UPWARD
                           : (d_graze && !EXACT) ? CKV_DROP_GRAZING : -1;
                // slow: traced exactly, cell by cell (grazing bunches; every bunch when curved,
                // whose upward and turning drops the tracer decides)
                bool slow = kept && (CURVED || (EXACT && d_graze));
                if (SLOWPATH && slow) {
                    alive = true;
                    if (PREC == 1) {
                        // a grazing ray magnifies a direction error by 1/w^2 on the
                        // ground: redo the direction in FP64 (frame of the step, FP64
                        // azimuth), as the FP64 path has it
                        const double Dz = -tw, sgn = copysign(1.0, Dz);
                        const double ia = -1.0 / (sgn + Dz), ib = tu * tv * ia;
                        const double b1x = 1.0 + sgn * tu * tu * ia, b1y = sgn * ib, b1z = -sgn * tu;
                        const double b2x = ib, b2y = sgn + tv * tv * ia, b2z = -tv;
                        const double st_ = sqrt((1.0 - ct) * (1.0 + ct));
                        double sp, cp;
                        sincos_turns64(r1, sp, cp);
                        pu = ct * tu + st_ * (cp * b1x + sp * b2x);
                        pv = ct * tv + st_ * (cp * b1y + sp * b2y);
                        pw = ct * tw - st_ * (cp * b1z + sp * b2z);
                    }
                    double T_x = 0.0;
                    if (CURVED) {
                        const SlowRay r = propagate_curved_call((uint64_t)__builtin_amdgcn_kernarg_segment_ptr(), xe,
                                                                ye, ze, he, pu, pv, pw);
                        xg = r.xg; yg = r.yg; T_x = r.T; uod = r.uo; vod = r.vo;
                        if (r.status >= 0) {
                            drop_why = r.status;
                            alive = false;
                        }
                    } else {
                        const SlowRay r = propagate_exact_call((uint64_t)__builtin_amdgcn_kernarg_segment_ptr(), xe,
                                                               ye, he, pu, pv, pw);
                        xg = r.xg; yg = r.yg; T_x = r.T;
                        uod = pu * r.uo / a.n_obs;
                        vod = pv * r.uo / a.n_obs;
                    }
                    t_rec = (te - t_ref) + T_x;
                }
                if (drop_why < 0 && !slow) {
                    alive = true;
                    // ---- atmosphere at the emission altitude (uniform table, no search)
                    const T f = (T)fcell;
                    const CellMoments m = cell_moments(ci, f, dcell);
                    const IndexTerms ix = index_terms(m.psi_e, pw);
                    // horizontal advance: S = dh + sum_{k>=1} a_k q^k D_k
                    const double dh = he - a.h_obs;
                    const T s_corr = advance_series(m, ix.q);
                    const double S = dh + (double)s_corr;
                    const double adv = ix.inv_w * S;
                    if (SCREEN) {
                        // bound of this path's ground-point error (direction error of the
                        // FP32 cone vector through 1/w and u/w^2, FP32 series corrections
                        // through q ~ 1/w^2 and 1/w): where it passes half the screening
                        // margin the sphere test cannot be trusted and the bunch is listed
                        const double e_g = dh * ix.inv_w * (kScreenErrDir * (1.0 + ix.inv_w) +
                                                            kScreenErrSeries * ix.inv_w * ix.inv_w);
                        screen_all = e_g > 0.5 * kScreenMargin;
                    }
                    xg = fma(pu, adv, xe);
                    yg = fma(pv, adv, ye);
                    // the sphere test takes the observed direction at the path's
                    // precision (FP64 path: before the record's FP32 rounding)
                    const T uT = (T)pu * ix.ratio, vT = (T)pv * ix.ratio;
                    uod = (double)uT;
                    vod = (double)vT;
                    if constexpr (PREC == 0) {
                        // FP64: the arrival time at once (keeping the inputs of its
                        // recomputation live costs this build more than it saves)
                        t_rec = (te - t_ref) + travel_time(m, ix, s_corr, dh);
                    } else {
                        t_rec = te - t_ref;
                        w_rec = pw;
                        f_rec = f;
                        fast_rec = true;
                    }
                }
            }
            {
                const int d0 = __popcll(__ballot(drop_why == CKV_DROP_BELOW_OBS));
                const int d1 = __popcll(__ballot(drop_why == CKV_DROP_ABOVE_TOP));
                const int d2 = __popcll(__ballot(drop_why == CKV_DROP_UPWARD));
                const int d3 = __popcll(__ballot(drop_why == CKV_DROP_GRAZING));
                if (lane == 0 && (d0 | d1 | d2 | d3)) {
                    wcnt[kWcDrop0 + CKV_DROP_BELOW_OBS] += d0;
                    wcnt[kWcDrop0 + CKV_DROP_ABOVE_TOP] += d1;
                    wcnt[kWcDrop0 + CKV_DROP_UPWARD] += d2;
                    wcnt[kWcDrop0 + CKV_DROP_GRAZING] += d3;
                }
            }
            // ---- candidate spheres (ascending telescope index)
            int cur = 0, cend = 0;
            int first = -1;          // the cell's first sphere, known without a list read
            bool brute = false;
            if (alive) {
                const double wo2 = 1.0 - uod * uod - vod * vod;
                if (wo2 >= kLevelW2[0]) {
                    const double fx = (xg - a.gx0) * a.inv_cell, fy = (yg - a.gy0) * a.inv_cell;
                    if (fx >= 0.0 && fy >= 0.0 && fx < (double)a.nx && fy < (double)a.ny) {
                        const int cidx = grid_level(wo2) * a.level_cells + (int)fx * a.ny + (int)fy;
                        const uint2 ce = a.cell_ent[cidx];
                        cur = (int)ce.x;
                        cend = cur + (int)(ce.y & 0xFFFFu);
                        first = (int)(ce.y >> 16);
                    }
                } else {
                    brute = true;
                }
            }
            int my_next = INT_MAX;
            auto crosses = [&](int kt) {
                const double* tq = tel_sh + 3 * kt;     // sphere table in LDS
                const double tX = tq[0], tY = tq[1], tR2 = tq[2];
                const double dx = xg - tX, dy = yg - tY;
                const double b = dx * uod + dy * vod;
                const double disc = b * b - (dx * dx + dy * dy - tR2);
                return disc >= 0.0;
            };
            // a chunk with a flat ray (below the grid's lowest w) sweeps all spheres, 32 at a
            // time and the same in all lanes, into a bitmask per lane: lane by lane, each
            // record's search for the lane's next sphere ran alone in its wave (3000
            // near-horizontal steps, 400 spheres, two crossings a bunch: 38 ms, now 3.8)
            const bool sweep = __ballot(brute) != 0ull;
            uint32_t hits = 0;
            auto sweep_from = [&](int kb) {
                hits = 0;
                if (alive) {
                    const int nk = min(32, a.n_tel - kb);
#pragma unroll 2
                    for (int q = 0; q < nk; ++q) hits |= crosses(kb + q) ? 1u << q : 0u;
                }
                my_next = hits ? kb + __builtin_ctz(hits) : INT_MAX;
            };
            auto advance = [&](int kb) {
                my_next = INT_MAX;
                if (sweep) {
                    hits &= hits - 1;
                    if (hits) my_next = kb + __builtin_ctz(hits);
                    return;
                }
                while (cur < cend) {
                    const int kt = first >= 0 ? first : (int)a.cell_list[cur];
                    first = -1;
                    ++cur;
                    if (crosses(kt)) { my_next = kt; break; }
                }
            };
            if (!sweep) advance(0);
            if constexpr (SCREEN) {
                // candidates of the soft response: gathered in the wave's buffer, which goes
                // to the list when full (one atomic on the list's count for each 256 or so:
                // claims of all waves come 13 ns apart)
                const uint64_t step = (uint64_t)(a.shower_first[s] + (t0 - a.tiles_before[s]) * (int64_t)TS +
                                                 stash[active ? si : 0].sidx);
                bool cand = my_next != INT_MAX || screen_all;
                if (sweep)
                    for (int kb = 0; kb < a.n_tel; kb += 32) {
                        sweep_from(kb);
                        cand = cand || hits != 0u;
                    }
                if (cand && ((uint32_t)k >= (1u << kSoftIdBits) || step >= (1ull << (64 - kSoftIdBits)))) {
                    atomicOr((unsigned long long*)a.list_count, kSoftListInvalid);
                    cand = false;
                }
                const uint64_t m = __ballot(cand);
                if (buf_n + __popcll(m) > kScreenBuf) {
                    flush_list(a, buf, buf_n, lane);
                    buf_n = 0;
                }
                if (cand) buf[buf_n + lanes_below(m)] = (step << kSoftIdBits) | (uint64_t)(uint32_t)k;
                buf_n += __popcll(m);
            } else {
                // ---- the records of the crossing bunches.  About one chunk in five holds
                // a crossing, so the wavelength and the record's roundings are done here,
                // for those lanes; the mixed path also takes the arrival time's series
                // (the only user of D_5 and 1/n_e) here, recomputed from the table rather
                // than kept live through the sphere tests.
                float uo = any_of<float>(), vo = any_of<float>(), t_f = any_of<float>(), he_f = any_of<float>();
                float photons = any_of<float>(), lam = any_of<float>();
                int32_t sidx_rec = (int32_t)any_u32();
                if (sweep || __ballot(my_next != INT_MAX)) {
                    if (sweep ? alive : my_next != INT_MAX) {
                        const Entry& er = stash[si];
                        sidx_rec = er.sidx;
                        photons = (float)er.photons;
                        if (PREC == 0) {
                            lam = (float)rcp64(a.inv_l1 - fma((double)r2_rec, 2.3283064365386963e-10,
                                                              1.1641532182693481e-10) * a.dl);
                        } else {
                            const float u2 = fmaf((float)r2_rec, 2.3283064365386963e-10f,
                                                  1.16415321826934814e-10f);
                            lam = __builtin_amdgcn_rcpf(fmaf(-u2, (float)a.dl, (float)a.inv_l1));
                        }
                        double tarr = t_rec;
                        if constexpr (PREC == 1) {
                            if (fast_rec) {
                                const CellMoments m = cell_moments(ci, f_rec, dcell);
                                const IndexTerms ix = index_terms(m.psi_e, w_rec);
                                tarr += travel_time(m, ix, advance_series(m, ix.q), he - a.h_obs);
                            }
                        }
                        uo = (float)uod;
                        vo = (float)vod;
                        t_f = (float)tarr;
                        he_f = (float)he;
                    }
                }
                // ---- record crossings.  A turn takes lanes with one sphere each, all lanes of a
                // sphere in the same turn, in bunch order: every crossing lane when none has
                // another sphere to come, else those of the lowest sphere.
                for (int kb = 0; kb < (sweep ? a.n_tel : 1); kb += 32) {
                    if (sweep) sweep_from(kb);
                    for (;;) {
                        const uint64_t any = __ballot(my_next != INT_MAX);
                        if (!any) break;
                        bool more = sweep ? (hits & (hits - 1)) != 0u : false;
                        if (!sweep && my_next != INT_MAX && cur < cend) {
                            // the rest of the lane's list, up to its next sphere
                            int c = cur;
                            while (c < cend && !more) more = crosses((int)a.cell_list[c++]);
                            cur = more ? c - 1 : cend;
                        }
                        const bool last = __ballot(more && my_next != INT_MAX) == 0ull;
                        const bool mine = my_next == (last ? my_next : wave_min_sparse(my_next, INT_MAX)) &&
                                          my_next != INT_MAX;
                        const uint64_t mask = __ballot(mine);
                        const int nmine = __popcll(mask);
                        const int below = lanes_below(mask);
                        // rank among the turn's crossings of the same tile and sphere, then the
                        // crossings of earlier turns
                        const int key = mine ? (sidx_rec / TS - h) * a.n_tel + my_next : -1;
                        int rank = 0, of_key = 0;
                        for (uint64_t rest = mask; rest;) {
                            const int kk = __builtin_amdgcn_readlane(key, __builtin_ctzll(rest));
                            const uint64_t same = __ballot(key == kk);
                            if (key == kk) {
                                rank = lanes_below(same);
                                of_key = __popcll(same);
                            }
                            rest &= ~same;
                        }
                        if (mine) {
                            const int before = tcount[key];
                            if (rank == 0) tcount[key] = before + of_key;
                            rank += before;
                        }
                        // staging slots: the first `room` crossings fill the current
                        // block, the rest start a newly claimed one
                        const int room = blk >= 0 ? kStageBlock - blk_fill : 0;
                        int64_t nbk = -2;
                        if (nmine > room && blk != -2) {
                            if (blk >= 0 && lane == 0) a.stage_fill[blk] = kStageBlock;
                            if (lane == 0) nbk = (int64_t)atomicAdd((unsigned long long*)&a.ctrl[kBlockCounter], 1ull);
                            nbk = uniform(nbk);
                            if (nbk >= a.stage_blocks) nbk = -2;
                        }
                        if (nmine > room && nbk < 0) {
                            // crossings find no slot: the run's written prefix ends before the
                            // first one's tile (lanes are in tile order)
                            const uint64_t none = __ballot(mine && below >= room);
                            const int64_t tl = t0 + __builtin_amdgcn_readlane(sidx_rec, __builtin_ctzll(none)) / TS;
                            if (tl < lost) {
                                lost = tl;
                                if (lane == 0) atomicMin((unsigned long long*)&a.ctrl[kFirstLost], (unsigned long long)tl);
                            }
                        }
                        if (mine) {
                            int64_t slot = -1;
                            if (below < room) slot = blk * kStageBlock + blk_fill + below;
                            else if (nbk >= 0) slot = nbk * kStageBlock + (below - room);
                            if (slot >= 0) {
                                StageEntry* se = a.stage + slot;
                                const double* tp = tel_sh + 3 * my_next;
                                float4* ef = reinterpret_cast<float4*>(se);
                                ef[0] = make_float4((float)(xg - tp[0]), (float)(yg - tp[1]), uo, vo);
                                ef[1] = make_float4(t_f, he_f, photons, lam);
                                uint4* eu = reinterpret_cast<uint4*>(se);
                                eu[2] = make_uint4((uint32_t)(t0 + sidx_rec / TS),
                                                   (uint32_t)my_next | ((uint32_t)(sidx_rec & (TS - 1)) << 16),
                                                   (uint32_t)rank, (uint32_t)k);
                            }
                        }
                        if (nmine > room) {
                            if (blk != -2) {
                                blk = nbk;               // -2 when the staging area is full
                                blk_fill = nmine - room;
                            }
                        } else {
                            blk_fill += nmine;
                        }
                        if (mine) advance(kb);
                    }
                }
            }
        }
        // the next unit's claim, on its way during the rest (claimed any earlier, the launch
        // ends unevenly: shells at 70 degrees 398 -> 480 us)
        if (h_next == h_all && lane == 0)
            claimed = (int64_t)atomicAdd((unsigned long long*)&a.claims[kClaimStride * cls], 1ull);
        // ---- per-telescope crossings of each tile as runs (ascending telescope)
        wave_lds_sync();
        for (int hh = h; !SCREEN && hh < h_next; ++hh) {
            const int64_t t = t0 + hh;
            int32_t* const tc = tcount + (hh - h) * a.n_tel;
            int nz = 0;
            int64_t found = 0;
            for (int k0 = 0; k0 < a.n_tel; k0 += kWave) {
                const int kk = k0 + lane;
                const int32_t c = kk < a.n_tel ? tc[kk] : 0;
                nz += __popcll(__ballot(c != 0));
                found += c;
            }
            const int32_t thits = (int32_t)wave_last(wave_incl_scan(found));
            // run slots from the wave's current block of kRunBlock (a tile with more
            // runs than a block takes enough whole blocks of its own)
            int64_t base = 0;
            if (nz > 0) {
                if (rblk < 0 || rfill + nz > kRunBlock) {
                    const int nblk = (nz + kRunBlock - 1) / kRunBlock;
                    int64_t b = 0;
                    if (lane == 0) b = (int64_t)atomicAdd((unsigned long long*)&a.ctrl[kRunCounter],
                                                          (unsigned long long)nblk);
                    rblk = scalar64(uniform(b));
                    rfill = 0;
                }
                base = rblk * kRunBlock + rfill;
                rfill = nz > kRunBlock ? kRunBlock : rfill + nz;
            }
            const bool fits = base + nz <= a.run_cap;
            if (!fits && t < lost) {
                lost = t;
                if (lane == 0) atomicMin((unsigned long long*)&a.ctrl[kFirstLost], (unsigned long long)t);
            }
            int done = 0;
            for (int k0 = 0; k0 < a.n_tel; k0 += kWave) {
                const int kk = k0 + lane;
                const int32_t c = kk < a.n_tel ? tc[kk] : 0;
                const uint64_t m = __ballot(c != 0);
                if (c != 0) {
                    if (fits)
                        a.runs[base + done + lanes_below(m)] = ((int64_t)kk << kRunTelShift) | c;
                    tc[kk] = 0;
                }
                done += __popcll(m);
            }
            if (lane == 0) {
                a.tile_run_off[t] = base;
                a.tile_run_n[t] = fits ? nz : 0;
                a.tile_hits[t] = thits;
            }
            if (lane == 0) wcnt[kWcHits] += thits;
        }
        wave_lds_sync();
        }
        unit = cls + n_cls * (cls_waves + scalar64(claimed));
    }

    if (SCREEN) flush_list(a, buf, buf_n, lane);
    // ---- close the staging block and publish counters: the workgroup's waves are
    // summed in LDS and the first wave adds the sums, one atomic per counter and
    // workgroup (one per wave queued thousands of atomics on the counters' line at
    // the end of every launch)
    if (blk >= 0 && lane == 0) a.stage_fill[blk] = blk_fill;
    __syncthreads();
    if (PROF) {
        // the waves' bins, summed over waves that end on the same shower
        const int nw = (int)(blockDim.x / kWave);
        for (int kk = threadIdx.x; kk < prof_bins; kk += blockDim.x) {
            double ph = 0.0;
            unsigned long long bu = 0;
            for (int w = 0; w < nw; ++w) {
                const WaveArea<PREC, TS> ww(lds + srch_bytes + tel_bytes(a.n_tel) + (size_t)w * wv_stride, n_count,
                                            prof_bins);
                ph += ww.hph[kk];
                bu += ww.hbu[kk];
                const int64_t s = ww.prof[0];
                bool last = w + 1 == nw;
                if (!last) {
                    const WaveArea<PREC, TS> wn(lds + srch_bytes + tel_bytes(a.n_tel) + (size_t)(w + 1) * wv_stride,
                                                n_count, prof_bins);
                    last = wn.prof[0] != s;
                }
                if (last) {
                    if (bu) {
                        atomicAdd(&a.prof_ph[s * prof_bins + kk], ph);
                        atomicAdd((unsigned long long*)&a.prof_bu[s * prof_bins + kk], bu);
                    }
                    ph = 0.0;
                    bu = 0;
                }
            }
        }
    }
    if (wave == 0 && lane < kWcCount) {
        const unsigned char* w0 = reinterpret_cast<const unsigned char*>(wcnt);
        int64_t v = 0;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w)
            v += reinterpret_cast<const int64_t*>(w0 + (size_t)w * wv_stride)[lane];
        const int slot = lane == kWcBunches ? kBunches
                       : lane == kWcEmitting ? kEmitting
                       : lane == kWcHits ? kHits
                       : kDrop0 + (lane - kWcDrop0);
        if (v) atomicAdd((unsigned long long*)&a.ctrl[slot], (unsigned long long)v);
    }
}

// The builds whose lanes leave the moment series (kFeatExact, kFeatCurved) are
// compiled by ckv_slowpath.hip, all others here.  Here the compiler must not keep
// loop-invariant values, mostly FP64 constants, in registers around the loops (the
// flag is with the file's name in build.py): at 128 registers (16 waves) they push
// tile state into scratch, and the soft kernels lose waves to them.  Kept against
// not kept: 2e6 TeV steps FP64 330 -> 288 us, mixed 298 -> 289 us; candidates of a
// 1.6e6-step fit 165 -> 123 us (220 -> 126 registers, two -> four waves per SIMD).
// The serial FP64 chains of the slow paths, 8 waves with registers to spare, are
// better with them in registers: curved 378 against 386 us, grazing 894 against 908.
#define CKV_SLOWPATH_TS(M, PREC, TS)                                               \
    M template __global__ void emit_kernel<PREC, TS, kFeatExact>(Args);            \
    M template __global__ void emit_kernel<PREC, TS, kFeatProfile | kFeatExact>(Args);
#define CKV_SLOWPATH_PREC(M, PREC)                                                 \
    M template __global__ void emit_kernel<PREC, 2, kFeatExact>(Args);             \
    M template __global__ void emit_kernel<PREC, 32, kFeatCurved>(Args);           \
    CKV_SLOWPATH_TS(M, PREC, 8)                                                    \
    CKV_SLOWPATH_TS(M, PREC, 16)                                                   \
    CKV_SLOWPATH_TS(M, PREC, 32)                                                   \
    CKV_SLOWPATH_TS(M, PREC, 64)

#ifdef CKV_SLOWPATH
CKV_SLOWPATH_PREC(, 0)
CKV_SLOWPATH_PREC(, 1)
#else
CKV_SLOWPATH_PREC(extern, 0)
CKV_SLOWPATH_PREC(extern, 1)

// --------------------------------------------------------------------------
// init: control block, shower validation, tile and row-block counts
// --------------------------------------------------------------------------
// Tiles of the report's size with 2^30 bunches or more are refused whole, also where the run
// works in smaller ones.  One of a refused tile's steps has 2^25 or more, so a workgroup
// looks at the lengths of its steps and of their neighbours; only where one is that long are
// the tiles counted.  Called by a whole workgroup of kHeavySteps threads (the wave that works
// on a tile would have to wait for its neighbours' lengths; here it takes no time beside the
// first workgroup's).
__device__ __forceinline__ void mark_heavy(const Args& a, int64_t block)
{
    constexpr int kTile = 32;
    const int64_t i = block * kHeavySteps + threadIdx.x;
    // (a count is at most k_ft L / bunch_size + 1)
    const double most = ((double)(1 << 25) - 2.0) * a.bunch_size;
    auto may = [&](int64_t j) {
        const double N = j >= 0 && j < a.n ? a.k_ft * a.len[j] : 0.0;
        return N >= most && isfinite(N) ? 1 : 0;
    };
    int any = may(i);
    if (threadIdx.x < kTile) any |= may(i - kTile) | may(i + kHeavySteps);
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) a.heavy[block] = any;
    if (!any || i >= a.n) return;
    int s = 0;
    for (int hi = a.n_showers; hi - s > 1;) {
        const int mid = (s + hi) >> 1;
        if (a.seg_offsets[mid] <= i) s = mid; else hi = mid;
    }
    // the step's tile (kept inside the arrays: the offsets are not validated yet)
    int64_t first = max(a.seg_offsets[s], (int64_t)0), end = min(a.seg_offsets[s + 1], a.n);
    if (s == a.cur_shower) first = max(first, a.cur_step);
    int64_t nb = 0;
    if (i >= first && i < end) {
        first += (i - first) / kTile * kTile;
        for (int64_t j = first; j < min(first + kTile, end); ++j) {
            Setup st;
            step_setup(a, j, st);
            if (st.status < 0) nb += st.nb;
        }
    }
    a.heavy_step[i] = nb >= ((int64_t)1 << 30) ? 1 : 0;
}

__global__ void __launch_bounds__(1024) init_kernel(Args a)
{
    if (blockIdx.x > 0) {
        mark_heavy(a, (int64_t)blockIdx.x - 1);
        return;
    }
    __shared__ int64_t sh_t[1024], sh_b[1024];
    __shared__ unsigned long long report;
    __shared__ int err;
    for (int q = threadIdx.x; q < kCtrlSlots; q += blockDim.x) a.ctrl[q] = 0;
    if (a.claims)
        for (int q = threadIdx.x; q < kTileClasses; q += blockDim.x) a.claims[kClaimStride * q] = 0;
    if (threadIdx.x == 0) { err = 0; report = 0; }
    __syncthreads();
    const int64_t TS = a.tile_segs;
    int64_t run_t = 0, run_b = 0;
    for (int base = 0; base < a.n_showers; base += blockDim.x) {
        const int s = base + threadIdx.x;
        int64_t nt = 0, nbk = 0;
        if (s < a.n_showers) {
            const int64_t lo = a.seg_offsets[s], hi = a.seg_offsets[s + 1];
            if (lo < 0 || hi < lo || hi > a.n || (s == 0 && lo != 0) ||
                (s == a.n_showers - 1 && hi != a.n))
                err = 1;
            // the run starts at the cursor: showers before its shower have no tiles,
            // its shower starts at the cursor's step
            int64_t first = lo;
            if (s < a.cur_shower) {
                first = hi;
            } else if (s == a.cur_shower) {
                if (a.cur_step < lo || a.cur_step > hi) err = 1;
                first = a.cur_step < lo ? lo : (a.cur_step > hi ? hi : a.cur_step);
            }
            if (a.shower_first) a.shower_first[s] = first;
            const int64_t cnt = hi >= first ? hi - first : 0;
            nt = (cnt + TS - 1) / TS;
            nbk = (nt + kRowBlock - 1) / kRowBlock;
            if (TS != a.report_segs)
                atomicAdd(&report, (unsigned long long)((cnt + a.report_segs - 1) / a.report_segs));
        }
        sh_t[threadIdx.x] = nt;
        sh_b[threadIdx.x] = nbk;
        __syncthreads();
        for (int d = 1; d < (int)blockDim.x; d <<= 1) {
            int64_t xt = 0, xb = 0;
            if ((int)threadIdx.x >= d) { xt = sh_t[threadIdx.x - d]; xb = sh_b[threadIdx.x - d]; }
            __syncthreads();
            sh_t[threadIdx.x] += xt;
            sh_b[threadIdx.x] += xb;
            __syncthreads();
        }
        if (s < a.n_showers) {
            a.tiles_before[s] = run_t + sh_t[threadIdx.x] - nt;
            a.blocks_before[s] = run_b + sh_b[threadIdx.x] - nbk;
        }
        run_t += sh_t[blockDim.x - 1];
        run_b += sh_b[blockDim.x - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.tiles_before[a.n_showers] = run_t;
        a.blocks_before[a.n_showers] = run_b;
        if (run_t > a.max_tiles || run_b > a.max_row_blocks) err = 1;
        a.ctrl[kNumTiles] = err ? 0 : run_t;
        a.ctrl[kNumRowBlocks] = err ? 0 : run_b;
        a.ctrl[kReportTiles] = err ? 0 : TS != a.report_segs ? (int64_t)report : run_t;
        a.ctrl[kFirstLost] = err ? 0 : run_t;      // no lost tile yet
        int64_t dealt = 0;
        if (!err && a.static_blocks > 0) {
            dealt = min(units_of(run_t, a.head_units, a.grid_waves, a.tile_segs).count, (int64_t)a.static_blocks);
        }
        a.ctrl[kBlockCounter] = dealt;
        a.ctrl[kRunCounter] = dealt;
        if (a.result) {
            // the bunch path's finalize fills the rest; the soft entry points report
            // the error word only
            ckv_result* r = a.result;
            r->n_bunches = r->n_hits = r->n_records = r->n_emitting = r->n_tiles = 0;
            for (int d = 0; d < CKV_N_DROP; ++d) r->drops[d] = 0;
            r->resume_step = a.n;
            r->resume_shower = a.n_showers;
            r->overflow = 0;
            r->error = err;
            r->reserved = 0;
        }
    }
}

// --------------------------------------------------------------------------
// finalize
// --------------------------------------------------------------------------
__device__ __forceinline__ int find_shower(const int64_t* before, int n_showers, int64_t x)
{
    int lo = 0, hi = n_showers;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (before[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Row block b of shower s holds the shower's tiles [t0, t1) below; blocks and tiles
// are both numbered shower by shower, so block order is tile order.
__device__ __forceinline__ void block_tiles(const Args& a, int64_t b, int& s, int64_t& t0, int64_t& t1)
{
    s = find_shower(a.blocks_before, a.n_showers, b);
    t0 = a.tiles_before[s] + (b - a.blocks_before[s]) * kRowBlock;
    t1 = min(t0 + (int64_t)kRowBlock, a.tiles_before[s + 1]);
}

// Tile of the j-th run (0 <= q < the lanes' total) among lanes 0..m-1 holding
// inclusive run counts `incl` (one tile per lane): the first lane whose count
// passes q.  m is a power of two, the same in every lane.
__device__ __forceinline__ int run_tile(int64_t incl, int64_t q, int m)
{
    int lo = 0;
    for (int step = m >> 1; step > 0; step >>= 1)
        if (__shfl(incl, lo + step - 1) <= q) lo += step;
    return lo;
}

// A: per row block, one workgroup: each run's count becomes the crossings of its telescope
// in the block's earlier tiles, and the block's crossings per telescope (block_sums,
// telescope-major: block_sums[k * max_row_blocks + b]) and in all (block_hits) are kept.
// The block's runs go into a dense tiles x telescopes count matrix in LDS, each
// telescope's column is scanned, and each run takes its entry: nothing is serial over the
// block's tiles but one register sum per column, and the runs are read once (sums and
// prefixes in kernels of their own: 17.6 us on the TeV shower, now 11).
constexpr int kPrefixDenseTel = 512;           // 128 KB of LDS

__global__ void __launch_bounds__(1024) block_prefix_dense_kernel(Args a)
{
    extern __shared__ int32_t mat[];               // kRowBlock x n_tel, row = tile
    __shared__ int64_t s_incl[kRowBlock], s_off[kRowBlock];
    const int tid = threadIdx.x, nt = a.n_tel;
    const int64_t nblk = a.ctrl[kNumRowBlocks];
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        int s;
        int64_t t0, t1;
        block_tiles(a, b, s, t0, t1);
        const int ntl = (int)(t1 - t0);
        if (tid < kWave) {
            // lane l: tile t0 + l; inclusive run counts over the block's tiles
            const bool mine = tid < ntl;
            const int n = mine ? a.tile_run_n[t0 + tid] : 0;
            s_off[tid] = mine ? a.tile_run_off[t0 + tid] : 0;
            const int64_t hits = mine ? (int64_t)a.tile_hits[t0 + tid] : 0;
            s_incl[tid] = wave_incl_scan((int64_t)n);
            const int64_t sum = wave_last(wave_incl_scan(hits));
            if (tid == 0) a.block_hits[b] = sum;
        }
        for (int q = tid; q < ntl * nt; q += blockDim.x) mat[q] = 0;
        __syncthreads();
        const int64_t total = s_incl[kRowBlock - 1];
        // the block's runs in flat order: run q's tile is the first whose inclusive
        // count passes q
        auto run_at = [&](int64_t q, int& j) {
            j = 0;
            for (int step = kRowBlock / 2; step > 0; step >>= 1)
                if (s_incl[j + step - 1] <= q) j += step;
            return s_off[j] + (q - (j ? s_incl[j - 1] : 0));
        };
        for (int64_t q = tid; q < total; q += blockDim.x) {
            int j;
            const int64_t r = a.runs[run_at(q, j)];
            mat[j * nt + (int)(r >> kRunTelShift)] = (int32_t)(r & kRunValueMask);
        }
        __syncthreads();
        // exclusive scan down each telescope's column
        for (int k = tid; k < nt; k += blockDim.x) {
            int32_t acc = 0;
            for (int j = 0; j < ntl; ++j) {
                const int32_t v = mat[j * nt + k];
                mat[j * nt + k] = acc;
                acc += v;
            }
            a.block_sums[(int64_t)k * a.max_row_blocks + b] = acc;
        }
        __syncthreads();
        for (int64_t q = tid; q < total; q += blockDim.x) {
            int j;
            const int64_t g = run_at(q, j);
            const int tel = (int)(a.runs[g] >> kRunTelShift);
            a.runs[g] = ((int64_t)tel << kRunTelShift) | mat[j * nt + tel];
        }
        __syncthreads();
    }
}

// The same for more telescopes: per row block, one wave.  The block's runs are gathered
// into LDS when they fit (one load round per tile list), walked tile by tile there, and
// written back.
constexpr int kPrefixLdsRuns = 4096;

__global__ void __launch_bounds__(64) block_prefix_kernel(Args a)
{
    extern __shared__ int32_t ctr[];               // n_tel counters, then the run buffer
    int64_t* buf = reinterpret_cast<int64_t*>(ctr + ((a.n_tel + 1) & ~1));
    const int lane = lane_id();
    const int64_t nblk = a.ctrl[kNumRowBlocks];
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        int s;
        int64_t t0, t1;
        block_tiles(a, b, s, t0, t1);
        for (int k = lane; k < a.n_tel; k += kWave) ctr[k] = 0;
        // lane l: tile t0 + l (a block has at most 64 tiles)
        const int64_t tl = t0 + lane;
        const int n = tl < t1 ? a.tile_run_n[tl] : 0;
        const int64_t off = tl < t1 ? a.tile_run_off[tl] : 0;
        const int64_t hits = wave_last(wave_incl_scan(tl < t1 ? (int64_t)a.tile_hits[tl] : 0));
        if (lane == 0) a.block_hits[b] = hits;
        const int64_t incl = wave_incl_scan((int64_t)n);
        const int64_t total = wave_last(incl);
        const int my0 = (int)(incl - n);
        const bool in_lds = total <= kPrefixLdsRuns;
        // the block's runs into LDS in flat order, a run per lane (the loads of
        // different tiles are not chained)
        if (in_lds)
            for (int64_t q0 = 0; q0 < total; q0 += kWave) {
                const int64_t q = q0 + lane;
                const int j = run_tile(incl, q, kWave);
                const int64_t off_j = __shfl(off, j), first_j = __shfl(incl, j) - __shfl((int64_t)n, j);
                if (q < total) buf[q] = a.runs[off_j + (q - first_j)];
            }
        wave_lds_sync();
        for (int64_t t = t0; t < t1; ++t) {
            // the tile's count, offset and first slot from its lane (a uniform lane
            // index: a register read, not an LDS round trip)
            const int j = (int)(t - t0);
            const int nj = __builtin_amdgcn_readlane(n, j);
            const int64_t offj = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(off >> 32), j) << 32) |
                                           (uint32_t)__builtin_amdgcn_readlane((int)off, j));
            const int bj = __builtin_amdgcn_readlane(my0, j);
            for (int i = lane; i < nj; i += kWave) {
                const int64_t r = in_lds ? buf[bj + i] : a.runs[offj + i];
                const int tel = (int)(r >> kRunTelShift);
                const int32_t v = ctr[tel];
                const int64_t w = ((int64_t)tel << kRunTelShift) | v;
                if (in_lds) buf[bj + i] = w; else a.runs[offj + i] = w;
                ctr[tel] = v + (int32_t)(r & kRunValueMask);
            }
            wave_lds_sync();
        }
        if (in_lds)
            for (int64_t q0 = 0; q0 < total; q0 += kWave) {
                const int64_t q = q0 + lane;
                const int j = run_tile(incl, q, kWave);
                const int64_t off_j = __shfl(off, j), first_j = __shfl(incl, j) - __shfl((int64_t)n, j);
                if (q < total) a.runs[off_j + (q - first_j)] = buf[q];
            }
        for (int k = lane; k < a.n_tel; k += kWave) a.block_sums[(int64_t)k * a.max_row_blocks + b] = ctr[k];
        wave_lds_sync();
    }
}

// B: the written prefix.  Without a lost tile and with every crossing within the
// capacity it is the whole run.  Otherwise it ends at the first tile that is
// lost or whose crossings would pass the capacity; the row block holding that
// tile gets its sums again over the tiles before it (acc: n_tel counters in LDS).
// Called by a whole workgroup of 1024 threads.
__device__ __forceinline__ void find_cutoff(const Args& a, int32_t* acc)
{
    __shared__ int64_t part[1024];
    __shared__ int first_thread;
    __shared__ int64_t cut_tile, cut_block, cut_records, blk_b, blk_before;
    const int64_t n_tiles = a.ctrl[kNumTiles], nblk = a.ctrl[kNumRowBlocks];
    const int64_t lost = a.ctrl[kFirstLost];
    const int64_t hits = a.ctrl[kHits];
    if (lost >= n_tiles && hits <= a.capacity) {
        if (threadIdx.x == 0) {
            a.ctrl[kCutTile] = n_tiles;
            a.ctrl[kCutBlocks] = nblk;
            a.ctrl[kRecords] = hits;
        }
        return;
    }
    // the row block holding the lost tile bounds the search
    int64_t b_lim = nblk;
    if (lost < n_tiles) {
        const int sl = find_shower(a.tiles_before, a.n_showers, lost);
        b_lim = a.blocks_before[sl] + (lost - a.tiles_before[sl]) / kRowBlock + 1;
    }
    // first block whose crossings, added to those before it, pass the capacity
    const int nt = blockDim.x;
    const int64_t chunk = (b_lim + nt - 1) / nt;
    const int64_t lo = (int64_t)threadIdx.x * chunk, hi = min(lo + chunk, b_lim);
    int64_t mine = 0;
    for (int64_t b = lo; b < hi; ++b) mine += a.block_hits[b];
    part[threadIdx.x] = mine;
    if (threadIdx.x == 0) first_thread = nt;
    __syncthreads();
    for (int d = 1; d < nt; d <<= 1) {
        const int64_t y = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += y;
        __syncthreads();
    }
    const int64_t before = part[threadIdx.x] - mine;
    if (lo < hi && part[threadIdx.x] > a.capacity) atomicMin(&first_thread, (int)threadIdx.x);
    __syncthreads();
    if ((int)threadIdx.x == (first_thread < nt ? first_thread : nt - 1)) {
        // walk this thread's blocks to the first that passes (the lost tile's block
        // when none does)
        int64_t cum = first_thread < nt ? before : part[nt - 1] - a.block_hits[b_lim - 1];
        int64_t b = first_thread < nt ? lo : b_lim - 1;
        if (first_thread < nt)
            while (b + 1 < hi && cum + a.block_hits[b] <= a.capacity) cum += a.block_hits[b++];
        blk_b = b;
        blk_before = cum;
    }
    __syncthreads();
    // the tile: first of block blk_b that is lost or passes the capacity
    if (threadIdx.x == 0) {
        int s;
        int64_t t0, t1;
        block_tiles(a, blk_b, s, t0, t1);
        int64_t cum = blk_before, t = t0;
        while (t < t1 && t < lost && cum + a.tile_hits[t] <= a.capacity) cum += a.tile_hits[t++];
        // (a cut inside a tile of the report's size goes back to its start)
        if (t < t1)
            for (int64_t back = (t - a.tiles_before[s]) % (a.report_segs / a.tile_segs); back > 0; --back)
                cum -= a.tile_hits[--t];
        cut_tile = t;
        cut_block = t > t0 ? blk_b + 1 : blk_b;
        cut_records = cum;
    }
    __syncthreads();
    // sums of the boundary block over its tiles before the cut
    const int64_t b = blk_b;
    int s;
    int64_t t0, t1;
    block_tiles(a, b, s, t0, t1);
    for (int k = threadIdx.x; k < a.n_tel; k += blockDim.x)
        acc[k] = a.block_sums[(int64_t)k * a.max_row_blocks + b];
    __syncthreads();
    // a telescope's first run at or past the cut holds its crossings before the cut
    for (int64_t t = max(t0, cut_tile) + threadIdx.x; t < t1; t += blockDim.x) {
        const int64_t off = a.tile_run_off[t];
        for (int i = 0; i < a.tile_run_n[t]; ++i) {
            const int64_t r = a.runs[off + i];
            atomicMin(&acc[(int)(r >> kRunTelShift)], (int32_t)(r & kRunValueMask));
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < a.n_tel; k += blockDim.x)
        a.block_sums[(int64_t)k * a.max_row_blocks + b] = acc[k];
    if (threadIdx.x == 0) {
        a.ctrl[kCutTile] = cut_tile;
        a.ctrl[kCutBlocks] = cut_block;
        a.ctrl[kRecords] = cut_records;
    }
}

__global__ void __launch_bounds__(1024) cutoff_kernel(Args a)
{
    extern __shared__ int32_t acc[];
    find_cutoff(a, acc);
}

// C: per (shower, telescope), one wave: exclusive scan over the shower's row
// blocks below the cut, 8 x 64 blocks per round
__device__ __forceinline__ void scan_row_blocks(const Args& a, int64_t wave0, int64_t waves)
{
    const int lane = lane_id();
    const int64_t nst = (int64_t)a.n_showers * a.n_tel;
    const bool have_tiles = a.ctrl[kNumTiles] > 0;
    const int64_t cutb = a.ctrl[kCutBlocks];
    for (int64_t q = wave0; q < nst; q += waves) {
        const int s = (int)(q / a.n_tel), k = (int)(q % a.n_tel);
        int64_t run = 0;
        if (have_tiles) {
            int32_t* col = a.block_sums + (int64_t)k * a.max_row_blocks;
            const int64_t b_end = min(a.blocks_before[s + 1], cutb);
            // the loads issue before the first store and one wave scan of the lane
            // sums serves all
            constexpr int G = 8;
            for (int64_t b0 = a.blocks_before[s]; b0 < b_end; b0 += G * kWave) {
                const int64_t bl = b0 + (int64_t)G * lane;
                int32_t x[G];
                int64_t lsum = 0;
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    x[j] = bl + j < b_end ? col[bl + j] : 0;
                    lsum += x[j];
                }
                const int64_t incl = wave_incl_scan(lsum);
                int64_t pre = run + incl - lsum;
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    if (bl + j < b_end) col[bl + j] = (int32_t)pre;
                    pre += x[j];
                }
                run += wave_last(incl);
            }
        }
        if (lane == 0) a.shower_tel[q] = (int32_t)run;
    }
}

__global__ void __launch_bounds__(256) rowblock_scan_kernel(Args a)
{
    const int64_t per = blockDim.x / kWave;
    scan_row_blocks(a, blockIdx.x * per + threadIdx.x / kWave, (int64_t)gridDim.x * per);
}

// D: CSR offsets over (shower, telescope) and the run report.  Each thread takes up to
// kCsrPer consecutive entries, so 256 showers x 100 telescopes are four rounds of one
// scan.  Called by a whole workgroup of 1024 threads.
constexpr int kCsrPer = 8;

__device__ __forceinline__ void write_offsets(const Args& a)
{
    __shared__ int64_t sums[1024 / kWave];
    const int lane = lane_id(), wave = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const int64_t nst = (int64_t)a.n_showers * a.n_tel;
    int64_t run = 0;
    for (int64_t base = 0; base < nst; base += (int64_t)blockDim.x * kCsrPer) {
        const int64_t q0 = base + (int64_t)threadIdx.x * kCsrPer;
        int64_t x[kCsrPer], mine = 0;
#pragma unroll
        for (int i = 0; i < kCsrPer; ++i) {
            x[i] = q0 + i < nst ? (int64_t)a.shower_tel[q0 + i] : 0;
            mine += x[i];
        }
        const int64_t incl = wave_incl_scan(mine);
        if (lane == kWave - 1) sums[wave] = incl;
        __syncthreads();
        int64_t at = run + incl - mine, all = 0;
        for (int w = 0; w < nw; ++w) {
            if (w < wave) at += sums[w];
            all += sums[w];
        }
#pragma unroll
        for (int i = 0; i < kCsrPer; ++i) {
            if (q0 + i < nst) a.tel_offsets[q0 + i] = at;
            at += x[i];
        }
        run += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.tel_offsets[nst] = run;
        ckv_result* r = a.result;
        const int64_t n_tiles = a.ctrl[kNumTiles], cut = a.ctrl[kCutTile];
        r->n_bunches = a.ctrl[kBunches];
        r->n_hits = a.ctrl[kHits];
        r->n_records = a.ctrl[kRecords];
        r->n_emitting = a.ctrl[kEmitting];
        r->n_tiles = a.ctrl[kReportTiles];
        for (int d = 0; d < CKV_N_DROP; ++d) r->drops[d] = a.ctrl[kDrop0 + d];
        if (cut < n_tiles) {
            const int sc = find_shower(a.tiles_before, a.n_showers, cut);
            r->resume_shower = sc;
            r->resume_step = a.shower_first[sc] + (cut - a.tiles_before[sc]) * (int64_t)a.tile_segs;
            r->overflow = 1;
        } else {
            r->resume_shower = a.n_showers;
            r->resume_step = a.n;
            r->overflow = 0;
        }
    }
}

__global__ void __launch_bounds__(1024) csr_kernel(Args a) { write_offsets(a); }

// Cutoff, row-block scan and offsets in one workgroup, for at most kFinishPairs (shower,
// telescope) pairs (8 columns a wave) and kFinishBlocks row blocks (130 000 steps): 6.7 us
// instead of three launches of 4.7 and their gaps.  With 977 row blocks and 100 spheres
// its columns take 82 us against 17 in three kernels.
constexpr int kFinishPairs = 128;
constexpr int kFinishBlocks = 64;

__global__ void __launch_bounds__(1024) finish_kernel(Args a)
{
    extern __shared__ int32_t acc[];               // n_tel
    find_cutoff(a, acc);
    __threadfence_block();
    __syncthreads();
    scan_row_blocks(a, threadIdx.x / kWave, blockDim.x / kWave);
    __threadfence_block();
    __syncthreads();
    write_offsets(a);
}

// E: scatter the staged records of the written tiles to their final slots.  A
// slot's place is its (shower, telescope) offset, plus its telescope's crossings
// in earlier row blocks of the shower and in earlier tiles of its block (its run's
// value), plus its rank in the tile.
// Each thread takes kScatterSlots slots a round and issues the loads that do not
// depend on one another together: the block fills, then the entries (record and
// placement at once), then the tile's run list, the shower's offset and the
// shower (tile bounds staged in LDS for up to kScatterShowerLds showers), then the
// searches over the runs side by side.
constexpr int kScatterSlots = 2;
constexpr int kScatterShowerLds = 2048;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // plain 16-byte vector

struct ScatterSlot {
    u32x4 rec0, rec1, meta;
    int64_t off, base;
    int n, tel, shower, lo, len;
    bool live;
};

__device__ __forceinline__ void scatter_fill(const Args& a, ScatterSlot& x, int64_t q, int64_t nslots)
{
    const int64_t b = q < nslots ? q / kStageBlock : 0;
    x.live = q < nslots && (int)(q - b * kStageBlock) < a.stage_fill[b];
}

// (a slot that is not live reads slot 0, which every such slot shares)
__device__ __forceinline__ void scatter_entry(const Args& a, ScatterSlot& x, int64_t q)
{
    const u32x4* e = reinterpret_cast<const u32x4*>(a.stage + (x.live ? q : 0));
    x.rec0 = e[0];
    x.rec1 = e[1];
    x.meta = e[2];
}

__device__ __forceinline__ void scatter_tile(const Args& a, ScatterSlot& x, const int64_t* before, int64_t cut)
{
    const int64_t tile = x.meta.x;
    x.tel = (int)(x.meta.y & 0xFFFFu);
    x.live = x.live && tile < cut && x.tel < a.n_tel;
    x.n = 0;
    x.lo = 0;
    if (x.live) {
        x.shower = find_shower(before, a.n_showers, tile);
        x.off = a.tile_run_off[tile];
        x.n = a.tile_run_n[tile];
        const int64_t b = a.blocks_before[x.shower] + (tile - before[x.shower]) / kRowBlock;
        x.base = a.tel_offsets[(int64_t)x.shower * a.n_tel + x.tel] +
                 a.block_sums[(int64_t)x.tel * a.max_row_blocks + b];
    }
    x.len = x.n;
}

// one halving step of the search for the tile's run of the slot's telescope (runs
// ascend by telescope)
__device__ __forceinline__ void scatter_halve(const Args& a, ScatterSlot& x)
{
    if (x.len > 1) {
        const int half = x.len >> 1;
        if ((int)(a.runs[x.off + x.lo + half] >> kRunTelShift) <= x.tel) x.lo += half;
        x.len -= half;
    }
}

__device__ __forceinline__ void scatter_store(const Args& a, const ScatterSlot& x, const int64_t* before)
{
    if (!x.live || x.n <= 0) return;
    const int64_t r = a.runs[x.off + x.lo];
    if ((int)(r >> kRunTelShift) != x.tel) return;
    const int64_t pos = x.base + (r & kRunValueMask) + x.meta.z;
    if (pos < 0 || pos >= a.capacity) return;
    u32x4* dst = reinterpret_cast<u32x4*>(a.records + 8 * pos);
    dst[0] = x.rec0;
    dst[1] = x.rec1;
    if (a.ids) {
        const int s = x.shower;
        a.ids[2 * pos] = a.shower_first[s] + ((int64_t)x.meta.x - before[s]) * (int64_t)a.tile_segs +
                         (int)(x.meta.y >> 16);
        a.ids[2 * pos + 1] = x.meta.w;
    }
}

__device__ __forceinline__ void scatter_pair(const Args& a, const int64_t* before, int64_t q0,
                                             int64_t stride, int64_t nslots, int64_t cut)
{
    ScatterSlot x, y;
    const int64_t q1 = q0 + stride;
    scatter_fill(a, x, q0, nslots);
    scatter_fill(a, y, q1, nslots);
    scatter_entry(a, x, q0);
    scatter_entry(a, y, q1);
    scatter_tile(a, x, before, cut);
    scatter_tile(a, y, before, cut);
    while (x.len > 1 || y.len > 1) {
        scatter_halve(a, x);
        scatter_halve(a, y);
    }
    scatter_store(a, x, before);
    scatter_store(a, y, before);
}

__global__ void __launch_bounds__(256) scatter_kernel(Args a)
{
    __shared__ int64_t s_before[kScatterShowerLds + 1];
    const bool lds_showers = a.n_showers <= kScatterShowerLds;
    if (lds_showers)
        for (int q = threadIdx.x; q <= a.n_showers; q += blockDim.x) s_before[q] = a.tiles_before[q];
    __syncthreads();
    const int64_t cut = a.ctrl[kCutTile];
    const int64_t nblk = min(a.ctrl[kBlockCounter], a.stage_blocks);
    const int64_t nslots = nblk * kStageBlock;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q0 < nslots; q0 += kScatterSlots * stride) {
        if (lds_showers) scatter_pair(a, s_before, q0, stride, nslots, cut);
        else scatter_pair(a, a.tiles_before, q0, stride, nslots, cut);
    }
}

// standalone bunch count per step (FP64, same operations as the bunch kernel)
__global__ void __launch_bounds__(256) count_kernel(Args a, int64_t* n_b)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.n;
         i += (int64_t)gridDim.x * blockDim.x) {
        Setup st;
        step_setup(a, i, st);
        n_b[i] = st.status >= 0 ? 0 : st.nb;
    }
}

// --------------------------------------------------------------------------
// Soft telescope response and its adjoint (differentiation pattern), FP64.
//   S_sk = sum photons * Phi(z),  A_sk = sum photons * Phi(z) * t,
//   z = (R^2 - rho^2) / (2 R sigma),
// with bunch counts frozen per step.  MODE 0 accumulates S and A; MODE 1
// recomputes every bunch from its random numbers and accumulates dL/dpsi_i and
// dL/dP_j(h_i) given dL/dS and dL/dA.
// --------------------------------------------------------------------------
struct SoftArgs {
    const int64_t* nb_frozen;
    double sigma;
    const double* gS;
    const double* gA;
    double* S;
    double* A;
    double* g_psi;
    double* g_P;
    double gx0, gy0, inv_cell;
    int32_t nx, ny, level_cells;
    const uint16_t* cell_list;
    const uint2* cell_ent;      // per cell: {offset, count | first sphere << 16}
    // list of the bunches with a nonzero weight: written by the forward, read by the
    // adjoint (ids (step << kSoftIdBits) | k; count > capacity: incomplete)
    uint64_t* ids;
    int64_t ids_cap;
    int64_t* ids_count;
    int32_t skip_if_listed;     // tile kernels: exit when the list is complete
    int32_t cand_lds_acc;       // candidate kernel: S, A of all (shower, sphere) pairs in LDS
    int32_t shower_lds;         // listed kernels: the per-shower table in LDS
};

// Per shower, for the listed kernels: first step, counter-word base (the counter
// word of step i is ctr_base + i without caller step ids), t_ref and the shower id.
struct ShowerRec {
    int64_t first;
    int64_t ctr_base;
    double t_ref;
    uint32_t id;
    uint32_t pad;
};


__device__ __forceinline__ bool soft_list_complete(const SoftArgs& sa)
{
    const int64_t n = *sa.ids_count;
    return n >= 0 && n <= sa.ids_cap;
}

struct alignas(16) SoftStep {
    double x0, y0, h0, t0, u, v, w;
    double cos_t, sin_t, photons, ds, inv_bc;
    double b1x, b1y, b1z, b2x, b2y, b2z;
    double r2, g1, f_m, kl_nb;
    double g_cos, g_sin, g_phot;     // adjoint accumulators of the step
    int32_t i_m, boff, sidx;
    uint32_t ctr1;                   // counter word 1 of the step's random numbers
};
static_assert(sizeof(SoftStep) % 16 == 0, "soft step entry alignment");

constexpr int kSoftTS = 32;
// 8 waves for both directions, two per SIMD: the forward keeps 143 registers, the
// adjoint 198
__host__ __device__ constexpr int soft_max_waves(int) { return 8; }
// adjoint bins (dL/dpsi_i, dL/dP_j(h_i)) of the lowest kSoftBinNodes nodes live in
// LDS (h_obs + 51 km on a 50 m grid); the rare contributions above go to HBM
constexpr int kSoftBinNodes = 1024;

__host__ __device__ inline int soft_bin_nodes(int n_nodes)
{
    return n_nodes < kSoftBinNodes ? n_nodes : kSoftBinNodes;
}

// per wave: step stash, flag row and (forward only) S, A per telescope
__host__ __device__ inline size_t soft_wave_bytes(int mode, int n_tel)
{
    return kSoftTS * sizeof(SoftStep) + kWave * sizeof(int32_t) +
           (mode == 0 ? (size_t)2 * n_tel * sizeof(double) : 0);
}

// per workgroup: adjoint bins, then {X, Y, R^2, 1 / (2 R sigma)} per telescope, then the waves
// node records {psi, P1..P5} of the lowest kSoftNodeLds nodes staged in LDS for the
// bunch lookups of the forward and of the listed adjoint
constexpr int kSoftNodeLds = 1024;

__host__ __device__ inline int soft_node_lds(int n_nodes)
{
    return n_nodes < kSoftNodeLds ? n_nodes : kSoftNodeLds;
}

__host__ __device__ inline size_t soft_lds_bytes(int mode, int n_nodes, int n_tel, int waves)
{
    const size_t bins = mode == 1 ? (size_t)6 * soft_bin_nodes(n_nodes) * sizeof(double) : 0;
    const size_t nodes = mode == 0 ? (size_t)kNode64 * soft_node_lds(n_nodes) * sizeof(double) : 0;
    return bins + (size_t)n_tel * 4 * sizeof(double) + nodes + (size_t)waves * soft_wave_bytes(mode, n_tel);
}

// step setup with a frozen bunch count; false when the step emits nothing
__device__ inline bool soft_step_setup(const Args& a, int64_t i, int64_t nb, SoftStep& e,
                                       const double* node_lds = nullptr, int n_lds = 0)
{
    // no contraction: the threshold decision is the one of the FP64 definition and
    // of the screening pass's step setup
#pragma clang fp contract(off)
    const double x0 = a.x0[i], y0 = a.y0[i], h0 = a.h0[i];
    const double u = a.u[i], v = a.v[i], w = a.w[i];
    const double L = a.len[i], t0 = a.t0[i], E = a.energy[i];
    const double m = a.ptype[i] == CKV_MUON ? kMassMuon : kMassElectron;
    // every test evaluated (no short circuit) and the mass inside one of them (E c
    // with c = m / 1 GeV in (0, 1) is finite exactly when E is): all the step's loads
    // go out in one round
    const int n_finite = (int)isfinite(x0) + (int)isfinite(y0) + (int)isfinite(h0) + (int)isfinite(u) +
                         (int)isfinite(v) + (int)isfinite(w) + (int)isfinite(L) + (int)isfinite(t0) +
                         (int)isfinite(E * (m * 1e-3));
    if (n_finite != 9 || !(L > 0.0) || nb <= 0) return false;
    const double r = m / E;
    const double r2 = r * r;
    if (!(r2 < 1.0)) return false;
    const double h_mid = h0 - (0.5 * L) * w;
    const double hc = h_mid < a.h_obs ? a.h_obs : (h_mid > a.h_top ? a.h_top : h_mid);
    const double x = (hc - a.h_obs) * a.inv_step;
    int64_t im = (int64_t)floor(x);
    if (im > a.n_nodes - 2) im = a.n_nodes - 2;
    const double fm = x - (double)im;
    // psi at the two nodes: from the LDS copy of the lowest nodes when it holds them
    double lo, hi;
    if (im + 1 < n_lds) {
        lo = as_lds(node_lds)[kNode64 * im];
        hi = as_lds(node_lds)[kNode64 * (im + 1)];
    } else {
        lo = as_hbm(a.node64)[kNode64 * im];
        hi = as_hbm(a.node64)[kNode64 * (im + 1)];
    }
    const double psi = lo + fm * (hi - lo);
    const double n2 = 1.0 + psi;
    const double num = psi - n2 * r2;
    if (!(num > 0.0)) return false;
    // past the threshold test the step's values take reciprocals from the hardware
    // estimate and two Newton steps (within an ulp or two of the quotient): nothing
    // decides on them, and S, A and the gradient move by a few ulps at most
    e.g1 = (1.0 - r2) * n2;
    const double sin2 = num * rcp64(e.g1);
    const double nbd = (double)nb;
    const double inv_nb = rcp64(nbd);
    e.x0 = x0; e.y0 = y0; e.h0 = h0; e.t0 = t0; e.u = u; e.v = v; e.w = w;
    e.kl_nb = (a.k_ft * L) * inv_nb;
    e.photons = e.kl_nb * sin2;
    e.cos_t = rcp64(sqrt(e.g1));
    e.sin_t = sqrt(sin2);
    e.ds = L * inv_nb;
    e.inv_bc = rcp64(sqrt(1.0 - r2) * kSpeedOfLight);
    const double Dx = u, Dy = v, Dz = -w;
    const double sgn = copysign(1.0, Dz);
    const double ia = -rcp64(sgn + Dz);
    const double ib = Dx * Dy * ia;
    e.b1x = 1.0 + sgn * Dx * Dx * ia;
    e.b1y = sgn * ib;
    e.b1z = -sgn * Dx;
    e.b2x = ib;
    e.b2y = sgn + Dy * Dy * ia;
    e.b2z = -Dy;
    e.r2 = r2;
    e.f_m = fm;
    e.i_m = (int32_t)im;
    e.g_cos = e.g_sin = e.g_phot = 0.0;
    return true;
}

// One bunch k of a soft-response step e (its random numbers from the counter
// (k, seg_id, shower_id, 0)): emission, propagation and the soft weights over
// the candidate spheres.  MODE 0 adds photons * Phi and photons * Phi * t into
// acc (LDS, S then A per telescope); MODE 1 runs the adjoint of the bunch into
// the table bins and g_psi0 and returns the step-level adjoints (dL/dcos_t,
// dL/dsin_t, dL/dphotons) in o_cos, o_sin, o_phot.  Returns true when some
// sphere has z >= -kSoftZCut, i.e. the bunch enters S, A and the gradient.
// NODE_LDS: node records of the lowest n_lds nodes come from node_lds (LDS).
template <int MODE, bool NODE_LDS, bool ACC_LDS, typename AddBin>
__device__ __forceinline__ bool soft_bunch(const Args& a, const SoftArgs& sa, const SoftStep& e,
                                           int32_t k, uint32_t seg_id, uint32_t shower_id, int s,
                                           double t_ref, const double* tsh, double* acc,
                                           double* accA, AddBin& add_bin, double inv_nobs,
                                           double half_inv_nobs3,
                                           const double* node_lds, int n_lds,
                                           double& g_psi0, double& o_cos, double& o_sin,
                                           double& o_phot)
{
    const int N = a.n_nodes;
    constexpr double a1 = -0.5, a2 = 0.375, a3 = -0.3125, a4 = 0.2734375;
    const double ak[5] = {1.0, a1, a2, a3, a4};
    const double inv_c = 1.0 / kSpeedOfLight;
    constexpr double inv_sqrt2 = 0.70710678118654752440;
    constexpr double inv_sqrt2pi = 0.39894228040143267794;
    uint32_t r[4];
    philox4x32_10((uint32_t)k, seg_id, shower_id, 0u, a.key0, a.key1, r);
    const double u0 = ((double)r[0] + 0.5) * 2.3283064365386963e-10;
    const double s_along = ((double)k + u0) * e.ds;
    const double xe = e.x0 + s_along * e.u;
    const double ye = e.y0 + s_along * e.v;
    const double he = e.h0 - s_along * e.w;
    const double te = e.t0 + s_along * e.inv_bc;
    double sp, cp;
    sincos_turns64(r[1], sp, cp);
    const double Ex = cp * e.b1x + sp * e.b2x;
    const double Ey = cp * e.b1y + sp * e.b2y;
    const double Ez = cp * e.b1z + sp * e.b2z;
    const double pu = e.cos_t * e.u + e.sin_t * Ex;
    const double pv = e.cos_t * e.v + e.sin_t * Ey;
    const double pw = e.cos_t * e.w - e.sin_t * Ez;
    if (he < a.h_obs || he >= a.h_top || pw <= a.w_min) return false;
    // atmosphere at emission
    const double x = (he - a.h_obs) * a.inv_step;
    int ie = (int)x;
    ie = min(ie, N - 2);
    const double fe = x - (double)ie;
    double pa, pb, X1, X2, X3, X4, X5;
    if (NODE_LDS) {
        // the cell from the LDS copy when it holds it, else from HBM, each through
        // its own address space (no generic load)
        if (ie + 1 < n_lds) {
            const LdsF64* nl = as_lds(node_lds) + (size_t)kNode64 * ie;
            pa = nl[0]; X1 = nl[1]; X2 = nl[2]; X3 = nl[3]; X4 = nl[4]; X5 = nl[5];
            pb = nl[kNode64];
        } else {
            const HbmF64* nd = as_hbm(a.node64) + (size_t)kNode64 * ie;
            pa = nd[0]; X1 = nd[1]; X2 = nd[2]; X3 = nd[3]; X4 = nd[4]; X5 = nd[5];
            pb = nd[kNode64];
        }
    } else {
        const double* nd = a.node64 + (size_t)kNode64 * ie;
        pa = nd[0]; X1 = nd[1]; X2 = nd[2]; X3 = nd[3]; X4 = nd[4]; X5 = nd[5];
        pb = nd[kNode64];
    }
    const double psi_e = pa + fe * (pb - pa);
    const double dz = fe * a.step;
    const double dh = he - a.h_obs;
    // D_k = int (psi - psi_e)^k dh: node moments shifted to psi_e (Pascal
    // triangle, P_0(h_i) = h_i - h_obs) plus the in-cell part of the linear
    // profile, dz (psi_i - psi_e)^k / (k+1)
    const double c = -psi_e, del = pa - psi_e;
    const double X0 = (double)ie * a.step;
    X5 += c * X4; X4 += c * X3; X3 += c * X2; X2 += c * X1; X1 += c * X0;
    X5 += c * X4; X4 += c * X3; X3 += c * X2; X2 += c * X1;
    X5 += c * X4; X4 += c * X3; X3 += c * X2;
    X5 += c * X4; X4 += c * X3;
    X5 += c * X4;
    const double dl2 = del * del, dl3 = dl2 * del, dl4 = dl3 * del;
    double D[6];
    D[0] = dh;
    D[1] = X1 + dz * 0.5 * del;
    D[2] = X2 + dz * (1.0 / 3.0) * dl2;
    D[3] = X3 + dz * 0.25 * dl3;
    D[4] = X4 + dz * 0.2 * dl4;
    D[5] = X5 + dz * (1.0 / 6.0) * (dl4 * del);
    const double ne2 = 1.0 + psi_e;
    const double ne = sqrt(ne2);
    const double inv_ne = rcp64(ne), inv_pw = rcp64(pw);
    const double q = (inv_pw * inv_pw) * (inv_ne * inv_ne);
    const double Sser = D[0] + q * (a1 * D[1] + q * (a2 * D[2] + q * (a3 * D[3] + q * a4 * D[4])));
    const double U = (ne2 * D[0] + D[1]) +
                     q * (a1 * (ne2 * D[1] + D[2]) +
                          q * (a2 * (ne2 * D[2] + D[3]) +
                               q * (a3 * (ne2 * D[3] + D[4]) + q * a4 * (ne2 * D[4] + D[5]))));
    const double T = U * inv_ne * inv_pw * inv_c;
    const double adv = Sser * inv_pw;
    const double xg = xe + pu * adv;
    const double yg = ye + pv * adv;
    const double tt = te + T - t_ref;
    const double uo = pu * ne * inv_nobs;
    const double vo = pv * ne * inv_nobs;
    const double p = e.photons;

    // soft weights over candidate spheres
    double g_xg = 0, g_yg = 0, g_uo = 0, g_vo = 0, g_t = 0, g_p = 0;
    bool seen = false;
    int cur = 0, cend = 0;
    int first = -1;          // the cell's first sphere, known without a list read
    bool brute = false;
    const double wo2 = 1.0 - uo * uo - vo * vo;
    if (wo2 >= kLevelW2[0]) {
        const double fx = (xg - sa.gx0) * sa.inv_cell, fy = (yg - sa.gy0) * sa.inv_cell;
        if (fx >= 0.0 && fy >= 0.0 && fx < (double)sa.nx && fy < (double)sa.ny) {
            const int cidx = grid_level(wo2) * sa.level_cells + (int)fx * sa.ny + (int)fy;
            const uint2 ce = sa.cell_ent[cidx];
            cur = (int)ce.x;
            cend = cur + (int)(ce.y & 0xFFFFu);
            first = (int)(ce.y >> 16);
        }
    } else {
        brute = true;
        cend = a.n_tel;
    }
    for (; cur < cend; ++cur) {
        const int kt = brute ? cur : (first >= 0 ? first : (int)sa.cell_list[cur]);
        first = -1;
        const double* tp = tsh + 4 * kt;                  // LDS
        const double dx = xg - tp[0], dy = yg - tp[1];
        const double b = dx * uo + dy * vo;
        const double rho2 = dx * dx + dy * dy - b * b;
        const double z = (tp[2] - rho2) * tp[3];
        if (z < -kSoftZCut) continue;
        seen = true;
        const double W = 0.5 * erfc(-z * inv_sqrt2);
        if (MODE == 0) {
            if (ACC_LDS) {
                lds_add(&acc[kt], p * W);
                lds_add(&accA[kt], p * W * tt);
            } else {
                hbm_add(&acc[kt], p * W);
                hbm_add(&accA[kt], p * W * tt);
            }
        } else {
            const double gSk = sa.gS[(int64_t)s * a.n_tel + kt];
            const double gAk = sa.gA[(int64_t)s * a.n_tel + kt];
            g_p += gSk * W + gAk * W * tt;
            g_t += gAk * p * W;
            const double g_z = (gSk * p + gAk * p * tt) * inv_sqrt2pi * exp(-0.5 * z * z);
            const double g_r2 = -g_z * tp[3];
            g_xg += g_r2 * (2.0 * dx - 2.0 * b * uo);
            g_yg += g_r2 * (2.0 * dy - 2.0 * b * vo);
            g_uo += g_r2 * (-2.0 * b * dx);
            g_vo += g_r2 * (-2.0 * b * dy);
        }
    }
    if (MODE == 1 && (g_xg != 0.0 || g_yg != 0.0 || g_uo != 0.0 || g_vo != 0.0 || g_t != 0.0 ||
                      g_p != 0.0)) {
        // ---- reverse through propagation
        double g_pu = g_uo * ne * inv_nobs + g_xg * adv;
        double g_pv = g_vo * ne * inv_nobs + g_yg * adv;
        double g_ne = (g_uo * pu + g_vo * pv) * inv_nobs;
        // n_obs = sqrt(1 + psi_0): d(1/n_obs)/d psi_0 = -1 / (2 n_obs^3)
        g_psi0 -= (g_uo * pu + g_vo * pv) * ne * half_inv_nobs3;
        const double g_U = g_t * inv_c * inv_ne * inv_pw;
        g_ne -= g_t * T * inv_ne;
        double g_pw = -g_t * T * inv_pw;
        const double XS = g_xg * pu + g_yg * pv;
        const double g_S = XS * inv_pw;
        g_pw -= XS * adv * inv_pw;
        const double qk[5] = {1.0, q, q * q, q * q * q, q * q * q * q};
        double gD[6] = {0, 0, 0, 0, 0, 0};
        double g_q = 0.0;
        for (int kk = 0; kk < 5; ++kk) {
            const double akq = ak[kk] * qk[kk];
            gD[kk] += g_S * akq + g_U * akq * ne2;
            gD[kk + 1] += g_U * akq;
            if (kk >= 1)
                g_q += (g_S * D[kk] + g_U * (ne2 * D[kk] + D[kk + 1])) * (double)kk * ak[kk] * qk[kk - 1];
        }
        double g_ne2 = g_U * Sser;
        g_ne2 -= g_q * q * inv_ne * inv_ne;
        g_pw -= 2.0 * g_q * q * inv_pw;
        g_ne2 += g_ne * 0.5 * inv_ne;
        // D_k as a function of (P_j(h_i), psi_i, psi_e):
        //   dD_k/dpsi_e = -k D_{k-1} + dz del^(k-1) / (k+1)
        //   dD_k/dpsi_i = dz k del^(k-1) / (k+1)
        const double dpow[5] = {1.0, del, dl2, dl3, dl4};
        double g_psie = g_ne2, g_pa = 0.0;
#pragma unroll
        for (int kk = 1; kk <= 5; ++kk) {
            const double inc = dz * dpow[kk - 1] * (1.0 / (double)(kk + 1));
            g_psie += gD[kk] * (inc - (double)kk * D[kk - 1]);
            g_pa += gD[kk] * ((double)kk * inc);
        }
        // dL/dP_j(h_i): the Pascal shift transposed
        double G1 = gD[1], G2 = gD[2], G3 = gD[3], G4 = gD[4], G5 = gD[5];
        G4 += c * G5;
        G3 += c * G4; G4 += c * G5;
        G2 += c * G3; G3 += c * G4; G4 += c * G5;
        G1 += c * G2; G2 += c * G3; G3 += c * G4; G4 += c * G5;
        G1 += c * G2; G2 += c * G3; G3 += c * G4; G4 += c * G5;
        add_bin(1, ie, G1);
        add_bin(2, ie, G2);
        add_bin(3, ie, G3);
        add_bin(4, ie, G4);
        add_bin(5, ie, G5);
        add_bin(0, ie, g_pa + (1.0 - fe) * g_psie);
        add_bin(0, ie + 1, fe * g_psie);
        // ---- reverse through the direction on the cone and the yield
        const double g_cos = g_pu * e.u + g_pv * e.v + g_pw * e.w;
        const double g_sin = g_pu * Ex + g_pv * Ey - g_pw * Ez;
        o_cos = g_cos;
        o_sin = g_sin;
        o_phot = g_p;
    }
    return seen;
}

// Step-level part of the soft adjoint: dL/dcos_t, dL/dsin_t and dL/dphotons of
// bunches of step es to dL/dpsi at the two table nodes around the step's
// midpoint (cos_t = g1^(-1/2), sin^2 = 1 - 1/g1, g1 = (1 - r^2) n^2; linear in
// the three inputs, so per-bunch and per-step application agree).
template <typename AddBin>
__device__ __forceinline__ void soft_step_reverse(const SoftStep& es, double g_cos, double g_sin,
                                                  double g_phot, AddBin& add_bin)
{
    const double sin2 = es.sin_t * es.sin_t;
    double g_sin2 = g_phot * es.kl_nb;
    if (sin2 > 0.0) g_sin2 += g_sin / (2.0 * es.sin_t);
    const double g_g1 = -0.5 * g_cos * es.cos_t * es.cos_t * es.cos_t + g_sin2 / (es.g1 * es.g1);
    const double g_psim = g_g1 * (1.0 - es.r2);
    if (g_psim != 0.0) {
        add_bin(0, es.i_m, (1.0 - es.f_m) * g_psim);
        add_bin(0, es.i_m + 1, es.f_m * g_psim);
    }
}

template <int MODE>
__global__ void __launch_bounds__(soft_max_waves(MODE) * kWave) soft_kernel(Args a, SoftArgs sa)
{
    extern __shared__ __align__(16) unsigned char lds[];
    // with a complete list soft_list_kernel (adjoint) or soft_cand_kernel (forward
    // after the screening pass) does the work (the same decision in every thread)
    if (sa.skip_if_listed && soft_list_complete(sa)) return;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int N = a.n_nodes;
    const int NB = soft_bin_nodes(N);
    double* bins = reinterpret_cast<double*>(lds);                 // MODE 1: 6 x NB
    double* tsh = bins + (MODE == 1 ? 6 * NB : 0);     // n_tel x {X, Y, R^2, 1 / (2 R sigma)}
    double* nlds = tsh + 4 * a.n_tel;                 // MODE 0: lowest node records
    const int NL = soft_node_lds(N);
    unsigned char* wbase = reinterpret_cast<unsigned char*>(nlds + (MODE == 0 ? kNode64 * NL : 0)) +
                           (size_t)wave * soft_wave_bytes(MODE, a.n_tel);
    SoftStep* stash = reinterpret_cast<SoftStep*>(wbase);
    int32_t* flags = reinterpret_cast<int32_t*>(wbase + kSoftTS * sizeof(SoftStep));
    double* acc = reinterpret_cast<double*>(flags + kWave);     // MODE 0: S then A per telescope
    if (MODE == 1)
        for (int q = threadIdx.x; q < 6 * NB; q += blockDim.x) bins[q] = 0.0;
    for (int q = threadIdx.x; q < a.n_tel; q += blockDim.x) {
        tsh[4 * q] = a.tel[4 * q];
        tsh[4 * q + 1] = a.tel[4 * q + 1];
        tsh[4 * q + 2] = a.tel[4 * q + 3];
        tsh[4 * q + 3] = 1.0 / (2.0 * a.tel[4 * q + 2] * sa.sigma);
    }
    if (MODE == 0)
        for (int q = threadIdx.x; q < kNode64 * NL; q += blockDim.x) nlds[q] = a.node64[q];
    if (MODE == 0)
        for (int q = lane; q < 2 * a.n_tel; q += kWave) acc[q] = 0.0;
    flags[lane] = 0;
    __syncthreads();
    // j = 0: dL/dpsi_i, j = 1..5: dL/dP_j(h_i)
    auto add_bin = [&](int j, int i, double v) {
        if (i < NB) lds_add(&bins[j * NB + i], v);
        else hbm_add(j == 0 ? &sa.g_psi[i] : &sa.g_P[(size_t)(j - 1) * N + i], v);
    };

    const double inv_nobs = 1.0 / a.n_obs;
    const double half_inv_nobs3 = 0.5 * inv_nobs * inv_nobs * inv_nobs;
    double g_psi0 = 0.0;
    const int64_t n_tiles = a.ctrl[kNumTiles];

    for (;;) {
        int64_t t = 0;
        if (lane == 0) t = (int64_t)atomicAdd((unsigned long long*)&a.ctrl[kTileCounter], 1ull);
        t = uniform(t);
        if (t >= n_tiles) break;
        int lo = 0, hi = a.n_showers;
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (a.tiles_before[mid] <= t) lo = mid; else hi = mid;
        }
        const int s = lo;
        const int64_t sfirst = a.seg_offsets[s];
        const int64_t g0 = a.shower_first[s] + (t - a.tiles_before[s]) * (int64_t)kSoftTS;
        const int64_t gend = min(g0 + (int64_t)kSoftTS, a.seg_offsets[s + 1]);
        const int nseg = (int)(gend - g0);
        const uint32_t shower_id = a.shower_ids ? a.shower_ids[s] : (uint32_t)s;
        const int64_t seg_id0 = (a.seg_id_base ? a.seg_id_base[s] : 0) + (g0 - sfirst);
        const double t_ref = a.t_ref[s];

        SoftStep st;
        int64_t nb = 0;
        bool emits = false;
        double len = 0.0;
        if (lane < nseg) {
            const int64_t nbf = sa.nb_frozen[g0 + lane];
            len = a.len[g0 + lane];
            emits = soft_step_setup(a, g0 + lane, nbf, st);
            if (emits) nb = nbf;
        }
        // the tile limit on the frozen counts, then the cull of the steps whose
        // bunches can weight no sphere (screen_annulus)
        if (wave_last(wave_incl_scan(nb)) >= ((int64_t)1 << 30)) {
            if (lane == 0 && a.result) atomicOr(&a.result->error, 2);
            continue;
        }
        if (a.cull_rmax > 0.0) {
            double cgx = 0.0, cgy = 0.0, cmid = 0.0, chalf = -1.0;
            const int ok = emits && screen_annulus(a, st.x0, st.y0, st.h0, st.u, st.v, st.w, len, st.cos_t,
                                                   st.sin_t, cgx, cgy, cmid, chalf) ? 1 : 0;
            // (called by the whole wave: the upper half-wave tests spheres for the lower one)
            const bool reached = annulus_holds_centre<4>(tsh, a.n_tel, lane, ok, cgx, cgy, cmid, chalf);
            if (ok && !reached) {
                emits = false;
                nb = 0;
            }
        }
        const int64_t incl = wave_incl_scan(nb);
        const int64_t total = wave_last(incl);
        const uint64_t emit_mask = __ballot(emits);
        const int excl = (int)(incl - nb);
        if (emits) {
            st.boff = excl;
            st.sidx = lane;
            st.ctr1 = a.step_id ? a.step_id[g0 + lane] : (uint32_t)(seg_id0 + lane);
            stash[lanes_below(emit_mask)] = st;
        }
        wave_lds_sync();

        for (int64_t c0 = 0; c0 < total; c0 += kWave) {
            const int32_t j = (int32_t)(c0 + lane);
            const bool active = j < total;
            const int cnt0 = __popcll(__ballot(emits && excl <= (int)c0));
            if (emits && excl > (int)c0 && excl < (int)c0 + kWave) flags[excl - (int)c0] = 1;
            wave_lds_sync();
            const uint64_t starts = __ballot(flags[lane] != 0);
            flags[lane] = 0;
            const int si = cnt0 - 1 + lanes_upto(starts);
            if (active) {
                SoftStep& e = stash[si];
                const int32_t k = j - e.boff;
                double o_cos = 0.0, o_sin = 0.0, o_phot = 0.0;
                soft_bunch<MODE, MODE == 0, true>(a, sa, e, k, e.ctr1, shower_id,
                                                   s, t_ref, tsh, acc, acc + a.n_tel, add_bin, inv_nobs,
                                                   half_inv_nobs3, nlds, NL, g_psi0, o_cos, o_sin,
                                                   o_phot);
                if (MODE == 1 && (o_cos != 0.0 || o_sin != 0.0 || o_phot != 0.0)) {
                    lds_add(&e.g_cos, o_cos);
                    lds_add(&e.g_sin, o_sin);
                    lds_add(&e.g_phot, o_phot);
                }
            }
        }
        wave_lds_sync();
        if (MODE == 0) {
            for (int kk = lane; kk < a.n_tel; kk += kWave) {
                const double vs = acc[kk], va = acc[a.n_tel + kk];
                if (vs != 0.0) atomicAdd(&sa.S[(int64_t)s * a.n_tel + kk], vs);
                if (va != 0.0) atomicAdd(&sa.A[(int64_t)s * a.n_tel + kk], va);
                acc[kk] = 0.0;
                acc[a.n_tel + kk] = 0.0;
            }
        } else if (emits) {
            // ---- reverse through the step setup (index at the step midpoint)
            const SoftStep& es = stash[lanes_below(emit_mask)];
            soft_step_reverse(es, es.g_cos, es.g_sin, es.g_phot, add_bin);
        }
        wave_lds_sync();
    }
    if (MODE == 1) {
        if (g_psi0 != 0.0) add_bin(0, 0, g_psi0);
        __syncthreads();
        for (int qq = threadIdx.x; qq < 6 * NB; qq += blockDim.x) {
            const double v = bins[qq];
            const int j = qq / NB, i = qq - j * NB;
            if (v != 0.0) atomicAdd(j == 0 ? &sa.g_psi[i] : &sa.g_P[(size_t)(j - 1) * N + i], v);
        }
    }
}

constexpr int kSoftListThreads = 512;   // listed adjoint: workgroup size
// listed forward: at most 16 waves a compute unit, in two workgroups where the LDS holds
// two, else in one (64 showers x 100 spheres, 102 KB of S and A: 3.18 ms with one of 512
// threads, 2.45 with 1024; 16 showers, where two fit: 122 us in two, 127 in one)
constexpr int kSoftCandThreads = 1024;

// Listed bunches of a wave (consecutive list entries, one per lane; id is the
// lane's entry, loaded by the caller): the step setup and the shower lookup are
// done once per run of lanes that name the same step (the screening pass lists a
// step's bunches together) and passed to the run's other lanes by lane shuffles.
// shr: the per-shower table in LDS, or null (then from HBM); node_lds: the lowest
// n_lds node records in LDS.  REV: also the step-level values of the reverse sweep.
// True for lanes whose id names a bunch of the inputs on a step that gives light.
// Called by the whole wave.
template <bool REV>
__device__ __forceinline__ bool listed_setup(const Args& a, const SoftArgs& sa, uint64_t id, bool have,
                                             int lane, const ShowerRec* shr, const double* node_lds,
                                             int n_lds, SoftStep& e, int& shower, uint32_t& ctr1,
                                             uint32_t& shower_id, double& t_ref, int32_t& k)
{
    const int64_t i = have ? (int64_t)(id >> kSoftIdBits) : -1;
    k = (int32_t)(id & ((1u << kSoftIdBits) - 1));
    const bool named = have && i < a.n;
    const int64_t nbf = named ? sa.nb_frozen[i] : 0;
    const int64_t i_prev = __shfl_up(i, 1);
    const bool head = named && (lane == 0 || i_prev != i);
    int lit = 0, lo = 0;
    uint32_t c1 = 0, sid = 0;
    double tr = 0.0;
    if (head) {
        int hi = a.n_showers;                   // the shower holding step i
        if (shr) {
            // the LDS table through its own address space (no generic loads)
            using LdsRec = const __attribute__((address_space(3))) ShowerRec;
            LdsRec* sh = (LdsRec*)shr;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (sh[mid].first <= i) lo = mid; else hi = mid;
            }
            c1 = a.step_id ? a.step_id[i] : (uint32_t)(sh[lo].ctr_base + i);
            sid = sh[lo].id;
            tr = sh[lo].t_ref;
        } else {
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (a.seg_offsets[mid] <= i) lo = mid; else hi = mid;
            }
            c1 = a.step_id ? a.step_id[i]
                           : (uint32_t)((a.seg_id_base ? a.seg_id_base[lo] : 0) + (i - a.seg_offsets[lo]));
            sid = a.shower_ids ? a.shower_ids[lo] : (uint32_t)lo;
            tr = a.t_ref[lo];
        }
        lit = soft_step_setup(a, i, nbf, e, node_lds, n_lds) ? 1 : 0;
    }
    // the run's head: the nearest head lane at or below this one
    const uint64_t heads = __ballot(head);
    const uint64_t le = lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1);
    const uint64_t mine = heads & le;
    const int src = mine ? 63 - __builtin_clzll(mine) : lane;
    lit = __shfl(lit, src);
    shower = __shfl(lo, src);
    ctr1 = __shfl(c1, src);
    shower_id = __shfl(sid, src);
    t_ref = __shfl(tr, src);
    e.x0 = __shfl(e.x0, src); e.y0 = __shfl(e.y0, src); e.h0 = __shfl(e.h0, src);
    e.t0 = __shfl(e.t0, src); e.u = __shfl(e.u, src); e.v = __shfl(e.v, src); e.w = __shfl(e.w, src);
    e.cos_t = __shfl(e.cos_t, src); e.sin_t = __shfl(e.sin_t, src);
    e.photons = __shfl(e.photons, src); e.ds = __shfl(e.ds, src); e.inv_bc = __shfl(e.inv_bc, src);
    e.b1x = __shfl(e.b1x, src); e.b1y = __shfl(e.b1y, src); e.b1z = __shfl(e.b1z, src);
    e.b2x = __shfl(e.b2x, src); e.b2y = __shfl(e.b2y, src); e.b2z = __shfl(e.b2z, src);
    if (REV) {
        e.r2 = __shfl(e.r2, src); e.g1 = __shfl(e.g1, src); e.f_m = __shfl(e.f_m, src);
        e.kl_nb = __shfl(e.kl_nb, src); e.i_m = __shfl(e.i_m, src);
    }
    return named && lit && k < nbf;
}

// Per-shower table of the listed kernels, staged into LDS by the workgroup.
__device__ __forceinline__ void stage_showers(const Args& a, ShowerRec* shr)
{
    for (int q = threadIdx.x; q < a.n_showers; q += blockDim.x) {
        ShowerRec r;
        r.first = a.seg_offsets[q];
        r.ctr_base = (a.seg_id_base ? a.seg_id_base[q] : 0) - a.seg_offsets[q];
        r.t_ref = a.t_ref[q];
        r.id = a.shower_ids ? a.shower_ids[q] : (uint32_t)q;
        r.pad = 0;
        shr[q] = r;
    }
}

// Bound like soft_cand_kernel below, at two waves per SIMD: 7.0e7 VALU instructions, 114 us
// of issue, take 258 us for a 1.6e6-step fit.  The reverse sweep keeps 192 registers; held
// to the 168 of three waves it spills (323 us).
// Adjoint over the forward's list: one listed bunch per thread, its step set up
// again (bunch count frozen), the bunch recomputed from its random numbers and
// reversed into the table bins, the step-level part applied per bunch.  Runs only
// when the list is complete; ids that do not name a bunch of the inputs are skipped.
__global__ void __launch_bounds__(kSoftListThreads) soft_list_kernel(Args a, SoftArgs sa)
{
    extern __shared__ __align__(16) unsigned char lds[];
    if (!soft_list_complete(sa)) return;
    const int64_t n_ids = *sa.ids_count;
    const int N = a.n_nodes;
    const int NB = soft_bin_nodes(N);
    double* bins = reinterpret_cast<double*>(lds);               // 6 x NB
    double* tsh = bins + 6 * NB;                                 // n_tel x {X, Y, R^2, 1 / (2 R sigma)}
    double* nlds = tsh + 4 * a.n_tel;                            // lowest node records
    const int NL = soft_node_lds(N);
    for (int q = threadIdx.x; q < 6 * NB; q += blockDim.x) bins[q] = 0.0;
    for (int q = threadIdx.x; q < kNode64 * NL; q += blockDim.x) nlds[q] = a.node64[q];
    for (int q = threadIdx.x; q < a.n_tel; q += blockDim.x) {
        tsh[4 * q] = a.tel[4 * q];
        tsh[4 * q + 1] = a.tel[4 * q + 1];
        tsh[4 * q + 2] = a.tel[4 * q + 3];
        tsh[4 * q + 3] = 1.0 / (2.0 * a.tel[4 * q + 2] * sa.sigma);
    }
    ShowerRec* shr = sa.shower_lds ? reinterpret_cast<ShowerRec*>(nlds + kNode64 * NL) : nullptr;
    if (shr) stage_showers(a, shr);
    __syncthreads();
    auto add_bin = [&](int j, int i, double v) {
        if (i < NB) lds_add(&bins[j * NB + i], v);
        else hbm_add(j == 0 ? &sa.g_psi[i] : &sa.g_P[(size_t)(j - 1) * N + i], v);
    };
    const double inv_nobs = 1.0 / a.n_obs;
    const double half_inv_nobs3 = 0.5 * inv_nobs * inv_nobs * inv_nobs;
    double g_psi0 = 0.0;
    const int lane = lane_id();
    // each lane's next list entry is loaded one round ahead, while the current
    // bunch is computed
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t q0 = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~(kWave - 1));
    uint64_t id = q0 + lane < n_ids ? sa.ids[q0 + lane] : ~0ull;
    for (; q0 < n_ids; q0 += stride) {
        const int64_t q = q0 + lane;
        const uint64_t id_next = q + stride < n_ids ? sa.ids[q + stride] : ~0ull;
        SoftStep e;
        int lo;
        uint32_t seg_id, shower_id;
        double t_ref;
        int32_t k;
        if (listed_setup<true>(a, sa, id, q < n_ids, lane, shr, nlds, NL, e, lo, seg_id, shower_id,
                               t_ref, k)) {
            double o_cos = 0.0, o_sin = 0.0, o_phot = 0.0;
            soft_bunch<1, true, true>(a, sa, e, k, seg_id, shower_id, lo, t_ref, tsh, nullptr, nullptr,
                                add_bin, inv_nobs, half_inv_nobs3, nlds, NL, g_psi0, o_cos, o_sin,
                                o_phot);
            if (o_cos != 0.0 || o_sin != 0.0 || o_phot != 0.0)
                soft_step_reverse(e, o_cos, o_sin, o_phot, add_bin);
        }
        id = id_next;
    }
    if (g_psi0 != 0.0) add_bin(0, 0, g_psi0);
    __syncthreads();
    for (int qq = threadIdx.x; qq < 6 * NB; qq += blockDim.x) {
        const double v = bins[qq];
        const int j = qq / NB, i = qq - j * NB;
        if (v != 0.0) atomicAdd(j == 0 ? &sa.g_psi[i] : &sa.g_P[(size_t)(j - 1) * N + i], v);
    }
}

// Bound by FP64 issue and the latency of its serial chains: 4.9e7 VALU instructions, 80 us
// of issue, take 122 us for a 1.6e6-step fit at four waves per SIMD (126 registers).
// Soft forward over the screening pass's candidate list: one candidate bunch per
// thread, its step set up again with the frozen count and the bunch recomputed in
// FP64 exactly as in the tile kernel; S and A are added straight into HBM.  Runs
// only when the list is complete; ids that name no bunch are skipped.
__global__ void __launch_bounds__(kSoftCandThreads) soft_cand_kernel(Args a, SoftArgs sa)
{
    extern __shared__ __align__(16) unsigned char lds[];
    if (!soft_list_complete(sa)) return;
    const int64_t n_ids = *sa.ids_count;
    const int N = a.n_nodes;
    double* tsh = reinterpret_cast<double*>(lds);                // n_tel x {X, Y, R^2, 1 / (2 R sigma)}
    double* nlds = tsh + 4 * a.n_tel;                            // lowest node records
    const int NL = soft_node_lds(N);
    for (int q = threadIdx.x; q < a.n_tel; q += blockDim.x) {
        tsh[4 * q] = a.tel[4 * q];
        tsh[4 * q + 1] = a.tel[4 * q + 1];
        tsh[4 * q + 2] = a.tel[4 * q + 3];
        tsh[4 * q + 3] = 1.0 / (2.0 * a.tel[4 * q + 2] * sa.sigma);
    }
    for (int q = threadIdx.x; q < kNode64 * NL; q += blockDim.x) nlds[q] = a.node64[q];
    // S and A summed per workgroup in LDS when they fit (added to HBM once at the
    // end): bunches near one sphere would otherwise all update the same two words
    const int64_t nsk = (int64_t)a.n_showers * a.n_tel;
    double* accS = nlds + kNode64 * NL;
    double* accA = accS + nsk;
    if (sa.cand_lds_acc)
        for (int64_t q = threadIdx.x; q < 2 * nsk; q += blockDim.x) accS[q] = 0.0;
    ShowerRec* shr = sa.shower_lds
                         ? reinterpret_cast<ShowerRec*>(sa.cand_lds_acc ? accA + nsk : accS)
                         : nullptr;
    if (shr) stage_showers(a, shr);
    __syncthreads();
    auto no_bins = [](int, int, double) {};
    const double inv_nobs = 1.0 / a.n_obs;
    const double half_inv_nobs3 = 0.5 * inv_nobs * inv_nobs * inv_nobs;
    double g_psi0 = 0.0;
    const int lane = lane_id();
    // each lane's next list entry is loaded one round ahead, while the current
    // bunch is computed
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t q0 = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~(kWave - 1));
    uint64_t id = q0 + lane < n_ids ? sa.ids[q0 + lane] : ~0ull;
    for (; q0 < n_ids; q0 += stride) {
        const int64_t q = q0 + lane;
        const uint64_t id_next = q + stride < n_ids ? sa.ids[q + stride] : ~0ull;
        SoftStep e;
        int lo;
        uint32_t seg_id, shower_id;
        double t_ref;
        int32_t k;
        if (listed_setup<false>(a, sa, id, q < n_ids, lane, shr, nlds, NL, e, lo, seg_id, shower_id,
                                t_ref, k)) {
            double o_cos = 0.0, o_sin = 0.0, o_phot = 0.0;
            // S and A into the workgroup's LDS rows, or straight into HBM (a uniform
            // choice; each branch keeps its address space)
            if (sa.cand_lds_acc)
                soft_bunch<0, true, true>(a, sa, e, k, seg_id, shower_id, lo, t_ref, tsh,
                                          accS + (int64_t)lo * a.n_tel, accA + (int64_t)lo * a.n_tel, no_bins,
                                          inv_nobs, half_inv_nobs3, nlds, NL, g_psi0, o_cos, o_sin, o_phot);
            else
                soft_bunch<0, true, false>(a, sa, e, k, seg_id, shower_id, lo, t_ref, tsh,
                                           sa.S + (int64_t)lo * a.n_tel, sa.A + (int64_t)lo * a.n_tel, no_bins,
                                           inv_nobs, half_inv_nobs3, nlds, NL, g_psi0, o_cos, o_sin, o_phot);
        }
        id = id_next;
    }
    if (sa.cand_lds_acc) {
        __syncthreads();
        for (int64_t q = threadIdx.x; q < nsk; q += blockDim.x) {
            if (accS[q] != 0.0) atomicAdd(&sa.S[q], accS[q]);
            if (accA[q] != 0.0) atomicAdd(&sa.A[q], accA[q]);
        }
    }
}

__global__ void zero_kernel(double* p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
namespace {

// Raises a kernel's dynamic-LDS limit the first time it is launched on a device
// (once per kernel and device; safe when several host threads launch).
void allow_lds(const void* kernel, int bytes)
{
    static std::mutex mu;
    static std::set<std::pair<const void*, int>> done;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lock(mu);
    if (done.insert({kernel, dev}).second)
        (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

Args make_args(const RunPlan& p)
{
    Args a{};
    const ckv_segments& s = p.segs;
    a.x0 = s.x0; a.y0 = s.y0; a.h0 = s.h0; a.u = s.u; a.v = s.v; a.w = s.w;
    a.len = s.length; a.t0 = s.t0; a.energy = s.energy; a.ptype = s.ptype; a.n = s.n;
    a.step_id = s.step_id;
    a.seg_offsets = p.showers.seg_offsets;
    a.t_ref = p.showers.t_ref;
    a.shower_ids = p.showers.shower_ids;
    a.seg_id_base = p.showers.seg_id_base;
    a.n_showers = p.showers.n_showers;
    const ckv_atmo* at = p.atmo;
    a.n_nodes = (int32_t)at->n_nodes;
    a.h_obs = at->h_obs; a.step = at->step; a.inv_step = at->inv_step; a.h_top = at->h_top;
    a.n_obs = at->n_obs;
    a.node64 = at->d_node64;
    a.cell32 = at->d_cell32;
    a.hnodes = at->d_hnodes;
    a.search_pow2 = 0;
    while ((a.search_pow2 ? 2 * a.search_pow2 : 1) < a.n_nodes - 1)
        a.search_pow2 = a.search_pow2 ? 2 * a.search_pow2 : 1;
    a.depth = at->d_depth;
    if (p.prof_bins > 0) {
        a.prof_ph = p.out.profile_photons;
        a.prof_bu = p.out.profile_bunches;
        a.inv_bin = 1.0 / p.params.depth_bin_gcm2;
        a.prof_bins = p.prof_bins;
    }
    const ckv_array* ar = p.arr;
    if (ar) {
        a.n_tel = ar->n_tel;
        a.tel = ar->d_tel;
        a.gx0 = ar->hit.gx0; a.gy0 = ar->hit.gy0; a.inv_cell = ar->hit.inv_cell;
        a.nx = ar->hit.nx; a.ny = ar->hit.ny; a.level_cells = ar->hit.level_cells;
        a.cell_list = ar->hit.d_cell_list;
        a.cell_ent = reinterpret_cast<const uint2*>(ar->hit.d_cell_ent);
        const ckv_reach& rg = ar->reach;
        if (rg.d_data) {
            a.reach_lev = reinterpret_cast<const ReachLevel*>(rg.d_data);
            a.reach_rec = reinterpret_cast<const uint2*>(rg.d_data + rg.rec_at);
            a.reach_list = reinterpret_cast<const uint2*>(rg.d_data + rg.list_at);
            a.reach_levels = rg.levels;
        }
    }
    a.bunch_size = p.params.bunch_size;
    a.k_ft = p.k_ft;
    a.inv_l1 = 1.0 / p.params.lambda_min_nm;
    a.dl = 1.0 / p.params.lambda_min_nm - 1.0 / p.params.lambda_max_nm;
    a.w_min = p.params.w_min;
    a.grazing_exact = p.params.grazing_exact;
    a.earth_r = p.params.earth_radius_m;
    a.r_obs = a.earth_r + a.h_obs;
    a.key0 = (uint32_t)p.params.seed;
    a.key1 = (uint32_t)(p.params.seed >> 32);
    a.tile_segs = p.tile_segs;
    a.report_segs = p.report_segs;
    a.heavy = p.heavy;
    a.heavy_step = p.heavy_step;
    a.cur_step = p.cursor.step;
    a.cur_shower = p.cursor.shower;
    a.ctrl = p.ctrl;
    a.claims = p.claims;
    a.tiles_before = p.tiles_before;
    a.blocks_before = p.blocks_before;
    a.shower_first = p.shower_first;
    a.tile_run_off = p.tile_run_off;
    a.tile_run_n = p.tile_run_n;
    a.tile_hits = p.tile_hits;
    a.runs = p.runs;
    a.run_cap = p.run_cap;
    a.block_hits = p.block_hits;
    a.block_sums = p.block_sums;
    a.shower_tel = p.shower_tel;
    a.stage_fill = p.stage_fill;
    a.stage = p.stage;
    a.stage_blocks = p.stage_slots / kStageBlock;
    a.max_tiles = p.max_tiles;
    a.max_row_blocks = p.max_row_blocks;
    a.records = p.out.records;
    a.ids = p.out.ids;
    a.capacity = p.out.capacity;
    a.tel_offsets = p.out.tel_offsets;
    a.result = p.out.result;
    return a;
}

// The azimuth sectors' bound constants (light_cone) for spheres of radius up to rmax
// with centres up to dmax from the origin.
void set_sectors(Args& a, const ckv_atmo* at, double rmax, double dmax)
{
    if (!(1.0 + at->psi_min >= 0.5)) return;
    a.sec_rmax = rmax;
    a.sec_dmax = dmax;
    a.sec_falls = at->psi_falls ? 1 : 0;
    a.sec_slope = at->psi_slope;
    a.sec_psi_max = at->psi_max;
    a.sec_psi_min = at->psi_min;
}

int check_launch(const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error(std::string(what) + ": " + hipGetErrorString(e));
        return CKV_ERR_HIP;
    }
    return CKV_OK;
}

}  // namespace

int emit_config(int precision, int n_tel, int prof_bins, const ckv_atmo* atmo, int tile_segs,
                int limit_segs, int max_waves, int* waves, size_t* lds_bytes, bool many_nodes_ok)
{
    const size_t srch = atmo->h_nodes.empty() ? 0 : search_bytes((int)atmo->n_nodes);
    const size_t cap = 160 * 1024;
    const size_t per = wave_bytes(precision, tile_segs, n_tel, prof_bins);
    auto beside_table = [&](bool part, int wv) {
        return ((table_bytes(precision, (int)atmo->n_nodes, part) + 15) & ~(size_t)15) + srch + tel_bytes(n_tel) +
                   (size_t)wv * limit_wave_bytes(precision, limit_segs, n_tel, prof_bins) <= cap;
    };
    if (beside_table(prof_bins > 0, 1) || (many_nodes_ok && beside_table(true, kMaxEmitWaves)))
        for (int wv = kMaxEmitWaves; wv >= 1; wv /= 2) {
            if (wv > max_waves) continue;
            const size_t tot = srch + tel_bytes(n_tel) + (size_t)wv * per;
            if (tot <= cap) {
                *waves = wv;
                *lds_bytes = tot;
                return CKV_OK;
            }
        }
    set_error("atmosphere table beyond the largest that the library takes");
    return CKV_ERR_TABLE;
}

namespace {

template <int PREC, int TS, int FEAT>
int launch_emit(const Args& a, int grid, int waves, size_t lds, hipStream_t st)
{
    allow_lds((const void*)emit_kernel<PREC, TS, FEAT>, 160 * 1024);
    emit_kernel<PREC, TS, FEAT><<<grid, waves * kWave, lds, st>>>(a);
    return check_launch("emit");
}

template <int PREC, int TS>
int launch_emit_feat(const Args& a, int grid, int waves, size_t lds, hipStream_t st)
{
    if (a.hnodes) {
        // node tables run alone (checked by the caller) and with 32-step tiles
        if (TS == 32) return launch_emit<PREC, 32, kFeatSearch>(a, grid, waves, lds, st);
        set_error("node tables need tile_segments 32");
        return CKV_ERR_ARG;
    }
    if (a.earth_r > 0.0) {
        // the curved atmosphere runs alone (checked by the caller) and with 32-step tiles
        if (TS == 32) return launch_emit<PREC, 32, kFeatCurved>(a, grid, waves, lds, st);
        set_error("the curved atmosphere needs tile_segments 32");
        return CKV_ERR_ARG;
    }
    const int feat = (a.prof_bins > 0 ? kFeatProfile : 0) | (a.grazing_exact ? kFeatExact : 0);
    switch (feat) {
        case 0: return launch_emit<PREC, TS, 0>(a, grid, waves, lds, st);
        case kFeatProfile: return launch_emit<PREC, TS, kFeatProfile>(a, grid, waves, lds, st);
        case kFeatExact: return launch_emit<PREC, TS, kFeatExact>(a, grid, waves, lds, st);
        default: return launch_emit<PREC, TS, kFeatProfile | kFeatExact>(a, grid, waves, lds, st);
    }
}

template <int PREC>
int launch_emit_ts(const Args& a, int ts, int grid, int waves, size_t lds, hipStream_t st)
{
    switch (ts) {
        case 2:
            if (a.grazing_exact && a.prof_bins == 0 && !a.hnodes && a.earth_r <= 0.0)
                return launch_emit<PREC, 2, kFeatExact>(a, grid, waves, lds, st);
            break;
        case 8: return launch_emit_feat<PREC, 8>(a, grid, waves, lds, st);
        case 16: return launch_emit_feat<PREC, 16>(a, grid, waves, lds, st);
        case 32: return launch_emit_feat<PREC, 32>(a, grid, waves, lds, st);
        case 64: return launch_emit_feat<PREC, 64>(a, grid, waves, lds, st);
    }
    set_error("tile_segments must be 8, 16, 32 or 64");
    return CKV_ERR_ARG;
}

}  // namespace

int launch_run(RunPlan& p)
{
    Args a = make_args(p);
    hipStream_t st = p.stream;
    int waves = 0;
    size_t lds = 0;
    int cap = p.emit_waves;
    if (p.params.grazing_exact || p.params.earth_radius_m > 0.0)
        cap = std::min(cap, emit_threads(p.params.precision, kFeatExact) / kWave);
    const bool many_nodes_ok = p.params.precision == 0 && p.params.waves_per_group == kMaxEmitWaves &&
                               p.prof_bins == 0 && !p.params.grazing_exact &&
                               p.params.earth_radius_m <= 0.0 && p.atmo->h_nodes.empty();
    if (int rc = emit_config(p.params.precision, a.n_tel, p.prof_bins, p.atmo, p.tile_segs, p.report_segs, cap,
                             &waves, &lds, many_nodes_ok))
        return rc;
    // as many tiles taken together as their crossing counters find room for
    const size_t fixed = (p.atmo->h_nodes.empty() ? 0 : search_bytes(a.n_nodes)) + tel_bytes(a.n_tel);
    int span = kWave / p.tile_segs;
    for (; span > 1; span >>= 1) {
        const size_t tot = fixed + (size_t)waves * wave_bytes(p.params.precision, p.tile_segs, a.n_tel * span,
                                                              p.prof_bins);
        if (tot <= 160 * 1024) {
            lds = tot;
            break;
        }
    }
    set_sectors(a, p.atmo, p.arr->rmax, p.arr->dmax);
    a.span_tiles = span;
    a.grid_waves = p.emit_grid * waves;
    // A run whose crossings pass its capacity writes the tiles before the first one that found
    // no room in the staging area, and the waves' first units are all worked on at once: if
    // they fill it, next to nothing is written and a resume gains as little.  4e5 steps over
    // 400 spheres, 9.5 crossings a step, wrote 346 records of a capacity of 300 000; in units
    // of 32 steps the 299 826 that whole tiles allow.  So the first round goes by these where
    // the area holds less than kDenseHits a step of units of 64; with more room it goes by 64
    // (32 there: 6e5 TeV steps 141 -> 147 us, 3e5 over the 400 spheres 301 -> 334).
    a.head_units = (int64_t)a.stage_blocks * kStageBlock < (int64_t)a.grid_waves * kWave * kDenseHits ? a.grid_waves : 0;
    // a block per wave of the launch, as far as the workspace holds them beside the claims'
    // (a grid of whole class rounds: the waves' first tiles are then 0 .. waves - 1, each
    // block with an owner that leaves its fill)
    a.static_blocks = p.emit_grid % kTileClasses != 0
                          ? 0
                          : (int32_t)std::min<int64_t>((int64_t)p.emit_grid * waves,
                                                       std::min(a.stage_blocks, p.run_cap / kRunBlock));
    const int64_t heavy_blocks = p.heavy ? (p.segs.n + kHeavySteps - 1) / kHeavySteps : 0;
    init_kernel<<<1 + (int)heavy_blocks, kHeavySteps, 0, st>>>(a);
    if (int rc = check_launch("init")) return rc;
    if (p.prof_bins > 0) {
        // the profile accumulates by atomics: clear it (a kernel, so the run stays capturable)
        const int64_t m = (int64_t)a.n_showers * p.prof_bins;
        zero_kernel<<<64, 256, 0, st>>>(a.prof_ph, m);
        zero_kernel<<<64, 256, 0, st>>>(reinterpret_cast<double*>(a.prof_bu), m);
        if (int rc = check_launch("zero")) return rc;
    }
    if (p.params.event_begin) (void)hipEventRecord((hipEvent_t)p.params.event_begin, st);
    int rc = p.params.precision == 0
                 ? launch_emit_ts<0>(a, p.tile_segs, p.emit_grid, waves, lds, st)
                 : launch_emit_ts<1>(a, p.tile_segs, p.emit_grid, waves, lds, st);
    if (rc) return rc;
    if (p.params.event_end) (void)hipEventRecord((hipEvent_t)p.params.event_end, st);
    const int fin_grid = 1024;
    const size_t tel_lds = (size_t)a.n_tel * sizeof(int32_t);
    if (a.n_tel <= kPrefixDenseTel) {
        // (256 threads for up to 128 telescopes: several workgroups share a compute unit)
        allow_lds((const void*)block_prefix_dense_kernel, kRowBlock * kPrefixDenseTel * sizeof(int32_t));
        block_prefix_dense_kernel<<<fin_grid, a.n_tel <= 128 ? 256 : 1024,
                                    (size_t)kRowBlock * a.n_tel * sizeof(int32_t), st>>>(a);
    } else {
        const size_t prefix_lds = (size_t)((a.n_tel + 1) & ~1) * sizeof(int32_t) +
                                  (size_t)kPrefixLdsRuns * sizeof(int64_t);
        block_prefix_kernel<<<fin_grid, kWave, prefix_lds, st>>>(a);
    }
    if (int rc2 = check_launch("block_prefix")) return rc2;
    if ((int64_t)a.n_showers * a.n_tel <= kFinishPairs && a.max_row_blocks <= kFinishBlocks) {
        finish_kernel<<<1, 1024, tel_lds, st>>>(a);
        if (int rc2 = check_launch("finish")) return rc2;
    } else {
        cutoff_kernel<<<1, 1024, tel_lds, st>>>(a);
        if (int rc2 = check_launch("cutoff")) return rc2;
        rowblock_scan_kernel<<<fin_grid, 256, 0, st>>>(a);
        if (int rc2 = check_launch("rowblock_scan")) return rc2;
        csr_kernel<<<1, 1024, 0, st>>>(a);
        if (int rc2 = check_launch("csr")) return rc2;
    }
    scatter_kernel<<<4096, 256, 0, st>>>(a);
    return check_launch("scatter");
}

int launch_soft(RunPlan& p, const SoftPlan& sp, int mode)
{
    Args a = make_args(p);
    a.tile_segs = a.report_segs = kSoftTS;          // the soft kernels walk 32-step tiles
    hipStream_t st = p.stream;
    const ckv_array* ar = p.arr;
    // the per-step cull's bound constants (screen_annulus) of the FP64 tile kernels
    {
        const ckv_atmo* at = p.atmo;
        if (ar->screen_rmax > 0.0 && 1.0 + at->psi_min >= 0.5) {
            a.cull_rmax = ar->screen_rmax;
            a.cull_x0 = (at->psi_max - at->psi_min) / (1.0 + at->psi_min);
            a.cull_b0 = (at->psi_falls ? 0.5 : 0.8) * a.cull_x0;
            a.cull_rho2 = at->psi_falls ? 1.0 : (1.0 + at->psi_max) / (1.0 + at->psi_min);
        }
    }
    SoftArgs s{};
    s.nb_frozen = sp.n_b_frozen;
    s.sigma = sp.sigma;
    s.gS = sp.gS;
    s.gA = sp.gA;
    s.S = sp.S;
    s.A = sp.A;
    s.g_psi = sp.g_psi;
    s.g_P = sp.g_P;
    s.gx0 = ar->soft.gx0;
    s.gy0 = ar->soft.gy0;
    s.inv_cell = ar->soft.inv_cell;
    s.nx = ar->soft.nx;
    s.ny = ar->soft.ny;
    s.level_cells = ar->soft.level_cells;
    s.cell_list = ar->soft.d_cell_list;
    s.cell_ent = reinterpret_cast<const uint2*>(ar->soft.d_cell_ent);
    s.ids = sp.ids;
    s.ids_cap = sp.ids_cap;
    s.ids_count = sp.ids_count;
    // listed adjoint: bins, spheres and the lowest node records in LDS (at most
    // 128 KB for CKV_MAX_TEL spheres); beyond the LDS the adjoint recomputes everything
    size_t lds_l = (size_t)6 * soft_bin_nodes(a.n_nodes) * sizeof(double) +
                   (size_t)a.n_tel * 4 * sizeof(double) +
                   (size_t)kNode64 * soft_node_lds(a.n_nodes) * sizeof(double);
    if (mode == 1 && lds_l > 160 * 1024) s.ids_count = nullptr;
    // the listed kernels keep the per-shower table in LDS when it fits beside the rest
    const size_t shr_b = (size_t)a.n_showers * sizeof(ShowerRec);
    s.skip_if_listed = s.ids_count ? 1 : 0;
    // forward with a list: the screening pass (mixed bunch kernel against spheres of
    // the cut radius plus a margin, frozen counts) lists the candidates, FP64
    // recomputes them (soft_cand_kernel); the FP64 tile forward runs only if the
    // list overflowed
    Args e = a;
    int e_waves = 0;
    size_t e_lds = 0;
    if (mode == 0 && s.ids_count) {
        e.tel = ar->d_tel_screen;
        e.gx0 = ar->soft.gx0;
        e.gy0 = ar->soft.gy0;
        e.inv_cell = ar->soft.inv_cell;
        e.nx = ar->soft.nx;
        e.ny = ar->soft.ny;
        e.level_cells = ar->soft.level_cells;
        e.cell_list = ar->soft.d_cell_list;
        e.cell_ent = reinterpret_cast<const uint2*>(ar->soft.d_cell_ent);
        set_sectors(e, p.atmo, ar->screen_rmax, ar->dmax);
        e.nb_frozen = sp.n_b_frozen;
        e.list_ids = sp.ids;
        e.list_cap = sp.ids_cap;
        e.list_count = sp.ids_count;
        const size_t tab = (table_bytes(1, e.n_nodes, true) + 15) & ~(size_t)15;
        const size_t per = wave_bytes(1, kSoftTS, 0, 0) + kScreenBuf * sizeof(uint64_t);
        if (tab + tel_bytes(e.n_tel) + limit_wave_bytes(1, kSoftTS, e.n_tel, 0) + kLimitScreenBytes <= 160 * 1024)
            for (int wv = kMaxEmitWaves; wv >= 1 && !e_waves; wv /= 2)
                if (tel_bytes(e.n_tel) + (size_t)wv * per <= 160 * 1024) {
                    e_waves = wv;
                    e_lds = tel_bytes(e.n_tel) + (size_t)wv * per;
                }
        if (!e_waves || e.n_nodes - 1 < 2) {
            set_error("soft response: atmosphere table beyond the largest that the screening pass takes");
            return CKV_ERR_TABLE;
        }
    }
    // as many waves as the kernel's launch bounds allow and the LDS holds
    const int wmax = soft_max_waves(mode);
    int waves = p.emit_waves > 0 && p.emit_waves < wmax ? p.emit_waves : wmax;
    while (waves > 1 && soft_lds_bytes(mode, a.n_nodes, a.n_tel, waves) > 160 * 1024) waves >>= 1;
    const size_t lds = soft_lds_bytes(mode, a.n_nodes, a.n_tel, waves);
    if (lds > 160 * 1024) {
        set_error("soft response: telescope count too large for LDS");
        return CKV_ERR_TABLE;
    }
    init_kernel<<<1, 1024, 0, st>>>(a);
    if (int rc = check_launch("init")) return rc;
    const int64_t nst = (int64_t)a.n_showers * a.n_tel;
    if (mode == 0) {
        zero_kernel<<<64, 256, 0, st>>>(s.S, nst);
        zero_kernel<<<64, 256, 0, st>>>(s.A, nst);
        // the list count starts at zero (all-zero bits: 0.0 is integer 0)
        if (s.ids_count) zero_kernel<<<1, 64, 0, st>>>(reinterpret_cast<double*>(s.ids_count), 1);
    } else {
        zero_kernel<<<64, 256, 0, st>>>(s.g_psi, a.n_nodes);
        zero_kernel<<<64, 256, 0, st>>>(s.g_P, (int64_t)5 * a.n_nodes);
    }
    if (int rc = check_launch("zero")) return rc;
    if (p.params.event_begin) (void)hipEventRecord((hipEvent_t)p.params.event_begin, st);
    if (mode == 0) {
        allow_lds((const void*)soft_kernel<0>, 160 * 1024);
        if (s.ids_count) {
            allow_lds((const void*)emit_kernel<1, kSoftTS, kFeatScreen>, 160 * 1024);
            e.span_tiles = kWave / kSoftTS;
            e.grid_waves = p.emit_grid * e_waves;
            emit_kernel<1, kSoftTS, kFeatScreen><<<p.emit_grid, e_waves * kWave, e_lds, st>>>(e);
            if (int rc = check_launch("screen")) return rc;
            size_t lds_c = (size_t)a.n_tel * 4 * sizeof(double) +
                           (size_t)kNode64 * soft_node_lds(a.n_nodes) * sizeof(double);
            const size_t acc_b = (size_t)2 * a.n_showers * a.n_tel * sizeof(double);
            s.cand_lds_acc = lds_c + acc_b <= 160 * 1024 ? 1 : 0;
            if (s.cand_lds_acc) lds_c += acc_b;
            s.shower_lds = lds_c + shr_b <= 160 * 1024 ? 1 : 0;
            if (s.shower_lds) lds_c += shr_b;
            allow_lds((const void*)soft_cand_kernel, 160 * 1024);
            const int groups = lds_c <= 80 * 1024 ? 2 : 1;
            soft_cand_kernel<<<groups * p.emit_grid, kSoftCandThreads / groups, lds_c, st>>>(a, s);
            if (int rc = check_launch("soft candidates")) return rc;
        }
        soft_kernel<0><<<p.emit_grid, waves * kWave, lds, st>>>(a, s);
    } else {
        allow_lds((const void*)soft_kernel<1>, 160 * 1024);
        soft_kernel<1><<<p.emit_grid, waves * kWave, lds, st>>>(a, s);
        if (s.ids_count) {
            if (int rc = check_launch("soft")) return rc;
            s.shower_lds = lds_l + shr_b <= 160 * 1024 ? 1 : 0;
            if (s.shower_lds) lds_l += shr_b;
            allow_lds((const void*)soft_list_kernel, 160 * 1024);
            soft_list_kernel<<<2 * p.emit_grid, kSoftListThreads, lds_l, st>>>(a, s);
        }
    }
    if (int rc = check_launch("soft")) return rc;
    if (p.params.event_end) (void)hipEventRecord((hipEvent_t)p.params.event_end, st);
    return CKV_OK;
}

int launch_count(const ckv_segments* segs, const ckv_params* prm, const ckv_atmo* atmo, double k_ft,
                 int64_t* n_b, hipStream_t stream)
{
    RunPlan p{};
    p.segs = *segs;
    p.params = *prm;
    p.atmo = atmo;
    p.arr = nullptr;
    p.k_ft = k_ft;
    p.tile_segs = p.report_segs = 1;
    Args a = make_args(p);
    if (segs->n == 0) return CKV_OK;
    const int64_t blocks = std::min<int64_t>((segs->n + 255) / 256, 65536);
    count_kernel<<<(unsigned)blocks, 256, 0, stream>>>(a, n_b);
    return check_launch("count");
}

#endif  // CKV_SLOWPATH

}  // namespace ckv
