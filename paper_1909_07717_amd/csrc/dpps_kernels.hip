// dpps_kernels.hip -- HIP kernels (gfx950) of the SBIP-DPPS passing-point search.
//
// Work decomposition
//   One workgroup per tile of candidate points (persistent workgroups pull
//   tiles from an atomic counter, or one workgroup per tile).  A wave
//   evaluates two neighbouring candidate points at a time, one per half, with
//   the 32 lanes of a half spread over the K path samples (K/32 per lane):
//
//   1. robot stage   for every interceptor and every sample, the robot's
//                    arrival time (straight line, bounded acceleration and
//                    speed, at rest on the sample); the minimum over teammates
//                    and over opponents is kept per sample.  Sample positions
//                    depend on the point only, so this stage is shared by all
//                    pass variants (Sec. 4.2 traverses speeds for fixed paths).
//   2. critical speed per sample, the kick speed at which the ball reaches the
//                    sample exactly when the first teammate (opponent) does;
//                    a slower kick is intercepted there, a faster one is not
//                    (the ball model of Sec. 4.1 is monotone in the kick speed).
//   3. first crossing per variant (SBIP, Sec. 4.2): the lowest sample whose
//                    critical speed is at least v0; the running maximum of the
//                    critical speeds over the samples is non-decreasing, so
//                    every variant lane finds its crossing by binary search in
//                    the wave's LDS row of running maxima.
//   4. finish        lanes become variants: ball time at the crossing sample
//                    (float64), margin, feasibility and the Eq. (3) score
//                    (Sec. 4.3); results are staged in LDS and written as whole
//                    rows per tile.  Each tile records its best pass; a small
//                    finalize kernel reduces the records of each frame.
//
// The open goal angle (Sec. 4.3/4.4) is computed with lanes = opponents.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dpps_internal.h"

namespace dpps {

#define MAX_ROB (2 * DPPS_MAX_SIDE)
#define MAX_VAR DPPS_MAX_VARIANTS
#define MAX_TILE 64
#define MAX_WAVES 8
#define MAX_K 256
#define PM_ROWS 4  // running-maximum rows per wave: flat team / opp, chip team / opp

// Running-maximum floats of one half of a search wave: a team and an opponent
// row of K, and 32 floats so that the halves' rows start in different banks.
constexpr int half_rows(int K) { return 2 * K + 32; }

// Dynamic LDS of the ray kernel: PM_ROWS rows of K floats per wave.  (Both
// kernels' dynamic LDS is read as 16-byte words: it is declared on 16 bytes,
// which pads the static LDS before it.)
static size_t pm_bytes(int K, int waves) { return (size_t)waves * PM_ROWS * K * sizeof(float); }

// The kernel's arguments, read anew from the kernarg segment: the laundered
// pointer keeps the compiler from holding every constant in scalar registers
// over a whole tile loop, where they do not fit and spill to vector lanes
// (two VALU instructions per spilled use); a scalar load from the cache costs
// no VALU issue.
template <class Args>
__device__ __forceinline__ const Args &fresh_args()
{
    typedef const __attribute__((address_space(4))) Args *KernArgs;
    KernArgs k = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *(const Args *)k;
}

struct VarConst {
    double va1, a1, va2, a2, soff2, toff2, split, D, sf_reach;
};

struct StageLDS {
    float4 rob[MAX_ROB];      // (x, y, vx, vy): team interceptors, then opponents
    float v0[MAX_VAR];
    int32_t type[MAX_VAR];
    int32_t vidx[MAX_VAR];    // the caller's index of each staged variant
    VarConst vc[MAX_VAR];
    int32_t n_tm, n_op, n_var, has_flat, has_chip, frame;
    int32_t vel_ok;           // every robot's speed is at most vmax
    float bx, by;
    float lim[4];             // arrival limit per quarter of a path, over sqrt(length)
};

// A wave's path-frame block: MAX_ROB entries, then 64 words of bound keys.
#define PR_ENTRIES (MAX_ROB + 16)
#define SPLIT_ROB 16  // most robots whose bounds are kept per quarter of the path

// Dynamic LDS of the search kernel, sized by the launch: each wave's
// running-maximum rows and path-frame blocks of two points, then the tile's staged
// score and mask maps (a row of tile_points per variant of the frame with the
// most, so that few variants leave room for more workgroups).
static size_t search_lds_bytes(int K, int waves, int tile_points, int max_variants)
{
    const size_t maps = (size_t)max_variants * tile_points * (sizeof(float) + 1);
    return (size_t)waves * 2 * (half_rows(K) * sizeof(float) + PR_ENTRIES * sizeof(float4)) +
           ((maps + 15) & ~(size_t)15);
}
__device__ __forceinline__ uint32_t *bound_keys(float4 *pr) { return (uint32_t *)(pr + MAX_ROB); }
__device__ __forceinline__ const uint32_t *bound_keys(const float4 *pr)
{
    return (const uint32_t *)(pr + MAX_ROB);
}

struct OutLDS {
    TileRec wbest[MAX_WAVES];  // each wave's best pass
};

__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float hsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float hrcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float med3(float x, float lo, float hi)
{
    return __builtin_amdgcn_fmed3f(x, lo, hi);
}
__device__ __forceinline__ int lane_id() { return __lane_id(); }
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float unif(float x)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ float readlane_f(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ int readlane_i(int x, int l) { return __builtin_amdgcn_readlane(x, l); }

// Ball constants of one variant (float64): phase split, speeds and
// decelerations, offsets, stopping distance D and the minimum reachable
// distance (the carry of a chip).
__device__ VarConst var_const(const BallParams64 &B, int type, float v0f)
{
    VarConst c;
    double v0 = (double)v0f;
    if (type == DPPS_CHIP) {
        double vh = v0 * B.cos_th, vz = v0 * B.sin_th;
        double tf = 2.0 * vz / B.g;
        double sf = vh * tf;
        c.va1 = vh; c.a1 = B.a_r;             // unused: split < 0
        c.va2 = vh; c.a2 = B.a_r; c.soff2 = sf; c.toff2 = tf;
        c.split = -1.0;
        c.D = sf + vh * vh / (2.0 * B.a_r);
        c.sf_reach = sf;
    } else {
        double v1 = B.ratio * v0;
        double t1 = (v0 - v1) / B.a_s;
        double d1 = (v0 * v0 - v1 * v1) / (2.0 * B.a_s);
        c.va1 = v0; c.a1 = B.a_s;
        c.va2 = v1; c.a2 = B.a_r; c.soff2 = d1; c.toff2 = t1;
        c.split = d1;
        c.D = d1 + v1 * v1 / (2.0 * B.a_r);
        c.sf_reach = 0.0;
    }
    return c;
}

// Stage frame f (its record F) into LDS: interceptors (passer dropped), the
// per-variant ball constants in float64, the counts and flags.  Done by the
// block's first wave with one round of loads: the lanes are robots and
// variants, the flags ballots, the variants' ranks lane reads (the block waits
// for this, so its length is latency; loops of dependent loads on one thread
// cost several microseconds).
__device__ void stage_frame(const DevParams &P, const FrameDev &F, const dpps_robot *robots,
                            const dpps_variant *variants, int f, StageLDS &S)
{
    const int tid = threadIdx.x;
    if (tid >= 64) return;
    const int nrob = F.n_team + F.n_opp, nv = F.n_variants;
    dpps_robot r = {0.0f, 0.0f, 0.0f, 0.0f};
    dpps_variant v = {-1, 0.0f};
    if (tid < nrob) r = robots[F.robot_off + tid];
    if (tid < nv) v = variants[F.variant_off + tid];
    if (tid < nrob && tid != F.passer)
        S.rob[tid < F.passer ? tid : tid - 1] = make_float4(r.x, r.y, r.vx, r.vy);
    const bool over = tid < nrob && !(fmaf(r.vx, r.vx, r.vy * r.vy) <= P.V * P.V);
    const bool all_slow = __ballot(over) == 0ull;
    const bool hf = __ballot(v.type == DPPS_FLAT) != 0ull;
    const bool hc = __ballot(v.type == DPPS_CHIP) != 0ull;
    // staged in order of kick type, then speed (stable): within a type the
    // first crossing never moves earlier as the speed grows
    int rank = 0;
    for (int j = 0; j < nv; ++j) {
        const int tj = readlane_i(v.type, j);
        const float vj = readlane_f(v.v0, j);
        rank += tj < v.type || (tj == v.type && (vj < v.v0 || (vj == v.v0 && j < tid)));
    }
    if (tid < nv) {
        S.v0[rank] = v.v0;
        S.type[rank] = v.type;
        S.vidx[rank] = tid;
        S.vc[rank] = var_const(P.bp, v.type, v.v0);
    }
    if (tid < 4) S.lim[tid] = fmaxf(hf ? P.f_lim[tid] : 0.0f, hc ? P.c_lim[tid] : 0.0f);
    if (tid == 0) {
        S.n_tm = F.n_team - 1;
        S.n_op = F.n_opp;
        S.n_var = nv;
        S.has_flat = hf;
        S.has_chip = hc;
        S.vel_ok = all_slow;
        S.frame = f;
        S.bx = F.ball_x;
        S.by = F.ball_y;
    }
}

// Inclusive prefix maximum over the 64 lanes of a wave (lane l gets the
// maximum of lanes 0..l): four DPP row shifts give it within each row of 16
// lanes (lanes without a source see the identity), then two DPP row
// broadcasts carry lane 15 into row 1 and row 3, and lane 31 into rows 2
// and 3.  The maxima of critical speeds and arrival times are taken on the
// bit patterns: those are non-negative floats or +inf, which order as their
// bits read as signed integers, and an integer max needs no NaN quieting, so
// each DPP lane shift fuses into its max (identity INT_MIN, the bits of
// -0.0).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_imax(int v)
{
    const int u = __builtin_amdgcn_update_dpp(INT_MIN, v, CTRL, ROW_MASK, 0xf, false);
    return max(v, u);
}

// half_prefix_imax stops before the last step: the prefix maximum within each
// half of 32 lanes.
__device__ __forceinline__ int half_prefix_imax(int v)
{
    v = dpp_imax<0x111, 0xf>(v);  // row_shr:1
    v = dpp_imax<0x112, 0xf>(v);  // row_shr:2
    v = dpp_imax<0x114, 0xf>(v);  // row_shr:4
    v = dpp_imax<0x118, 0xf>(v);  // row_shr:8
    return dpp_imax<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
}

__device__ __forceinline__ int wave_prefix_imax(int v)
{
    return dpp_imax<0x143, 0xc>(half_prefix_imax(v));  // row_bcast:31 into rows 2 and 3
}

// Lane l gets lane l - 1's value, lane 0 gets INT_MIN (DPP wave_shr:1).
__device__ __forceinline__ int wave_shift_up_i(int v)
{
    return __builtin_amdgcn_update_dpp(INT_MIN, v, 0x138, 0xf, 0xf, false);
}

// Order this wave's accesses to its own LDS row.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The constants of the robot model, by value: read once before a robot loop.
struct RobotK {
    float RA, Vh, V2, inv2V, halfV;
    __device__ __forceinline__ explicit RobotK(const DevParams &P)
        : RA(P.RA), Vh(P.Vh), V2(P.V2), inv2V(P.inv2V), halfV(P.halfV)
    {
    }
};

// Arrival time of one robot at one sample.  Lengths are scaled by amax (a
// distance d becomes A d) and speeds by 1/sqrt(2); with that scaling the
// time-optimal straight-line motion that ends at rest takes
//   A T = R(D') + sigma sqrt(2) u',
//   R(D) = 2 sqrt(D) if D <= V^2, else D / V + V (cruising at vmax = V),
// where u' is the (scaled) speed toward the point, s = u'^2 the scaled
// stopping distance, delta the scaled distance still to cover, and either
// (overshoot: the robot cannot stop before the point, or is already there at
// rest) D' = s - delta, sigma = +1, or D' = s + delta, sigma = -1 (moving
// toward) / +1 (moving away).  The function returns A T / 2.
//
// The sample and the robot are given in the path frame of the candidate
// point: the sample lies at distance fq * LA along the path from the ball;
// r = (t, q^2, w.e, q w.n) holds the robot's own coordinate along the path
// (t) and across it (q), and its scaled velocity w projected on the path
// direction e and on the normal n.  The offset from the robot to the sample
// is then h e + q n with h = fq LA - t, its length sqrt(h^2 + q^2), and the
// speed toward the sample (h w.e + q w.n) / length.  With CLAMP that speed is
// limited to vmax; without it the caller knows that no robot is faster.
template <bool CLAMP>
__device__ __forceinline__ float robot_time_h(float4 r, float fq, float LA, const RobotK &P)
{
    const float h = fmaf(fq, LA, -r.x);
    const float r2 = fmaf(h, h, r.y);
    const float inv = rsq(r2);
    const float del = fmaxf(fmaf(r2, inv, -P.RA), 0.0f);
    float u = fmaf(h, r.z, r.w) * inv;
    if (CLAMP) u = med3(u, -P.Vh, P.Vh);
    const float ss = u * fabsf(u);  // its magnitude is u^2 (the add's abs modifier)
    const bool over = ss >= del;
    const float Dp = fabsf(ss) + (over ? -del : del);
    const float sg = over ? u : -u;
    const float rh = Dp > P.V2 ? fmaf(Dp, P.inv2V, P.halfV) : hsqrt(Dp);
    return fmaf(sg, 0.70710678118654752f, rh);
}

// How a wave's lanes hold a path's samples: HALF_WAVE, lanes 0-31 one
// point's and lanes 32-63 another's; FULL_WAVE, all 64 lanes one path's.
enum { HALF_WAVE, FULL_WAVE };

// Greatest of the lanes' values over groups of 8 lanes (8: row_half_mirror
// last) or rows of 16, on every lane of the group.
template <int CTRL>
__device__ __forceinline__ int dpp_swap_imax(int v)
{
    return max(v, __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ int group8_imax(int v)
{
    return dpp_swap_imax<0x141>(dpp_swap_imax<0x4E>(dpp_swap_imax<0xB1>(v)));
}
__device__ __forceinline__ int row_mirror_i(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true);
}

// Which robots of the path's sorted order (bit = rank) may still lower an
// arrival minimum T that matters, those not yet taken among them.  With the
// bounds kept per quarter of the path (n_rob <= SPLIT_ROB) robot r is needed
// in a quarter when its bound there is below both the latest of the minima
// over the quarter's samples and the quarter's limit `lim` (in the same units;
// lane's own quarter and, HALF_WAVE, the other one of its row).  With HALF_WAVE
// the result covers both points.  Otherwise one bound per robot is compared
// with the latest minimum of the whole path.  Arrival times are
// non-negative or +inf, bounds non-negative: all compare as their bits.
template <int KPL, int MODE>
__device__ __forceinline__ uint32_t robots_needed(const float4 *pr, bool split, float lim,
                                                  float lim_other, const float (&T)[KPL])
{
    const int l = lane_id();
    int m = __float_as_int(T[0]);
#pragma unroll
    for (int q = 1; q < KPL; ++q) m = max(m, __float_as_int(T[q]));
    bool below;
    if (split) {
        if (MODE == HALF_WAVE) {
            m = group8_imax(m);
            const int mo = min(row_mirror_i(m), __float_as_int(lim_other));
            m = min(m, __float_as_int(lim));
            const int b = (l & 31) >> 3, r = l & 15;
            below = (int)bound_keys(pr)[b * 16 + r] < m || (int)bound_keys(pr)[(b ^ 1) * 16 + r] < mo;
        } else {
            m = dpp_swap_imax<0x140>(group8_imax(m));
            below = (int)bound_keys(pr)[l] < m;
        }
        const unsigned long long b = __ballot(below);
        const uint32_t x = (uint32_t)b | (uint32_t)(b >> 32);
        return (x | (x >> 16)) & 0xFFFFu;
    }
    if (MODE == HALF_WAVE) {
        m = half_prefix_imax(m);
        const int m0 = __builtin_amdgcn_readlane(m, 31), m1 = __builtin_amdgcn_readlane(m, 63);
        m = l < 32 ? m0 : m1;
    } else {
        m = __builtin_amdgcn_readlane(wave_prefix_imax(m), 63);
    }
    const unsigned long long b = __ballot((int)bound_keys(pr)[l & 31] < m);
    return (uint32_t)b | (uint32_t)(b >> 32);
}

// Earliest arrival (A T / 2) of robots [j0, j0 + n) of the path frame, in
// their sorted order, at each of the lane's samples: the first two, then,
// pair by pair, those that robots_needed keeps.  A robot left out has, in
// every quarter, a bound that is not below the latest minimum there, so it
// lowers no sample's minimum; or not below the quarter's limit.  The limit is
// 1.03 times the ball's time to the quarter's end for the slowest kick that
// gets to the end of the path at all, of the frame's kick types: a robot that
// is no earlier meets only slower kicks there, which no reachable variant
// is, so minima at or past the limit may stay later than they would be and
// every reachable variant's first crossing is still the same (critical speeds
// at the limit are below that slowest kick by 2^-12 at least, or there is no
// limit; in the last quarter it is past its stop, where the critical speed does
// not depend on the arrival any more).  Pass +inf where the minima themselves
// are used.
template <int KPL, bool CLAMP, int MODE>
__device__ __forceinline__ void robot_stage(const float4 *pr, const RobotK &P, int j0, int n,
                                            bool split, float lim, float lim_other,
                                            const float (&fs)[KPL], float LA, float (&T)[KPL])
{
    uint32_t todo = ((1u << n) - 1u) << j0;  // n <= 16
    // one copy of each body (the kernel's code stays small enough for the
    // instruction cache)
    while (todo) {
        const float4 ra = pr[__builtin_ctz(todo)];
        todo &= todo - 1;
        if (!todo) {
#pragma unroll
            for (int q = 0; q < KPL; ++q)
                T[q] = fminf(T[q], robot_time_h<CLAMP>(ra, fs[q], LA, P));
            break;
        }
        const float4 rb = pr[__builtin_ctz(todo)];
        todo &= todo - 1;
#pragma unroll
        for (int q = 0; q < KPL; ++q)
            T[q] = fminf(T[q], fminf(robot_time_h<CLAMP>(ra, fs[q], LA, P),
                                     robot_time_h<CLAMP>(rb, fs[q], LA, P)));
        if (todo) todo &= robots_needed<KPL, MODE>(pr, split, lim, lim_other, T);
    }
}

// A lower bound on a robot's arrival time (robot stage units) at every sample
// of the segment [s0, s1] of the path along e.  With delta = max(dist - RA,
// 0) for its distance to the segment, and u' the speed toward a sample
// (clamped to +-vmax/sqrt 2 as the stage clamps it), the time -u'/sqrt 2 +
// R(u'^2 + delta) falls as u' grows up to sqrt(delta) and grows with delta,
// so with U the largest u' toward any sample: U < sqrt(delta) bounds it by
// -U/sqrt 2 + R(U^2 + delta); otherwise, whatever the velocity, by
// sqrt(delta / 2) for delta <= vmax^2 / 2 and else delta / (2 vmax) + vmax /
// 4.  U: the scaled velocity w' = (w.e, w.n) against the directions (h, q) to
// the samples, h in [s0 - t, s1 - t]: |w'| when w' lies among them, else the
// larger end.  Less 2^-12 for the rounding of both computations.
__device__ __forceinline__ float arrival_bound(const RobotK &P, double t, double q, float wef,
                                               float wnf, double s0, double s1)
{
    const double tc = fmax(fmax(s0 - t, t - s1), 0.0);
    const float dseg = hsqrt((float)(q * q + tc * tc));
    const float del = fmaxf(dseg - P.RA, 0.0f);
    const float qf = (float)q, h0 = (float)(s0 - t), h1 = (float)(s1 - t);
    const float sq = qf < 0.0f ? -1.0f : 1.0f;
    const bool among = ((h1 * wnf - qf * wef) * sq >= 0.0f) & ((wef * qf - wnf * h0) * sq >= 0.0f);
    const float u0 = fmaf(h0, wef, qf * wnf) * rsq(fmaxf(fmaf(h0, h0, qf * qf), 1e-30f));
    const float u1 = fmaf(h1, wef, qf * wnf) * rsq(fmaxf(fmaf(h1, h1, qf * qf), 1e-30f));
    const float ww = hsqrt(fmaf(wef, wef, wnf * wnf));
    const float U = med3(among ? ww : fmaxf(u0, u1), -P.Vh, P.Vh);
    // every form, then selects (the lanes are robots: branches would split)
    const float D = fmaf(U, U, del);
    const float rd = hsqrt(D), rh = hsqrt(0.5f * del);
    const float fast = fmaf(D, P.inv2V, P.halfV), far = fmaf(del, P.inv2V, 0.5f * P.halfV);
    const float lb0 = fmaf(-0.70710678118654752f, U, D > P.V2 ? fast : rd);
    const float lb1 = del <= 0.5f * P.V2 ? rh : far;
    return (U * fabsf(U) < del ? lb0 : lb1) * (1.0f - 1.0f / 4096.0f);
}

// A robot in the frame of a path from (bx, by) along (ux, uy), in units of
// its acceleration: (along, across^2, velocity along, across x velocity
// across); t, q and wn are the unrounded along and across and the velocity
// across.
__device__ __forceinline__ float4 robot_frame(const float4 &r, double A, double bx, double by,
                                              double ux, double uy, double &t, double &q,
                                              double &wn)
{
    const double ax = bx - (double)r.x, ay = by - (double)r.y;
    t = -(ax * ux + ay * uy) * A;
    q = (ay * ux - ax * uy) * A;
    const double we = ((double)r.z * ux + (double)r.w * uy) * 0.70710678118654752;
    wn = ((double)r.w * ux - (double)r.z * uy) * 0.70710678118654752;
    return make_float4((float)t, (float)(q * q + 1e-30), (float)we, (float)(q * wn));
}

// Path frame of a ball path along the unit direction e = (ux, uy) for the
// staged robots, in float64 and then rounded once: for robot j with offset a
// = ball - x_j and normal n = (-e_y, e_x): t = -a.e and q = a.n (scaled by
// amax), w = velocity / sqrt(2), and its entry (t, q^2, w.e, q w.n).  The
// entries are written in the order of the robots' arrival bounds, each side's
// by ascending bound, the team's first.  l is the lane's index among the
// lanes that share the path (32 with HALF_WAVE, else 64).  With `split` (at
// most SPLIT_ROB robots) every row of 16 of those lanes takes all robots and
// bounds them over its own part of the path: with FULL_WAVE row b the
// b-th quarter, with HALF_WAVE row b the quarters 2b and 2b + 1; the bounds
// go to the key block as [quarter][rank], and the order is by the least.
// Otherwise lane l takes robot l and bounds it over the whole path; keys by
// rank.  Every lane of the wave takes part (the syncs are wave-wide).
template <int MODE>
__device__ __forceinline__ void path_frame_dir(const StageLDS &S, const DevParams &P, float4 *pr,
                                               int n_rob, int n_tm, double LA, double ux,
                                               double uy, double bx, double by, int l)
{
    const bool split = n_rob <= SPLIT_ROB;
    const int r0 = split ? l & 15 : l, row = l >> 4;
    const RobotK rk(P);
    uint32_t *const pk = bound_keys(pr);
    float4 fr = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    uint32_t key = 0xFFFFFFFFu;
    float lb0 = INFINITY, lb1 = INFINITY;  // the row's bounds (split)
    if (r0 < n_rob) {
        const float4 r = S.rob[r0];
        double t, q, wn;
        fr = robot_frame(r, (double)P.A, bx, by, ux, uy, t, q, wn);
        double s0 = 0.0, s1 = LA;
        if (split) {
            s0 = 0.25 * LA * (double)(MODE == HALF_WAVE ? 2 * row : row);
            s1 = s0 + 0.25 * LA;
        }
        lb0 = arrival_bound(rk, t, q, fr.z, (float)wn, s0, s1);
        if (MODE == HALF_WAVE && split)
            lb1 = arrival_bound(rk, t, q, fr.z, (float)wn, s1, s1 + 0.25 * LA);
    }
    if (split) {
        // the robot's least bound over the rows
        float lb = fminf(lb0, lb1);
        lb = fminf(lb, __shfl_xor(lb, 16, 64));
        if (MODE == FULL_WAVE) lb = fminf(lb, __shfl_xor(lb, 32, 64));
        if (r0 < n_rob) key = __float_as_uint(lb);
    } else if (r0 < n_rob) {
        key = __float_as_uint(lb0);
    }
    // Rank by key: the bound's bits, with the robot in the low bits and the
    // side in the top bit
    if (r0 < n_rob)
        key = (key & ~(uint32_t)(MAX_ROB - 1)) | (uint32_t)r0 | (r0 >= n_tm ? 0x80000000u : 0u);
    if (split ? row == 0 : l < MAX_ROB) pk[r0] = key;
    wave_lds_sync();
    int rank = 0;
    for (int j = 0; j < n_rob; j += 4) {
        const uint4 k4 = *(const uint4 *)(pk + j);
        rank += (k4.x < key) + (k4.y < key) + (k4.z < key) + (k4.w < key);
    }
    if (r0 < n_rob && (!split || row == 0)) pr[rank] = fr;
    wave_lds_sync();  // the ranks are formed: the key block takes the bounds by rank
    if (r0 < n_rob) {
        if (!split) {
            pk[rank] = __float_as_uint(lb0) & ~(uint32_t)(MAX_ROB - 1);
        } else if (MODE == HALF_WAVE) {
            pk[(2 * row) * 16 + rank] = __float_as_uint(lb0);
            pk[(2 * row + 1) * 16 + rank] = __float_as_uint(lb1);
        } else {
            pk[row * 16 + rank] = __float_as_uint(lb0);
        }
    }
    // the row is written and read by this wave only
    wave_lds_sync();
}

// The same for the path from the ball to candidate point c: e = (c - ball) /
// |c - ball| (a point on the ball gets e = (1, 0); it is never reachable).
// 1 / |c - ball| is the hardware estimate refined by one Newton step
// (relative error far below the float32 rounding that follows).  Returns
// |c - ball| A.
__device__ __forceinline__ float path_frame(const StageLDS &S, const DevParams &P, float4 *pr,
                                            int n_rob, int n_tm, double cx64, double cy64,
                                            double bx, double by, int l)
{
    const double ex = cx64 - bx, ey = cy64 - by;
    const double L2 = ex * ex + ey * ey;
    double iL = __builtin_amdgcn_rsq(L2);
    iL = iL * (1.5 - 0.5 * L2 * iL * iL);
    const bool pos = L2 > 0.0;
    const double L = pos ? L2 * iL : 0.0;
    const double ux = pos ? ex * iL : 1.0, uy = pos ? ey * iL : 0.0;
    path_frame_dir<HALF_WAVE>(S, P, pr, n_rob, n_tm, L * (double)P.A, ux, uy, bx, by, l);
    return (float)(L * (double)P.A);
}

// First crossings by running maxima.  The first crossing of a variant on
// one side is the lowest sample k whose critical speed vc_k is at least the
// kick speed v0 (K: none).  The running maximum of vc over the samples is
// non-decreasing, so that crossing is the number of samples whose running
// maximum is still below v0.  The wave writes each side's running maxima to a
// row of its LDS block (samples are lane-major: lane l holds k = l KPL + q),
// then every variant lane counts by binary search in its kick type's two rows,
// the team's and the opponents' searches interleaved.  The decisions are the
// comparisons v0 <= vc_k of a scan over k.
// With HALF each half of the wave holds a point's samples and `row` is the
// lane's own half's row.
template <int KPL, bool HALF>
__device__ __forceinline__ void store_running_max(const float (&vc)[KPL], float *row)
{
    const int l = HALF ? lane_id() & 31 : lane_id();
    int run[KPL];
    run[0] = __float_as_int(vc[0]);
#pragma unroll
    for (int q = 1; q < KPL; ++q) run[q] = max(run[q - 1], __float_as_int(vc[q]));
    int excl = wave_shift_up_i(HALF ? half_prefix_imax(run[KPL - 1]) : wave_prefix_imax(run[KPL - 1]));
    if (HALF) excl = l == 0 ? INT_MIN : excl;
#pragma unroll
    for (int q = 0; q < KPL; ++q) row[l * KPL + q] = __int_as_float(max(excl, run[q]));
}

template <int K>
__device__ __forceinline__ void count_below(const float *rt, const float *ro, float v0, int &kt,
                                            int &ko)
{
    // a search over 2^n >= K entries, those past K read as the last one (the
    // rows are non-decreasing, so the count only exceeds K when every entry
    // is below v0, and is then clamped); no branches, both sides interleaved.
    // The search moves row pointers (the step's offset goes into the LDS
    // read's immediate); when K is a power of two no read can pass the end.
    constexpr int S0 = K > 128 ? 128 : K / 2;  // half of 2^n
    constexpr bool POW2 = (K & (K - 1)) == 0;
    const float *pt = rt, *po = ro;
    const float *const et = rt + (K - 1), *const eo = ro + (K - 1);
#pragma unroll
    for (int st = S0; st > 0; st >>= 1) {
        const float mt = POW2 ? pt[st - 1] : *min(pt + (st - 1), et);
        const float mo = POW2 ? po[st - 1] : *min(po + (st - 1), eo);
        pt += mt < v0 ? st : 0;
        po += mo < v0 ? st : 0;
    }
    const float mt = POW2 ? *pt : *min(pt, et);
    const float mo = POW2 ? *po : *min(po, eo);
    const int lt = (int)(pt - rt) + (mt < v0 ? 1 : 0);
    const int lo = (int)(po - ro) + (mo < v0 ? 1 : 0);
    kt = POW2 ? lt : min(lt, K);
    ko = POW2 ? lo : min(lo, K);
}

// Kick speed at which the ball covers distance s in exactly time T (the
// ball's distance at a fixed time grows with the kick speed).  Regimes at
// time T: stopped (s <= cA T^2), decelerating at the slower rate
// (quadratic in v0), or still in the fast phase (s >= cB T^2: sliding for a
// flat kick, in the air for a chip).  Stopped, the ball has covered its
// whole range cD v0^2, so v0 = sqrt(s / cD), which depends on the sample
// only.  In the fast phase a flat kick slides, v0 = (s + hfast T^2) / T, and
// a chip flies, v0 = s / (pfast T).  The slow root 2Q / (beta T +
// sqrt(4 alpha Q + beta^2 T^2)) is taken with numerator and denominator
// halved (Q / (hbeta T + sqrt(alpha Q + hbeta^2 T^2)), hbeta = beta / 2:
// power-of-two scalings, so the same value).  The terms that depend on the
// sample only, s / cA, s / cB and the stopped root, come precomputed, so
// that both sides share them.  T must be finite (a side with no robot has
// no crossing; the caller skips it).  Every regime's terms are formed first
// and then picked by plain selects (the fast and slow roots share one
// division), so that the lanes of a wave (samples in different regimes) do
// not split into branches.
template <bool CHIP>
__device__ __forceinline__ float vcrit(float T, float s, float s_icA, float s_icB, float v_stop,
                                       float alpha, float hbeta, float hbeta2, float hfast,
                                       float pfast, float half_ar)
{
    const float T2 = T * T;
    const float Q = fmaf(half_ar, T2, s);
    const bool stop = s_icA <= T2;
    const bool fast = s_icB >= T2;
    // Never negative for a flat kick in this regime.  A chip's can be, by
    // rounding, where its roll is a few 1e-5 of its flight (at 100 m/s^2 or 1.57
    // rad): no root of a negative number may reach the minima that follow.
    const float m = fmaf(alpha, Q, hbeta2 * T2);
    const float m_slow = CHIP ? fmaxf(m, 0.0f) : m;
    const float d_slow = fmaf(hbeta, T, hsqrt(m_slow));
    const float N = fast ? (CHIP ? s : fmaf(hfast, T2, s)) : Q;
    const float D = fast ? (CHIP ? pfast * T : T) : d_slow;
    return stop ? v_stop : N * hrcp(D);
}

// The side-independent terms of the inversion at the lane's samples for one
// kick type.  With TARGET the path ends at the point passed to, so the variants
// that count reach its last sample: they are faster than the stopped root of
// every earlier sample (less by a factor sqrt((K - 1) / K) at least), which is
// then taken as 0, and only the lane's last one is formed.
template <int KPL, bool CHIP, bool TARGET>
struct SampleTerms {
    float icA[KPL], icB[KPL], vst[KPL];
    __device__ __forceinline__ SampleTerms(const DevParams &P, const float (&sk)[KPL])
    {
#pragma unroll
        for (int q = 0; q < KPL; ++q) {
            icA[q] = sk[q] * (CHIP ? P.c_icA : P.f_icA);
            icB[q] = sk[q] * (CHIP ? P.c_icB : P.f_icB);
            vst[q] = TARGET && q < KPL - 1 ? 0.0f : hsqrt(sk[q] * (CHIP ? P.c_icD : P.f_icD));
        }
    }
};

// Critical speeds of one side at the lane's samples for one kick type (0 for
// every sample when the side has no robot).
template <int KPL, bool CHIP, bool TARGET>
__device__ __forceinline__ void side_vcrit(const DevParams &P, int n_side, const float (&T)[KPL],
                                           const float (&sk)[KPL],
                                           const SampleTerms<KPL, CHIP, TARGET> &st,
                                           const float (&vair)[KPL], float (&v)[KPL])
{
    if (n_side == 0) {
#pragma unroll
        for (int q = 0; q < KPL; ++q) v[q] = 0.0f;
        return;
    }
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        if (CHIP)
            v[q] = fminf(vair[q], vcrit<true>(T[q], sk[q], st.icA[q], st.icB[q], st.vst[q],
                                              P.c_alpha, P.c_hbeta, P.c_hbeta2, P.c_hfast,
                                              P.c_pfast, P.half_ar));
        else
            v[q] = vcrit<false>(T[q], sk[q], st.icA[q], st.icB[q], st.vst[q], P.f_alpha,
                                P.f_hbeta, P.f_hbeta2, P.f_hfast, P.f_pfast, P.half_ar);
    }
}

// Square root of a non-negative float64 from the hardware reciprocal square
// root estimate with two Newton steps (0 for 0): within a few units in the
// last place, in about half the instructions of the correctly rounded sqrt.
__device__ __forceinline__ double sqrt64(double q)
{
    double y = __builtin_amdgcn_rsq(q);
    y = y * fma(-0.5 * q, y * y, 1.5);
    y = y * fma(-0.5 * q, y * y, 1.5);
    return q > 0.0 ? q * y : 0.0;
}

// Ball time (float64) to distance s for staged variant c.
__device__ __forceinline__ double ball_time64(const VarConst &c, double s)
{
    bool ph1 = s <= c.split;
    double va = ph1 ? c.va1 : c.va2;
    double ac = ph1 ? c.a1 : c.a2;
    double so = ph1 ? 0.0 : c.soff2;
    double to = ph1 ? 0.0 : c.toff2;
    double x = s - so;
    double q = fmax(va * va - 2.0 * ac * x, 0.0);
    // sqrt(q) and the division from the hardware estimates with two Newton
    // steps each (relative error far below the float32 results need)
    double y = __builtin_amdgcn_rsq(q);
    y = y * fma(-0.5 * q, y * y, 1.5);
    y = y * fma(-0.5 * q, y * y, 1.5);
    const double den = va + (q > 0.0 ? q * y : 0.0);
    double r = __builtin_amdgcn_rcp(den);
    r = r * fma(-den, r, 2.0);
    r = r * fma(-den, r, 2.0);
    return fma(2.0 * x, r, to);
}

// Order-preserving map of a float's bits to an unsigned key (negative scores
// order below positive ones); a finite score never maps to 0, which marks
// "no feasible pass" in the argmax keys.
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    return u ^ ((u & 0x80000000u) ? 0xFFFFFFFFu : 0x80000000u);
}

__device__ __forceinline__ float unordered_bits(uint32_t k)
{
    return __uint_as_float(k ^ ((k & 0x80000000u) ? 0x80000000u : 0xFFFFFFFFu));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned long long dpp_max_u64(unsigned long long x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, ROW_MASK, 0xf,
                                               false);
    const unsigned long long y = ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo;
    return y > x ? y : x;
}

// Largest 64-bit key over the wave, on every lane: the DPP scan steps of
// wave_prefix_imax (lanes without a source see 0), then lane 63's total.
// half_prefix_max_u64 leaves each half's largest on its lane 31.
__device__ __forceinline__ unsigned long long half_prefix_max_u64(unsigned long long x)
{
    x = dpp_max_u64<0x111, 0xf>(x);
    x = dpp_max_u64<0x112, 0xf>(x);
    x = dpp_max_u64<0x114, 0xf>(x);
    x = dpp_max_u64<0x118, 0xf>(x);
    return dpp_max_u64<0x142, 0xa>(x);
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x)
{
    x = dpp_max_u64<0x143, 0xc>(half_prefix_max_u64(x));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}

// Passing power (Sec. 4.1, Eq. 1-2) for a pass over d64 metres whose
// receiver arrives after t_recv seconds: the ball should arrive t_recv +
// buffer; ignoring the sliding phase, the speed after it is (d + a t^2/2) / t
// while the ball still rolls at t, else the slowest ball that reaches the
// point, sqrt(2 a d); the kick speed is that over the slide ratio, clamped to
// [vmin, vmax]; 0 when no teammate can receive.
__device__ __forceinline__ double pass_power(const DevParams &P, double d64, float t_recv,
                                             double buffer, double vmin, double vmax)
{
    if (!(t_recv < INFINITY)) return 0.0;
    const double t = (double)t_recv + buffer;
    const double a = P.bp.a_r;
    const double v1 = d64 >= 0.5 * a * t * t ? (d64 + 0.5 * a * t * t) / t : sqrt(2.0 * a * d64);
    return fmin(fmax(v1 / P.bp.ratio, vmin), vmax);
}

// SBIP of every staged variant along one path of length d (metres; LA = d
// scaled by amax) whose path frame is in pr: robot stage over the lane's
// samples (lanes = samples, K/64 consecutive samples per lane), critical
// speeds, first crossings (pm: this wave's LDS block of 4 K floats).  On
// return lane v (a staged variant) holds its first team / opponent crossing
// samples (K: none).
template <int KPL>
__device__ __forceinline__ void sbip_crossings(const StageLDS &S, const float4 *pr, float *pm,
                                               float myv0,
                                               int mytype, float d, float LA, int &my_kt,
                                               int &my_ko)
{
    const int l = lane_id();
    const int K = KPL * 64;
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
    const float invK = 1.0f / (float)K;
    int k0 = l * KPL + 1;  // (fractions formed anew for each ray: fewer registers)
    asm volatile("" : "+v"(k0));

    float fs[KPL], sk[KPL], Tt[KPL], To[KPL];
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        fs[q] = (float)(k0 + q) * invK;
        Tt[q] = INFINITY;
        To[q] = INFINITY;
    }
    // 1. robot stage, in the path frame
    const bool split = n_tm + n_op <= SPLIT_ROB;
    const RobotK rk(fresh_args<RayArgs>().P);
    if (uni(S.vel_ok)) {
        robot_stage<KPL, false, FULL_WAVE>(pr, rk, 0, n_tm, split, INFINITY, INFINITY, fs, LA, Tt);
        robot_stage<KPL, false, FULL_WAVE>(pr, rk, n_tm, n_op, split, INFINITY, INFINITY, fs, LA, To);
    } else {
        robot_stage<KPL, true, FULL_WAVE>(pr, rk, 0, n_tm, split, INFINITY, INFINITY, fs, LA, Tt);
        robot_stage<KPL, true, FULL_WAVE>(pr, rk, n_tm, n_op, split, INFINITY, INFINITY, fs, LA, To);
    }
    // 2-3. critical kick speeds per sample, then the first crossing of each
    // lane's variant (a side with no robot never intercepts: critical speed 0)
    const float invA2 = fresh_args<RayArgs>().P.invA2;
#pragma unroll
    for (int q = 0; q < KPL; ++q) {
        sk[q] = fs[q] * d;
        Tt[q] *= invA2;  // seconds
        To[q] *= invA2;
    }
    const unsigned long long flat_m = __ballot(mytype == DPPS_FLAT);
    const unsigned long long chip_m = __ballot(mytype == DPPS_CHIP);
    float *const pf = pm, *const pc = pm + 2 * K;  // flat rows, chip rows
    wave_lds_sync();  // the previous path's searches are done with the rows
    if (flat_m) {
        const DevParams &P = fresh_args<RayArgs>().P;
        float vt[KPL], vo[KPL];
        const SampleTerms<KPL, false, false> st(P, sk);
        side_vcrit<KPL, false, false>(P, n_tm, Tt, sk, st, sk, vt);
        side_vcrit<KPL, false, false>(P, n_op, To, sk, st, sk, vo);
        store_running_max<KPL, false>(vt, pf);
        store_running_max<KPL, false>(vo, pf + K);
    }
    if (chip_m) {
        const DevParams &P = fresh_args<RayArgs>().P;
        float vt[KPL], vo[KPL], vair[KPL];
#pragma unroll
        for (int q = 0; q < KPL; ++q) vair[q] = hsqrt(sk[q] * P.lam1_inv);
        const SampleTerms<KPL, true, false> st(P, sk);
        side_vcrit<KPL, true, false>(P, n_tm, Tt, sk, st, vair, vt);
        side_vcrit<KPL, true, false>(P, n_op, To, sk, st, vair, vo);
        store_running_max<KPL, false>(vt, pc);
        store_running_max<KPL, false>(vo, pc + K);
    }
    wave_lds_sync();
    my_kt = K;
    my_ko = K;
    if ((mytype == DPPS_FLAT) | (mytype == DPPS_CHIP)) {
        const float *r = mytype == DPPS_CHIP ? pc : pf;
        count_below<KPL * 64>(r, r + K, myv0, my_kt, my_ko);
    }
}

// Value of x held by lane `src` (0-31) of the lane's own half of the wave.
__device__ __forceinline__ float half_read(float x, int src)
{
    const int a = ((lane_id() & 32) | src) << 2;
    return __int_as_float(__builtin_amdgcn_ds_bpermute(a, __float_as_int(x)));
}

// Open goal angle at two points, one per half of the wave (lane's own cx, cy),
// against the staged opponents: lane o < n_op of a half holds opponent o, its
// lanes 30 and 31 the goal posts.  Each interval contributes what the
// half's intervals sorted before it (by start, then index) have not already
// covered.  Returns on every lane the angle of its half's point.  Costs a
// wave about what one point alone did.
__device__ float open_angle_pair(const StageLDS &S, const DevParams &P, float cx, float cy,
                                 int n_op, int n_tm)
{
    const int l = lane_id(), hl = l & 31;
    const float dxg = fmaxf(P.goal_x - cx, P.goal_eps);
    const float4 o = S.rob[n_tm + (hl < n_op ? hl : 0)];
    const float ox = o.x - cx, oy = o.y - cy;
    const float Y = hl < n_op ? oy : (hl == 30 ? -P.half_goal_w - cy : P.half_goal_w - cy);
    const float X = hl < n_op ? ox : dxg;
    const float ang = atan2f(Y, X);
    const float lo = half_read(ang, 30);
    const float hi = half_read(ang, 31);
    const bool valid = hl < n_op && o.x < P.goal_x;
    const float rho2 = fmaf(ox, ox, oy * oy);
    const unsigned long long in = __ballot(valid && rho2 <= P.R * P.R);
    const float al = asinf(fminf(P.R * rsq(fmaxf(rho2, 1e-30f)), 1.0f));
    const float s = fmaxf(ang - al, lo);
    const float e = fminf(ang + al, hi);
    const bool has = valid && e > s;
    const unsigned long long hm = __ballot(has);
    const uint32_t any = (uint32_t)hm | (uint32_t)(hm >> 32);
    const float sh = has ? s : INFINITY;  // a start of +inf marks no interval
    float M = -INFINITY;
    for (uint32_t m = any; m; m &= m - 1) {
        const int k = __builtin_ctz(m);
        const float sk = half_read(sh, k), ek = half_read(e, k);
        const bool before = sk < sh || (sk == sh && k < hl);
        M = before ? fmaxf(M, ek) : M;
    }
    const float contrib = has ? fmaxf(e - fmaxf(s, M), 0.0f) : 0.0f;
    float blocked = 0.0f;
    for (uint32_t m = any; m; m &= m - 1) blocked += half_read(contrib, __builtin_ctz(m));
    const bool inside = (l < 32 ? (uint32_t)in : (uint32_t)(in >> 32)) != 0u;
    return inside ? 0.0f : (hi - lo) - blocked;
}

// SBIP crossings of two candidate points at once, one per half of the wave:
// the 32 lanes of a half hold the K samples of its point (K/32 consecutive
// ones per lane), pr and pm are the lane's own half's path frame and its two
// running-maximum rows (K floats each, used for the flat kicks and then for
// the chips).  On return kt[c] / ko[c] are the first team / opponent crossing
// samples (K: none) of the lane's variant of chunk c (variant 32 c + lane of
// the half).  With POWER the frame's variants are replaced by one flat pass
// at the power of Eq. 1-2 (lane 0 of the half), whose receiver is the first
// teammate at the last sample, the point itself; its speed is returned in v0.
template <int KPH, bool POWER>
__device__ __forceinline__ void pair_crossings(const StageLDS &S, const float4 *pr, float *pm,
                                               float d, float LA, int (&kt)[2], int (&ko)[2],
                                               double d64, double &v0)
{
    constexpr int K = KPH * 32;
    const int hl = lane_id() & 31;
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
    const int n_var = POWER ? 1 : uni(S.n_var);
    // (the sample fractions are formed anew for each pair of points: kept
    // across the tile loop they would hold KPH registers)
    int k0 = hl * KPH + 1;
    asm volatile("" : "+v"(k0));
    float fs[KPH], Tt[KPH], To[KPH];
#pragma unroll
    for (int q = 0; q < KPH; ++q) {
        fs[q] = (float)(k0 + q) * (1.0f / (float)K);
        Tt[q] = INFINITY;
        To[q] = INFINITY;
    }
    {
    const RobotK rk(fresh_args<SearchLaunch>().a.P);
    const bool split = n_tm + n_op <= SPLIT_ROB;
    // arrival limits of the lane's quarter of the path and the other of its
    // row; with POWER the team's minimum at the last sample is the
    // receiver's time itself
    const float rd = hsqrt(d);
    const int b = hl >> 3;
    const float lim = rd * S.lim[b], limx = rd * S.lim[b ^ 1];
    const float lim_t = POWER && b == 3 ? INFINITY : lim;
    const float limx_t = POWER && b == 2 ? INFINITY : limx;
    if (uni(S.vel_ok)) {
        robot_stage<KPH, false, HALF_WAVE>(pr, rk, 0, n_tm, split, lim_t, limx_t, fs, LA, Tt);
        robot_stage<KPH, false, HALF_WAVE>(pr, rk, n_tm, n_op, split, lim, limx, fs, LA, To);
    } else {
        robot_stage<KPH, true, HALF_WAVE>(pr, rk, 0, n_tm, split, lim_t, limx_t, fs, LA, Tt);
        robot_stage<KPH, true, HALF_WAVE>(pr, rk, n_tm, n_op, split, lim, limx, fs, LA, To);
    }
    }
    const LaunchArgs &a = fresh_args<SearchLaunch>().a;
    const float invA2 = a.P.invA2;
    float sk[KPH];
#pragma unroll
    for (int q = 0; q < KPH; ++q) {
        sk[q] = fs[q] * d;
        Tt[q] *= invA2;  // seconds
        To[q] *= invA2;
    }
    if (POWER) {
        v0 = pass_power(a.P, d64, half_read(Tt[KPH - 1], 31), (double)a.p_buffer, (double)a.p_vmin,
                        (double)a.p_vmax);
    }
    kt[0] = kt[1] = ko[0] = ko[1] = K;
    if (POWER || uni(S.has_flat)) {
        const DevParams &P = fresh_args<SearchLaunch>().a.P;
        float vc[KPH];
        const SampleTerms<KPH, false, true> st(P, sk);
        wave_lds_sync();  // the previous searches are done with the rows
        side_vcrit<KPH, false, true>(P, n_tm, Tt, sk, st, sk, vc);
        store_running_max<KPH, true>(vc, pm);
        side_vcrit<KPH, false, true>(P, n_op, To, sk, st, sk, vc);
        store_running_max<KPH, true>(vc, pm + K);
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int v = 32 * c + hl;
            if (POWER && c == 0 && hl == 0 && v0 > 0.0)
                count_below<K>(pm, pm + K, (float)v0, kt[0], ko[0]);
            if (!POWER && 32 * c < n_var && v < n_var && S.type[v] == DPPS_FLAT)
                count_below<K>(pm, pm + K, S.v0[v], kt[c], ko[c]);
        }
    }
    if (!POWER && uni(S.has_chip)) {
        const DevParams &P = fresh_args<SearchLaunch>().a.P;
        float vc[KPH], vair[KPH];
#pragma unroll
        for (int q = 0; q < KPH; ++q) vair[q] = hsqrt(sk[q] * P.lam1_inv);
        const SampleTerms<KPH, true, true> st(P, sk);
        wave_lds_sync();
        side_vcrit<KPH, true, true>(P, n_tm, Tt, sk, st, vair, vc);
        store_running_max<KPH, true>(vc, pm);
        side_vcrit<KPH, true, true>(P, n_op, To, sk, st, vair, vc);
        store_running_max<KPH, true>(vc, pm + K);
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int v = 32 * c + hl;
            if (32 * c < n_var && v < n_var && S.type[v] == DPPS_CHIP)
                count_below<K>(pm, pm + K, S.v0[v], kt[c], ko[c]);
        }
    }
}

// The wave's best pass (the lane with the largest key) into its record.
__device__ __forceinline__ void wave_best(OutLDS &O, int w, unsigned long long key, float tt,
                                          float to, float v0)
{
    const unsigned long long wk = wave_max_u64(key);
    const unsigned long long who = __ballot(key == wk);
    if (lane_id() == (int)__builtin_ctzll(who)) {
        O.wbest[w].key = wk;
        O.wbest[w].t_team = wk ? tt : INFINITY;
        O.wbest[w].t_opp = wk ? to : INFINITY;
        O.wbest[w].v0 = wk ? v0 : 0.0f;
        O.wbest[w].pad = 0.0f;
    }
}

// The largest of the waves' records (keys of different waves differ unless
// both are 0), written by one wave.
__device__ __forceinline__ unsigned long long group_best(const OutLDS &O, int nw, TileRec *rec)
{
    const int l = lane_id();
    const unsigned long long k = l < nw ? O.wbest[l].key : 0ull;
    const unsigned long long tk = wave_max_u64(k);
    const unsigned long long at = __ballot(k == tk && l < nw);
    if (l == (int)__builtin_ctzll(at)) *rec = O.wbest[l];
    return tk;
}

// Tile t of the launch: from the list, or implicit (tables built on the device).
__device__ __forceinline__ TileDev tile_at(const LaunchArgs &a, int t)
{
    if (a.tiles_per_frame == 0) return a.tiles[t];
    const int win = (int)((unsigned)t / (unsigned)a.tiles_per_frame);
    return TileDev{win, t - win * a.tiles_per_frame};
}

// The greatest score found so far of a frame, -inf if none.
__device__ __forceinline__ float frame_best_score(const uint32_t *p)
{
    const uint32_t b = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return b ? unordered_bits(b) : -INFINITY;
}

// The score that no pass to (cx, cy) exceeds: the goal's whole angle open and
// the greatest margin (the same operations as the score's).
__device__ __forceinline__ float score_bound(const DevParams &P, float cx, float cy)
{
    const float dxg = fmaxf(P.goal_x - cx, P.goal_eps);
    const float ang = atan2f(P.half_goal_w - cy, dxg) - atan2f(-P.half_goal_w - cy, dxg);
    const float gx = cx - P.goal_x;
    const float dg = hsqrt(fmaf(gx, gx, cy * cy));
    const float dterm = fmaf(-dg, P.inv_dist_norm, 1.0f);
    return fmaf(P.w_ang_pi, ang, fmaf(P.w_dist, dterm, P.w_margin * P.margin_cap));
}

// Greatest of the lanes' values, none negative.
__device__ __forceinline__ float wave_max_pos(float x)
{
    return __int_as_float(__builtin_amdgcn_readlane(wave_prefix_imax(__float_as_int(x)), 63));
}

// Word l of a window's record in lane l.
__device__ __forceinline__ int window_words(const LaunchArgs &a, bool inl, int win)
{
    static_assert(sizeof(WinDev) == 48, "12 words");
    const int l = lane_id();
    const WinDev *const w = inl ? &fresh_args<SearchLaunch>().one.win : a.wins + win;
    return l < 12 ? ((const int *)w)[l] : 0;
}

// Bound by VALU issue.  One point per half of a wave rather than per wave: the
// bound tests, prefix maxima, searches, the float64 finish (32 lanes are
// variants) and the open angle cost a pair of points what they cost one,
// the robot stage and the inversions cost the same per sample.  With the bounds
// kept per quarter of the path, its arrival limits and the arguments read
// where they are used the default-shape full frame (8v8, 43 621 points, 32
// variants, K = 256) went from 142 to 123 us and from 66.9 M to 52.5 M VALU
// instructions, 256 uneven windows at 8 variants, K = 128, from 4.42 to 3.40 ms,
// the passing power of the full frame from 122 to 96 us; with tiles by request,
// runs of tiles and the 16-byte LDS to 113 us, 3.25 ms and 89 us.
// Registers: at most 128 VGPRs, so that four waves fit on each SIMD.  13 to 20
// scalars stay spilled to lanes (57 to 100 without the late argument reads) and
// at K = 256 18 to 27 VGPRs to scratch (K = 192: 9 to 14, K = 64: 2 or none);
// three waves without spills took 124 us for the full frame against 118.  K =
// 128 with maps or power runs five waves in 96 VGPRs, spilling 34 to 40 of them
// (256 windows 3.56 -> 3.39 ms, five full frames of passing power 262 -> 244 us);
// BEST does not (30 frames of 64 windows 132 us a call with five, 103 with four; 300
// frames 414 and 314).  At K = 64 five were slower for one small frame, 16.2 ->
// 19.0 us.
// POWER: one flat pass per point at the point's own passing power (Eq. 1-2).
// BEST: only the best record is asked for, and points that cannot hold it are
// left out (1000 frames of 64 windows of 16 points, one flat kick: 940 -> 457
// us, their exact fallback of 18 frames 710 -> 486).
template <int KPH, bool POWER, bool BEST>
__global__ void __launch_bounds__(512, KPH == 4 && !BEST ? 5 : 4) search_kernel(SearchLaunch launch)
{
    const LaunchArgs &args = launch.a;
    __shared__ StageLDS S;
    __shared__ OutLDS O;
    // dynamic: each wave's running maxima (two rows of K for each half), its
    // path frames of two points, the tile's staged score and mask maps
    extern __shared__ __attribute__((aligned(16))) float PMX[];
    __shared__ int s_tile;
    __shared__ float s_least[2];  // least score worth finding (this tile's, the next's)
    const int nw = blockDim.x >> 6;
    const int w = threadIdx.x >> 6;
    const int l = lane_id();
    const int TP = args.tile_points;
    constexpr int K = KPH * 32, HROWS = half_rows(K);
    static_assert(HROWS % 4 == 0, "the rows keep the entries behind them on 16 bytes");
    const int h = l >> 5, hl = l & 31;  // half of the wave, lane in it
    float4 *const PR = (float4 *)(PMX + nw * 2 * HROWS);
    float *const OS = (float *)(PR + nw * 2 * PR_ENTRIES);
    uint8_t *const OM = (uint8_t *)(OS + args.max_variants * TP);
    const bool reduced = (args.P.out_flags & DPPS_OUT_REDUCED) != 0;
    int cur_frame = -1;
    const int G = (int)gridDim.x, b = (int)blockIdx.x;
    const int n_tiles = args.n_frames_dev ? *args.n_frames_dev * args.tiles_per_frame : args.n_tiles;
    // One workgroup per tile, or a persistent grid: every workgroup takes its
    // own n_own tiles (first, first + stride, ...) and then pulls from a work
    // counter as it finishes, so that the last tiles go to the workgroups that
    // are free.
    // One frame: round-robin for all but the last one or two rounds.
    // Workgroup b of the grid sits on XCD b % 8, and so do its own tiles when
    // the grid is a multiple of 8; its pulled tiles keep that class too, from
    // one counter per class, so that the tiles an XCD runs together write
    // neighbouring chunks (below) and its L2 merges their lines.  C classes:
    // every class has a workgroup (a grid under 8 workgroups uses G classes).
    // Several frames: a run of consecutive tiles (n_own, chosen by the host; three
    // quarters of the even share where there are many: frames differ in cost),
    // then groups of `claim` tiles, so that a workgroup stages few frames; the
    // chunks of a run fill whole lines by themselves.
    // BEST, small tiles (16 points): a pulled tile waits for the counter and
    // then for its window and its frame, which cost more than the tile, so up to
    // 11 tiles a workgroup are its own (30 frames of 128 windows: 168 us a call
    // with one of 3.75 tiles its own, 115 with 3; 200 of 64: 350 and 253).
    // Beyond, a quarter, since frames with a poor best leave few points out and
    // cost many times the others (1000 of 64: the kernel took 631 us with three
    // quarters, 457 with one, 472 with an eighth), then groups of as many, up to
    // 8 (300 of 64: 476 us a call with single tiles, 294 with 4; 1000 of 64:
    // groups of 4 593 us, of 8 457).
    // BEST, large tiles (64 points, whole lattices): a quarter, at least one,
    // then one tile each, or 8 from 32 tiles a workgroup on, where the last
    // round weighs less than the pulls (9 lattices: 1 or 8 alike; 18: 486 us with
    // 1, 526 with 4; 60: 2030 with 1, 1780 with 8; 200: 5550 and 3700).
    const int C = min(G, 8), xcd = (int)((unsigned)b % (unsigned)C);
    const bool runs = args.persistent && args.n_frames > 1;
    const int even = n_tiles / G;
    const bool small = TP <= 16;
    const int own = !BEST ? args.n_own
                          : small && even < 12 ? even : max(even / 4, min(even, 1));
    const int n_own = !args.persistent ? 1 : runs ? own : max(even - 1, 0);
    const int first = runs ? b * n_own : b, stride = runs ? 1 : G;
    const int n_static = n_own * G;
    const int claim = !BEST ? min(max(even / 16, 1), 8)
                            : small ? min(max(even / 4, 1), 8) : even >= 32 ? 8 : 1;
    // the lane's best pass of the tile, or of all the workgroup's tiles with
    // one record per workgroup
    unsigned long long bkey = 0ull;
    float btt = INFINITY, bto = INFINITY, bv0 = 0.0f;
    // the next own tile and its window's record (word i in lane i) are loaded
    // while the current tile is searched
    const bool inl = launch.one.on != 0;  // the tables come with the launch
    TileDev ta = {0, 0}, tb = {0, 0};
    int words = 0;
    if (n_own > 0) {
        ta = tile_at(args, first);
        if (n_own > 1) tb = tile_at(args, first + stride);
        words = window_words(args, inl, ta.win);
    }
    if (args.n_frames == 1 && !args.n_frames_dev) {  // known without the tile: one round trip less
        const OneFrame &o = fresh_args<SearchLaunch>().one;
        stage_frame(args.P, inl ? o.frame : args.frames[0], inl ? o.robots : args.robots,
                    inl ? o.variants : args.variants, 0, S);
        cur_frame = 0;
    }
    if (BEST) {
        if (n_tiles == 0) return;  // no frame took the fallback
        if (threadIdx.x == 0) s_least[0] = s_least[1] = -INFINITY;
    }
    int it = 0, pull = 0, pull_end = 0, turn = 0;
    while (true) {
        // the previous tile (its staged results and records) is finished
        __syncthreads();
        const LaunchArgs &a = fresh_args<SearchLaunch>().a;
        int t, at, cw;
        if (it < n_own) {
            t = first + it * stride;
            at = ta.at;
            cw = words;
            ++it;
            if (it < n_own) {
                ta = tb;
                words = window_words(a, inl, ta.win);
                if (it + 1 < n_own) tb = tile_at(a, first + (it + 1) * stride);
            }
        } else {
            if (!a.persistent) break;
            if (pull < pull_end) {
                t = pull++;
            } else {
                if (threadIdx.x == 0)
                    s_tile = runs ? n_static + claim * (int)atomicAdd(a.counter, 1u)
                                  : n_static + C * (int)atomicAdd(a.counter + xcd, 1u) + xcd;
                __syncthreads();
                t = uni(s_tile);
                pull = t + 1;
                pull_end = runs ? min(t + claim, n_tiles) : 0;
            }
            if (t >= n_tiles) break;
            const TileDev tile = tile_at(a, t);
            at = tile.at;
            cw = window_words(a, inl, tile.win);
        }
        const int tk = uni(at);
        WinDev W;  // the same for every lane: scalar
        W.h = readlane_f(__int_as_float(cw), 0);
        W.i0 = readlane_i(cw, 1);
        W.j0 = readlane_i(cw, 2);
        W.nx = readlane_i(cw, 3);
        W.n_tiles = readlane_i(cw, 4);
        W.halfNx = readlane_f(__int_as_float(cw), 5);
        W.halfNy = readlane_f(__int_as_float(cw), 6);
        W.frame = readlane_i(cw, 7);
        W.npts = readlane_i(cw, 8);
        W.elem_base = readlane_i(cw, 9);
        W.out_base = (int64_t)(((uint64_t)(uint32_t)readlane_i(cw, 11) << 32) |
                               (uint32_t)readlane_i(cw, 10));
        if (W.frame != cur_frame) {
            stage_frame(a.P, a.frames[W.frame], a.robots, a.variants, W.frame, S);
            if (BEST && threadIdx.x == 0) s_least[turn] = frame_best_score(a.frame_best + W.frame);
            __syncthreads();
            cur_frame = W.frame;
        }
        const int n_var = uni(S.n_var);
        // the window's points in chunks of CH; tile k of a window cut into T
        // tiles holds chunks pk, pk + T, pk + 2T, ...: every tile samples the
        // whole window, so tiles cost alike (neighbouring points cost alike,
        // distant ones do not) and the last round of tiles ends together,
        // while each chunk's outputs are still written as one 16-byte piece
        // per variant.  pk ranks the tiles by (k % 8, k / 8), so the tiles of
        // one class mod 8 (one XCD's, when the window's tiles start the
        // launch's tile list) hold neighbouring chunks.  Slot s of the tile
        // is point (pk + (s / CH) T) CH + s % CH; only the window's last
        // chunk can be short, and it is the last chunk of its tile.
        constexpr int CH = 4;
        const int NC = (int)((unsigned)(W.npts + CH - 1) / CH), cpt = TP / CH;
        const int Tw = W.n_tiles;  // ceil(npts / TP)
        const int pk = (tk & 7) * (Tw >> 3) + min(tk & 7, Tw & 7) + (tk >> 3);
        int nch = tk < Tw ? cpt : 0;
        while (nch > 0 && (int64_t)pk + (int64_t)(nch - 1) * Tw >= NC) --nch;
        const int npts =
            nch > 0 ? (nch - 1) * CH + min(CH, W.npts - (pk + (nch - 1) * Tw) * CH) : 0;
        if (!args.wg_records) {
            bkey = 0ull;
            btt = bto = INFINITY;
            bv0 = 0.0f;
        }
        // The tile's points that are worth evaluating, slot list[k] in lane k:
        // all of them, or, where only the frame's best is asked for, those
        // within some variant's reach whose score with an open goal and the
        // greatest margin is not below the best found so far (the score's
        // roundings are monotone in both terms).  Every wave forms the same
        // list.
        int n_list = npts, list = 0;
        float least = -INFINITY;
        uint32_t others = 0u;
        if (BEST) {
            least = s_least[turn];
            const int p = (pk + (l / CH) * Tw) * CH + (l & (CH - 1));
            const int j = (int)((unsigned)p / (unsigned)W.nx), i = p - j * W.nx;
            const float cx = W.h * ((float)(W.i0 + i) - W.halfNx);
            const float cy = W.h * ((float)(W.j0 + j) - W.halfNy);
            const float ex = cx - unif(S.bx), ey = cy - unif(S.by);
            const float reach =
                wave_max_pos(l < n_var ? (float)S.vc[l].D : 0.0f) * (1.0f + 1.0f / 65536.0f);
            const bool in = l < npts && hsqrt(fmaf(ex, ex, ey * ey)) <= reach &&
                            score_bound(fresh_args<SearchLaunch>().a.P, cx, cy) >= least;
            const unsigned long long m = __ballot(in);
            n_list = __builtin_popcountll(m);
            const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            list = __builtin_amdgcn_ds_permute((in ? before : n_list + l - before) << 2, l);
            turn ^= 1;
            if (n_list == 0) {
                if (threadIdx.x == 0) {
                    s_least[turn] = least;
                    const TileRec none = {0ull, INFINITY, INFINITY, 0.0f, 0.0f};
                    args.tile_rec[t] = none;
                }
                continue;
            }
            if (threadIdx.x == 0)
                others = __hip_atomic_load(args.frame_best + W.frame, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
        // the wave's points in pairs of neighbours, slots s0 and s0 + 1, one
        // per half of the wave (a lone last point is taken by both halves,
        // which write the same values)
        for (int s0 = 2 * w; s0 < n_list; s0 += 2 * nw) {
            const int k = min(s0 + h, n_list - 1);
            const int slot = BEST ? __builtin_amdgcn_ds_bpermute(k << 2, list) : k;
            const int p = (pk + (slot / CH) * Tw) * CH + (slot & (CH - 1));
            const int j = (int)((unsigned)p / (unsigned)W.nx), i = p - j * W.nx;
            const float mi = (float)(W.i0 + i) - W.halfNx;
            const float mj = (float)(W.j0 + j) - W.halfNy;
            const float cx = W.h * mi, cy = W.h * mj;
            const double cx64 = (double)W.h * (double)mi, cy64 = (double)W.h * (double)mj;
            const float bx = unif(S.bx), by = unif(S.by);
            const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
            float4 *const pr = PR + (w * 2 + h) * PR_ENTRIES;
            const float LA = path_frame(S, fresh_args<SearchLaunch>().a.P, pr, n_tm + n_op, n_tm, cx64, cy64, (double)bx,
                                        (double)by, hl);
            const float ex = cx - bx, ey = cy - by;
            const float d = hsqrt(fmaf(ex, ex, ey * ey));
            const double ex64 = cx64 - (double)bx, ey64 = cy64 - (double)by;
            const double d64 = sqrt64(ex64 * ex64 + ey64 * ey64);
            int kt[2], ko[2];
            double v0 = 0.0;
            pair_crossings<KPH, POWER>(S, pr, PMX + (w * 2 + h) * HROWS, d, LA, kt, ko, d64, v0);
            // finish: the lanes of a half are its point's variants
            const LaunchArgs &a = fresh_args<SearchLaunch>().a;
            const DevParams &P = a.P;
            float tt[2], to[2], mc[2];
            bool feas[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                tt[c] = INFINITY;
                to[c] = INFINITY;
                mc[c] = 0.0f;
                feas[c] = false;
                const int v = 32 * c + hl;
                if (c > 0 && (POWER || n_var <= 32)) continue;
                if (v < n_var && (!POWER || v0 > 0.0)) {
                    const VarConst vc = POWER ? var_const(P.bp, DPPS_FLAT, (float)v0) : S.vc[v];
                    const bool reach = d64 >= 1e-9 && d64 <= vc.D && d64 >= vc.sf_reach;
                    double t1 = INFINITY, t2 = INFINITY;
                    if (reach) {
                        if (kt[c] < K) t1 = ball_time64(vc, (double)(kt[c] + 1) * P.invK_d * d64);
                        if (ko[c] < K) t2 = ball_time64(vc, (double)(ko[c] + 1) * P.invK_d * d64);
                    }
                    const bool tfin = t1 < INFINITY;
                    const double m = !tfin ? -INFINITY : (t2 < INFINITY ? t2 - t1 : INFINITY);
                    feas[c] = reach && tfin && m >= P.margin_d;
                    tt[c] = (float)t1;
                    to[c] = (float)t2;
                    mc[c] = fminf(fmaxf((float)m, 0.0f), P.margin_cap);
                }
            }
            // the open goal angle (lanes = opponents) and the distance to the
            // goal enter only feasible scores
            float ang = 0.0f, dterm = 0.0f;
            if (__ballot(feas[0] || feas[1])) {
                ang = open_angle_pair(S, P, cx, cy, n_op, n_tm);
                const float gx = cx - P.goal_x;
                const float dg = hsqrt(fmaf(gx, gx, cy * cy));
                dterm = fmaf(-dg, P.inv_dist_norm, 1.0f);
            }
            if (POWER && hl == 0 && a.v0_out) a.v0_out[W.out_base + p] = (float)v0;
            unsigned long long pkey = 0ull;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (c > 0 && (POWER || n_var <= 32)) continue;
                const int v = 32 * c + hl;
                const int vid = v < n_var ? S.vidx[v] : 0;  // the caller's index
                float sc = -INFINITY;
                unsigned long long key = 0ull;
                if (feas[c]) {
                    sc = fmaf(P.w_ang_pi, ang, fmaf(P.w_dist, dterm, P.w_margin * mc[c]));
                    const uint32_t lin = (uint32_t)(W.elem_base + vid * W.npts + p);
                    key = ((unsigned long long)ordered_bits(sc) << 32) |
                          (unsigned long long)(0xFFFFFFFFu - lin);
                }
                if (key > bkey) {
                    bkey = key;
                    btt = tt[c];
                    bto = to[c];
                    bv0 = POWER ? (float)v0 : S.v0[v];
                }
                if (reduced) {
                    pkey = key > pkey ? key : pkey;
                } else if (!BEST && v < n_var) {
                    OS[vid * TP + slot] = sc;
                    OM[vid * TP + slot] = (uint8_t)feas[c];
                    const int64_t e = W.out_base + (int64_t)vid * W.npts + p;
                    if (a.t_team) a.t_team[e] = tt[c];
                    if (a.t_opp) a.t_opp[e] = to[c];
                }
            }
            if (reduced) {
                pkey = half_prefix_max_u64(pkey);
                if (hl == 31) {
                    const int64_t o = W.out_base + p;
                    if (a.score)
                        a.score[o] = pkey ? unordered_bits((uint32_t)(pkey >> 32)) : -INFINITY;
                    if (a.mask) {
                        const uint32_t lin = 0xFFFFFFFFu - (uint32_t)pkey;
                        a.mask[o] = pkey ? (uint8_t)((lin - (uint32_t)W.elem_base) /
                                                     (uint32_t)W.npts)
                                         : (uint8_t)255;
                    }
                }
            }
        }
        // the staged maps are complete; with one record per tile so are the
        // waves' best passes
        if (!args.wg_records) wave_best(O, w, bkey, btt, bto, bv0);
        __syncthreads();
        if (!args.wg_records && w == 0) {
            const uint32_t found = (uint32_t)(group_best(O, nw, args.tile_rec + t) >> 32);
            if (BEST && l == 0) {
                if (found > others) atomicMax(args.frame_best + W.frame, found);
                others = max(others, found);
                s_least[turn] = others ? fmaxf(least, unordered_bits(others)) : least;
            }
        }
        if (!reduced && !BEST) {
            // one variant's piece of one chunk per thread: four scores in one
            // store and their flags in another (the last chunk of the window
            // may be short)
            const LaunchArgs &a = fresh_args<SearchLaunch>().a;
            const float rn = hrcp((float)nch);
            for (int e = threadIdx.x; e < n_var * nch; e += blockDim.x) {
                const int v = (int)(((float)e + 0.5f) * rn), c = e - v * nch;
                const int first = (pk + c * Tw) * CH;
                const int64_t o = W.out_base + (int64_t)v * W.npts + first;
                const float *const sv = OS + v * TP + c * CH;
                const uint8_t *const mv = OM + v * TP + c * CH;
                if (first + CH <= W.npts) {
                    const float4 x = *(const float4 *)sv;
                    const uint32_t y = *(const uint32_t *)mv;
                    if (a.score) __builtin_memcpy(a.score + o, &x, sizeof x);
                    if (a.mask) __builtin_memcpy(a.mask + o, &y, sizeof y);
                } else {
                    for (int q = 0; q < W.npts - first; ++q) {
                        if (a.score) a.score[o + q] = sv[q];
                        if (a.mask) a.mask[o + q] = mv[q];
                    }
                }
            }
        }
    }
    if (args.wg_records) {
        wave_best(O, w, bkey, btt, bto, bv0);
        __syncthreads();
        if (w == 0) group_best(O, nw, args.tile_rec + blockIdx.x);
    }
}

// One workgroup per frame: reduce the frame's tile records to its best pass;
// block 0 also rearms the persistent work counter for the next launch.
// INL: the tables come with the launch (a kernel of its own: pointers that may
// lead to either memory would be slower for both).
template <bool INL>
__global__ void __launch_bounds__(256) finalize_kernel(SearchLaunch launch)
{
    const LaunchArgs &a = launch.a;
    const OneFrame &one = fresh_args<SearchLaunch>().one;
    const WinDev *const wins = INL ? &one.win : a.wins;
    const dpps_variant *const variants = INL ? one.variants : a.variants;
    __shared__ TileRec red[256 / 64];
    __shared__ int s_wi;
    const int f = blockIdx.x;
    const int tid = threadIdx.x;
    if (f == 0 && tid < 8 && a.counter) a.counter[tid] = 0u;  // the search's 8 counters
    if (f == 0 && tid == 0 && a.count_host) *a.count_host = *a.n_frames_dev;
    if (a.n_frames_dev && f >= *a.n_frames_dev) return;
    // (by reference: a copy is kept in private memory, and the kernel takes 17
    // us instead of 5 over 256 frames)
    const FrameDev &F = INL ? one.frame : a.frames[f];
    // the frame's tile records, or one record per workgroup of a one-frame
    // launch
    const int rc = a.wg_records ? a.wg_records : F.tile_count;
    const int rb = a.wg_records ? 0 : F.tile_begin;
    TileRec r;
    r.key = 0ull;
    r.v0 = 0.0f;
    r.pad = 0.0f;
    r.t_team = INFINITY;
    r.t_opp = INFINITY;
    // four records in flight per thread (the keys are unique: order-free)
    for (int k0 = tid; k0 < rc; k0 += 4 * blockDim.x) {
        TileRec x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = k0 + q * blockDim.x;
            x[q].key = 0ull;
            if (k < rc) x[q] = a.tile_rec[rb + k];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (x[q].key > r.key) r = x[q];
    }
    // each wave's largest key by DPP, the waves' winners through LDS
    const unsigned long long wk = wave_max_u64(r.key);
    const unsigned long long who = __ballot(r.key == wk);
    if ((tid & 63) == (int)__builtin_ctzll(who)) red[tid >> 6] = r;
    if (tid == 0) s_wi = 0;
    __syncthreads();
    TileRec bestr = red[0];
    for (int q = 1; q < (int)(blockDim.x >> 6); ++q)
        if (red[q].key > bestr.key) bestr = red[q];
    // the window of the best element: the last window whose element base is
    // not above it (bases increase with the window), searched in parallel
    const uint32_t lin = 0xFFFFFFFFu - (uint32_t)bestr.key;
    if (bestr.key != 0ull)
        for (int k = tid; k < F.n_windows; k += blockDim.x)
            if ((uint32_t)wins[F.win_off + k].elem_base <= lin) atomicMax(&s_wi, k);
    __syncthreads();
    if (tid != 0) return;
    dpps_best b;
    b.found = 0; b.window = -1; b.variant = -1; b.i = -1; b.j = -1; b.type = -1;
    b.x = b.y = b.v0 = 0.0f;
    b.score = -INFINITY; b.t_team = INFINITY; b.t_opp = INFINITY; b.t_ball = INFINITY;
    b.pad = 0;
    if (bestr.key != 0ull) {
        const int wi = s_wi;
        const WinDev W = wins[F.win_off + wi];
        const uint32_t rel = lin - (uint32_t)W.elem_base;
        const int v = (int)(rel / (uint32_t)W.npts);
        const int p = (int)(rel - (uint32_t)v * (uint32_t)W.npts);
        const int j = p / W.nx, i = p - j * W.nx;
        const float mi = (float)(W.i0 + i) - W.halfNx;
        const float mj = (float)(W.j0 + j) - W.halfNy;
        const dpps_variant var = variants[F.variant_off + v];
        // the per-point power search passes one flat kick at the point's power
        const int ptype = a.power ? DPPS_FLAT : var.type;
        const float pv0 = a.power ? bestr.v0 : var.v0;
        const VarConst c = var_const(a.P.bp, ptype, pv0);
        double ex64 = (double)W.h * (double)mi - (double)F.ball_x;
        double ey64 = (double)W.h * (double)mj - (double)F.ball_y;
        b.found = 1;
        b.window = wi;
        b.variant = v;
        b.i = i;
        b.j = j;
        b.type = ptype;
        b.x = W.h * mi;
        b.y = W.h * mj;
        b.v0 = pv0;
        b.score = unordered_bits((uint32_t)(bestr.key >> 32));
        b.t_team = bestr.t_team;
        b.t_opp = bestr.t_opp;
        b.t_ball = (float)ball_time64(c, sqrt(ex64 * ex64 + ey64 * ey64));
    }
    const int slot_b = a.best_map ? a.best_map[f] : f;
    a.best[slot_b] = b;
    if (a.best_host) a.best_host[slot_b] = b;
    if (a.fb_on && (!b.found || b.score < a.fb.below)) {
        // this frame takes the exact fallback: one window over the whole lattice
        const int slot = atomicAdd(a.fb.count, 1);
        FrameDev G = F;
        G.n_windows = 1;
        G.win_off = slot;
        G.tile_begin = slot * a.fb.tiles_per_frame;
        G.tile_count = a.fb.tiles_per_frame;
        a.fb.frames[slot] = G;
        WinDev V;
        V.h = a.fb.h;
        V.i0 = 0;
        V.j0 = 0;
        V.nx = a.fb.nx;
        V.halfNx = 0.5f * (float)(a.fb.nx - 1);
        V.halfNy = 0.5f * (float)(a.fb.ny - 1);
        V.frame = slot;
        V.npts = a.fb.nx * a.fb.ny;
        V.n_tiles = a.fb.tiles_per_frame;
        V.elem_base = 0;
        V.out_base = 0;
        a.fb.wins[slot] = V;
        a.fb.map[slot] = f;
    }
}


template <int KPL>
static int launch_kpl(const SearchLaunch &s, int waves_per_wg, int grid, hipStream_t st,
                      hipEvent_t e0, hipEvent_t e1)
{
    const LaunchArgs &a = s.a;
    if (e0) (void)hipEventRecord(e0, st);
    if (a.n_tiles > 0 && grid > 0) {
        const size_t lds = search_lds_bytes(KPL * 64, waves_per_wg, a.tile_points,
                                            a.max_variants);
        if (a.power)
            hipLaunchKernelGGL((search_kernel<2 * KPL, true, false>), dim3(grid),
                               dim3(64 * waves_per_wg), lds, st, s);
        else if (a.frame_best)
            hipLaunchKernelGGL((search_kernel<2 * KPL, false, true>), dim3(grid),
                               dim3(64 * waves_per_wg), lds, st, s);
        else
            hipLaunchKernelGGL((search_kernel<2 * KPL, false, false>), dim3(grid),
                               dim3(64 * waves_per_wg), lds, st, s);
    }
    if (e1) (void)hipEventRecord(e1, st);
    if (a.n_frames > 0)
        hipLaunchKernelGGL(s.one.on ? finalize_kernel<true> : finalize_kernel<false>,
                           dim3(a.n_frames), dim3(256), 0, st, s);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ----------------------------------------------------------------------------
// The paper's direction x power form (Sec. 4.2): rays from the ball, the pass
// received at the first teammate's interception, five-feature score.
// ----------------------------------------------------------------------------

// Lane n of each row of 16 lanes, broadcast to its row (DPP row_newbcast).
template <int N>
__device__ __forceinline__ float row_newbcast(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xf, 0xf, true));
}

// Lane l ^ m within each group of 4 lanes (m = 1, 2, 3; DPP quad_perm; every
// source lane exists, so no old value is needed).
template <int M>
__device__ __forceinline__ float quad_xor(float v)
{
    constexpr int ctrl = M == 1 ? 0xB1 : M == 2 ? 0x4E : 0x1B;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true));
}

// Lane l ^ 7 within each group of 8 lanes (DPP row_half_mirror).
__device__ __forceinline__ float half_mirror(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, true));
}

// Lane l ^ 15 within each row of 16 lanes (DPP row_mirror).
__device__ __forceinline__ float row_mirror(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, true));
}

// Sum over each group of GS (8 or 16) lanes, on every lane of the group:
// pairs, then quads, then halves (each partner holds the same partial sum,
// so every lane gets the same bits).
template <int GS>
__device__ __forceinline__ float group_sum(float c)
{
    c += quad_xor<1>(c);
    c += quad_xor<2>(c);
    c += half_mirror(c);
    if (GS == 16) c += row_mirror(c);
    return c;
}

// Least of the lanes' values over each half of the wave, on all its lanes.
__device__ __forceinline__ float half_min(float x)
{
    x = fminf(x, quad_xor<1>(x));
    x = fminf(x, quad_xor<2>(x));
    x = fminf(x, half_mirror(x));
    x = fminf(x, row_mirror(x));
    // rows 0 and 1 (2 and 3) exchanged
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Least value over the wave (DPP within each row of 16 lanes,
// then the four rows), on every lane.
__device__ __forceinline__ float wave_min_dpp(float x)
{
    x = fminf(x, quad_xor<1>(x));
    x = fminf(x, quad_xor<2>(x));
    x = fminf(x, half_mirror(x));
    x = fminf(x, row_mirror(x));
    return fminf(fminf(readlane_f(x, 0), readlane_f(x, 16)),
                 fminf(readlane_f(x, 32), readlane_f(x, 48)));
}

// Covered length of the union of the intervals [s, e] held by the lanes of
// each group of GS lanes (GS = 8, or 16 for up to n <= 16 intervals; lane o of
// a group holds interval o, has marks a real interval, no end exceeds hi), on
// every lane of the group: each interval adds what the group's intervals
// sorted before it (by start, then index) have not covered.  M, the largest
// end among those, is formed with a median against hi, which needs no NaN
// quieting.
template <int GS>
__device__ __forceinline__ float group_cover(float s, float e, bool has, float hi, int o, int n)
{
    const float sh = has ? s : INFINITY;  // a start of +inf marks no interval
    float M = -INFINITY;
    if (GS == 8) {
        // interval of lane o ^ m of the group for m = 1..7 by DPP lane swaps
        // (l ^ m = l ^ 7 ^ (m ^ 7) for m >= 4); that lane sorts before this
        // one on equal starts when o has the highest bit of m set
        const float hs = half_mirror(sh), he = half_mirror(e);
        const bool hb1 = (o & 1) != 0, hb2 = (o & 2) != 0, hb4 = (o & 4) != 0;
#define GC_UNION(SJ, EJ, HB)                                             \
    {                                                                    \
        const float sj = (SJ), ej = (EJ);                                \
        const bool before = (sj < sh) || ((sj == sh) && (HB));           \
        M = before ? __builtin_amdgcn_fmed3f(M, ej, hi) : M;             \
    }
        GC_UNION(quad_xor<1>(sh), quad_xor<1>(e), hb1)
        GC_UNION(quad_xor<2>(sh), quad_xor<2>(e), hb2)
        GC_UNION(quad_xor<3>(sh), quad_xor<3>(e), hb2)
        GC_UNION(quad_xor<3>(hs), quad_xor<3>(he), hb4)
        GC_UNION(quad_xor<2>(hs), quad_xor<2>(he), hb4)
        GC_UNION(quad_xor<1>(hs), quad_xor<1>(he), hb4)
        GC_UNION(hs, he, hb4)
#undef GC_UNION
    } else {
        // interval j of the group by a row broadcast of lane j
#define GC_STEP(J)                                                                    \
    if (J < n) {                                                                      \
        const float sj = row_newbcast<J>(sh), ej = row_newbcast<J>(e);                \
        const bool before = (sj < sh) || ((sj == sh) && (J < o));                     \
        M = before ? __builtin_amdgcn_fmed3f(M, ej, hi) : M;                          \
    }
        GC_STEP(0) GC_STEP(1) GC_STEP(2) GC_STEP(3)
        GC_STEP(4) GC_STEP(5) GC_STEP(6) GC_STEP(7)
        GC_STEP(8) GC_STEP(9) GC_STEP(10) GC_STEP(11)
        GC_STEP(12) GC_STEP(13) GC_STEP(14) GC_STEP(15)
#undef GC_STEP
    }
    return group_sum<GS>(has ? fmaxf(e - fmaxf(s, M), 0.0f) : 0.0f);
}

// Open goal angle at up to 64 / GS points at once: lane GS g + o looks at
// point g (its own cx, cy, and the point's goal-post angles lo, hi) and
// opponent o (GS = 16 for up to 16 opponents, 8 for up to 8).  The same
// construction as open_angle_pair within each group of GS lanes; returns on every
// lane the angle of its group's point.
template <int GS>
__device__ float open_angle_groups(const StageLDS &S, const DevParams &P, float cx, float cy,
                                   float lo, float hi, int n_op, int n_tm)
{
    const int l = lane_id();
    const int o = l & (GS - 1), base = l & (64 - GS);
    const float4 r = S.rob[n_tm + (o < n_op ? o : 0)];
    const float ox = r.x - cx, oy = r.y - cy;
    const bool valid = o < n_op && r.x < P.goal_x;
    const float rho2 = fmaf(ox, ox, oy * oy);
    const bool inside = valid && rho2 <= P.R * P.R;
    const float ang = atan2f(oy, ox);
    const float al = asinf(fminf(P.R * rsq(fmaxf(rho2, 1e-30f)), 1.0f));
    const float s = fmaxf(ang - al, lo);
    const float e = fminf(ang + al, hi);
    const bool has = valid && e > s;
    const float c = group_cover<GS>(s, e, has, hi, o, n_op);
    const unsigned long long gmask = GS == 16 ? 0xFFFFull : 0xFFull;
    const bool gin = ((__ballot(inside) >> base) & gmask) != 0ull;
    return gin ? 0.0f : (hi - lo) - c;
}

// Open goal angles at the passing points of a direction's feasible variants
// (lanes): a feasible lane whose passing sample differs from the previous
// feasible lane's leads.  The leaders write their points and goal-post
// angles, in lane order, to the wave's LDS block scr (64 float4; free once
// the crossings are known), their points go 64 / GS at a time through
// open_angle_groups, each angle goes back to its leader's entry, and every
// feasible lane reads its leader's.
template <int GS>
__device__ float leader_angles(const StageLDS &S, const DevParams &P, float *scr, bool feas,
                               int my_k, float px, float py, int n_op, int n_tm)
{
    constexpr int NG = 64 / GS;
    const int l = lane_id();
    const unsigned long long fm = __ballot(feas);
    const unsigned long long below = fm & ((1ull << l) - 1ull);
    const int prevl = below ? 63 - __builtin_clzll(below) : 0;
    const int kprev = __shfl(my_k, prevl, 64);
    const bool lead = feas && (below == 0ull || kprev != my_k);
    const unsigned long long lm = __ballot(lead);
    const int n_lead = __popcll(lm);
    float4 *const pts = (float4 *)scr;
    wave_lds_sync();  // the crossing searches are done with the block
    if (lead) {
        const float dxg = fmaxf(P.goal_x - px, P.goal_eps);
        pts[__popcll(lm & ((1ull << l) - 1ull))] =
            make_float4(px, py, atan2f(-P.half_goal_w - py, dxg), atan2f(P.half_goal_w - py, dxg));
    }
    wave_lds_sync();
    for (int c0 = 0; c0 < n_lead; c0 += NG) {
        const int idx = c0 + l / GS;
        const float4 q = pts[min(idx, n_lead - 1)];
        const float a = open_angle_groups<GS>(S, P, q.x, q.y, q.z, q.w, n_op, n_tm);
        if ((l & (GS - 1)) == 0 && idx < n_lead) scr[4 * idx + 2] = a;
    }
    wave_lds_sync();
    // a feasible lane's leader is the last leader at or below it
    const unsigned long long upto = l == 63 ? lm : lm & ((2ull << l) - 1ull);
    const float la = feas ? scr[4 * (__popcll(upto) - 1) + 2] : 0.0f;
    return la;
}

// Distance from the ball along (ux, uy) to the edge of the field (0 when the
// ray leaves at once).
__device__ __forceinline__ double ray_length(const DevParams &P, double bx, double by,
                                             double ux, double uy)
{
    const double hl = 0.5 * (double)P.field_len, hw = 0.5 * (double)P.field_wid;
    double L = INFINITY;
    if (ux > 0.0) L = fmin(L, (hl - bx) / ux);
    if (ux < 0.0) L = fmin(L, (-hl - bx) / ux);
    if (uy > 0.0) L = fmin(L, (hw - by) / uy);
    if (uy < 0.0) L = fmin(L, (-hw - by) / uy);
    return L > 0.0 ? L : 0.0;
}

struct RayOut {
    unsigned long long key;  // 0: not feasible
    float score, t_team, t_opp, s_recv, open_angle, refract;
    int feas;
};

// Every staged variant (lanes) for direction d of the staged frame.
// Unit vector of each kick direction, theta_d = 2 pi d / n from +x
// (computed once per direction count, read by every ray).
__global__ void __launch_bounds__(256) ray_dirs_kernel(double2 *dirs, int n)
{
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n) return;
    const double xd = 2.0 * (double)d / (double)n;  // theta_d / pi
    dirs[d] = make_double2(cospi(xd), sinpi(xd));
}

int launch_ray_dirs(double2 *dirs, int n, void *stream)
{
    hipLaunchKernelGGL(ray_dirs_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       dirs, n);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int KPL>
__device__ RayOut ray_direction(const StageLDS &S, float4 *pr, float *pm, float myv0, int mytype,
                                int myvid, int d)
{
    const int l = lane_id();
    const int K = KPL * 64;
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op), n_var = uni(S.n_var);
    const double bx = (double)unif(S.bx), by = (double)unif(S.by);
    double ux, uy, L, LA;
    {
        const RayArgs &a = fresh_args<RayArgs>();
        const double2 u = a.dirs[d];
        ux = u.x;
        uy = u.y;
        L = ray_length(a.P, bx, by, ux, uy);
        LA = L * (double)a.P.A;
        path_frame_dir<FULL_WAVE>(S, a.P, pr, n_tm + n_op, n_tm, LA, ux, uy, bx, by, l);
    }
    int my_kt, my_ko;
    sbip_crossings<KPL>(S, pr, pm, myv0, mytype, (float)L, (float)LA, my_kt, my_ko);
    const RayArgs &a = fresh_args<RayArgs>();
    const DevParams &P = a.P;

    RayOut o;
    o.key = 0ull;
    o.score = -INFINITY;
    o.t_team = INFINITY;
    o.t_opp = INFINITY;
    o.s_recv = INFINITY;
    o.open_angle = 0.0f;
    o.refract = 0.0f;
    o.feas = 0;
    double px = 0.0, py = 0.0, m = -INFINITY;
    if (l < n_var) {
        // a crossing counts only where the ball gets to (within its stop)
        const VarConst c = S.vc[l];
        const double st = (double)(my_kt + 1) * P.invK_d * L;
        const double so = (double)(my_ko + 1) * P.invK_d * L;
        const double tt = (my_kt < K && st <= c.D) ? ball_time64(c, st) : INFINITY;
        const double to = (my_ko < K && so <= c.D) ? ball_time64(c, so) : INFINITY;
        const bool tfin = tt < INFINITY;
        m = !tfin ? -INFINITY : (to < INFINITY ? to - tt : INFINITY);
        o.feas = tfin && m >= P.margin_d;
        o.t_team = (float)tt;
        o.t_opp = (float)to;
        o.s_recv = tfin ? (float)st : INFINITY;
        px = bx + st * ux;
        py = by + st * uy;
    }
    // open goal angle at each feasible passing point
    const float my_ang = n_op <= 8 ? leader_angles<8>(S, P, pm, o.feas != 0, my_kt, (float)px,
                                                      (float)py, n_op, n_tm)
                                   : leader_angles<16>(S, P, pm, o.feas != 0, my_kt, (float)px,
                                                       (float)py, n_op, n_tm);
    if (o.feas) {
        const double gx = (double)P.goal_x - px, gy = -py;
        const float dg = (float)sqrt(gx * gx + gy * gy);
        const float refr = dg > 0.0f ? atan2f((float)fabs(ux * gy - uy * gx), (float)(ux * gx + uy * gy))
                                     : 0.0f;
        const float mc = fminf(fmaxf((float)m, 0.0f), P.margin_cap);
        const float sc = fmaf(P.w_ang_pi, my_ang,
                              fmaf(P.w_dist, fmaf(-dg, P.inv_dist_norm, 1.0f),
                                   fmaf(P.w_margin, mc,
                                        fmaf(-a.w_time, o.t_team, -a.w_refract * refr * 0.318309886183790672f))));
        o.score = sc;
        o.open_angle = my_ang;
        o.refract = refr;
        const uint32_t lin = (uint32_t)(d * n_var + myvid);
        o.key = ((unsigned long long)ordered_bits(sc) << 32) | (unsigned long long)(0xFFFFFFFFu - lin);
    }
    return o;
}

template <int KPL>
__global__ void __launch_bounds__(512, 4) ray_kernel(RayArgs args)
{
    __shared__ StageLDS S;
    __shared__ float4 PR[MAX_WAVES][PR_ENTRIES];
    extern __shared__ __attribute__((aligned(16))) float PMX[];
    __shared__ RayRec WB[MAX_WAVES];
    __shared__ int s_tile;
    __shared__ int s_dir;  // next unclaimed direction slot of the tile
    const int nw = blockDim.x >> 6;
    const int w = threadIdx.x >> 6;
    const int l = lane_id();
    int cur_frame = -1;
    float myv0 = 0.0f;
    int mytype = -1, myvid = 0;
    // a contiguous run of tiles per workgroup (consecutive tiles share a
    // frame, so it is staged once per run) for all but the last one or two
    // rounds' worth, then the work counter
    const int G = (int)gridDim.x;
    const int R = max(args.n_tiles / G - 1, 0);
    const int n_static = R * G;
    int iter = 0;
    if (threadIdx.x == 0) s_dir = nw;  // read after the loop's first barrier
    while (true) {
        __syncthreads();  // the previous tile is finished
        const RayArgs &a = fresh_args<RayArgs>();
        int t = iter < R ? (int)blockIdx.x * R + iter : n_static;
        if (t >= n_static) {
            if (threadIdx.x == 0) s_tile = n_static + (int)atomicAdd(a.counter, 1u);
            __syncthreads();
            t = uni(s_tile);
        }
        if (t >= a.n_tiles) break;
        ++iter;
        const TileDev tile = a.tiles[t];
        const int f = uni(tile.win), d0 = uni(tile.at);
        if (f != cur_frame) {
            stage_frame(a.P, a.frames[f], a.robots, a.variants, f, S);
            __syncthreads();
            cur_frame = f;
            const int nv = S.n_var;
            myv0 = l < nv ? S.v0[l] : 0.0f;
            mytype = l < nv ? S.type[l] : -1;
            myvid = l < nv ? S.vidx[l] : 0;
        }
        const int n_var = uni(S.n_var);
        const int64_t base = a.frames[f].ray_base;
        const int nd = min(a.tile_dirs, a.n_dirs - d0);
        // the wave's best so far: its key in a uniform register, its record
        // in the wave's LDS slot (written by the lane that holds it)
        unsigned long long wbk = 0ull;
        if (l == 0) {
            WB[w].key = 0ull;
            WB[w].t_team = WB[w].t_opp = WB[w].s_recv = INFINITY;
            WB[w].open_angle = WB[w].refract = WB[w].pad = 0.0f;
        }
        // each wave takes slot w, then claims the tile's next free slot as it
        // finishes one (directions differ in cost: the waves end together)
        for (int slot = w; slot < nd;) {
            const int d = d0 + slot;
            const RayOut o = ray_direction<KPL>(S, PR[w], PMX + w * PM_ROWS * KPL * 64, myv0,
                                                mytype, myvid, d);
            const RayArgs &a = fresh_args<RayArgs>();
            if (l < n_var) {
                const int64_t e = base + (int64_t)d * n_var + myvid;
                if (a.mask) a.mask[e] = (uint8_t)o.feas;
                if (a.score) a.score[e] = o.score;
                if (a.t_team) a.t_team[e] = o.t_team;
                if (a.t_opp) a.t_opp[e] = o.t_opp;
                if (a.s_recv) a.s_recv[e] = o.s_recv;
            }
            const unsigned long long dk = wave_max_u64(o.key);
            if (dk > wbk) {
                wbk = dk;
                const int src = __builtin_ctzll(__ballot(o.key == dk));
                if (l == src) {
                    WB[w].key = dk;
                    WB[w].t_team = o.t_team;
                    WB[w].t_opp = o.t_opp;
                    WB[w].s_recv = o.s_recv;
                    WB[w].open_angle = o.open_angle;
                    WB[w].refract = o.refract;
                }
            }
            int nx = 0;
            if (l == 0) nx = atomicAdd(&s_dir, 1);
            slot = uni(nx);
        }
        // the tile's best of the waves' records (keys of different waves
        // differ unless both are 0); the slot counter is rearmed for the
        // next tile, whose first barrier orders it before any claim
        __syncthreads();
        if (threadIdx.x == 0) s_dir = nw;
        if (w == 0) {
            const unsigned long long k = l < nw ? WB[l].key : 0ull;
            const unsigned long long tk = wave_max_u64(k);
            const unsigned long long at = __ballot(k == tk && l < nw);
            if (l == (int)__builtin_ctzll(at)) a.tile_rec[t] = WB[l];
        }
    }
}

// One workgroup per frame: reduce the frame's tile records into its best
// pass; block 0 also rearms the persistent work counter.
__global__ void __launch_bounds__(256) ray_finalize_kernel(RayArgs a)
{
    __shared__ RayRec red[256];
    const int f = blockIdx.x;
    const int tid = threadIdx.x;
    if (f == 0 && tid == 0) *a.counter = 0u;
    const FrameDev F = a.frames[f];
    RayRec r;
    r.key = 0ull;
    r.t_team = r.t_opp = r.s_recv = INFINITY;
    r.open_angle = r.refract = r.pad = 0.0f;
    for (int k = tid; k < F.tile_count; k += blockDim.x) {
        const RayRec x = a.tile_rec[F.tile_begin + k];
        if (x.key > r.key) r = x;
    }
    red[tid] = r;
    __syncthreads();
    for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
        if (tid < s && red[tid + s].key > red[tid].key) red[tid] = red[tid + s];
        __syncthreads();
    }
    if (tid != 0) return;
    const RayRec b = red[0];
    dpps_ray_best o;
    o.found = 0; o.dir = -1; o.variant = -1; o.type = -1;
    o.theta = 0.0f; o.v0 = 0.0f; o.x = 0.0f; o.y = 0.0f;
    o.score = -INFINITY; o.t_team = INFINITY; o.t_opp = INFINITY;
    o.open_angle = 0.0f; o.refract = 0.0f; o.pad = 0;
    if (b.key != 0ull) {
        const uint32_t lin = 0xFFFFFFFFu - (uint32_t)b.key;
        const int d = (int)(lin / (uint32_t)F.n_variants);
        const int v = (int)(lin - (uint32_t)d * (uint32_t)F.n_variants);
        const dpps_variant var = a.variants[F.variant_off + v];
        const double th = 6.283185307179586476925 * (double)d / (double)a.n_dirs;
        const double xd = 2.0 * (double)d / (double)a.n_dirs;
        const double ux = cospi(xd), uy = sinpi(xd);
        o.found = 1;
        o.dir = d;
        o.variant = v;
        o.type = var.type;
        o.theta = (float)th;
        o.v0 = var.v0;
        o.x = (float)((double)F.ball_x + (double)b.s_recv * ux);
        o.y = (float)((double)F.ball_y + (double)b.s_recv * uy);
        o.score = unordered_bits((uint32_t)(b.key >> 32));
        o.t_team = b.t_team;
        o.t_opp = b.t_opp;
        o.open_angle = b.open_angle;
        o.refract = b.refract;
    }
    a.best[f] = o;
}

template <int KPL>
static int launch_ray_kpl(const RayArgs &a, int waves_per_wg, int grid, hipStream_t st,
                          hipEvent_t e0, hipEvent_t e1)
{
    if (e0) (void)hipEventRecord(e0, st);
    if (a.n_tiles > 0 && grid > 0)
        hipLaunchKernelGGL(ray_kernel<KPL>, dim3(grid), dim3(64 * waves_per_wg),
                           pm_bytes(KPL * 64, waves_per_wg), st, a);
    if (e1) (void)hipEventRecord(e1, st);
    if (a.n_frames > 0)
        hipLaunchKernelGGL(ray_finalize_kernel, dim3(a.n_frames), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_ray(const RayArgs &a, int waves_per_wg, int grid, void *stream, void *ev_start,
               void *ev_stop)
{
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0 = (hipEvent_t)ev_start, e1 = (hipEvent_t)ev_stop;
    switch (a.P.K / 64) {
    case 1: return launch_ray_kpl<1>(a, waves_per_wg, grid, st, e0, e1);
    case 2: return launch_ray_kpl<2>(a, waves_per_wg, grid, st, e0, e1);
    case 3: return launch_ray_kpl<3>(a, waves_per_wg, grid, st, e0, e1);
    case 4: return launch_ray_kpl<4>(a, waves_per_wg, grid, st, e0, e1);
    default: return -2;
    }
}

int ray_occupancy(int K, int waves_per_wg)
{
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    const int bs = 64 * waves_per_wg;
    switch (K / 64) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, ray_kernel<1>, bs, pm_bytes(1 * 64, waves_per_wg)); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, ray_kernel<2>, bs, pm_bytes(2 * 64, waves_per_wg)); break;
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, ray_kernel<3>, bs, pm_bytes(3 * 64, waves_per_wg)); break;
    case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, ray_kernel<4>, bs, pm_bytes(4 * 64, waves_per_wg)); break;
    default: break;
    }
    return e == hipSuccess && n > 0 ? n : 1;
}

// ----------------------------------------------------------------------------
// Shooting decision (Sec. 4.4): the widest open gap of the goal mouth, then
// the opponents' interception along a flat shot through its centre.
// ----------------------------------------------------------------------------

// A kick's ball-time constants in float32.
struct BallTime {
    float split, va1, va2, na1, na2, so2, to2;  // na = -2 a
    __device__ __forceinline__ explicit BallTime(const VarConst &c)
        : split(unif((float)c.split)), va1(unif((float)c.va1)), va2(unif((float)c.va2)),
          na1(unif(-2.0f * (float)c.a1)), na2(unif(-2.0f * (float)c.a2)),
          so2(unif((float)c.soff2)), to2(unif((float)c.toff2))
    {
    }
    __device__ __forceinline__ float at(float s) const
    {
        const bool ph1 = s <= split;
        const float va = ph1 ? va1 : va2;
        const float x = s - (ph1 ? 0.0f : so2);
        const float q = fmaxf(fmaf(ph1 ? na1 : na2, x, va * va), 0.0f);
        return fmaf(2.0f * x, hrcp(va + hsqrt(q)), ph1 ? 0.0f : to2);
    }
};

// Staging of up to SHOT_TILE shooter positions of one frame.
struct ShotLDS {
    double cx[SHOT_TILE], cy[SHOT_TILE], ux[SHOT_TILE], uy[SHOT_TILE], L[SHOT_TILE];
    // each opponent's shadow (start and end angle, empty: start > end), later
    // its bound; the gap behind each shadow and (last) above the lower post
    float s[DPPS_MAX_SIDE][SHOT_TILE], e[DPPS_MAX_SIDE][SHOT_TILE];
    float w[DPPS_MAX_SIDE + 1][SHOT_TILE];
    float lo[SHOT_TILE], hi[SHOT_TILE];
    float tb[4][SHOT_TILE];                      // latest ball time of each quarter
    int blocked[SHOT_TILE];                      // the position is inside an opponent
    dpps_shot rec[SHOT_TILE];
    float4 fr[SHOT_TILE][DPPS_MAX_SIDE + 1];     // opponents by ascending bound (a column
    float sl[SHOT_TILE][DPPS_MAX_SIDE + 1];      // more: rows on different banks)
};

// The least, over the lane's samples, of the opponents' earliest arrival less
// the ball's time; lanes of one half share a position (row of H) and have its
// least slack.  Opponents are taken by ascending lower bound on the slack they
// leave; one whose bound is not below the slack so far cannot lower it, nor
// can those after it (every rounding in between is monotone): they are left
// out.  1.8 of 8 opponents per position are evaluated on average.
template <int KPH, bool CLAMP>
__device__ __forceinline__ float shot_slack(const ShotLDS &H, const RobotK &rk, const BallTime &bt,
                                            float D, float A, float invA2, int n_op, int p)
{
    const int hl = lane_id() & 31;
    const float Lf = (float)H.L[p], LA = (float)(H.L[p] * (double)A);
    float fs[KPH], tb[KPH];
#pragma unroll
    for (int q = 0; q < KPH; ++q) {
        fs[q] = (float)(q * 32 + hl + 1) * (1.0f / (float)(KPH * 32));
        const float sk = fs[q] * Lf;
        const float t = bt.at(sk);
        tb[q] = sk <= D ? t : -INFINITY;  // past the ball's reach: no slack
    }
    const float bound = hl < n_op ? H.sl[p][hl] : INFINITY;
    float m = INFINITY;
    for (int j = 0; j < n_op; ++j) {
        const float4 r = H.fr[p][j];
#pragma unroll
        for (int q = 0; q < KPH; ++q) {
            const float d = robot_time_h<CLAMP>(r, fs[q], LA, rk) * invA2 - tb[q];
            m = fminf(m, d);
        }
        m = half_min(m);
        if (__ballot(hl > j && bound < m) == 0ull) break;
    }
    return m;
}

// A lone position's decision (a frame's ball), by one wave from the staged
// frame; the lanes of the record agree.  The same operations as the tiles'
// below, but with the opponents' values in lanes instead of LDS rows (the loops
// over them are lane reads, not waits for LDS), the quarters' bounds spread over
// the lanes too and the samples over the whole wave.  Where only the balls are
// asked for, the call waits for this chain and not for the ALUs: 10 balls at K =
// 256 take 11.1 us as tiles of one, 7.2 this way (the call 16.0 and 13.8), 1000
// balls 37.1 and 32.3 a call.
template <int KPH, bool CLAMP>
__device__ __forceinline__ float lone_slack(const RobotK &rk, const BallTime &bt, const float4 &fr,
                                            float bound, int rank, int n_op, float Lf, float LA,
                                            float D, float invA2)
{
    const int l = lane_id();
    float fs[KPH / 2], tb[KPH / 2];
#pragma unroll
    for (int q = 0; q < KPH / 2; ++q) {
        fs[q] = (float)(q * 64 + l + 1) * (1.0f / (float)(KPH * 32));
        const float sk = fs[q] * Lf;
        const float t = bt.at(sk);
        tb[q] = sk <= D ? t : -INFINITY;  // past the ball's reach: no slack
    }
    float m = INFINITY;
    for (int j = 0; j < n_op; ++j) {
        const int o = __builtin_ctzll(__ballot(l < n_op && rank == j));
        const float4 r = make_float4(readlane_f(fr.x, o), readlane_f(fr.y, o), readlane_f(fr.z, o),
                                     readlane_f(fr.w, o));
#pragma unroll
        for (int q = 0; q < KPH / 2; ++q)
            m = fminf(m, robot_time_h<CLAMP>(r, fs[q], LA, rk) * invA2 - tb[q]);
        m = wave_min_dpp(m);
        if (__ballot(l < n_op && rank > j && bound < m) == 0ull) break;
    }
    return m;
}

template <int KPH>
__device__ __forceinline__ dpps_shot shot_lone(const StageLDS &S, const DevParams &P, double cx,
                                               double cy, float min_angle, float margin)
{
    const int l = lane_id();
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
    // shadows: lanes are opponents, then the posts
    const float fx = (float)cx, fy = (float)cy;
    const float dxf = fmaxf(P.goal_x - fx, P.goal_eps);
    const float4 r = S.rob[n_tm + (l < n_op ? l : 0)];
    const float ox = r.x - fx, oy = r.y - fy;
    const float Y = l < n_op ? oy : (l == n_op ? -P.half_goal_w - fy : P.half_goal_w - fy);
    const float X = l < n_op ? ox : dxf;
    const float ang = atan2f(Y, X);
    const float lo = readlane_f(ang, n_op), hi = readlane_f(ang, n_op + 1);
    const bool valid = l < n_op && r.x < P.goal_x;
    const float rho2 = fmaf(ox, ox, oy * oy);
    const bool blocked = __ballot(valid && rho2 <= P.R * P.R) != 0ull;
    const float al = asinf(fminf(P.R * rsq(fmaxf(rho2, 1e-30f)), 1.0f));
    const float s = fmaxf(ang - al, lo), e = fminf(ang + al, hi);
    const bool has = valid && e > s;
    // the gap behind each shadow, and (lane n_op) above the lower post
    const float st = l < n_op ? e : lo;
    bool cov = false;
    float nxt = hi;
    for (unsigned long long m = __ballot(has); m; m &= m - 1) {
        const int k = __builtin_ctzll(m);
        const float sk = readlane_f(s, k), ek = readlane_f(e, k);
        cov = cov || (sk <= st && ek > st);
        nxt = sk > st ? fminf(nxt, sk) : nxt;
    }
    const float w = (has || l == n_op) && !cov && !blocked ? fmaxf(nxt - st, 0.0f) : 0.0f;
    // widest gap (ties to the lower start) and the sum of the gaps
    float gap = 0.0f, g0 = lo, open = 0.0f;
    for (unsigned long long m = __ballot(w > 0.0f); m; m &= m - 1) {
        const int k = __builtin_ctzll(m);
        const float wk = readlane_f(w, k), sk = readlane_f(st, k);
        open += wk;
        if (wk > gap || (wk == gap && sk < g0)) {
            gap = wk;
            g0 = sk;
        }
    }
    const double dxg = fmax((double)P.goal_x - cx, (double)P.goal_eps);
    const float aim = gap > 0.0f ? fmaf(0.5f, gap, g0) : atan2f(-fy, (float)dxg);
    const double ux = (double)cosf(aim), uy = (double)sinf(aim);
    const double L = dxg / ux;
    const float Lf = (float)L;
    const VarConst &vc = S.vc[0];  // the shot: the frame's only variant
    const BallTime bt(vc);
    const float D = unif((float)vc.D);
    // lane (o, k): opponent o's bound over quarter k, then the least over k
    const int o = l & 15;
    const float k = (float)(l >> 4);
    const float s1 = fminf(0.25f * (k + 1.0f) * Lf * (1.0f + 1.0f / 1048576.0f), D);
    const bool in = 0.25f * k * Lf * (1.0f - 1.0f / 1048576.0f) <= D;
    const float tb = in ? bt.at(s1) * (1.0f + 1.0f / 65536.0f) : -INFINITY;
    const RobotK rk(P);
    const double LA = L * (double)P.A, q0 = 0.25 * LA * (double)k;
    double tq, qq, wn;
    const float4 fr = robot_frame(S.rob[n_tm + (o < n_op ? o : 0)], (double)P.A, cx, cy, ux, uy, tq,
                                  qq, wn);
    const float lb = arrival_bound(rk, tq, qq, fr.z, (float)wn, q0, q0 + 0.25 * LA);
    float bd = fmaf(lb * (1.0f - 1.0f / 65536.0f), P.invA2, -tb);
    bd = fminf(bd, __shfl_xor(bd, 16, 64));
    bd = fminf(bd, __shfl_xor(bd, 32, 64));
    const uint32_t key = ordered_bits(bd);
    int rank = 0;
    for (int j = 0; j < n_op; ++j) {
        const uint32_t y = (uint32_t)readlane_i((int)key, j);
        rank += y < key || (y == key && j < o);
    }
    const float m =
        uni(S.vel_ok)
            ? lone_slack<KPH, false>(rk, bt, fr, bd, rank, n_op, Lf, (float)LA, D, P.invA2)
            : lone_slack<KPH, true>(rk, bt, fr, bd, rank, n_op, Lf, (float)LA, D, P.invA2);
    dpps_shot res;
    res.reachable = L <= vc.D;
    res.aim = aim;
    res.gap = gap;
    res.open_angle = open;
    res.length = Lf;
    res.t_goal = res.reachable ? (float)ball_time64(vc, L) : INFINITY;
    res.slack = m;
    res.shoot = gap >= min_angle && res.reachable && m > margin;
    return res;
}

// The balls alone: one wave per frame.
template <int KPH, bool INL>
__global__ void __launch_bounds__(64) shot_ball_kernel(ShotLaunch launch)
{
    __shared__ StageLDS S;
    const ShotArgs &a = launch.a;
    const OneFrame &one = fresh_args<ShotLaunch>().one;
    const int f = blockIdx.x;
    stage_frame(a.P, INL ? one.frame : a.frames[f], INL ? one.robots : a.robots,
                INL ? one.variants : a.variants, f, S);
    wave_lds_sync();
    const dpps_shot r = shot_lone<KPH>(S, a.P, (double)unif(S.bx), (double)unif(S.by), a.min_angle,
                                       a.margin);
    if (threadIdx.x == 0) a.ball[f] = r;
}

// Shooting decisions of one frame per workgroup: a tile of its window's
// points, or (the first n_frames workgroups) its ball, as a tile of one.
//
// Bound by VALU issue.  What differs by position and opponent -- the shadow's
// angles, the opponent in the shot's frame, its bounds -- has a lane per
// (position, opponent), and what differs by position only -- the widest gap,
// the aim's sine and cosine, the path's length -- a lane per position, rather
// than a wave per position with a lane per opponent; the samples of two
// positions share a wave, one per half.  The bounds are on the slack of each
// quarter of the path.  241 x 181 positions, 8 opponents, K = 256:
// 84 -> 35 us (profiled), the whole call 51 -> 18 us.  Tiles of 16: 35 us too,
// but 64 frames of 61 x 46 positions 197 us a call against 176.
template <int KPH, bool INL>
__global__ void __launch_bounds__(256) shot_kernel(ShotLaunch launch)
{
    __shared__ StageLDS S;
    __shared__ ShotLDS H;
    const ShotArgs &a = launch.a;
    const OneFrame &one = fresh_args<ShotLaunch>().one;
    const int tid = threadIdx.x, nt = blockDim.x;
    const bool map = (int)blockIdx.x >= a.n_frames;
    const int t = map ? (int)blockIdx.x - a.n_frames : (int)blockIdx.x;
    WinDev W = {};
    int f = t, p0 = 0, np = 1;
    if (map) {
        const TileDev tile = INL ? TileDev{0, t} : a.tiles[t];
        W = INL ? one.win : a.wins[tile.win];
        f = W.frame;
        p0 = tile.at * SHOT_TILE;
        np = min(SHOT_TILE, W.npts - p0);
    }
    const FrameDev F = INL ? one.frame : a.frames[f];
    stage_frame(a.P, F, INL ? one.robots : a.robots, INL ? one.variants : a.variants, f, S);
    // (the last threads: the first wave stages the frame)
    for (int p = nt - 1 - tid; p < np; p += nt) {
        const int j = map ? (p0 + p) / W.nx : 0, i = p0 + p - j * W.nx;
        H.cx[p] = map ? (double)W.h * ((double)(W.i0 + i) - (double)W.halfNx) : (double)F.ball_x;
        H.cy[p] = map ? (double)W.h * ((double)(W.j0 + j) - (double)W.halfNy) : (double)F.ball_y;
        H.blocked[p] = 0;
    }
    __syncthreads();
    const DevParams &P = a.P;
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
    // pairs (position, row): a power of two of lanes per row
    const int sh = np > 1 ? 32 - __builtin_clz(np - 1) : 0, pm = (1 << sh) - 1;
    // Shadows seen from the position: angle of the opponent, -+ asin(R / distance)
    // (rows n_op and n_op + 1: the posts).
    for (int x = tid; x < (n_op + 2) << sh; x += nt) {
        const int p = x & pm, o = x >> sh;
        if (p >= np) continue;
        const float cx = (float)H.cx[p], cy = (float)H.cy[p];
        const float dxg = fmaxf(P.goal_x - cx, P.goal_eps);
        const float4 r = S.rob[n_tm + (o < n_op ? o : 0)];
        const float ox = r.x - cx, oy = r.y - cy;
        const float Y = o < n_op ? oy : (o == n_op ? -P.half_goal_w - cy : P.half_goal_w - cy);
        const float X = o < n_op ? ox : dxg;
        const float ang = atan2f(Y, X);
        if (o >= n_op) {
            (o == n_op ? H.lo : H.hi)[p] = ang;
            continue;
        }
        const bool valid = r.x < P.goal_x;
        const float rho2 = fmaf(ox, ox, oy * oy);
        if (valid && rho2 <= P.R * P.R) H.blocked[p] = 1;
        const float al = asinf(fminf(P.R * rsq(fmaxf(rho2, 1e-30f)), 1.0f));
        H.s[o][p] = valid ? ang - al : INFINITY;
        H.e[o][p] = valid ? ang + al : -INFINITY;
    }
    __syncthreads();
    // Gap behind each shadow within the mouth, and above the lower post (row
    // n_op): none if another shadow covers its start, else up to the next
    // shadow's start or the upper post.
    for (int x = tid; x < (n_op + 1) << sh; x += nt) {
        const int p = x & pm, o = x >> sh;
        if (p >= np) continue;
        const float lo = H.lo[p], hi = H.hi[p];
        bool cand = true;
        float st = lo;
        if (o < n_op) {
            st = fminf(H.e[o][p], hi);
            cand = st > fmaxf(H.s[o][p], lo);
        }
        bool cov = false;
        float nxt = hi;
        for (int k = 0; k < n_op; ++k) {
            const float sk = fmaxf(H.s[k][p], lo), ek = fminf(H.e[k][p], hi);
            const bool has = ek > sk;
            cov = cov || (has && sk <= st && ek > st);
            nxt = has && sk > st ? fminf(nxt, sk) : nxt;
        }
        H.w[o][p] = cand && !cov ? fmaxf(nxt - st, 0.0f) : 0.0f;
    }
    __syncthreads();
    const VarConst &vc = S.vc[0];  // the shot: the frame's only variant
    const BallTime bt(vc);
    const float D = unif((float)vc.D);
    for (int p = tid; p < np; p += nt) {
        const double cx = H.cx[p], cy = H.cy[p];
        const float lo = H.lo[p], hi = H.hi[p];
        // widest gap (ties to the lower start) and the sum of the gaps
        float gap = 0.0f, g0 = lo, open = 0.0f;
        if (!H.blocked[p]) {
            for (int o = 0; o <= n_op; ++o) {
                const float wk = H.w[o][p];
                const float sk = o < n_op ? fminf(H.e[o][p], hi) : lo;
                open += wk;
                if (wk > gap || (wk == gap && wk > 0.0f && sk < g0)) {
                    gap = wk;
                    g0 = sk;
                }
            }
        }
        const double dxg = fmax((double)P.goal_x - cx, (double)P.goal_eps);
        const float aim = gap > 0.0f ? fmaf(0.5f, gap, g0) : atan2f(-(float)cy, (float)dxg);
        const double ux = (double)cosf(aim), uy = (double)sinf(aim);
        const double L = dxg / ux;
        const float Lf = (float)L;
        H.ux[p] = ux;
        H.uy[p] = uy;
        H.L[p] = L;
        // Latest ball time over each quarter's samples, raised by 2^-16 for the
        // float form's roundings; -inf where the ball stops before the quarter.
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const float s1 = fminf(0.25f * (float)(b + 1) * Lf * (1.0f + 1.0f / 1048576.0f), D);
            const bool in = 0.25f * (float)b * Lf * (1.0f - 1.0f / 1048576.0f) <= D;
            H.tb[b][p] = in ? bt.at(s1) * (1.0f + 1.0f / 65536.0f) : -INFINITY;
        }
        dpps_shot r;
        r.reachable = L <= vc.D;
        r.aim = aim;
        r.gap = gap;
        r.open_angle = open;
        r.length = Lf;
        r.t_goal = r.reachable ? (float)ball_time64(vc, L) : INFINITY;
        r.slack = INFINITY;
        r.shoot = 0;
        H.rec[p] = r;
    }
    __syncthreads();
    // The opponents in the shot's frame and their bounds: on the arrival over
    // each quarter (shaved by 2^-16) less the latest ball time there.
    const RobotK rk(P);
    float4 fr[2];  // 16 x 32 pairs on 256 threads
    float bd[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int x = tid + q * nt, p = x & pm, o = x >> sh;
        if (o >= n_op || p >= np) continue;
        double tq, qq, wn;
        const double ux = H.ux[p], uy = H.uy[p], LA = H.L[p] * (double)P.A;
        fr[q] = robot_frame(S.rob[n_tm + o], (double)P.A, H.cx[p], H.cy[p], ux, uy, tq, qq,
                            wn);
        float b = INFINITY;
        for (int k = 0; k < 4; ++k) {
            const double s0 = 0.25 * LA * (double)k;
            const float lb = arrival_bound(rk, tq, qq, fr[q].z, (float)wn, s0, s0 + 0.25 * LA);
            b = fminf(b, fmaf(lb * (1.0f - 1.0f / 65536.0f), P.invA2, -H.tb[k][p]));
        }
        bd[q] = b;
        H.s[o][p] = b;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int x = tid + q * nt, p = x & pm, o = x >> sh;
        if (o >= n_op || p >= np) continue;
        const uint32_t key = ordered_bits(bd[q]);
        int rank = 0;
        for (int k = 0; k < n_op; ++k) {
            const uint32_t y = ordered_bits(H.s[k][p]);
            rank += y < key || (y == key && k < o);
        }
        H.fr[p][rank] = fr[q];
        H.sl[p][rank] = bd[q];
    }
    __syncthreads();
    const int h = lane_id() >> 5;
    for (int p2 = 2 * (tid >> 6); p2 < np; p2 += 2 * (nt >> 6)) {
        const int p = min(p2 + h, np - 1);
        const float m = uni(S.vel_ok)
                            ? shot_slack<KPH, false>(H, rk, bt, D, P.A, P.invA2, n_op, p)
                            : shot_slack<KPH, true>(H, rk, bt, D, P.A, P.invA2, n_op, p);
        if ((tid & 31) == 0 && p2 + h < np) {
            H.rec[p].slack = m;
            H.rec[p].shoot = H.rec[p].gap >= a.min_angle && H.rec[p].reachable && m > a.margin;
        }
    }
    __syncthreads();
    static_assert(sizeof(dpps_shot) == 32, "eight words");
    int *const out = (int *)(map ? a.map + W.out_base + p0 : a.ball + f);
    for (int x = tid; x < 8 * np; x += nt) out[x] = ((const int *)H.rec)[x];
}

// Workgroups of four waves, one per frame's ball and tile; the balls alone in a
// kernel of their own.  (With the balls beside a map by that kernel's way, maps
// of 64 frames at K = 256 took 120.4 us a call instead of 117.8.)
template <int KPH, bool INL>
static void launch_shot_kph(const ShotLaunch &s, hipStream_t st)
{
    const dim3 grid(s.a.n_frames + (s.a.map ? s.a.n_tiles : 0));
    if (s.a.map)
        hipLaunchKernelGGL((shot_kernel<KPH, INL>), grid, dim3(256), 0, st, s);
    else
        hipLaunchKernelGGL((shot_ball_kernel<KPH, INL>), grid, dim3(64), 0, st, s);
}

template <bool INL>
static int launch_shot_inl(const ShotLaunch &s, hipStream_t st)
{
    switch (s.a.P.K / 64) {
    case 1: launch_shot_kph<2, INL>(s, st); break;
    case 2: launch_shot_kph<4, INL>(s, st); break;
    case 3: launch_shot_kph<6, INL>(s, st); break;
    case 4: launch_shot_kph<8, INL>(s, st); break;
    default: return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_shot(const ShotLaunch &s, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (s.a.n_frames <= 0) return 0;
    return s.one.on ? launch_shot_inl<true>(s, st) : launch_shot_inl<false>(s, st);
}

// ----------------------------------------------------------------------------
// Running points (Sec. 5.2): five criteria per zone vertex, weighted (Eq. 4);
// lanes are points, the opponents are looped over from LDS.
// ----------------------------------------------------------------------------

// Arrival time (A T / 2) of staged robot r = (x, y, vx, vy) at (px, py): the
// scaled model of robot_time_h with the offset taken directly.
__device__ __forceinline__ float robot_time_pt(const DevParams &P, float4 r, float px, float py)
{
    const float dx = (px - r.x) * P.A, dy = (py - r.y) * P.A;
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, 1e-30f));
    const float inv = rsq(r2);
    const float del = fmaxf(fmaf(r2, inv, -P.RA), 0.0f);
    float u = fmaf(dx, r.z, dy * r.w) * (0.70710678118654752f * inv);
    u = med3(u, -P.Vh, P.Vh);
    const float ss = u * fabsf(u);  // its magnitude is u^2 (the add's abs modifier)
    const bool over = ss >= del;
    const float Dp = fabsf(ss) + (over ? -del : del);
    const float sg = over ? u : -u;
    const float rh = Dp > P.V2 ? fmaf(Dp, P.inv2V, P.halfV) : hsqrt(Dp);
    return fmaf(sg, 0.70710678118654752f, rh);
}

// Entry parameter of the segment from c along (dx, dy) into the rectangle
// [x0, x1] x [y0, y1] that holds its end point (slab form, FP64: a segment
// that grazes an edge must be decided as the oracle decides it).
__device__ __forceinline__ double slab_enter(double cx, double cy, double dx, double dy,
                                             double x0, double x1, double y0, double y1)
{
    // the slab's near side chosen before the one division per axis (the
    // same quotients; lanes whose dy signs differ share one division)
    double t = 0.0;
    if (dx != 0.0) t = fmax(t, ((dx > 0.0 ? x0 : x1) - cx) / dx);
    if (dy != 0.0) t = fmax(t, ((dy > 0.0 ? y0 : y1) - cy) / dy);
    return fmin(t, 1.0);
}

// The same for a rectangle that need not hold the end point: 1, the end, when
// the segment passes it by (the entry by the slabs is then not on its edge).
__device__ __forceinline__ double slab_enter_or_end(double cx, double cy, double dx, double dy,
                                                    double x0, double x1, double y0, double y1)
{
    double tx = 0.0, ty = 0.0;
    if (dx != 0.0) tx = fmax(tx, ((dx > 0.0 ? x0 : x1) - cx) / dx);
    if (dy != 0.0) ty = fmax(ty, ((dy > 0.0 ? y0 : y1) - cy) / dy);
    const double t = fmax(tx, ty), x = cx + t * dx, y = cy + t * dy;
    const bool in_x = x >= x0 && x <= x1, in_y = y >= y0 && y <= y1;
    const bool met = t == 0.0 ? in_x && in_y : (t == tx && in_y) || (t == ty && in_x);
    return met ? fmin(t, 1.0) : 1.0;
}

// What the points of a zone share: the opponents (bit o) that can be the
// earliest at some place that P or Q can take, and those within the marking
// radius of some point of the zone.
struct RunZone {
    uint32_t guard, mark;
};

// Lanes are opponents.  P and Q lie in the rectangle as deep as the defense
// area and as wide as the area or the goal, whichever is wider (a segment that
// passes a narrow area by ends at a post beside it), so an opponent whose
// arrival bound over that rectangle is past the latest arrival of another one
// anywhere in it never sets t_P or t_Q.  With D the least and E the greatest
// distance to the rectangle (widened by 1 mm, and by 2^-20 of its coordinates
// and the robot's, for the rounding of P and Q and of the differences), less
// the radius, both scaled by amax: whatever its velocity the
// robot needs at least sqrt(D / 2) (D <= vmax^2 / 2) or D / 2vmax + vmax / 4,
// and at most the time when it first stops moving away at its full speed,
// |w| / sqrt 2 + R(|w|^2 + E), in the robot stage's units; 2^-12 apart for
// rounding.  About three of eight opponents are left in random frames.  The
// marking weight is 0 beyond mark_radius.
__device__ __forceinline__ RunZone run_zone(const StageLDS &S, const DevParams &P,
                                            const dpps_run_params &R, const WinDev &W, int ny,
                                            int n_tm, int n_op)
{
    const int l = lane_id();
    const float4 r = S.rob[n_tm + (l < n_op ? l : 0)];
    const float x0 = P.goal_x - R.def_depth, x1 = P.goal_x;
    const float hw = fmaxf(0.5f * R.def_width, P.half_goal_w);
    const float wide = 1e-3f + (fabsf(x0) + fabsf(x1) + hw + fabsf(r.x) + fabsf(r.y)) *
                                   (1.0f / 1048576.0f);
    const float nx = fmaxf(fmaxf(x0 - r.x, r.x - x1), 0.0f), nyd = fmaxf(fabsf(r.y) - hw, 0.0f);
    const float fx = fmaxf(fabsf(r.x - x0), fabsf(r.x - x1)), fy = fabsf(r.y) + hw;
    const float D = P.A * fmaxf(hsqrt(fmaf(nx, nx, nyd * nyd)) - wide - P.R, 0.0f);
    const float E = P.A * (hsqrt(fmaf(fx, fx, fy * fy)) + wide);
    const float w2 = fminf(0.5f * fmaf(r.z, r.z, r.w * r.w), 0.5f * P.V2);
    const float F = w2 + E;
    float lb = D <= 0.5f * P.V2 ? hsqrt(0.5f * D) : fmaf(D, P.inv2V, 0.25f * P.V);
    float ub = fmaf(0.70710678118654752f, hsqrt(w2),
                    F > P.V2 ? fmaf(F, P.inv2V, P.halfV) : hsqrt(F));
    lb *= 1.0f - 1.0f / 4096.0f;
    ub = l < n_op ? ub * (1.0f + 1.0f / 4096.0f) : INFINITY;
    const float latest = wave_min_dpp(ub);
    // the zone's rectangle
    const float zx0 = W.h * ((float)W.i0 - W.halfNx), zx1 = W.h * ((float)(W.i0 + W.nx - 1) - W.halfNx);
    const float zy0 = W.h * ((float)W.j0 - W.halfNy), zy1 = W.h * ((float)(W.j0 + ny - 1) - W.halfNy);
    const float mx = fmaxf(fmaxf(zx0 - r.x, r.x - zx1), 0.0f);
    const float my = fmaxf(fmaxf(zy0 - r.y, r.y - zy1), 0.0f);
    RunZone z;
    z.guard = (uint32_t)__ballot(l < n_op && lb <= latest);
    z.mark = (uint32_t)__ballot(l < n_op && hsqrt(fmaf(mx, mx, my * my)) - 1e-3f <= R.mark_radius);
    return z;
}

// The five criteria and the score at (cx, cy); returns -inf inside the
// defense area (crit untouched).  ball2: each opponent's squared distance to
// the ball.
__device__ __forceinline__ float run_eval(const StageLDS &S, const DevParams &P,
                                          const dpps_run_params &R, const double *ball2,
                                          const RunZone &z, double cx, double cy, int n_tm,
                                          int n_op, float (&crit)[5])
{
    const double x0d = (double)P.goal_x - (double)R.def_depth;
    const double hwd = 0.5 * (double)R.def_width;
    if (cx > x0d && cx < (double)P.goal_x && cy > -hwd && cy < hwd) return -INFINITY;
    const float fx = (float)cx, fy = (float)cy;
    // the offset to the goal centre in FP64, then rounded once: its sign
    // decides the bearing's branch for points on the goal line
    const float gx = (float)((double)P.goal_x - cx), gy = (float)(-cy);
    crit[0] = fmaf(-sqrtf(fmaf(gx, gx, gy * gy)), P.inv_dist_norm, 1.0f);
    const double bx = cx - (double)S.bx, by = cy - (double)S.by;
    const double db2 = bx * bx + by * by;
    crit[1] = fminf(sqrtf((float)db2) / R.ball_norm, 1.0f);
    const float phi = fabsf(atan2f(gy, gx));
    const float off = phi < R.ang_lo ? R.ang_lo - phi : (phi > R.ang_hi ? phi - R.ang_hi : 0.0f);
    crit[2] = fmaxf(1.0f - off / R.ang_fall, 0.0f);
    const double gxd = (double)P.goal_x - cx, hwg = (double)P.half_goal_w;
    const double dpy = hwg - cy, dqy = -hwg - cy;
    double tp_, tq_;
    if (hwd < hwg) {  // an area narrower than the goal
        tp_ = slab_enter_or_end(cx, cy, gxd, dpy, x0d, (double)P.goal_x, -hwd, hwd);
        tq_ = slab_enter_or_end(cx, cy, gxd, dqy, x0d, (double)P.goal_x, -hwd, hwd);
    } else {
        tp_ = slab_enter(cx, cy, gxd, dpy, x0d, (double)P.goal_x, -hwd, hwd);
        tq_ = slab_enter(cx, cy, gxd, dqy, x0d, (double)P.goal_x, -hwd, hwd);
    }
    const float px = (float)(cx + tp_ * gxd), py = (float)(cy + tp_ * dpy);
    const float qx = (float)(cx + tq_ * gxd), qy = (float)(cy + tq_ * dqy);
    float tP = INFINITY, tQ = INFINITY;
    for (uint32_t m = z.guard; m; m &= m - 1) {
        const float4 r = S.rob[n_tm + __builtin_ctz(m)];
        tP = fminf(tP, robot_time_pt(P, r, px, py));
        tQ = fminf(tQ, robot_time_pt(P, r, qx, qy));
    }
    // the largest marking weight is that of the nearest opponent that counts
    // (sqrt, division and subtraction are monotone)
    float near2 = INFINITY;
    for (uint32_t m = z.mark; m; m &= m - 1) {
        const int o = __builtin_ctz(m);
        const float4 r = S.rob[n_tm + o];
        const float ex = r.x - fx, ey = r.y - fy;
        near2 = ball2[o] < db2 ? fminf(near2, fmaf(ex, ex, ey * ey)) : near2;
    }
    const float mark = fmaxf(1.0f - sqrtf(near2) / R.mark_radius, 0.0f);
    crit[3] = n_op > 0 ? fminf((tP * P.invA2 + tQ * P.invA2) / R.guard_norm, 1.0f) : 1.0f;
    crit[4] = 1.0f - mark;
    return fmaf(R.w_goal, crit[0],
                fmaf(R.w_ball, crit[1],
                     fmaf(R.w_angle, crit[2], fmaf(R.w_guard, crit[3], R.w_defense * crit[4]))));
}

// One workgroup per zone, lanes = points.  Bound by VALU issue (float64
// geometry, three divisions and the transcendentals of a point, two arrival
// times per opponent): the opponents that cannot matter in the zone are left
// out, squared ball distances are formed once, the marking weight once per
// point from the nearest opponent, and the best point's criteria stay with
// its lane instead of being computed again.  2048 frames x 4 zones (10.2 M
// points): 318 -> 178 us.
__global__ void __launch_bounds__(1024) run_kernel(RunArgs a)
{
    __shared__ StageLDS S;
    __shared__ double ball2[DPPS_MAX_SIDE];
    __shared__ unsigned long long red[16];
    const DevParams &P = a.P;
    const WinDev W = a.wins[blockIdx.x];
    stage_frame(P, a.frames[W.frame], a.robots, a.variants, W.frame, S);
    __syncthreads();
    const int n_tm = uni(S.n_tm), n_op = uni(S.n_op);
    if ((int)threadIdx.x < n_op) {
        const float4 r = S.rob[n_tm + threadIdx.x];
        const double ox = (double)r.x - (double)S.bx, oy = (double)r.y - (double)S.by;
        ball2[threadIdx.x] = ox * ox + oy * oy;
    }
    const int ny = W.nx > 0 ? W.npts / W.nx : 0;
    const RunZone z = run_zone(S, P, a.R, W, ny, n_tm, n_op);
    __syncthreads();
    unsigned long long best = 0ull;
    float bc[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int p = threadIdx.x; p < W.npts; p += blockDim.x) {
        const int j = (int)((unsigned)p / (unsigned)W.nx), i = p - j * W.nx;
        const double cx = (double)W.h * ((double)(W.i0 + i) - (double)W.halfNx);
        const double cy = (double)W.h * ((double)(W.j0 + j) - (double)W.halfNy);
        float crit[5];
        const float sc = run_eval(S, P, a.R, ball2, z, cx, cy, n_tm, n_op, crit);
        if (a.score) a.score[W.out_base + p] = sc;
        if (sc > -INFINITY) {
            const unsigned long long k = ((unsigned long long)ordered_bits(sc) << 32) |
                                         (unsigned long long)(0xFFFFFFFFu - (uint32_t)p);
            if (k > best) {
                best = k;
#pragma unroll
                for (int q = 0; q < 5; ++q) bc[q] = crit[q];
            }
        }
    }
    const unsigned long long wb = wave_max_u64(best);
    if (lane_id() == 0) red[threadIdx.x >> 6] = wb;
    __syncthreads();
    unsigned long long top = red[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) top = red[w] > top ? red[w] : top;
    // the lane that holds the best point (keys are unique), or the first
    // thread when no point is usable
    if (top != 0ull ? best != top : threadIdx.x != 0) return;
    dpps_run_best r;
    r.found = 0; r.i = -1; r.j = -1; r.reserved = 0;
    r.x = 0.0f; r.y = 0.0f; r.score = -INFINITY;
    r.goal = r.ball = r.angle = r.guard = r.defense = 0.0f;
    if (top != 0ull) {
        const int p = (int)(0xFFFFFFFFu - (uint32_t)top);
        const int j = p / W.nx, i = p - j * W.nx;
        r.score = unordered_bits((uint32_t)(top >> 32));
        r.found = 1; r.i = i; r.j = j;
        r.x = (float)((double)W.h * ((double)(W.i0 + i) - (double)W.halfNx));
        r.y = (float)((double)W.h * ((double)(W.j0 + j) - (double)W.halfNy));
        r.goal = bc[0]; r.ball = bc[1]; r.angle = bc[2]; r.guard = bc[3];
        r.defense = bc[4];
    }
    a.best[blockIdx.x] = r;
}

// Threads per zone: 256 where the zones fill the chip; twice and four times as
// many for up to two zones and one a CU, where a call waits for one zone's
// points (4 frames x 4 zones of 1200 points, 11 opponents: 29.4 us a call with
// 256, 22.4 with 512, 20.1 with 1024; one opponent 20.4, 16.7 and 16.2; 100
// frames, 400 zones: 52.0, 45.6 with 512; 130 frames, 520 zones, 53.5 with any).
int launch_run(const RunArgs &a, int n_cu, void *stream)
{
    const int threads = a.n_wins <= n_cu ? 1024 : a.n_wins <= 2 * n_cu ? 512 : 256;
    if (a.n_wins > 0)
        hipLaunchKernelGGL(run_kernel, dim3(a.n_wins), dim3(threads), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Clears n words (one thread each): a kernel rather than a memset node, so
// that a caller may capture it in a graph.
__global__ void __launch_bounds__(64) zero_words_kernel(uint32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

int launch_zero_words(uint32_t *p, int n, void *stream)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(zero_words_kernel, dim3((n + 63) / 64), dim3(64), 0, (hipStream_t)stream,
                       p, n);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_search(const SearchLaunch &s, int waves_per_wg, int grid, void *stream, void *ev_start,
                  void *ev_stop)
{
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0 = (hipEvent_t)ev_start, e1 = (hipEvent_t)ev_stop;
    switch (s.a.P.K / 64) {
    case 1: return launch_kpl<1>(s, waves_per_wg, grid, st, e0, e1);
    case 2: return launch_kpl<2>(s, waves_per_wg, grid, st, e0, e1);
    case 3: return launch_kpl<3>(s, waves_per_wg, grid, st, e0, e1);
    case 4: return launch_kpl<4>(s, waves_per_wg, grid, st, e0, e1);
    default: return -2;
    }
}

template <int KPL>
static int occupancy_kpl(int block, size_t lds, bool best)
{
    int n = 0;
    const hipError_t e =
        best ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, search_kernel<2 * KPL, false, true>,
                                                            block, lds)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, search_kernel<2 * KPL, false, false>,
                                                            block, lds);
    return e == hipSuccess && n > 0 ? n : 1;
}

int search_occupancy(int K, int waves_per_wg, int tile_points, int max_variants, bool best)
{
    const int bs = 64 * waves_per_wg;
    const size_t lds = search_lds_bytes(K, waves_per_wg, tile_points, max_variants);
    switch (K / 64) {
    case 1: return occupancy_kpl<1>(bs, lds, best);
    case 2: return occupancy_kpl<2>(bs, lds, best);
    case 3: return occupancy_kpl<3>(bs, lds, best);
    case 4: return occupancy_kpl<4>(bs, lds, best);
    default: return 1;
    }
}

}  // namespace dpps
