// Device helpers shared by the uniform-tree kernels (kernels.hip) and the adaptive-tree
// kernels (adaptive.hip): complex arithmetic on float2 / double2, the near-field
// particle records, the regularised pair kernel of the near field, and its mutual form
// for pairs of dense same-level leaves.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "fmm_internal.h"

namespace fmm {

constexpr double kInv2Pi = 0.15915494309189533576888376337251;

// ---------------------------------------------------------------------------------
// Small complex helpers on float2 / double2
// ---------------------------------------------------------------------------------
template <typename T> struct Vec2;
template <> struct Vec2<float> { using type = float2; };
template <> struct Vec2<double> { using type = double2; };
template <typename T> using c2 = typename Vec2<T>::type;

template <typename T> __device__ __forceinline__ c2<T> mk(T x, T y)
{
    c2<T> r;
    r.x = x;
    r.y = y;
    return r;
}

// acc + a * b
template <typename T> __device__ __forceinline__ c2<T> cmac(c2<T> acc, c2<T> a, c2<T> b)
{
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
    return acc;
}

template <typename T> __device__ __forceinline__ c2<T> cmul(c2<T> a, c2<T> b)
{
    return mk<T>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

template <typename TO, typename TI> __device__ __forceinline__ c2<TO> cvt(c2<TI> a)
{
    return mk<TO>((TO)a.x, (TO)a.y);
}

// ---------------------------------------------------------------------------------
// Per-particle records for the near field: {X, Y, Gamma, 0} with (X, Y) = alpha (z - c_leaf),
// alpha chosen per call so that the pair exponent needs no extra multiply:
//   FP64: alpha^2 = 1/(2 sigma^2)          -> g = 1 - exp(-s)
//   FP32: alpha^2 = log2(e)/(2 sigma^2)    -> g = 1 - exp2(-s)
// with s = |X_i - X_j|^2 (leaf offset added per neighbour leaf).  Leaf-local origins
// keep FP32 differences accurate at the blob scale.
// ---------------------------------------------------------------------------------
// Workgroups are dealt to the XCDs round-robin; this remaps block b so that XCD x walks
// the contiguous range [x per, (x + 1) per) of logical blocks (grids are launched as a
// multiple of nxcd), which keeps the memory windows each XCD touches few and in its L2.
__device__ __forceinline__ int xcd_block(int nxcd)
{
    const int per = gridDim.x / nxcd;
    return (blockIdx.x % nxcd) * per + blockIdx.x / nxcd;
}
inline unsigned xcd_grid(int64_t work, int per_block, int nxcd)
{
    const int64_t b = (work + per_block - 1) / per_block;
    return (unsigned)((std::max<int64_t>(b, 1) + nxcd - 1) / nxcd * nxcd);
}

template <typename T> struct Rec;
template <> struct Rec<float> { using type = float4; };
template <> struct Rec<double> { using type = double4; };
template <typename T> using rec_t = typename Rec<T>::type;
template <typename R> struct RecScalar;
template <> struct RecScalar<float4> { using type = float; };
template <> struct RecScalar<double4> { using type = double; };

// Where the near-field kernels read a particle's record {X, Y, Gamma, 0} from: the
// particles' coordinates relative to their leaf's centre, kept with the tree and scaled on
// load (the uniform tree: leaf-unit coordinates xi = (z - c_leaf)/w scaled by alpha w; the
// adaptive tree, whose leaves have several widths: z - c_leaf scaled by alpha), and the
// circulations in tree order, gathered per call (only they change between calls).
template <typename T> struct SoaRec {
    const c2<T> *__restrict__ pos;
    const T *__restrict__ gam;
    T scale;
    const c2<T> *__restrict__ q = nullptr;  // adjoint charges (the pair force)
    __device__ __forceinline__ rec_t<T> operator()(int64_t i) const
    {
        const c2<T> p = pos[i];
        rec_t<T> r;
        r.x = p.x * scale;
        r.y = p.y * scale;
        r.z = gam[i];
        r.w = (T)0;
        return r;
    }
};

// What the near field sums for a particle: its velocity, or in the adjoint the force on it
// (see pair_force), alone or with Phi.  The adjoint's records carry the adjoint charge: its
// real part as the record's fourth value, its imaginary part qy beside the record.
enum NearSums { kVelocity = 0, kForce = 1, kForcePhi = 2 };
template <int KIND> constexpr int kSums = KIND == kForcePhi ? 3 : 2;

template <int KIND, typename T> __device__ __forceinline__ rec_t<T> load_rec(const SoaRec<T> &rec, int64_t i, T &qy)
{
    rec_t<T> r = rec(i);
    if constexpr (KIND != kVelocity) {
        const c2<T> q = rec.q[i];
        r.w = q.x;
        qy = q.y;
    }
    return r;
}

// g(s) = 1 - exp(-|dz|^2/(2 sigma^2)) in the scaled variable s, and 1/s.
__device__ __forceinline__ float one_minus_exp(float s) { return 1.0f - __builtin_amdgcn_exp2f(-s); }
// FP64 e = exp(-s) and g = 1 - e for s >= 0, g without cancellation: Cody-Waite reduction
// s = k ln2 + r, |r| <= ln2/2 (ln2 as a high part with 21 trailing zero bits, so that k ln2_hi
// is exact, plus the rest), expm1(x) = x p(x) at x = -r with p of degree 10 (the Taylor series
// of expm1(x)/x economized by Chebyshev polynomials on |x| <= 0.3467, in exact rational
// arithmetic, coefficients rounded to double: within 2.3e-17 of p), then e = 2^-k (1 + em1)
// and g = (1 - 2^-k) - 2^-k em1, where 1 - 2^-k is exact.  Within about 2 ulp of both; 2^-k
// underflows to 0 for large s (e = 0, g = 1).  Branch-free, 19 instructions.
__device__ __forceinline__ void exp_pair(double s, double &e, double &g)
{
    constexpr double kInvLn2 = 1.4426950408889634, kLn2Hi = 6.93147180369123816490e-01,
                     kLn2Lo = 1.90821492927058770002e-10;
    const double k = rint(s * -kInvLn2);  // minus the k above: the exponent as ldexp takes it
    const double x = -fma(k, kLn2Lo, fma(k, kLn2Hi, s));  // -(s - k ln2)
    double p = 2.5110080609180445e-08;
    p = fma(p, x, 2.7626408708679167e-07);
    p = fma(p, x, 2.7557240802111588e-06);
    p = fma(p, x, 2.4801504223004426e-05);
    p = fma(p, x, 0.000198412698901562);
    p = fma(p, x, 0.0013888888932586684);
    p = fma(p, x, 0.00833333333331956);
    p = fma(p, x, 0.04166666666657286);
    p = fma(p, x, 0.1666666666666668);
    p = fma(p, x, 0.5000000000000006);
    p = fma(p, x, 1.0);
    const double em1 = p * x;  // expm1(-r)
    const double t = ldexp(1.0, (int)k);
    e = fma(t, em1, t);
    g = fma(-t, em1, 1.0 - t);
}
__device__ __forceinline__ double one_minus_exp(double s)
{
    double e, g;
    exp_pair(s, e, g);
    return g;
}
__device__ __forceinline__ float recip(float s) { return __builtin_amdgcn_rcpf(s); }
// FP64: the hardware reciprocal estimate (relative error below 2^-24, measured) refined by
// one cubic step r + r (d + d^2), d = 1 - s r, which triples the correct bits: within an ulp
// of 1/s (equal to the IEEE quotient on 4M sampled s in [1e-3, 1e6], measured; not
// guaranteed correctly rounded), 4 instructions against 5 for two Newton steps and about 10
// for the division, on a positive normal s (s >= tiny).
__device__ __forceinline__ double recip(double s)
{
    const double r = __builtin_amdgcn_rcp(s);
    const double d = fma(-s, r, 1.0);
    return fma(r, fma(d, d, d), r);
}
// Added to every s: a pair at distance 0 (the particle itself) then gives g = 0 and a
// finite Gamma/s (for |Gamma| < 1e18 in FP32), hence exactly zero, while any s above
// ~1e-13 (FP32) or ~1e-284 (FP64) is unchanged.
template <typename T> __device__ __forceinline__ T tiny();
template <> __device__ __forceinline__ float tiny<float>() { return 1e-20f; }
template <> __device__ __forceinline__ double tiny<double>() { return 1e-300; }

// f = Gamma (1 - e)/s evaluated as q - e q with q = Gamma/s (one fused multiply-add);
// on a far tile e rounds to 0 against 1 and f = q.
__device__ __forceinline__ float exp_neg_scaled(float s) { return __builtin_amdgcn_exp2f(-s); }

template <typename T, bool FAR>
__device__ __forceinline__ void p2p_pair(const rec_t<T> &rj, T tx, T ty, T &fu, T &fv)
{
    const T ddx = tx - rj.x;
    const T ddy = ty - rj.y;
    const T s = fma(ddx, ddx, fma(ddy, ddy, tiny<T>()));
    const T q = recip(s) * rj.z;
    T f;
    if (FAR) f = q;
    else if constexpr (sizeof(T) == 4) f = fma(-exp_neg_scaled(s), q, q);
    else f = one_minus_exp(s) * q;
    fu = fma(f, ddy, fu);
    fv = fma(f, ddx, fv);
}

template <typename T, int K, bool FAR>
__device__ __forceinline__ void p2p_tile(const rec_t<T> *tile, int len, int k, T tx, T ty, T &fu, T &fv)
{
    if (len == 64) {
#pragma unroll 8
        for (int it = 0; it < 64 / K; ++it) p2p_pair<T, FAR>(tile[k + it * K], tx, ty, fu, fv);
    } else {
        for (int j = k; j < len; j += K) p2p_pair<T, FAR>(tile[j], tx, ty, fu, fv);
    }
}

template <typename T, int K>
__device__ __forceinline__ void p2p_tile_any(const rec_t<T> *tile, int len, int k, T tx, T ty, T &fu, T &fv, bool far)
{
    if (far) p2p_tile<T, K, true>(tile, len, k, tx, ty, fu, fv);
    else p2p_tile<T, K, false>(tile, len, k, tx, ty, fu, fv);
}

// ---------------------------------------------------------------------------------
// The pair force.  For particles that move as evaluation point and as source at once, what a
// pair adds to dL/d(x, y) of its two particles is equal and opposite, since the kernel depends
// on their difference alone.  With dz' = (dx', dy') the scaled difference z_i - z_j, e and g as
// for the velocity, lambda ln 2 (FP32, whose exponent is base 2) or 1 (FP64),
//   h = (lambda e - g/s')/s' = d(g/s')/ds',  v = Gamma_j q_i - Gamma_i q_j,  c = v_y dx' - v_x dy',
//   dL/dx_i += ka sum_j [ v_y g/s' + 2 h c dx'],
//   dL/dy_i += ka sum_j [-v_x g/s' + 2 h c dy'],          ka = alpha^2/(2 pi),
// the gradient of (v_y dx' - v_x dy') g/s', and the sum of the evaluation part Gamma_j (q_i A, B)
// and the source part Gamma_i (q_j ..) of the separate sums below.  (As a turned product of v with
// h conj(dz')^2 +- lambda e a step took three operations more, 28 in FP32 instead of 25, 62 in FP64
// with Phi instead of 60: adjoint of 2^22 patch particles, mixed, 2.90 -> 2.77 ms; the errors are
// the same.)  Two sums per particle in place of seven, and both particles of a pair
// are served by one evaluation of the weights.  In FP32 it serves the mutual items; the
// target-centric units take the separate sums there (p2p_force_kernel says why).  The sums kept are -dL/dx/ka and dL/dy/ka, the
// signs of the velocity's.  Phi_i = alpha sum_j q_j (g/s') conj(dz') enters by its imaginary
// part alone.
//
// The difference lambda e - g/s' cancels for small s', but |c dz'/s'| <= |v| puts its error, a
// rounding of lambda e, beside v g/s' itself.  g/s' = r - e r loses 1/s' roundings
// in FP32 and is taken from its series below series_cut (class 0; class 1: the boxes of the
// two tiles keep every pair above it; class 2: e rounds to 0 against 1).
// ---------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ constexpr T exponent_base_log();  // lambda
template <> __device__ __forceinline__ constexpr float exponent_base_log<float>() { return 0.69314718055994530942f; }
template <> __device__ __forceinline__ constexpr double exponent_base_log<double>() { return 1.0; }

// The natural exponent x = |dz|^2/(2 sigma^2) below which FP32 takes the series
// g/s' = lambda (1 - x/2 + x^2/6 - x^3/24 + x^4/120): the next term is under a rounding there.
constexpr float kSeriesX = 0.125f;

// gr = g/s' and (of no use to class 2) k = 2 h.
template <typename T, int CLS> __device__ __forceinline__ void force_weights(T ddx, T ddy, T &gr, T &k)
{
    constexpr T lam = exponent_base_log<T>();
    const T s = fma(ddx, ddx, fma(ddy, ddy, tiny<T>()));
    const T r = recip(s);
    if constexpr (CLS == 2) {
        gr = r;
        k = 0;
    } else {
        T e;
        if constexpr (sizeof(T) == 4) {
            e = __builtin_amdgcn_exp2f(-s);
            gr = fma(-e, r, r);
            if constexpr (CLS == 0) {
                constexpr float l2 = lam * lam, l3 = l2 * lam;
                const float series = fma(s, fma(s, fma(s, fma(s, l3 * l2 / 120.0f, -l2 * l2 / 24.0f), l3 / 6.0f), -l2 / 2.0f), lam);
                gr = s < kSeriesX / lam ? series : gr;
            }
        } else {
            double g;
            exp_pair(s, e, g);
            gr = g * r;
        }
        const T t = fma(lam, e, -gr);
        k = (t + t) * r;
    }
}

// n (x, y) is the part of the pair's sums along dz', (x, y) being dz' or gr dz'.
template <typename T, int CLS>
__device__ __forceinline__ void force_along(T ddx, T ddy, T gr, T k, T vx, T vy, T &x, T &y, T &n)
{
    if constexpr (CLS == 2) {  // k = -2 gr^2
        x = gr * ddx;
        y = gr * ddy;
        n = (T)-2 * fma(vx, y, -(vy * x));
    } else {
        x = ddx;
        y = ddy;
        n = k * fma(vx, y, -(vy * x));
    }
}

// Source rj with qjy onto a particle at (tx, ty) with Gamma g and charge (qx, qy).
template <typename T, int KIND, int CLS>
__device__ __forceinline__ void force_pair(const rec_t<T> &rj, T qjy, const rec_t<T> &ti, T tiqy, T tx, T ty,
                                           T (&f)[kSums<KIND>])
{
    const T ddx = tx - rj.x;
    const T ddy = ty - rj.y;
    T gr, k;
    force_weights<T, CLS>(ddx, ddy, gr, k);
    const T vx = fma(rj.z, ti.w, -(ti.z * rj.w));
    const T vy = fma(rj.z, tiqy, -(ti.z * qjy));
    T x, y, n;
    force_along<T, CLS>(ddx, ddy, gr, k, vx, vy, x, y, n);
    f[0] = fma(n, x, f[0]);
    f[0] = fma(-gr, vy, f[0]);
    f[1] = fma(-n, y, f[1]);
    f[1] = fma(-gr, vx, f[1]);
    if constexpr (KIND == kForcePhi) {
        f[2] = fma(gr, fma(qjy, ddx, -(rj.w * ddy)), f[2]);
    }
}

// ---------------------------------------------------------------------------------
// Target-centric units over sparse source leaves.  Taken leaf by leaf, a 3x3 neighbourhood
// of ~16-particle leaves is nine dependent loads and barriers for nine steps of work each
// (1024^2 lattice, 16 per leaf, FP64: 0.40 ms; its pairs issue in 0.17 ms).  So the unit's
// source ranges are concatenated and staged 64 sources at a time, each moved into the
// frame of the target's leaf on the way into LDS.
// ---------------------------------------------------------------------------------

// How a unit's 64 lanes share its nt targets: lane = k tp + t takes target t and every K-th
// source from k on.  From 9 targets on tp = nt, so that no lane is left over but 64 mod nt;
// below, tp is a power of two, so that the partial sums meet in a butterfly.
struct UnitLanes {
    int tp, K, t, k;
    bool pow2;
    __device__ __forceinline__ UnitLanes(int lane, int nt, int logtp)
    {
        pow2 = nt <= 8 || nt > 32;
        tp = pow2 ? 1 << logtp : nt;
        k = pow2 ? lane >> logtp : (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)nt));
        K = pow2 ? 64 >> logtp : 64 / nt;
        t = lane - k * tp;
        if (k >= K) k = 0;  // a lane left over repeats the first share; its sums are not read
    }
    // the K partial sums of target t, complete in the lanes k = 0
    __device__ __forceinline__ double reduce(double v) const
    {
        if (pow2) {
            for (int o = tp; o < 64; o <<= 1) v += __shfl_xor(v, o);
            return v;
        }
        double r = v;
        for (int j = 1; j < K; ++j) r += __shfl(v, t + j * tp);
        return r;
    }
};

// The concatenation of up to E <= 64 source ranges, lane e < E holding the length of range e
// (lanes >= E zero), in batches of 64: stage(e, j) with this lane's source, the j-th of
// range e (j < 0: none), between two barriers, then work(count) over the staged sources.
template <int E, typename Stage, typename Work>
__device__ __forceinline__ void source_batches(int len, Stage stage, Work work)
{
    const int lane = threadIdx.x;
    int incl = len;
#pragma unroll
    for (int d = 1; d < E; d <<= 1) {
        const int o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    const int total = __builtin_amdgcn_readlane(incl, E - 1);
    const int excl = incl - len;
    for (int b = 0; b < total; b += 64) {
        const int g = b + lane;
        int e = 0;  // the last range that starts at or before g
#pragma unroll
        for (int d = E / 2; d >= 1; d >>= 1)
            if (__shfl(excl, e + d) <= g) e += d;
        const int j = g - __shfl(excl, e);
        __syncthreads();
        stage(e, g < total ? j : -1);
        __syncthreads();
        work(min(64, total - b));
    }
}

// Steps of one batch: lane share k of K over `count` staged sources (zero-charge records
// follow the last one up to 64 + K).
template <typename T, bool FAR>
__device__ __forceinline__ void p2p_batch(const rec_t<T> *tile, int count, int k, int K, T tx, T ty, T &fu, T &fv)
{
    const int steps = (count + K - 1) / K;
    const rec_t<T> *src = tile + k;
#pragma unroll 4
    for (int it = 0; it < steps; ++it, src += K) p2p_pair<T, FAR>(*src, tx, ty, fu, fv);
}

template <typename T, int KIND, int CLS>
__device__ __forceinline__ void force_batch(const rec_t<T> *tile, const T *qtile, int count, int k, int K,
                                            const rec_t<T> &ti, T tiqy, T (&f)[kSums<KIND>])
{
    const int steps = (count + K - 1) / K;
    const rec_t<T> *src = tile + k;
    const T *qsrc = qtile + k;
#pragma unroll 4
    for (int it = 0; it < steps; ++it, src += K, qsrc += K)
        force_pair<T, KIND, CLS>(*src, *qsrc, ti, tiqy, ti.x, ti.y, f);
}

// This lane's source of a batch into LDS, moved by (sx, sy), with a zero record 64 places on;
// at < 0: none.
template <int KIND, typename T>
__device__ __forceinline__ void stage_source(rec_t<T> *tile, T *qtile, const SoaRec<T> &rec, int64_t at, T sx, T sy)
{
    const int lane = threadIdx.x;
    rec_t<T> r, none;
    r.x = r.y = r.z = r.w = (T)0;
    none = r;
    T qy = (T)0;
    if (at >= 0) {
        r = load_rec<KIND>(rec, at, qy);
        r.x += sx;
        r.y += sy;
    }
    tile[lane] = r;
    tile[64 + lane] = none;
    qtile[lane] = qy;
    qtile[64 + lane] = (T)0;
}

// The squared gap in leaves from which two tiles of FP32 records need no series.
__host__ __device__ inline float force_series_leaf2(double step)
{
    return (float)(2.0 * (0.125 / 0.69314718055994530942) / (step * step));
}

// Smallest squared distance between two boxes {xmin, ymin, xmax, ymax}, the first
// shifted by (ox, oy).
__device__ __forceinline__ float box_gap2(float4 a, float ox, float oy, float4 b)
{
    const float gx = fmaxf(0.0f, fmaxf(b.x - (a.z + ox), (a.x + ox) - b.z));
    const float gy = fmaxf(0.0f, fmaxf(b.y - (a.w + oy), (a.y + oy) - b.w));
    return gx * gx + gy * gy;
}

// ---------------------------------------------------------------------------------
// Stage 9, mutual form for pairs of dense leaves.  The kernel of eq. regB-S2DGau is
// odd, K(-z) = -K(z), so one evaluation of g(s)/s serves both particles of a pair.
// One wavefront per item {S, R}: R is S itself or one of its neighbours (+1,0),
// (-1,+1), (0,+1), (+1,+1), so every unordered pair of neighbouring dense leaves is
// one item.  For each pair of 64-particle tiles (b of S, a of R), one tile is held one
// particle per lane ("resident") and the other is staged in LDS and streamed in chunks
// of 16 sources.  Within a chunk, lane l of a 16-lane row meets source (l + j) mod 16
// at step j; the resident sums stay in the lane, and each source's terms meet its sum by a
// rotation within the row: of the sum, one lane per step, or in FP32 velocities of the term (a
// DPP operand).  After 16 steps every row holds its partial sums of the chunk's sources;
// two butterfly steps across rows complete them.  Sums for tile b stay in registers
// over the tiles of R; sums for tile a accumulate in its particles' slot in memory.
// Slots: nine per particle, one per neighbour direction d = 3(dy+1) + (dx+1), written
// by exactly one item (the item of S = R writes its own particles' slot 4 from both
// ends, tile b folding in what the earlier tiles wrote).  The near field is the fixed
// order sum of the slots plus the target-centric part for sparse neighbours, so the
// result does not depend on scheduling.
// ---------------------------------------------------------------------------------

// Lane l receives the value of lane 16 (l / 16) + ((l + 1) mod 16): DPP row_ror:15.
__device__ __forceinline__ float row_rot(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x12F, 0xF, 0xF,
                                                                 false));
}
__device__ __forceinline__ double row_rot(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffff), 0x12F, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x12F, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Lane l receives the value of lane 16 (l / 16) + ((l - J) mod 16): DPP row_ror:J.
template <int J> __device__ __forceinline__ float row_back(float v)
{
    if constexpr (J == 0) return v;
    else
        return __builtin_bit_cast(float,
                                  __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + J, 0xF, 0xF, true));
}

// -Gamma of the resident particles as the chunk's steps take it.  FP32: of the lane J before in
// its row, for J < 8.
template <typename T> struct RowGamma;
template <> struct RowGamma<double> {
    double g;
    __device__ __forceinline__ explicit RowGamma(double v) : g(v) {}
};
template <> struct RowGamma<float> {
    float g[8];
    template <int J = 0> __device__ __forceinline__ void spread(float v)
    {
        g[J] = row_back<J>(v);
        if constexpr (J < 7) spread<J + 1>(v);
    }
    __device__ __forceinline__ explicit RowGamma(float v) { spread(v); }
};

// 16 steps of one chunk: src points at this lane's start in the chunk's doubled copy
// (src[j] = source (l + j) mod 16).  rg: -Gamma of the resident particles (zero for an idle
// lane).  On return (cu, cv)[l] = this row's sum for source l mod 16 of the chunk.
template <bool FAR>
__device__ __forceinline__ void mutual_chunk(const rec_t<double> *src, double rx, double ry,
                                             const RowGamma<double> &rg, double &fu, double &fv, double &cu,
                                             double &cv)
{
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const rec_t<double> sj = src[j];
        const double ddx = rx - sj.x;
        const double ddy = ry - sj.y;
        const double ss = fma(ddx, ddx, fma(ddy, ddy, tiny<double>()));
        const double r = recip(ss);
        const double h = FAR ? r : one_minus_exp(ss) * r;  // g(s)/s
        const double wt = h * sj.z;
        fu = fma(wt, ddy, fu);
        fv = fma(wt, ddx, fv);
        const double ws = h * rg.g;
        if (j == 0) {
            cu = ws * ddy;
            cv = ws * ddx;
        } else {
            cu = row_rot(cu) + ws * ddy;
            cv = row_rot(cv) + ws * ddx;
        }
    }
    cu = row_rot(cu);
    cv = row_rot(cv);
}

// FP32: the sums stay in their lanes and the terms move.  The terms of source s at step q come
// from the lane q before it, through the DPP operand of a fused multiply-add with that lane's
// Gamma: 11 vector operations besides the reciprocal and the exponential, where sums that
// travel with their source take a rounded product and a rotating add each, 13.  Sources l + 8 to
// l + 15 come first and their sums move by half a row before sources l to l + 7, so that eight
// of the row's Gamma do: with sixteen the kernel holds 70 registers, 7 wavefronts per SIMD
// instead of 8, and 1000003 patch particles at depth 8 took 0.452 ms against 0.433 before.
// Now 0.413; 2^22 at depth 9 1.76 -> 1.67, 2^24 at depth 10 7.06 -> 6.75.  (FP64 has no such
// operand: two moves per term either way, and its Gamma would take 16 registers more.)
//
// The compiler does not form the instruction, and does not look into the block for hazards: a
// DPP read needs two wait states after the write.  In front stand the resident's two sums;
// behind the last step before the move, an s_nop.
template <int Q>
__device__ __forceinline__ void mutual_add(float ux, float uy, float z, float g, float &fu, float &fv, float &cu,
                                           float &cv)
{
    if constexpr (Q == 0) {
        fu = fma(z, uy, fu);
        fv = fma(z, ux, fv);
        cu = g * uy;
        cv = g * ux;
    } else if constexpr (Q == 8) {
        fu = fma(z, uy, fu);
        fv = fma(z, ux, fv);
        cu = fma(g, uy, row_back<8>(cu));
        cv = fma(g, ux, row_back<8>(cv));
    } else {
        asm("v_fmac_f32_e32 %0, %4, %5\n\t"
            "v_fmac_f32_e32 %1, %4, %6\n\t"
            "v_fmac_f32_dpp %2, %5, %7 row_ror:%8 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %6, %7 row_ror:%8 row_mask:0xf bank_mask:0xf"
            : "+&v"(fu), "+&v"(fv), "+&v"(cu), "+&v"(cv)
            : "v"(z), "v"(uy), "v"(ux), "v"(g), "n"(Q % 8));
        if constexpr (Q == 7) asm("s_nop 1" : "+v"(cu), "+v"(cv));
    }
}

// (Two steps at a time: both chains up to the terms are in flight together.)
template <bool FAR, int Q = 0>
__device__ __forceinline__ void mutual_chunk(const rec_t<float> *src, float rx, float ry, const RowGamma<float> &rg,
                                             float &fu, float &fv, float &cu, float &cv)
{
    float ux[2], uy[2], z[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const rec_t<float> sj = src[(Q + k + 8) % 16];
        const float ddx = rx - sj.x;
        const float ddy = ry - sj.y;
        const float ss = fma(ddx, ddx, fma(ddy, ddy, tiny<float>()));
        const float r = recip(ss);
        const float h = FAR ? r : fma(-exp_neg_scaled(ss), r, r);  // g(s)/s
        ux[k] = h * ddx;
        uy[k] = h * ddy;
        z[k] = sj.z;
    }
    __builtin_amdgcn_sched_barrier(0);
    mutual_add<Q>(ux[0], uy[0], z[0], rg.g[Q % 8], fu, fv, cu, cv);
    mutual_add<Q + 1>(ux[1], uy[1], z[1], rg.g[Q % 8 + 1], fu, fv, cu, cv);
    if constexpr (Q < 14) mutual_chunk<FAR, Q + 2>(src, rx, ry, rg, fu, fv, cu, cv);
}

// The same for the pair force: qsrc the sources' qy; the source's sums are the negative of the
// resident's terms.
template <typename T, int KIND, int CLS>
__device__ __forceinline__ void force_chunk(const rec_t<T> *src, const T *qsrc, T rx, T ry, T rg, T rqx, T rqy,
                                            T (&f)[kSums<KIND>], T (&c)[kSums<KIND>])
{
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const rec_t<T> sj = src[j];
        const T sqy = qsrc[j];
        const T ddx = rx - sj.x;
        const T ddy = ry - sj.y;
        T gr, k;
        force_weights<T, CLS>(ddx, ddy, gr, k);
        const T vx = fma(sj.z, rqx, -(rg * sj.w));
        const T vy = fma(sj.z, rqy, -(rg * sqy));
        T x, y, n;
        force_along<T, CLS>(ddx, ddy, gr, k, vx, vy, x, y, n);
        const T fx = fma(n, x, -(gr * vy));
        const T fy = fma(-n, y, -(gr * vx));
        T tj = 0;
        if constexpr (KIND == kForcePhi) {
            const T cx = gr * ddx, cy = gr * ddy;
            f[2] = fma(sqy, cx, f[2]);
            f[2] = fma(-sj.w, cy, f[2]);
            tj = fma(rqx, cy, -(rqy * cx));
        }
        f[0] += fx;
        f[1] += fy;
        if (j == 0) {
            c[0] = -fx;
            c[1] = -fy;
            if constexpr (KIND == kForcePhi) c[2] = tj;
        } else {
            c[0] = row_rot(c[0]) - fx;
            c[1] = row_rot(c[1]) - fy;
            if constexpr (KIND == kForcePhi) c[2] = row_rot(c[2]) + tj;
        }
    }
#pragma unroll
    for (int m = 0; m < kSums<KIND>; ++m) c[m] = row_rot(c[m]);
}

// Records of one tile into LDS, each chunk of 16 stored twice in a row (so that the
// sources of step j are at a constant offset), zero records past the tile's end.
template <int KIND, typename T>
__device__ __forceinline__ rec_t<T> stage_doubled(rec_t<T> *dst, T *qdst, const SoaRec<T> &rec, int first, int len,
                                                  T &qy)
{
    const int lane = threadIdx.x;
    rec_t<T> r;
    r.x = r.y = r.z = r.w = (T)0;
    qy = (T)0;
    if (lane < len) r = load_rec<KIND>(rec, first + lane, qy);
    const int at = (lane >> 4) * 32 + (lane & 15);
    dst[at] = r;
    dst[at + 16] = r;
    if constexpr (KIND != kVelocity) {
        qdst[at] = qy;
        qdst[at + 16] = qy;
    }
    return r;
}

// One direction's slots: the first two sums of a particle together, the third by itself.
template <typename T, int KIND> struct NearSlot {
    c2<T> *uv;
    T *phi;
    __device__ __forceinline__ void load(int64_t i, T (&f)[kSums<KIND>]) const
    {
        const c2<T> o = uv[i];
        f[0] = o.x;
        f[1] = o.y;
        if constexpr (KIND == kForcePhi) f[2] = phi[i];
    }
    __device__ __forceinline__ void store(int64_t i, const T (&f)[kSums<KIND>]) const
    {
        uv[i] = mk<T>(f[0], f[1]);
        if constexpr (KIND == kForcePhi) phi[i] = f[2];
    }
};

// The LDS of a near-field workgroup.
template <typename T, int KIND> struct NearLds {
    rec_t<T> a[128], b[128];
    T qa[128], qb[128];
};
template <typename T> struct NearLds<T, kVelocity> {
    rec_t<T> a[128], b[128];
    static constexpr T *qa = nullptr, *qb = nullptr;
};

// What a mutual item reads of the tree, and the squared gaps (in leaves) from which a pair of
// tiles skips the exponential and the series.
struct MutualTree {
    const int *__restrict__ leaf_start;
    const int *__restrict__ tile_start;
    const float4 *__restrict__ tile_box;
    float cut_leaf2, series_leaf2;
};

// The tiles of R that an item takes (the particles from a0 to a1), and where its sums for the
// particles of S go: their slot, or for a part of an item (see MutualParts) an array of the part's
// own.
template <typename T, int KIND> struct MutualRange {
    int a0, a1;
    bool part;
    NearSlot<T, KIND> s, r;
};

// One tile b of S against every tile a of the range (a >= b when S = R).  Per block (b, a) the
// tile with more chunks of 16 sits in the lanes and the other is streamed from LDS, so
// that fewer steps are spent; either way both sums come out lane-indexed by particle.
template <int KIND, typename T>
__device__ __forceinline__ void mutual_resident_tile(const int4 it, NearLds<T, KIND> &lds, int b, int tb,
                                                     const SoaRec<T> &rec, const MutualTree &mt, T step,
                                                     const MutualRange<T, KIND> &range)
{
    constexpr int NS = kSums<KIND>;
    const int lane = threadIdx.x;
    const uint32_t S = (uint32_t)it.x, R = (uint32_t)it.y;
    const bool self = S == R;
    const int ds = it.z & 15;
    const int dx = ds % 3 - 1, dy = ds / 3 - 1;  // R - S in leaves
    const T ox = (T)dx * step, oy = (T)dy * step;
    const int s0 = mt.leaf_start[S], s1 = mt.leaf_start[S + 1];
    const int r0 = mt.leaf_start[R], r1 = range.a1;
    const int lenb = min(64, s1 - b);
    const int nchb = (lenb + 15) >> 4;
    __syncthreads();
    T qyb;
    const rec_t<T> rb = stage_doubled<KIND>(lds.b, lds.qb, rec, b, lenb, qyb);
    // tile b in the frame of leaf R (resident form); in the streamed form it stays in
    // the frame of S and tile a is moved there
    const T bx = rb.x - ox, by = rb.y - oy;
    const T bgn = lane < lenb ? -rb.z : (T)0;
    const float4 bbox = mt.tile_box[tb];
    T f[NS];
#pragma unroll
    for (int m = 0; m < NS; ++m) f[m] = 0;
    if (self && !range.part && b > s0 && lane < lenb) range.s.load(b + lane, f);  // what the earlier tiles of S wrote for this tile
    const bool first_touch = b == s0;  // the first resident tile creates the streamed slots
    const int from = self ? max(b, range.a0) : range.a0;
    int ta = mt.tile_start[R] + ((from - r0) >> 6);
    for (int a = from; a < r1; a += 64, ++ta) {
        const int lena = min(64, r1 - a);
        const int ncha = (lena + 15) >> 4;
        const bool diag = self && a == b;
        const float gap2 = box_gap2(bbox, (float)-dx, (float)-dy, mt.tile_box[ta]);
        const bool far = gap2 >= mt.cut_leaf2;
        if (diag) {
            // the tile with itself: every ordered pair from the resident end
            __syncthreads();
            for (int c = 0; c < nchb; ++c)
                if constexpr (KIND == kVelocity) {
                    if (far) {
#pragma unroll
                        for (int j = 0; j < 16; ++j) p2p_pair<T, true>(lds.b[c * 32 + j], bx, by, f[0], f[1]);
                    } else {
#pragma unroll
                        for (int j = 0; j < 16; ++j) p2p_pair<T, false>(lds.b[c * 32 + j], bx, by, f[0], f[1]);
                    }
                } else {
                    T fc[NS] = {};
                    if (far) {
#pragma unroll 2
                        for (int j = 0; j < 16; ++j)
                            force_pair<T, KIND, 2>(lds.b[c * 32 + j], lds.qb[c * 32 + j], rb, qyb, bx, by, fc);
                    } else {
#pragma unroll 4
                        for (int j = 0; j < 16; ++j)
                            force_pair<T, KIND, 0>(lds.b[c * 32 + j], lds.qb[c * 32 + j], rb, qyb, bx, by, fc);
                    }
#pragma unroll
                    for (int m = 0; m < NS; ++m) f[m] += fc[m];
                }
            continue;
        }
        T old[NS];
#pragma unroll
        for (int m = 0; m < NS; ++m) old[m] = 0;
        if (!first_touch && lane < lena) range.r.load(a + lane, old);
        const bool swap = ncha > nchb;  // tile a in the lanes, tile b streamed
        __syncthreads();
        T qya;
        const rec_t<T> ra = stage_doubled<KIND>(lds.a, lds.qa, rec, a, lena, qya);
        __syncthreads();
        T px, py, pgn, pqx = 0, pqy = 0;
        const rec_t<T> *src;
        const T *qsrc = nullptr;
        int nch;
        if (swap) {
            px = ra.x + ox;
            py = ra.y + oy;
            pgn = lane < lena ? -ra.z : (T)0;
            src = lds.b;
            nch = nchb;
        } else {
            px = bx;
            py = by;
            pgn = bgn;
            src = lds.a;
            nch = ncha;
        }
        if constexpr (KIND != kVelocity) {
            pqx = swap ? ra.w : rb.w;
            pqy = swap ? qya : qyb;
            qsrc = swap ? lds.qb : lds.qa;
        }
        const RowGamma<T> back(pgn);
        T r[NS], col[NS];
#pragma unroll
        for (int m = 0; m < NS; ++m) r[m] = col[m] = 0;
        for (int c = 0; c < nch; ++c) {
            T cs[NS];
            const int at = c * 32 + (lane & 15);
            if constexpr (KIND == kVelocity) {
                if (far) mutual_chunk<true>(src + at, px, py, back, r[0], r[1], cs[0], cs[1]);
                else mutual_chunk<false>(src + at, px, py, back, r[0], r[1], cs[0], cs[1]);
            } else {
                T rc[NS] = {};  // the chunk's terms apart from the running sums: see p2p_force_kernel
                if (far) force_chunk<T, KIND, 2>(src + at, qsrc + at, px, py, -pgn, pqx, pqy, rc, cs);
                else if (sizeof(T) == 8 || gap2 >= mt.series_leaf2)
                    force_chunk<T, KIND, 1>(src + at, qsrc + at, px, py, -pgn, pqx, pqy, rc, cs);
                else force_chunk<T, KIND, 0>(src + at, qsrc + at, px, py, -pgn, pqx, pqy, rc, cs);
#pragma unroll
                for (int m = 0; m < NS; ++m) r[m] += rc[m];
            }
#pragma unroll
            for (int m = 0; m < NS; ++m) cs[m] += __shfl_xor(cs[m], 16);
#pragma unroll
            for (int m = 0; m < NS; ++m) cs[m] += __shfl_xor(cs[m], 32);
            if ((lane >> 4) == c) {
#pragma unroll
                for (int m = 0; m < NS; ++m) col[m] = cs[m];
            }
        }
        // sums of tile b and of tile a, lane-indexed
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            f[m] += swap ? col[m] : r[m];
            old[m] += swap ? r[m] : col[m];
        }
        if (lane < lena) range.r.store(a + lane, old);
    }
    if (lane < lenb) range.s.store(b + lane, f);
}

// The item's slots: 9 x n pairs of sums in uv, 9 x n third sums in phi.
template <int KIND, typename T>
__device__ __forceinline__ void mutual_item(const int4 it, NearLds<T, KIND> &lds, const SoaRec<T> &rec,
                                            const MutualTree &mt, const MutualParts &parts, T step, int64_t n,
                                            c2<T> *__restrict__ uv, T *__restrict__ phi)
{
    const uint32_t S = (uint32_t)it.x;
    const int64_t at_s = (int64_t)(it.z & 15) * n, at_r = (int64_t)(it.z >> 4) * n;
    const int s0 = mt.leaf_start[S];
    int s1 = mt.leaf_start[S + 1];
    MutualRange<T, KIND> range{mt.leaf_start[it.y],
                               mt.leaf_start[it.y + 1],
                               false,
                               {uv + at_s, KIND == kForcePhi ? phi + at_s : nullptr},
                               {uv + at_r, KIND == kForcePhi ? phi + at_r : nullptr}};
    if (parts.list && it.w > 2 * kMutualItem) {
        const int4 q = parts.list[(it.w >> 9) - 1];
        range.a0 = q.x;
        range.a1 = q.y;
        range.part = true;
        const int64_t at = (int64_t)(unsigned)q.z - s0;
        range.s.uv = (c2<T> *)parts.sums + at;
        if (KIND == kForcePhi) range.s.phi = (T *)((c2<T> *)parts.sums + parts.count) + at;
        if (it.y == it.x) s1 = min(s1, q.y);  // (later tiles of S meet none of the range)
    }
    for (int b = s0, tb = mt.tile_start[S]; b < s1; b += 64, ++tb)
        mutual_resident_tile<KIND>(it, lds, b, tb, rec, mt, step, range);
}

// The sums of a split item's particles of S, in the order of its parts, to their slot: one
// workgroup per split item {S, direction of R, first part, parts}.
template <typename T, int KIND>
__global__ __launch_bounds__(256) void mutual_fold_kernel(const int4 *__restrict__ items, const MutualParts parts,
                                                          const int *__restrict__ leaf_start, int64_t n,
                                                          c2<T> *__restrict__ uv, T *__restrict__ phi)
{
    constexpr int NS = kSums<KIND>;
    const int4 it = items[blockIdx.x];
    const int s0 = leaf_start[it.x], s1 = leaf_start[it.x + 1];
    const bool self = it.y == 4;
    const NearSlot<T, KIND> slot{uv + it.y * n, KIND == kForcePhi ? phi + it.y * n : nullptr};
    c2<T> *const puv = (c2<T> *)parts.sums;
    const NearSlot<T, KIND> part{puv, KIND == kForcePhi ? (T *)(puv + parts.count) : nullptr};
    for (int i = s0 + threadIdx.x; i < s1; i += 256) {
        const int b = s0 + ((i - s0) & ~63);
        T f[NS], g[NS];
#pragma unroll
        for (int m = 0; m < NS; ++m) f[m] = 0;
        if (self && b > s0) slot.load(i, f);  // from the parts that hold the particle's own tile
        for (int p = 0; p < it.w; ++p) {
            const int4 q = parts.list[it.z + p];
            if (self && b >= q.y) continue;
            part.load((int64_t)(unsigned)q.z + (i - s0), g);
#pragma unroll
            for (int m = 0; m < NS; ++m) f[m] += g[m];
        }
        slot.store(i, f);
    }
}


// ---------------------------------------------------------------------------------
// Adjoint near field (shared by the uniform and the adaptive tree)
// ---------------------------------------------------------------------------------
// e = exp(-x) and g = 1 - e in the scaled variable: FP32 base 2 (g by subtraction,
// small x handled by the series below); FP64 base e by the exp_pair above.
__device__ __forceinline__ void exp_pair(float s, float &e, float &g)
{
    e = __builtin_amdgcn_exp2f(-s);
    g = 1.0f - e;
}

// Below this natural exponent the 5-term series of g/s' and (lambda e s' - g)/s'^2 is
// used: its truncation error x^5/720 is under the rounding unit of T there.
template <typename T> __device__ __forceinline__ T series_cut();
template <> __device__ __forceinline__ float series_cut<float>() { return 0.125f; }
template <> __device__ __forceinline__ double series_cut<double>() { return 1e-3; }

// acc: Im Phi (its real part enters no output); A as its real part and its imaginary part divided
// by -2 (the factor is applied in finalize); B; with SRC also the source-position sums with the
// adjoint charges, At = sum q_j conj(dz')^2 (lambda e s' - g)/s'^2 (2) and Bt = sum q_j e (2).
// conj(dz')^2 = (dx'^2 - dy'^2) - 2i dx' dy' reuses dy'^2 from s'.  SERIES false: the
// pair is known to lie beyond the series cut (its tile's bounding boxes say so), and the
// test is left out.  (With the real part of Phi summed too, two operations and 8 B per particle
// more: 2^22 patch particles, mixed, 3.75 ms, now 3.50; 700001, FP64, 1.32, now 1.20.)
template <typename T, bool FAR, bool SRC, bool SERIES = true>
__device__ __forceinline__ void p2p_bwd_pair(const rec_t<T> &rj, const c2<T> qj, T tx, T ty, T lambda,
                                             T (&acc)[SRC ? 8 : 4])
{
    T &fpi = acc[0], &far_r = acc[1], &far_ih = acc[2], &fb = acc[3];
    const T ddx = tx - rj.x;
    const T ddy = ty - rj.y;
    const T dy2 = fma(ddy, ddy, tiny<T>());
    const T s = fma(ddx, ddx, dy2);
    const T r = recip(s);
    if constexpr (FAR) {
        // e rounds to 0 against 1 (g = 1): the terms of the point vortex, Phi: q_j w and
        // A: -Gamma_j w^2 with w = 1/dz' = conj(dz')/s' = cx + i cy.  The A sums take
        // Re(-w^2) = d = cy^2 - cx^2 and Im(-w^2)/-2 = cx cy; the source-position sum takes
        // q_j (d - 2i cx cy).  (Three operations fewer than the general form below.)
        const T cx = r * ddx, cy = -r * ddy;
        fpi = fma(qj.x, cy, fpi);
        fpi = fma(qj.y, cx, fpi);
        const T d = fma(cy, cy, -cx * cx);
        const T m = cx * cy;
        far_r = fma(rj.z, d, far_r);
        far_ih = fma(rj.z, m, far_ih);
        if constexpr (SRC) {
            const T wi = (T)-2 * m;
            acc[4] = fma(qj.x, d, acc[4]);
            acc[4] = fma(-qj.y, wi, acc[4]);
            acc[5] = fma(qj.x, wi, acc[5]);
            acc[5] = fma(qj.y, d, acc[5]);
        }
        return;
    }
    T e, g;
    exp_pair(s, e, g);
    // g/s': in FP32 as r - e r (one fused multiply-add, as the forward's kernel); in FP64
    // from the accurate g of exp_pair
    T gr;
    if constexpr (sizeof(T) == 4) gr = fma(-e, r, r);
    else gr = g * r;
    T h = (lambda * e - gr) * r;  // lambda e/s' - g/s'^2
    // x = lambda s' is the natural exponent |dz|^2/(2 sigma^2).  For small x, 1 - e
    // cancels; there g/s' and (lambda e s' - g)/s'^2 come from their series
    //   g/s' = lambda (1 - x/2 + x^2/6 - x^3/24 + x^4/120),
    //   (lambda e s' - g)/s'^2 = lambda^2 (-1/2 + x/3 - x^2/8 + x^3/30 - x^4/144).
    // (The test is on s' against the cut divided by lambda, a loop invariant.)
    if (SERIES && s < series_cut<T>() / lambda) {
        const T x = lambda * s;
        gr = lambda * fma(x, fma(x, fma(x, fma(x, (T)(1.0 / 120), (T)(-1.0 / 24)), (T)(1.0 / 6)), (T)-0.5), (T)1);
        h = lambda * lambda *
            fma(x, fma(x, fma(x, fma(x, (T)(-1.0 / 144), (T)(1.0 / 30)), (T)(-1.0 / 8)), (T)(1.0 / 3)), (T)-0.5);
    }
    fb = fma(rj.z, e, fb);  // B: Gamma_j e
    if constexpr (SRC) {
        acc[6] = fma(qj.x, e, acc[6]);
        acc[7] = fma(qj.y, e, acc[7]);
    }
    // Phi: q_j (g/s') conj(dz')
    const T cx = gr * ddx, cy = -gr * ddy;
    fpi = fma(qj.x, cy, fpi);
    fpi = fma(qj.y, cx, fpi);
    // A: Gamma_j conj(dz')^2 (lambda e s' - g)/s'^2
    const T hg = h * rj.z;
    const T zr = fma((T)-2, dy2, s);  // dx'^2 - dy'^2
    const T zh = ddx * ddy;           // Im conj(dz')^2 / -2
    far_r = fma(hg, zr, far_r);
    far_ih = fma(hg, zh, far_ih);
    if constexpr (SRC) {
        const T wr = h * zr, wi = ((T)-2 * h) * zh;
        acc[4] = fma(qj.x, wr, acc[4]);
        acc[4] = fma(-qj.y, wi, acc[4]);
        acc[5] = fma(qj.x, wi, acc[5]);
        acc[5] = fma(qj.y, wr, acc[5]);
    }
}

template <typename T, int K, bool FAR, bool SRC, bool SERIES = true>
__device__ __forceinline__ void p2p_bwd_tile(const rec_t<T> *tile, const c2<T> *qtile, int len, int k, T tx, T ty,
                                             T lambda, T (&acc)[SRC ? 8 : 4])
{
    if (len == 64) {
#pragma unroll 4
        for (int it = 0; it < 64 / K; ++it)
            p2p_bwd_pair<T, FAR, SRC, SERIES>(tile[k + it * K], qtile[k + it * K], tx, ty, lambda, acc);
    } else {
        for (int j = k; j < len; j += K) p2p_bwd_pair<T, FAR, SRC, SERIES>(tile[j], qtile[j], tx, ty, lambda, acc);
    }
}

// cls 2: every pair of the tile is beyond the exponential's cut (point-vortex terms);
// 1: beyond the series cut (no per-pair test; units of one or two lanes per target,
// which carry nearly all pairs, so the other unrolled variants stay few); 0: the full form.
template <typename T, int K, bool SRC>
__device__ __forceinline__ void p2p_bwd_tile_any(const rec_t<T> *tile, const c2<T> *qtile, int len, int k, T tx, T ty,
                                                 T lambda, T (&acc)[SRC ? 8 : 4], int cls)
{
    if (cls == 2) p2p_bwd_tile<T, K, true, SRC>(tile, qtile, len, k, tx, ty, lambda, acc);
    else if (K <= 2 && cls == 1) p2p_bwd_tile<T, K, false, SRC, false>(tile, qtile, len, k, tx, ty, lambda, acc);
    else p2p_bwd_tile<T, K, false, SRC>(tile, qtile, len, k, tx, ty, lambda, acc);
}

// Steps of one batch of the adjoint, as p2p_batch.
template <typename T, bool FAR, bool SRC>
__device__ __forceinline__ void p2p_bwd_batch(const rec_t<T> *tile, const c2<T> *qtile, int count, int k, int K, T tx,
                                              T ty, T lambda, T (&acc)[SRC ? 8 : 4])
{
    const int steps = (count + K - 1) / K;
    const rec_t<T> *src = tile + k;
    const c2<T> *qsrc = qtile + k;
#pragma unroll 2
    for (int it = 0; it < steps; ++it, src += K, qsrc += K)
        p2p_bwd_pair<T, FAR, SRC>(*src, *qsrc, tx, ty, lambda, acc);
}

// The same over staged records that carry the adjoint charge (load_rec), source-position sums
// included: the FP32 units of the pair force.
template <typename T, bool FAR>
__device__ __forceinline__ void force_sums_batch(const rec_t<T> *tile, const T *qtile, int count, int k, int K, T tx,
                                                 T ty, T (&acc)[8])
{
    const int steps = (count + K - 1) / K;
    const rec_t<T> *src = tile + k;
    const T *qsrc = qtile + k;
#pragma unroll 2
    for (int it = 0; it < steps; ++it, src += K, qsrc += K)
        p2p_bwd_pair<T, FAR, true>(*src, mk<T>(src->w, *qsrc), tx, ty, exponent_base_log<T>(), acc);
}

// The pair force multiplies Gamma_j q_i in the records' precision.  So that FP32 neither
// overflows nor underflows where the separate sums (linear in each) did not, the FP32 charges
// carry the power of two that brings max|q| max|Gamma| near 1 (charge_scale): the maxima of every
// block here, reduced by every block of the pack kernel, which leaves the factor for the finalize
// kernel.
static __global__ __launch_bounds__(256) void adjoint_range_kernel(int64_t n, const double *__restrict__ gamma,
                                                            const double2 *__restrict__ dl, double scale,
                                                            double2 *__restrict__ range)
{
    double g = 0.0, q = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double2 d = dl[i];
        g = fmax(g, fabs(gamma[i]));
        q = fmax(q, fmax(fabs(scale * d.x), fabs(scale * d.y)));
    }
    __shared__ double2 part[4];
    for (int o = 32; o >= 1; o >>= 1) {
        g = fmax(g, __shfl_xor(g, o));
        q = fmax(q, __shfl_xor(q, o));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = make_double2(g, q);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k) {
            g = fmax(g, part[k].x);
            q = fmax(q, part[k].y);
        }
        range[blockIdx.x] = make_double2(g, q);
    }
}

// The factor, by a whole block of 256 threads; block 0 writes it to qscale.  range NULL: 1.
__device__ __forceinline__ double charge_scale(const double2 *__restrict__ range, double *__restrict__ qscale)
{
    if (!range) return 1.0;
    __shared__ double2 part[4];
    double g = 0.0, q = 0.0;
#pragma unroll
    for (int k = 0; k < kRangeBlocks / 256; ++k) {
        const double2 v = range[k * 256 + threadIdx.x];
        g = fmax(g, v.x);
        q = fmax(q, v.y);
    }
    for (int o = 32; o >= 1; o >>= 1) {
        g = fmax(g, __shfl_xor(g, o));
        q = fmax(q, __shfl_xor(q, o));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = make_double2(g, q);
    __syncthreads();
    for (int k = 0; k < 4; ++k) {
        g = fmax(g, part[k].x);
        q = fmax(q, part[k].y);
    }
    // (a zero, infinite or NaN maximum counts as 1.  Half of Gamma's exponent range in FP32: Phi
    // sums the charges themselves, and 2^60 of them and products down to 2^-66 both leave room)
    const int eg = g > 0.0 && g < 1e300 ? max(-60, min(60, ilogb(g))) : 0;
    const int eq = q > 0.0 && q < 1e300 ? ilogb(q) : 0;
    const double s = ldexp(1.0, -max(-900, min(900, eg + eq)));
    if (blockIdx.x == 0 && threadIdx.x == 0) *qscale = s;
    return s;
}

// ---------------------------------------------------------------------------------
// Sums over the lanes of a group, for the expansions made of particles.
// ---------------------------------------------------------------------------------
// v of a lane whose number differs in bit O (1, 2, 4 or 8) and in no higher bit, as a DPP move:
// within four lanes, mirrored within eight (O = 4), rotated by eight within sixteen.
template <int O> __device__ __forceinline__ int lane_partner(int v)
{
    constexpr int ctrl = O == 1 ? 0xB1 : O == 2 ? 0x4E : O == 4 ? 0x141 : 0x128;
    return __builtin_amdgcn_mov_dpp(v, ctrl, 0xF, 0xF, true);
}
template <int O> __device__ __forceinline__ float lane_partner(float v)
{
    return __builtin_bit_cast(float, lane_partner<O>(__builtin_bit_cast(int, v)));
}
template <int O> __device__ __forceinline__ double lane_partner(double v)
{
    const int2 b = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(lane_partner<O>(b.x), lane_partner<O>(b.y)));
}

// The sum over this lane and the one 16 away of lo in the lanes with bit 4 clear, of hi in the
// others: one exchange puts both lanes' copies side by side.
__device__ __forceinline__ uint2 lane_swap16(unsigned x, unsigned y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return make_uint2(r[0], r[1]);
}
__device__ __forceinline__ float swap_sum16(float lo, float hi)
{
    const uint2 r = lane_swap16(__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi));
    return __builtin_bit_cast(float, r.x) + __builtin_bit_cast(float, r.y);
}
__device__ __forceinline__ double swap_sum16(double lo, double hi)
{
    const uint2 x = __builtin_bit_cast(uint2, lo), y = __builtin_bit_cast(uint2, hi);
    const uint2 a = lane_swap16(x.x, y.x), b = lane_swap16(x.y, y.y);
    return __builtin_bit_cast(double, make_uint2(a.x, b.x)) + __builtin_bit_cast(double, make_uint2(a.y, b.y));
}

// Sum over the lanes of a group of G = 8, 16 or 32 of each of NC >= G values by recursive
// halving: at offset O a lane keeps the half of its values that its lane bit O selects and adds
// its partner's copy of that half.  Starting from O = G/2, lane g of a group ends with the
// totals of values g NC/G on in v[0 .. NC/G).  Lane exchanges of the vector unit throughout: no
// LDS, which a near field beside the kernel may hold, and no round trips to it (leaves of
// 3000001 clustered particles, FP64, 16 lanes each: 86 us with a shuffled sum of every
// coefficient in every lane, 39 us).
template <typename TC, int NC, int W, int O>
__device__ __forceinline__ void lane_halve(TC (&v)[NC], int lane)
{
    static_assert(O <= 16 && (O < 1 || W > 1), "at most 32 lanes, at least as many values");
    if constexpr (O >= 1) {
        const bool hi = (lane & O) != 0;
#pragma unroll
        for (int k = 0; k < W / 2; ++k) {
            if constexpr (O == 16) {
                v[k] = swap_sum16(v[k], v[k + W / 2]);
            } else {
                const TC send = hi ? v[k] : v[k + W / 2];
                const TC keep = hi ? v[k + W / 2] : v[k];
                v[k] = keep + lane_partner<O>(send);
            }
        }
        lane_halve<TC, NC, W / 2, O / 2>(v, lane);
    }
}

// Lane g of a group of G stores the totals that lane_halve left it, of n values in all.
template <typename TC, int NC, int G>
__device__ __forceinline__ void store_halved(const TC (&v)[NC], int g, int n, TC *__restrict__ out)
{
#pragma unroll
    for (int k = 0; k < NC / G; ++k)
        if (g * (NC / G) + k < n) out[g * (NC / G) + k] = v[k];
}

// ---------------------------------------------------------------------------------
// Per-particle gathers of the finalize kernels, written so that a wavefront waits for
// memory a few times rather than once per load.  A load guarded by a lane-dependent
// branch is followed by a wait inside the branch, so nine guarded slot loads cost nine
// memory round trips; a loop over coefficients with a run-time bound waits once per
// coefficient.
// ---------------------------------------------------------------------------------

// Near-field velocity of sorted particle i of n from the mutual form: the target-centric
// part near[i] when bit 9 of the leaf mask m is set, minus/plus scale times the slots
// d = 0..8 whose bits are set, summed in that order.  The slot loads go out together,
// unguarded: a slot the leaf's items did not write is read at the address of the lowest
// one they did (a line this particle reads anyway) and its value discarded by a select,
// so the wavefront waits once.  (Guarding each load by its bit made the compiler wait
// after each.)  su and sv start at +0 and never become -0, so adding +0 for an unset slot
// gives the bits of skipping it.
template <typename TS>
__device__ __forceinline__ double2 near_from_slots(int64_t i, int64_t n, int m, const double2 *__restrict__ near,
                                                   const c2<TS> *__restrict__ slots, double scale)
{
    double2 r = make_double2(0.0, 0.0);
    if ((m >> 9) & 1) r = near[i];
    const int set = m & 0x1FF;
    if (set) {
        const int64_t lowest = (int64_t)__builtin_ctz(set) * n + i;
        c2<TS> v[9];
#pragma unroll
        for (int d = 0; d < 9; ++d) v[d] = slots[(set >> d) & 1 ? (int64_t)d * n + i : lowest];
        double su = 0.0, sv = 0.0;
#pragma unroll
        for (int d = 0; d < 9; ++d) {
            const bool on = (set >> d) & 1;
            su += on ? (double)v[d].x : 0.0;
            sv += on ? (double)v[d].y : 0.0;
        }
        r.x -= scale * su;
        r.y += scale * sv;
    }
    return r;
}

// The third sum of the adjoint's near field, gathered the same way.
template <typename TS>
__device__ __forceinline__ double phi_from_slots(int64_t i, int64_t n, int m, const double *__restrict__ near,
                                                 const TS *__restrict__ slots)
{
    double r = 0.0;
    if ((m >> 9) & 1) r = near[i];
    const int set = m & 0x1FF;
    if (set) {
        const int64_t lowest = (int64_t)__builtin_ctz(set) * n + i;
        TS v[9];
#pragma unroll
        for (int d = 0; d < 9; ++d) v[d] = slots[(set >> d) & 1 ? (int64_t)d * n + i : lowest];
#pragma unroll
        for (int d = 0; d < 9; ++d) r += (set >> d) & 1 ? (double)v[d] : 0.0;
    }
    return r;
}

// Horner's rule b_{p-1} x^{p-1} + ... + b_0 (p >= 1), in the order l = p-2 .. 0, with the
// coefficients loaded eight at a time ahead of their use (an index below 0 re-reads b_0
// and is not used).
template <typename T>
__device__ __forceinline__ c2<T> horner_prefetch(const c2<T> *__restrict__ b, int p, c2<T> x)
{
    c2<T> acc = b[p - 1];
    for (int l0 = p - 2; l0 >= 0; l0 -= 8) {
        c2<T> c[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = b[l0 - k >= 0 ? l0 - k : 0];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (l0 - k >= 0) acc = cmac<T>(c[k], acc, x);
    }
    return acc;
}

// Horner's rule with weighted coefficients, sum_{l=lo}^{p-1} (l + add) b_l x^(l-lo)
// (p > lo), in the order l = p-2 .. lo, the coefficients loaded eight at a time ahead of
// their use: the derivative of the series above with lo = 1, add = 0.
template <typename T>
__device__ __forceinline__ c2<T> horner_weighted_prefetch(const c2<T> *__restrict__ b, int p, c2<T> x, int lo,
                                                          int add)
{
    const c2<T> top = b[p - 1];
    const T wt = (T)(p - 1 + add);
    c2<T> acc = mk<T>(wt * top.x, wt * top.y);
    for (int l0 = p - 2; l0 >= lo; l0 -= 8) {
        c2<T> c[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = b[l0 - k >= lo ? l0 - k : lo];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (l0 - k >= lo) {
                const T l = (T)(l0 - k + add);
                acc = cmac<T>(mk<T>(l * c[k].x, l * c[k].y), acc, x);
            }
    }
    return acc;
}

// A velocity row of user row o: the velocity itself, or with a base (the transport
// update of section "Test problem", dx/dt = u, one explicit stage) base + h u.
__device__ __forceinline__ void store_velocity(double *uv, int64_t o, double2 v, const double *base, double h)
{
    if (base) {
        v.x = fma(h, v.x, base[2 * o]);
        v.y = fma(h, v.y, base[2 * o + 1]);
    }
    uv[2 * o] = v.x;
    uv[2 * o + 1] = v.y;
}

// Second half of a staged finalize: (u, v) of sorted particle i, written in sorted order
// by the finalize kernel, to row perm[i] of the user-order output.  Reading the slot sums
// and writing rows in random order in one kernel took longer (840 us for 2^24 particles)
// than doing each in a kernel of its own (413 + 343 us).
namespace {
__global__ __launch_bounds__(256) void scatter_rows_kernel(int n, const int *__restrict__ perm,
                                                           const double2 *__restrict__ staged,
                                                           double *__restrict__ uv, const double *__restrict__ base,
                                                           double h)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    store_velocity(uv, perm[i], staged[i], base, h);
}
}  // namespace

__device__ __forceinline__ void store_adjoint(const AdjointOut &a, int64_t o, double g, double ex, double ey, double sx,
                                              double sy)
{
    if (a.dg) a.dg[o] = a.acc_g ? a.dg[o] + g : g;
    if (a.dxe) {
        a.dxe[2 * o] = ex;
        a.dxe[2 * o + 1] = ey;
    }
    if (a.dxs) {
        a.dxs[2 * o] = sx;
        a.dxs[2 * o + 1] = sy;
    }
    if (a.dxy) {
        double vx = ex + sx, vy = ey + sy;
        if (a.lam) {
            vx += a.lam[2 * o];
            vy += a.lam[2 * o + 1];
        }
        if (a.acc_xy) {
            vx += a.dxy[2 * o];
            vy += a.dxy[2 * o + 1];
        }
        a.dxy[2 * o] = vx;
        a.dxy[2 * o + 1] = vy;
    }
}

}  // namespace fmm
