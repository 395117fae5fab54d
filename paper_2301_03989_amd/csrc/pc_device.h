// pc_device.h -- device-side building blocks shared by the fused and the plain kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <type_traits>
#include "pc_internal.h"

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

#define PC_PI 3.14159265358979323846

// Moves inside a row of 16 lanes through DPP (no LDS round trip, unlike a lane shuffle).
// CTRL: 0xB1 quad_perm [1,0,3,2] (lane ^ 1), 0x4E quad_perm [2,3,0,1] (lane ^ 2),
// 0x128 row_ror:8 (lane ^ 8), 0x141 row_half_mirror (7 - lane in each 8),
// 0x140 row_mirror (15 - lane).  Callers keep the source lanes active.
template <int CTRL>
static __device__ __forceinline__ int pc_dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
static __device__ __forceinline__ float pc_dpp(float v)
{
    return __builtin_bit_cast(float, pc_dpp<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
static __device__ __forceinline__ double pc_dpp(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)pc_dpp<CTRL>((int)(unsigned)b);
    const unsigned hi = (unsigned)pc_dpp<CTRL>((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Sum (OR) over the 16 lanes of a row, the butterfly over lane ^ 1, ^ 2, ^ 4, ^ 8: after
// the two quad steps every quad holds one value, so the mirrored lanes (7 - lane within
// each 8, then 15 - lane) hold what lane ^ 4 and lane ^ 8 hold, and every lane ends with
// the butterfly's result bit for bit.
static __device__ __forceinline__ double pc_row_sum16(double v)
{
    v += pc_dpp<0xB1>(v);
    v += pc_dpp<0x4E>(v);
    v += pc_dpp<0x141>(v);
    v += pc_dpp<0x140>(v);
    return v;
}
static __device__ __forceinline__ int pc_row_or16(int v)
{
    v |= pc_dpp<0xB1>(v);
    v |= pc_dpp<0x4E>(v);
    v |= pc_dpp<0x141>(v);
    v |= pc_dpp<0x140>(v);
    return v;
}

static __device__ __forceinline__ f64x4 mfma16(double a, double b, f64x4 c)
{
    // D = A(16x4) B(4x16) + C.  Operand lanes: A[l%16][l/16], B[l/16][l%16];
    // result lanes on gfx950: D[l/16 + 4r][l%16] in element r.
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

static __device__ __forceinline__ f32x4 mfma16f(float a, float b, f32x4 c)
{
    // f32 16x16x4: same operand lanes as the f64 form; result D[4(l/16) + r][l%16] in element r
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// max that propagates NaN from either argument
static __device__ __forceinline__ double nmax(double a, double b)
{
    return (a > b || a != a) ? a : b;
}

// ---------------------------------------------------------------------------
// Two-body orbits (gravitational parameter 1)
// ---------------------------------------------------------------------------

// Eccentric anomaly from the mean anomaly (Kepler's equation, Newton's method).
// Returns E modulo 2 pi.
static __device__ double pc_ecc_anomaly(double M, double e)
{
    const double Mr = M - 2.0 * PC_PI * rint(M / (2.0 * PC_PI));
    double E = (e < 0.8) ? Mr : (Mr >= 0.0 ? PC_PI : -PC_PI);
    for (int it = 0; it < 60; ++it) {
        double sE, cE;
        sincos(E, &sE, &cE);
        const double dE = (E - e * sE - Mr) / (1.0 - e * cE);
        E -= dE;
        if (fabs(dE) <= 1e-10 * (1.0 + fabs(E))) break;   // quadratic: the next error is ~dE^2
    }
    return E;
}

static __device__ void pc_body_position(const PcBodyDev& B, double dt_epoch, double r[3])
{
    const double E = pc_ecc_anomaly(B.M0 + B.n * dt_epoch, B.e);
    double sE, cE;
    sincos(E, &sE, &cE);
    const double xp = B.a * (cE - B.e);
    const double yp = B.b * sE;
    for (int k = 0; k < 3; ++k) r[k] = xp * B.P[k] + yp * B.Q[k];
}

// Position and velocity of a body on its Keplerian orbit (gravitational parameter 1):
// the velocity is the time derivative of the position, dE/dt = n / (1 - e cos E).
static __device__ void pc_body_state(const PcBodyDev& B, double dt_epoch, double r[3], double v[3])
{
    const double E = pc_ecc_anomaly(B.M0 + B.n * dt_epoch, B.e);
    double sE, cE;
    sincos(E, &sE, &cE);
    const double Ed = B.n / (1.0 - B.e * cE);
    const double xp = B.a * (cE - B.e), yp = B.b * sE;
    const double xd = -B.a * sE * Ed, yd = B.b * cE * Ed;
    for (int k = 0; k < 3; ++k) {
        r[k] = xp * B.P[k] + yp * B.Q[k];
        v[k] = xd * B.P[k] + yd * B.Q[k];
    }
}

// 1/sqrt(x) in full FP64 for finite x > 0: the hardware estimate y, e = 1 - x y^2, and
// (1 - e)^(-1/2) = 1 + e/2 + 3e^2/8 + O(e^3) (|e| near 2^-22, dropped terms below 2^-63).
static __device__ __forceinline__ double pc_rsqrt_full(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x, y * y, 1.0);
    return y * fma(e, fma(0.375, e, 0.5), 1.0);
}

// sqrt(x) and 1/sqrt(x), each rounded about once (one more correction by the residual of each).
static __device__ __forceinline__ void pc_roots(double x, double& s, double& i)
{
    i = pc_rsqrt_full(x);
    s = x * i;
    s = fma(0.5 * i, fma(-s, s, x), s);
    i = fma(i, fma(-s, i, 1.0), i);
}

// 1/x by the hardware estimate (relative error near 2^-22) and one Newton step (2^-44) or two.
static __device__ __forceinline__ double pc_rcp1(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}
static __device__ __forceinline__ double pc_rcp_full(double x)
{
    const double y = pc_rcp1(x);
    return fma(y, fma(-x, y, 1.0), y);
}

// Sine and cosine: x - k pi/2 with pi/2 in two parts (off by k 1.5e-33, less than the rounding
// of x itself at any k), then the Taylor series on [-pi/4, pi/4], whose dropped terms are below
// 1e-18.  A third of the library call's instructions.  No call for large angles: with one on
// that path, never taken by an orbit, the solve saved and reloaded two dozen registers at every
// call; without it the 12000 eccentric ICs of 48 nodes went from 4.98 to 4.63 ms, a single
// orbit of 32 nodes from 215 to 209 us.
static __device__ __forceinline__ void pc_sincos(double x, double& s, double& c)
{
    const double k = rint(x * 0.63661977236758134308);
    double r = fma(-k, 6.12323399573676603587e-17, fma(-k, 1.57079632679489655800, x));
    r = fabs(r) > 1.0 ? r - r : r;   // beyond 2^52 turns x has no phase left: any on the circle
    const double z = r * r;
    double p = 1.0 / 355687428096000.0, q = 1.0 / 20922789888000.0;
    p = fma(p, z, -1.0 / 1307674368000.0);
    q = fma(q, z, -1.0 / 87178291200.0);
    p = fma(p, z, 1.0 / 6227020800.0);
    q = fma(q, z, 1.0 / 479001600.0);
    p = fma(p, z, -1.0 / 39916800.0);
    q = fma(q, z, -1.0 / 3628800.0);
    p = fma(p, z, 1.0 / 362880.0);
    q = fma(q, z, 1.0 / 40320.0);
    p = fma(p, z, -1.0 / 5040.0);
    q = fma(q, z, -1.0 / 720.0);
    p = fma(p, z, 1.0 / 120.0);
    q = fma(q, z, 1.0 / 24.0);
    p = fma(p, z, -1.0 / 6.0);
    q = fma(q, z, -0.5);
    const double sr = fma(r * z, p, r), cr = fma(z, q, 1.0);
    const int m = (int)fma(-4.0, rint(0.25 * k), k);   // k modulo 4, -2..2
    const double ss = (m & 1) ? cr : sr, cc = (m & 1) ? sr : cr;
    s = (m & 2) ? -ss : ss;
    c = ((m + 1) & 2) ? -cc : cc;
}

// Warm start (Sec. 2.1): propagate y0 by dt on its osculating ellipse, through the
// Lagrange coefficients f, g, fdot, gdot written in the eccentric-anomaly change x:
//   F(x) = x - (1 - r0/a) sin x + (r0.v0/sqrt(a)) (1 - cos x) - n dt = 0.
// Solved by Halley's iteration x -= 2 F F' / (2 F'^2 - F F''), cubically convergent; F''
// comes from the same sine and cosine as F and F'.  Three steps in FP32 on the hardware sine
// bring the start n dt to about 1e-6 (they only choose the starting point); the FP64 steps
// then go on until one is below 1e-5.  The error after a step is about K e^3, e the error
// before it (close to the step) and K = O(1) for e < 0.8, so that leaves an error near 1e-15,
// usually after the first; the sine and cosine at the final x follow from those of the last
// step by its second-order Taylor expansion (the dropped cubic term is under 2e-16).
// The square roots and divisions are the hardware estimates refined to full FP64, the roots to
// their last place (pc_roots), and 1/n is corrected against n: an ulp of either is multiplied by the
// angle n dt.  Steps of up to 8 time units, e = 0, 0.3 and 0.6: median error 1.0e-15, 1.0e-15 and
// 0.9e-15 with IEEE roots and divisions, 1.5e-15, 1.4e-15 and 1.2e-15 without these corrections,
// 0.9e-15, 1.0e-15 and 0.9e-15 with them (sixteen of 250 instructions).
// What bounds it is one wave's chain of dependent FP64 instructions: a column refill waits
// for one solve per lane.  Four FP64 steps from n dt with library sines and IEEE divisions
// took about 900 instructions, this about 250 without them: 12000 eccentric ICs of 48 nodes and 16 segments
// (a third of the sweeps refill a column) 5.20 -> 5.08 ms, the uneven 65536-IC batch 160.0 ->
// 157.8 ms (each before the sweeps themselves were shortened).
// The state goes in and out by value (registers, no stack traffic); a non-elliptic or
// degenerate state returns NaN components.
struct PcState6 {
    double c[6];
};

static __device__ __attribute__((noinline)) PcState6 pc_kepler_state(PcState6 s0, double dt)
{
    const double* y0 = s0.c;
    PcState6 out;
    const double r02 = y0[0] * y0[0] + y0[1] * y0[1] + y0[2] * y0[2];
    const double v02 = y0[3] * y0[3] + y0[4] * y0[4] + y0[5] * y0[5];
    double r0n, ir0;
    pc_roots(r02, r0n, ir0);
    const double alpha = fma(2.0, ir0, -v02);      // 1/a
    if (!(r0n > 0.0) || !isfinite(r0n) || !isfinite(v02) || !(alpha > 0.0)) {
#pragma unroll
        for (int k = 0; k < 6; ++k) out.c[k] = (double)NAN;
        return out;
    }
    double sqal, sqa;
    pc_roots(alpha, sqal, sqa);                    // sqa = sqrt(a)
    double a = sqa * sqa;
    a = fma(a, fma(-alpha, a, 1.0), a);
    const double n = alpha * sqal;                 // mean motion
    const double sig = y0[0] * y0[3] + y0[1] * y0[4] + y0[2] * y0[5];
    const double ec = fma(-r0n, alpha, 1.0);       // e cos E0
    const double es = sig * sqal;                  // e sin E0
    const double ndt = n * dt;
    double x = ndt;
    {
        // u = x - n dt; angles in turns, as the hardware sine takes them
        const float i2p = 0.15915494309189535f;
        const double t = ndt * 0.15915494309189533577;
        const float t0 = (float)(t - rint(t)), ecf = (float)ec, esf = (float)es;
        float u = 0.0f;
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const float an = fmaf(u, i2p, t0);
            const float sf = __builtin_amdgcn_sinf(an), cf = __builtin_amdgcn_cosf(an);
            const float F = u - ecf * sf + esf * (1.0f - cf);
            const float F1 = 1.0f - ecf * cf + esf * sf;
            const float F2 = ecf * sf + esf * cf;
            u -= 2.0f * F * F1 * __builtin_amdgcn_rcpf(2.0f * F1 * F1 - F * F2);
            u = fminf(fmaxf(u, -2.0f), 2.0f);   // |u| <= 2 e at the solution
        }
        x += (double)u;
    }
    // F rises with x: near e = 1 a step that leaves the bracket is replaced by its midpoint
    double lo = ndt - 2.0, hi = ndt + 2.0;
    double sx, cx;
    bool done = false;
    for (int it = 0; it < 60; ++it) {
        pc_sincos(x, sx, cx);
        const double F = x - ec * sx + es * (1.0 - cx) - ndt;
        const double F1 = 1.0 - ec * cx + es * sx;
        const double F2 = ec * sx + es * cx;
        double xn = x - 2.0 * F * F1 * pc_rcp1(2.0 * F1 * F1 - F * F2);
        lo = F > 0.0 ? lo : x;
        hi = F > 0.0 ? x : hi;
        if (!(xn >= lo && xn <= hi)) xn = 0.5 * (lo + hi);
        const double dx = x - xn;
        x = xn;
        if (fabs(dx) <= 1e-5) {
            // sin and cos of x = x_prev - dx
            const double h2 = 0.5 * dx * dx;
            const double s1 = sx - dx * cx - h2 * sx;
            const double c1 = cx + dx * sx - h2 * cx;
            sx = s1;
            cx = c1;
            done = true;
            break;
        }
    }
    if (!done) pc_sincos(x, sx, cx);
    const double rn = a + (r0n - a) * cx + sig * sqa * sx;
    const double irn = pc_rcp_full(rn);
    const double f = 1.0 - a * ir0 * (1.0 - cx);
    double in = sqa * a;                           // 1/n
    in = fma(in, fma(-n, in, 1.0), in);
    const double g = fma(sx - x, in, dt);
    const double irr = irn * ir0, fq = -sqa * sx;
    const double fd0 = fq * irr, fd = fma(fma(-fd0, rn * r0n, fq), irr, fd0);
    const double gd = 1.0 - a * irn * (1.0 - cx);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        out.c[k] = f * y0[k] + g * y0[3 + k];
        out.c[3 + k] = fd * y0[k] + gd * y0[3 + k];
    }
    return out;
}

// Array form of the warm start; false when the result is not finite (y then unspecified).
static __device__ __forceinline__ bool pc_kepler(const double (&y0)[6], double dt, double (&y)[6])
{
    PcState6 s0;
#pragma unroll
    for (int k = 0; k < 6; ++k) s0.c[k] = y0[k];
    const PcState6 r = pc_kepler_state(s0, dt);
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        y[k] = r.c[k];
        ok = ok && isfinite(r.c[k]);
    }
    return ok;
}

// From here on the multiply-adds of the sweeps are written out and contraction is off, so that
// every job body rounds alike: an IC's iterates do not depend on the body, job or column.
#pragma clang fp contract(off)

// mu / x^(3/2) in full FP64 for finite x > 0, the attraction factor of a point mass at
// squared distance x: from the hardware estimate y of 1/sqrt(x) and e = 1 - x y^2 (x y^2
// with y^2 rounded), x^(-3/2) = (y^2)^(3/2) (1 - e)^(-3/2) = y^3 (1 + 3e/2 + 15e^2/8 + O(e^3)).
// The series coefficients come premultiplied into the mass (mu1 = 3 mu / 2,
// mu2 = 15 mu / 8), so a point-body pair costs six operations after the estimate.  With
// |e| near 2^-22 the dropped terms are below 2^-63 relative.
static __device__ __forceinline__ double pc_mu_r3(double x, double mu, double mu1, double mu2)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double t = y * y;
    const double e = fma(-x, t, 1.0);
    return (y * t) * fma(e, fma(mu2, e, mu1), mu);
}

static __device__ __forceinline__ double pc_norm2(double x, double y, double z)
{
    return fma(z, z, fma(y, y, x * x));
}

// One attracting body's acceleration at offset d.
static __device__ __forceinline__ void pc_pull(double dx, double dy, double dz, double mu, double mu1, double mu2,
                                               double& ax, double& ay, double& az)
{
    const double s = pc_mu_r3(pc_norm2(dx, dy, dz), mu, mu1, mu2);
    ax = fma(-s, dx, ax);
    ay = fma(-s, dy, ay);
    az = fma(-s, dz, az);
}

// ---------------------------------------------------------------------------
// Force model: point masses in the heliocentric frame with the indirect term,
//   a = -mu_S r/|r|^3 - sum_p mu_p (r - r_p)/|r - r_p|^3 - sum_p mu_p r_p/|r_p|^3.
// rec[p] = (r_p, mu_p) for p < P; rec[P] = (precomputed indirect sum, 0).
// ---------------------------------------------------------------------------
static __device__ __forceinline__ void pc_accel(double x, double y, double z, const double4* rec,
                                                int P, double mu_sun, double& ax, double& ay,
                                                double& az)
{
    ax = ay = az = 0.0;
    pc_pull(x, y, z, mu_sun, 1.5 * mu_sun, 1.875 * mu_sun, ax, ay, az);
    for (int p = 0; p < P; ++p) {
        const double4 q = rec[p];
        pc_pull(x - q.x, y - q.y, z - q.z, q.w, 1.5 * q.w, 1.875 * q.w, ax, ay, az);
    }
    const double4 ind = rec[P];
    ax -= ind.x;
    ay -= ind.y;
    az -= ind.z;
}


// ---------------------------------------------------------------------------
// Shared pieces of the propagation kernels
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(1))) double* gconst_dp;
typedef const __attribute__((address_space(1))) char* gconst_cp;
typedef double pc_d2v __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) pc_d2v* gconst_d2p;

// Base address of per-segment records that is one value per wave (scalar registers): a
// load then adds only the lane's 32-bit byte offset, a global load with a scalar base and
// no per-lane 64-bit address arithmetic.  Callers pass records of one segment of one job,
// the same for every lane of the wave.
static __device__ __forceinline__ gconst_cp pc_wave_base(const void* e)
{
    const uint64_t v = reinterpret_cast<uint64_t>(e);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (gconst_cp)((((uint64_t)hi) << 32) | lo);
}
static __device__ __forceinline__ double4 pc_load_d4(gconst_cp q)
{
    const gconst_d2p p = (gconst_d2p)q;
    const pc_d2v a = p[0], b = p[1];
    return make_double4(a.x, a.y, b.x, b.y);
}
typedef __attribute__((address_space(1))) double* gdp;
typedef __attribute__((address_space(1))) int32_t* gi32p;

// Global-memory views of the buffers the kernel parameters point to.  Pointers read from
// the parameter block are generic, so the compiler emits flat loads and stores for them;
// a flat access counts against the LDS counter too, so the next wait for an LDS read also
// waits for it to reach memory, and it may alias LDS, so loads around LDS stores are
// issued one at a time.  Through these views the accesses are global instructions.
static __device__ __forceinline__ gdp pc_gd(double* q) { return (gdp)q; }
static __device__ __forceinline__ gconst_dp pc_gcd(const double* q) { return (gconst_dp)q; }
static __device__ __forceinline__ gi32p pc_gi(int32_t* q) { return (gi32p)q; }

// Shape of a job: NP padded nodes x T = PAIRS / NP ICs on NT threads in W waves.
//
// From 32 padded nodes on (PAR) the sweep works on pairs of mirrored nodes (row i: node i and
// node N-1-i, tau = -tau'), because integration maps the even and the odd part of F apart
// (pc_product).  A wave owns 16 rows x 8 ICs: both nodes of the pair, all six components.
// The 16 IC rows of an MFMA block are the position (rows 0..7) and the velocity (8..15)
// component b of the 8 ICs, and block 3h + b belongs to node h of the pair, so by the result
// layout (row l/16 + 4r in element r, column l%16) a lane holds the full states of two ICs at
// both nodes of one row: norms, force and gravity gradient need no other lane.
// At 16 padded nodes a pair block would be half padding; there a row is one node, and block
// 3h + b belongs to the h-th eight of a wave's 16 ICs.
//
// LDS layout of F: [row][group of ICs][b 3][i 16][h 2], i = 8 (component half) + IC of the
// group's eight, place i XOR-ed with row % 16.  One ds_read_b128 gives a lane the operands of
// both h; the 16 lanes of a k row read 256 consecutive bytes, and the 16 lanes that publish
// one IC at 16 rows write 16 different 16-byte places (without the XOR all would fall on the
// same banks, a row being a multiple of 256 bytes).
template <int PAIRS, int NP>
struct PcShape {
    static constexpr int NT = PAIRS / 4;
    static constexpr int W = NT / 64;
    static constexpr int T = PAIRS / NP;
    static constexpr bool PAR = NP >= 32;
    static constexpr int KR = PAR ? NP / 2 : NP;   // rows of F
    static constexpr int NQ = KR / 4;              // k steps of the 16x16x4 product
    static constexpr int STRIPS = KR / 16;
    static constexpr int COLS = PAR ? 8 : 16;      // ICs of one wave (a group)
    static constexpr int GN = T / COLS;            // groups
    static constexpr int ROW = GN * 96;            // doubles per row of F
    static constexpr int E = PAR ? 2 : 4;          // ICs a lane holds points of
    static_assert(T >= 8 && T <= PAIRS / 16 && W == STRIPS * GN, "unsupported job shape");
};

struct PcLane {
    int lane, wave, strip, grp;
    int g, c;        // lane / 16, lane % 16
    int row;         // the lane's row of F
    int jn[2];       // its nodes (past the last row: those of the last one)
    bool ok;         // the row holds nodes
    bool two;        // the row's nodes differ (not the middle node of an odd count, nor one-node rows)
    int nq;          // k steps the products run: up to the last block of 16 rows that holds nodes
};

// The fragments of the operators are zero past the last row, so the products stop after the
// last 16-row block holding one (4 k steps each; at least two blocks when the padded count
// has them, which the k loop's prologue needs).
// Waves of one group are consecutive: a job with few ICs keeps one wave per SIMD busy.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_lane_place(PcLane& L, int N)
{
    using Sh = PcShape<PAIRS, NP>;
    const int M = Sh::PAR ? (N + 1) >> 1 : N;
    L.g = L.lane >> 4;
    L.c = L.lane & 15;
    L.row = L.strip * 16 + L.c;
    L.ok = L.row < M;
    const int i = L.ok ? L.row : M - 1;
    L.jn[0] = i;
    L.jn[1] = Sh::PAR ? N - 1 - i : i;
    L.two = Sh::PAR && L.jn[1] != L.jn[0];
}
template <int PAIRS, int NP>
static __device__ __forceinline__ PcLane pc_lane_geometry(int tid, int N)
{
    using Sh = PcShape<PAIRS, NP>;
    PcLane L;
    const int M = Sh::PAR ? (N + 1) >> 1 : N;
    L.nq = Sh::NQ > 4 ? min(Sh::NQ, max(8, ((M + 15) >> 4) << 2)) : Sh::NQ;
    L.lane = tid & 63;
    L.wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // one value per wave: scalar registers and branches
    L.strip = L.wave % Sh::STRIPS;
    L.grp = L.wave / Sh::STRIPS;
    pc_lane_place<PAIRS, NP>(L, N);
    return L;
}
// The same lane, its places computed again from here on: a sweep loop then forms its LDS
// addresses where it uses them (a few integer instructions) instead of holding each across the
// loop, which spilled them to scratch.
template <int PAIRS, int NP>
static __device__ __forceinline__ PcLane pc_lane_again(const PcLane& L, int N)
{
    PcLane R = L;
    asm volatile("" : "+v"(R.lane));
    pc_lane_place<PAIRS, NP>(R, N);
    return R;
}

// Column (IC within the group) of the lane's e-th IC, and the IC (within the job) of its point
// (h, r).
template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_col(const PcLane& L, int e)
{
    return PcShape<PAIRS, NP>::PAR ? L.g + 4 * e : 8 * (e >> 1) + L.g + 4 * (e & 1);
}
template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_ic(const PcLane& L, int h, int r)
{
    using Sh = PcShape<PAIRS, NP>;
    return L.grp * Sh::COLS + (Sh::PAR ? 0 : 8 * h) + L.g + 4 * r;
}

// Place of (row, group, b, i) in F, in pairs of values.
template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_unit(int row, int grp, int b, int i)
{
    return row * (PcShape<PAIRS, NP>::ROW / 2) + grp * 48 + b * 16 + (i ^ (row & 15));
}

// Shared-memory arena of one workgroup (sized for the largest job shape).
// Past the 6T doubles in use, Y0 holds the weights of the job's rows (pc_weights).
template <int PAIRS>
struct PcSmem {
    static constexpr int REC = pc_rec_cap(PAIRS);
    alignas(16) double F[6 * PAIRS];
    alignas(16) double Rec[REC];  // [node][body 0..P][3]: perturber positions, then the indirect term
    double Y0[6 * (PAIRS / 16)];  // [comp][IC] initial state of the current segment
    alignas(16) double Mu[4 * PC_MAX_PERT_DEV];   // per perturber mu, 3 mu / 2, 15 mu / 8 (pc_mu_r3), 0
    int Flag[(PAIRS / 256) * 16]; // per wave, per IC: bit 0 not converged, bit 1 non-finite, bit 2 large change
    int Keep[PAIRS / 256];        // per wave: an iterating IC still changes by more than the FP32 switch
    int Go[PAIRS / 256];          // per wave (or IC group): some IC still iterates after this sweep
    int Active[PAIRS / 16];
    int Dead[PAIRS / 16];
};

template <int PAIRS, int NP>
static __device__ __forceinline__ double* pc_weights(PcSmem<PAIRS>& sm)
{
    return sm.Y0 + 6 * PcShape<PAIRS, NP>::T;
}

// The rows' weights into LDS, once per job: w (even part of the last node's integral) and w2
// (odd part of its double integral, second-order sweeps).
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_stage_weights(PcSmem<PAIRS>& sm, const double* wts)
{
    using Sh = PcShape<PAIRS, NP>;
    if constexpr (Sh::PAR) {
        for (int i = threadIdx.x; i < 2 * Sh::KR; i += Sh::NT) pc_weights<PAIRS, NP>(sm)[i] = pc_gcd(wts)[i];
    }
}

// After the stopping rule (taken by threads tid < T on their IC's status word), the waves
// that hold status words note whether some IC still iterates; the barrier that ends the
// sweep makes the notes visible to every wave (one barrier instead of a barrier-reduction).
// The notes are rewritten only after the next sweep's first barrier, when every wave has
// read them.
template <int PAIRS, int NP, class Lane>
static __device__ __forceinline__ void pc_note_active(PcSmem<PAIRS>& sm, const Lane& L)
{
    constexpr int T = PAIRS / NP;
    if (L.wave * 64 < T) {
        const int tid = L.wave * 64 + L.lane;
        const unsigned long long b = __ballot(tid < T && sm.Active[tid]);
        if (L.lane == 0) sm.Go[L.wave] = b != 0ull;
    }
}
template <int PAIRS, int NP>
static __device__ __forceinline__ bool pc_any_active(const PcSmem<PAIRS>& sm)
{
    constexpr int T = PAIRS / NP;
    int a = 0;
#pragma unroll
    for (int w = 0; w < (T + 63) / 64; ++w) a |= sm.Go[w];
    return a != 0;
}

// ---------------------------------------------------------------------------
// Force, gravity gradient and Hessian products at a lane's four points: point p = 2h + r is
// IC r at node jn[h].
// ---------------------------------------------------------------------------
// Accelerations with the records in LDS (compact [node][body][3], masses [body][4]): two
// bodies at a time, so that a wave waits on LDS once per eight body-point pairs.
template <int R>
static __device__ __forceinline__ void pc_force_lds(const double (&x)[2 * R], const double (&y)[2 * R], const double (&z)[2 * R],
                                                    const int (&jn)[2], int P, double mu_sun, const double* srec,
                                                    const double* smu, double (&ax)[2 * R], double (&ay)[2 * R],
                                                    double (&az)[2 * R])
{
#pragma unroll
    for (int p = 0; p < 2 * R; ++p) {
        ax[p] = ay[p] = az[p] = 0.0;
        pc_pull(x[p], y[p], z[p], mu_sun, 1.5 * mu_sun, 1.875 * mu_sun, ax[p], ay[p], az[p]);
    }
    const double* rec[2] = {srec + jn[0] * 3 * (P + 1), srec + jn[1] * 3 * (P + 1)};
    auto bodies = [&](int b, auto nb) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb)::value;
        double q[NB][2][3], mu[NB][3];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const pc_d2v m01 = *reinterpret_cast<const pc_d2v*>(smu + 4 * (b + k));
            mu[k][0] = m01.x;
            mu[k][1] = m01.y;
            mu[k][2] = smu[4 * (b + k) + 2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int c = 0; c < 3; ++c) q[k][h][c] = rec[h][3 * (b + k) + c];
            }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
#pragma unroll
            for (int p = 0; p < 2 * R; ++p)
                pc_pull(x[p] - q[k][p / R][0], y[p] - q[k][p / R][1], z[p] - q[k][p / R][2], mu[k][0], mu[k][1],
                        mu[k][2], ax[p], ay[p], az[p]);
        }
    };
    int b = 0;
    for (; b + 2 <= P; b += 2) bodies(b, std::integral_constant<int, 2>{});
    if (b < P) bodies(b, std::integral_constant<int, 1>{});
#pragma unroll
    for (int p = 0; p < 2 * R; ++p) {
        ax[p] -= rec[p / R][3 * P];
        ay[p] -= rec[p / R][3 * P + 1];
        az[p] -= rec[p / R][3 * P + 2];
    }
}

// FP32 variant for the early sweeps of the precision schedule: the differences to the
// perturbers are formed in FP64, everything after them in FP32.
static __device__ __forceinline__ void pc_force_lds32(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                      const int (&jn)[2], int P, double mu_sun, const double* srec,
                                                      const double* smu, double (&ax)[4], double (&ay)[4],
                                                      double (&az)[4])
{
    float fx[4], fy[4], fz[4];
    auto add = [&](int p, float dx, float dy, float dz, float mu) __attribute__((always_inline)) {
        const float id = rsqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        const float s = mu * (id * id * id);
        fx[p] = fmaf(-s, dx, fx[p]);
        fy[p] = fmaf(-s, dy, fy[p]);
        fz[p] = fmaf(-s, dz, fz[p]);
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        fx[p] = fy[p] = fz[p] = 0.0f;
        add(p, (float)x[p], (float)y[p], (float)z[p], (float)mu_sun);
    }
    const double* rec[2] = {srec + jn[0] * 3 * (P + 1), srec + jn[1] * 3 * (P + 1)};
    for (int b = 0; b < P; ++b) {
        const float mu = (float)smu[4 * b];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double* q = rec[p >> 1] + 3 * b;
            add(p, (float)(x[p] - q[0]), (float)(y[p] - q[1]), (float)(z[p] - q[2]), mu);
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const double* q = rec[p >> 1] + 3 * P;
        ax[p] = (double)(fx[p] - (float)q[0]);
        ay[p] = (double)(fy[p] - (float)q[1]);
        az[p] = (double)(fz[p] - (float)q[2]);
    }
}

// Same as pc_force_lds with the records read from global memory ((x, y, z, mu) per body, then
// the indirect term), each where it is used: the other wave on the SIMD covers the wait.
static __device__ __forceinline__ void pc_force_glb(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                    const int (&jn)[2], int P, double mu_sun, const double4* grec,
                                                    double (&ax)[4], double (&ay)[4], double (&az)[4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        ax[p] = ay[p] = az[p] = 0.0;
        pc_pull(x[p], y[p], z[p], mu_sun, 1.5 * mu_sun, 1.875 * mu_sun, ax[p], ay[p], az[p]);
    }
    const gconst_cp base = pc_wave_base(grec);
    const uint32_t vo[2] = {(uint32_t)jn[0] * (uint32_t)(P + 1) * 32u, (uint32_t)jn[1] * (uint32_t)(P + 1) * 32u};
    for (int b = 0; b < P; ++b) {
        double4 q[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) q[h] = pc_load_d4((base + (size_t)b * 32) + vo[h]);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double4& k = q[p >> 1];
            pc_pull(x[p] - k.x, y[p] - k.y, z[p] - k.z, k.w, 1.5 * k.w, 1.875 * k.w, ax[p], ay[p], az[p]);
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const double4 q = pc_load_d4((base + (size_t)P * 32) + vo[p >> 1]);
        ax[p] -= q.x;
        ay[p] -= q.y;
        az[p] -= q.z;
    }
}

// Record of body b at the lane's node h: from LDS (compact [node][body][3], masses in smu) or
// from global memory (double4 (x, y, z, mu)).
template <bool LDSREC>
static __device__ __forceinline__ double4 pc_record(const double* srec, const double* smu, const double4* grec, int P,
                                                    int j, int b)
{
    if constexpr (LDSREC) {
        const double* q = srec + j * 3 * (P + 1) + 3 * b;
        return make_double4(q[0], q[1], q[2], smu[4 * b]);
    } else {
        return pc_load_d4((pc_wave_base(grec) + (size_t)b * 32) + (uint32_t)j * (uint32_t)(P + 1) * 32u);
    }
}

// One attracting body's term of H w at offset d (squared length x): with A = mu/|d|^3 from
// the premultiplied series of pc_mu_r3 and 1/|d|^2 = y^2 (1 + e + e^2) from the same
// estimate y (error of order e^3), h -= A w - 3 A/|d|^2 (d.w) d.
static __device__ __forceinline__ void pc_hess_term(double dx, double dy, double dz, double wx, double wy,
                                                    double wz, double mu, double mu1, double mu2, double& hx,
                                                    double& hy, double& hz)
{
    const double x = pc_norm2(dx, dy, dz);
    const double y = __builtin_amdgcn_rsq(x);
    const double t = y * y;
    const double e = fma(-x, t, 1.0);
    const double A = (y * t) * fma(e, fma(mu2, e, mu1), mu);
    const double i2 = fma(t, fma(e, e, e), t);
    const double c = (A * i2) * (3.0 * fma(dz, wz, fma(dy, wy, dx * wx)));
    hx = fma(c, dx, fma(-A, wx, hx));
    hy = fma(c, dy, fma(-A, wy, hy));
    hz = fma(c, dz, fma(-A, wz, hz));
}

// H w for the symmetric force Jacobian H = da/dr at the lane's points: every attracting body
// with parameter mu at offset d contributes -mu (w/|d|^3 - 3 d (d.w)/|d|^5); the indirect term
// does not depend on r.
template <bool LDSREC>
static __device__ __forceinline__ void pc_hess_apply(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                     const double (&wx)[4], const double (&wy)[4],
                                                     const double (&wz)[4], const int (&jn)[2], int P, double mu_sun,
                                                     const double* srec, const double* smu, const double4* grec,
                                                     double (&hx)[4], double (&hy)[4], double (&hz)[4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        hx[p] = hy[p] = hz[p] = 0.0;
        pc_hess_term(x[p], y[p], z[p], wx[p], wy[p], wz[p], mu_sun, 1.5 * mu_sun, 1.875 * mu_sun, hx[p], hy[p], hz[p]);
    }
    for (int b = 0; b < P; ++b) {
        double4 q[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) q[h] = pc_record<LDSREC>(srec, smu, grec, P, jn[h], b);
        const double mu1 = LDSREC ? smu[4 * b + 1] : 1.5 * q[0].w, mu2 = LDSREC ? smu[4 * b + 2] : 1.875 * q[0].w;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double4& k = q[p >> 1];
            pc_hess_term(x[p] - k.x, y[p] - k.y, z[p] - k.z, wx[p], wy[p], wz[p], k.w, mu1, mu2, hx[p], hy[p], hz[p]);
        }
    }
}

// The Jacobian H = da/dr itself at the lane's points, (xx, yy, zz, xy, xz, yz): every attracting
// body adds 3 A/|d|^2 d d^T - A, A = mu/|d|^3.  The adjoint's points stay fixed over a segment's
// sweeps: forming H once and taking H w as 9 multiply-adds replaces a pass over the bodies (27
// FP64 instructions each) in every sweep, and H takes the registers of the iterate, which the
// sweeps no longer need: forward and gradient of 16384 ICs (128 nodes, 5 segments) 13.4 -> 11.8 ms.
template <bool LDSREC>
static __device__ __forceinline__ void pc_hess_matrix(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                      const int (&jn)[2], int P, double mu_sun, const double* srec,
                                                      const double* smu, const double4* grec, double (&H)[6][4])
{
    auto add = [&](int p, double dx, double dy, double dz, double mu, double mu1, double mu2)
                   __attribute__((always_inline)) {
        const double r2 = pc_norm2(dx, dy, dz);
        const double v = __builtin_amdgcn_rsq(r2);
        const double t = v * v;
        const double e = fma(-r2, t, 1.0);
        const double A = (v * t) * fma(e, fma(mu2, e, mu1), mu);
        const double B = 3.0 * (A * fma(t, fma(e, e, e), t));
        const double bx = B * dx, by = B * dy;
        H[0][p] += fma(bx, dx, -A);
        H[1][p] += fma(by, dy, -A);
        H[2][p] += fma(B * dz, dz, -A);
        H[3][p] = fma(bx, dy, H[3][p]);
        H[4][p] = fma(bx, dz, H[4][p]);
        H[5][p] = fma(by, dz, H[5][p]);
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int k = 0; k < 6; ++k) H[k][p] = 0.0;
        add(p, x[p], y[p], z[p], mu_sun, 1.5 * mu_sun, 1.875 * mu_sun);
    }
    for (int b = 0; b < P; ++b) {
        double4 q[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) q[h] = pc_record<LDSREC>(srec, smu, grec, P, jn[h], b);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double4& k = q[p >> 1];
            add(p, x[p] - k.x, y[p] - k.y, z[p] - k.z, k.w, 1.5 * k.w, 1.875 * k.w);
        }
    }
}

// Linear change of the point-mass acceleration over a position change at the lane's points:
// g = (da/dr)(r) dr, the Hessian product with w = dr.
static __device__ __forceinline__ void pc_grad_dot(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                   const double (&dx)[4], const double (&dy)[4], const double (&dz)[4],
                                                   const int (&jn)[2], int P, double mu_sun, bool rec_lds,
                                                   const double* srec, const double* smu, const double4* grec,
                                                   double (&gx)[4], double (&gy)[4], double (&gz)[4])
{
    if (rec_lds) pc_hess_apply<true>(x, y, z, dx, dy, dz, jn, P, mu_sun, srec, smu, grec, gx, gy, gz);
    else pc_hess_apply<false>(x, y, z, dx, dy, dz, jn, P, mu_sun, srec, smu, grec, gx, gy, gz);
}

// Gravity gradient da/dr of the force model at the lane's points, in FP32, as the six
// entries (xx, yy, zz, xy, xz, yz) of the symmetric 3x3 matrix: every point mass (the Sun
// at the origin, the perturbers at their record positions) adds mu (3 d d^T / |d|^5 -
// I / |d|^3), d the offset of the point from the mass; the indirect term does not depend
// on the position.  Used as the linear map of the increment sweeps, whose limit moves by
// the error of G times the distance of the anchor from the solution: d is formed in FP64
// and then rounded (near a close approach, rounding the positions first would leave an
// error of 1e-5 in G and of about 1e-12 in the result), the rest is FP32.
static __device__ __forceinline__ void pc_grad_lds32(const double (&x)[4], const double (&y)[4], const double (&z)[4],
                                                     const int (&jn)[2], int P, double mu_sun, const double* srec,
                                                     const double* smu, float (&G)[6][4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int e = 0; e < 6; ++e) G[e][p] = 0.0f;
    }
    auto add = [&](int p, float dx, float dy, float dz, float mu) __attribute__((always_inline)) {
        const float q = __builtin_amdgcn_rsqf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        const float q2 = q * q;
        const float m3 = mu * q * q2;          // mu / |d|^3
        const float m5 = 3.0f * m3 * q2;       // 3 mu / |d|^5
        const float tx = m5 * dx, ty = m5 * dy, tz = m5 * dz;
        G[0][p] += fmaf(tx, dx, -m3);
        G[1][p] += fmaf(ty, dy, -m3);
        G[2][p] += fmaf(tz, dz, -m3);
        G[3][p] = fmaf(tx, dy, G[3][p]);
        G[4][p] = fmaf(tx, dz, G[4][p]);
        G[5][p] = fmaf(ty, dz, G[5][p]);
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) add(p, (float)x[p], (float)y[p], (float)z[p], (float)mu_sun);
    for (int b = 0; b < P; ++b) {
        const float mu = (float)smu[4 * b];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double* q = srec + jn[p >> 1] * 3 * (P + 1) + 3 * b;
            add(p, (float)(x[p] - q[0]), (float)(y[p] - q[1]), (float)(z[p] - q[2]), mu);
        }
    }
}

// Records of the relativistic model per node: for every major body b = 0..P (0 = the
// central body, at rest at the origin) three double4, (r_b, U_b - 2 v_b^2), (4 v_b, mu_b),
// (7/2 a_b, 0), with U_b the potential of the other major bodies at b (the two terms of the
// bracket below that depend on body b alone, summed once per node; the factors are those the
// sums below need), then the indirect term (ax, ay, az, 0).  A
// segment's records are stored slot-major, [slot][node], so that the lanes of a wave,
// which hold consecutive nodes, read consecutive double4.
constexpr int pc_eih_rec(int P) { return 3 * (P + 1) + 1; }


// A segment's records read from a base address and a slot stride that are one value per
// wave (scalar registers): each load adds only the 32-bit byte offset of the lane's node,
// a global load with a scalar base and no per-lane address arithmetic.  Every caller's
// records are those of one segment of one group, the same for all lanes of the wave.
struct PcEihRecs {
    gconst_cp base;   // slot 0, node 0
    uint32_t slot;    // bytes per slot (ns double4)
};
static __device__ __forceinline__ PcEihRecs pc_eih_recs(const double4* e, int ns)
{
    PcEihRecs E;
    E.base = pc_wave_base(e);
    E.slot = (uint32_t)__builtin_amdgcn_readfirstlane(ns) * 32u;
    return E;
}
static __device__ __forceinline__ double4 pc_eih_load(const PcEihRecs& E, int k, uint32_t vo)
{
    return pc_load_d4(E.base + (size_t)k * E.slot + vo);
}

// Einstein-Infeld-Hoffmann acceleration of R massless points (x, y, z, vx, vy, vz) at one
// node (PPN beta = gamma = 1, Sec. 5.4.1): with d = r - r_b, rho = |d| and the potential
// Phi = sum_b mu_b / rho_b at the point,
//   a = sum_b -mu_b d / rho^3 [1 - (4 Phi + U_b - v^2 - 2 v_b^2 + 4 v.v_b
//                                   + 3/2 (d.v_b / rho)^2 + 1/2 d.a_b) / c^2]
//     + sum_b mu_b / (c^2 rho^3) [d.(4 v - 3 v_b)] (v - v_b) + 7/2 sum_b mu_b a_b / (c^2 rho)
// minus the Newtonian indirect term.  What does not depend on the body is taken out of the
// sums: with N = sum m3 d (m3 = mu_b / rho^3), s the bracket without 4 Phi - v^2 and
// k = m3 d.(4 v - 3 v_b) / 4,
//   a = -N + [ (4 Phi - v^2) N + 4 v sum k + sum (m3 s d - 4 k v_b + 7/2 mu_b a_b / rho) ] / c^2,
// one pass over the bodies and 48 FP64 instructions per body and point (22 for the central
// body, whose v_b and a_b are zero); the terms one by one took 65.  This force is about half of a
// relativistic sweep at 200 nodes: 13509 ICs 7.29 -> 6.17 ms.
// e: the segment's records, slot k of node j at e[k ns + j].
template <int R>
static __device__ __forceinline__ void pc_force_eih(const double (&x)[R], const double (&y)[R],
                                                    const double (&z)[R], const double (&vx)[R],
                                                    const double (&vy)[R], const double (&vz)[R],
                                                    const double4* __restrict__ e, int j, int ns, int P, double inv_c2,
                                                    double (&ax)[R], double (&ay)[R], double (&az)[R])
{
    const PcEihRecs E = pc_eih_recs(e, ns);
    const uint32_t vo = (uint32_t)j * 32u;
    auto rec = [&](int k) -> double4 { return pc_eih_load(E, k, vo); };
    double phi[R], nx[R], ny[R], nz[R], bx[R], by[R], bz[R], K[R];
    const double4 sun = rec(0);
    {
        const double mu = rec(1).w;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double i1 = pc_rsqrt_full(pc_norm2(x[r], y[r], z[r]));
            phi[r] = mu * i1;
            const double m3 = phi[r] * (i1 * i1), k1 = m3 * sun.w;
            nx[r] = m3 * x[r];
            ny[r] = m3 * y[r];
            nz[r] = m3 * z[r];
            bx[r] = k1 * x[r];
            by[r] = k1 * y[r];
            bz[r] = k1 * z[r];
            K[r] = m3 * fma(z[r], vz[r], fma(y[r], vy[r], x[r] * vx[r]));
        }
    }
    for (int b = 1; b <= P; ++b) {
        const double4 q = rec(3 * b), w = rec(3 * b + 1), g = rec(3 * b + 2);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double dx = x[r] - q.x, dy = y[r] - q.y, dz = z[r] - q.z;
            const double i1 = pc_rsqrt_full(pc_norm2(dx, dy, dz));
            const double i2 = i1 * i1;
            const double m1 = w.w * i1;
            const double m3 = m1 * i2;               // mu / rho^3
            phi[r] += m1;
            nx[r] = fma(m3, dx, nx[r]);
            ny[r] = fma(m3, dy, ny[r]);
            nz[r] = fma(m3, dz, nz[r]);
            const double dw = fma(dz, w.z, fma(dy, w.y, dx * w.x));   // 4 d.v_b
            const double dg = fma(dz, g.z, fma(dy, g.y, dx * g.x));   // 7/2 d.a_b
            const double dv = fma(dz, vz[r], fma(dy, vy[r], dx * vx[r]));
            const double c = 0.09375 * dw;                            // 3/32
            double s = fma(vz[r], w.z, fma(vy[r], w.y, fma(vx[r], w.x, q.w)));
            s = fma(c * i2, dw, s);
            s = fma(1.0 / 7.0, dg, s);
            const double k1 = m3 * s, k2 = m3 * fma(-2.0, c, dv);
            K[r] += k2;
            bx[r] = fma(m1, g.x, fma(-k2, w.x, fma(k1, dx, bx[r])));
            by[r] = fma(m1, g.y, fma(-k2, w.y, fma(k1, dy, by[r])));
            bz[r] = fma(m1, g.z, fma(-k2, w.z, fma(k1, dz, bz[r])));
        }
    }
    const double4 ind = rec(3 * (P + 1));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double f = fma(4.0, phi[r], -pc_norm2(vx[r], vy[r], vz[r])), k4 = 4.0 * K[r];
        ax[r] = fma(inv_c2, fma(k4, vx[r], fma(f, nx[r], bx[r])), -nx[r]) - ind.x;
        ay[r] = fma(inv_c2, fma(k4, vy[r], fma(f, ny[r], by[r])), -ny[r]) - ind.y;
        az[r] = fma(inv_c2, fma(k4, vz[r], fma(f, nz[r], bz[r])), -nz[r]) - ind.z;
    }
}

// Jacobian of that acceleration at one point, as the adjoint applies it: gr_i = sum_j R[i][j] u_j
// for (da/dr)^T u and gv_i = sum_j V[i][j] u_j for (da/dv)^T u.  Per body, with m3 = mu/rho^3,
// B = 3 mu/rho^5, s the bracket without 4 Phi - v^2, W = 4 v_b, G = 7/2 a_b, c = d.W/rho^2,
// q = d.v - (3/16) d.W and e = 1/c^2:
//   H = sum B d d^T - M,   N = sum m3 d,   M = sum m3,   K = sum m3 q,   S = sum m3 s,
//   R = H + e [ sum (d a^T + W b^T + G g^T) + S + v (4 M v - sum m3 W)^T - (4 Phi - v^2) H - 4 N N^T ],
//   a = -(s B + (3/16) m3 c^2) d - B q (4 v - W) - m3 G,   b = (3/16) m3 (c d - (4 v - W)),   g = m3 d / 7,
//   V = e [ 4 N v^T - 2 v N^T + 4 K + (cross product with Q from the right) ],   Q = sum m3 W x d.
// The adjoint's points stay fixed over a segment's sweeps, so R and V are formed once (about 105
// FP64 instructions per body) and a sweep takes 18 multiply-adds per point instead of a pass
// over the bodies (84 per body): gradients through 1237 x 200 nodes 5.77 -> 4.08 ms.  About a
// third of the 72 values per lane live in scratch; a sweep reads them once.  At e = 0, R is the point-mass Jacobian; the indirect term does
// not depend on the state.  Records as pc_force_eih.
static __device__ __forceinline__ void pc_eih_jacobian(double x, double y, double z, double vx, double vy, double vz,
                                                       const PcEihRecs& E, int j, int P, double inv_c2,
                                                       double (&R)[9], double (&V)[9])
{
    const uint32_t vo = (uint32_t)j * 32u;
    auto rec = [&](int k) -> double4 { return pc_eih_load(E, k, vo); };
    const double v[3] = {vx, vy, vz};
    double phi = 0.0, K = 0.0, M = 0.0, S = 0.0, n[3] = {}, Q[3] = {}, mw[3] = {}, H[6] = {}, A[9] = {};
    for (int b = 0; b <= P; ++b) {
        const double4 q4 = rec(3 * b), w4 = rec(3 * b + 1), g4 = rec(3 * b + 2);
        const double d[3] = {x - q4.x, y - q4.y, z - q4.z}, w[3] = {w4.x, w4.y, w4.z}, g[3] = {g4.x, g4.y, g4.z};
        const double i1 = pc_rsqrt_full(pc_norm2(d[0], d[1], d[2]));
        const double i2 = i1 * i1, m1 = w4.w * i1, m3 = m1 * i2;
        const double dw = fma(d[2], w[2], fma(d[1], w[1], d[0] * w[0]));
        const double dg = fma(d[2], g[2], fma(d[1], g[1], d[0] * g[0]));
        const double dv = fma(d[2], vz, fma(d[1], vy, d[0] * vx));
        const double c = dw * i2;
        double s = fma(vz, w[2], fma(vy, w[1], fma(vx, w[0], q4.w)));
        s = fma(0.09375 * c, dw, s);
        s = fma(1.0 / 7.0, dg, s);
        const double qd = fma(-0.1875, dw, dv), B = 3.0 * (m3 * i2);
        phi += m1;
        M += m3;
        K = fma(m3, qd, K);
        S = fma(s, m3, S);
        const double a1 = -fma(s, B, 0.1875 * (m3 * (c * c))), a2 = -(B * qd), b1 = 0.1875 * m3, g1 = (1.0 / 7.0) * m3;
        double al[3], be[3], ga[3], md[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double t = fma(4.0, v[k], -w[k]);
            md[k] = m3 * d[k];
            n[k] += md[k];
            mw[k] = fma(m3, w[k], mw[k]);
            al[k] = fma(a1, d[k], fma(a2, t, -(m3 * g[k])));
            be[k] = b1 * fma(c, d[k], -t);
            ga[k] = g1 * d[k];
        }
        Q[0] += fma(w[1], md[2], -(w[2] * md[1]));
        Q[1] += fma(w[2], md[0], -(w[0] * md[2]));
        Q[2] += fma(w[0], md[1], -(w[1] * md[0]));
        const double bx = B * d[0], by = B * d[1];
        H[0] = fma(bx, d[0], H[0]);
        H[1] = fma(by, d[1], H[1]);
        H[2] = fma(B * d[2], d[2], H[2]);
        H[3] = fma(bx, d[1], H[3]);
        H[4] = fma(bx, d[2], H[4]);
        H[5] = fma(by, d[2], H[5]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                A[3 * i + k] = fma(g[i], ga[k], fma(w[i], be[k], fma(d[i], al[k], A[3 * i + k])));
        }
    }
    const double f = fma(4.0, phi, -pc_norm2(vx, vy, vz));
    const double h[9] = {H[0] - M, H[3], H[4], H[3], H[1] - M, H[5], H[4], H[5], H[2] - M};
    const double X[9] = {0.0, Q[2], -Q[1], -Q[2], 0.0, Q[0], Q[1], -Q[0], 0.0};   // X u = u x Q
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int e = 3 * i + k;
            const double r = fma(v[i], fma(4.0 * M, v[k], -mw[k]), fma(-f, h[e], fma(-4.0 * n[i], n[k], A[e])));
            R[e] = fma(inv_c2, i == k ? r + S : r, h[e]);
            const double t = fma(4.0 * n[i], v[k], fma(-2.0 * v[i], n[k], X[e]));
            V[e] = inv_c2 * (i == k ? fma(4.0, K, t) : t);
        }
    }
}

// Software-pipelined k loop of a 16x16x4 product over nq steps (a multiple of 4, at most
// NQ, at least 8 when NQ is; NQ fixes the layout of the operands).  The A operand of step q
// (a K_N fragment, read from L2) is loaded DK steps ahead into a ring of DK registers, the
// B operands (LDS) one step ahead into two buffers, and the loop body is unrolled DK
// times, so both rings rotate by register renaming.  A register move out of a ring would
// make the wave wait for the load it copies right after issuing it.
// loadB(q, q % 4, buffer) gets the phase as a compile-time constant after unrolling;
// loadA0(u) supplies the first DK A operands (registers kept across calls, or loads).
// mma may take the phase as well.
// SG_DS / SG_MFMA / SG_VMEM > 0 pin the order of one step in the steady-state loop for
// the scheduler: the B reads of the next step, this step's MFMAs, then the A read DK
// steps ahead (left to itself, the scheduler sinks the reads below the MFMAs that free
// their registers, and the wave then waits on each read right after issuing it).
template <int NQ, class AT, class BT, int SG_DS = 0, int SG_MFMA = 0, int SG_VMEM = 0, class LA0,
          class LA, class LB, class MM>
static __device__ __forceinline__ void pc_kloop(int nq, LA0 loadA0, LA loadA, LB loadB, MM mma)
{
    constexpr int DK = 4;
    static_assert(NQ % DK == 0, "k steps must be a multiple of the A ring depth");
    AT ka[DK];
    BT bb[2];
#pragma unroll
    for (int u = 0; u < DK; ++u) ka[u] = loadA0(u);
    loadB(0, 0, bb[0]);
    auto steps = [&](int q0) {
#pragma unroll
        for (int u = 0; u < DK; ++u) {
            loadB(q0 + u + 1, (u + 1) & 3, bb[(u + 1) & 1]);
            if constexpr (std::is_invocable_v<MM, AT, BT, int>) mma(ka[u], bb[u & 1], u);
            else mma(ka[u], bb[u & 1]);
            ka[u] = loadA(q0 + u + DK);
            if constexpr (SG_MFMA > 0) {
                __builtin_amdgcn_sched_group_barrier(0x100, SG_DS, 0);     // DS reads
                __builtin_amdgcn_sched_group_barrier(0x008, SG_MFMA, 0);   // MFMA
                __builtin_amdgcn_sched_group_barrier(0x020, SG_VMEM, 0);   // VMEM reads
            }
        }
    };
    // the first DK steps outside the loop: their products start from the caller's
    // accumulators directly (a zero start becomes the MFMA's inline constant instead of
    // register moves on every sweep)
    if constexpr (NQ > DK) steps(0);
    auto rest = [&](int n) __attribute__((always_inline)) {
#pragma unroll 1
        for (int q0 = DK; q0 < n - DK; q0 += DK) steps(q0);
#pragma unroll
        for (int u = 0; u < DK; ++u) {   // the last DK steps load nothing past the end
            if (u + 1 < DK) loadB(n - DK + u + 1, (u + 1) & 3, bb[(u + 1) & 1]);
            if constexpr (std::is_invocable_v<MM, AT, BT, int>) mma(ka[u], bb[u & 1], u);
            else mma(ka[u], bb[u & 1]);
        }
    };
    // a job whose nodes fill every k step keeps the compile-time bound (constant B
    // offsets in the last steps); a shorter one runs to its own bound, one value per wave
    // (a scalar, which keeps the loop and the B addresses off the vector registers)
    if constexpr (NQ > 2 * DK) {
        if (nq < NQ) {
            rest(__builtin_amdgcn_readfirstlane(nq));
            return;
        }
    }
    rest(NQ);
}
// ---------------------------------------------------------------------------
// Products
// ---------------------------------------------------------------------------
// Integration from -1 of a function sampled at the mirrored nodes of a pair (l: node i, r: node
// N-1-i): with s = F_l + F_r and d = F_l - F_r the even and the odd part of F,
//   y_l = y0 + w2 (U s + O d),   y_r = y0 + w2 (W + O d - U s),
// where U and O hold (K[i][p] +- K[i][N-1-p]) / 2 and W = sum_p w_p s_p, the integral over the
// whole segment (w: U's row of the last node; the middle node of an odd count is its own
// mirror: F_l = F_r, its column of U and w is halved and its column of O zero).  Two products of
// half the size in each direction: half the MFMAs of y0 + w2 K_N F, which is what bounds a
// sweep (v_mfma_f64_16x16x4 takes 64 cycles of a SIMD, an FP64 VALU instruction between 4 and
// 5, and nothing else issues beside the MFMA).  Whole products before and this after: 4096
// Venus ICs (128 nodes, 8 segments) 2.07 -> 1.51 ms, the uneven 65536-IC batch 157.8 -> 107.1
// ms, 13509 relativistic ICs of 200 nodes 11.7 -> 7.3 ms, gradients of 16384 ICs 17.9 -> 13.4 ms.
// W comes from the same operands: each lane adds w_p s_p over its k rows (one VALU multiply-add
// per block and k step), and one MFMA against ones adds the four k rows and leaves the sum in
// the result layout.  Taking W from the strip that holds the last node instead would need a
// barrier between the product and the epilogue.

typedef float pc_f2v __attribute__((ext_vector_type(2)));

// A strip's fragments of one operator: the strip's address is one value per wave (scalar
// registers) and a load adds only the lane's byte offset.  With one 64-bit address per k step
// in vector registers those addresses were spilled, and every reload from scratch waited for
// the fragments still in flight.
template <class V>
struct PcFrag {
    gconst_cp base;
    uint32_t vo;
    __device__ __forceinline__ V operator[](int q) const
    {
        gconst_cp p = base + (size_t)q * (64 * sizeof(V));
        asm volatile("" : "+s"(p));   // the scalar sum stays one: base + vo is not formed per lane
        return *(const __attribute__((address_space(1))) V*)(p + vo);
    }
};
typedef PcFrag<pc_d2v> PcFragD;
typedef PcFrag<pc_f2v> PcFragF;
template <int PAIRS, int NP, class F>
static __device__ __forceinline__ F pc_frag(const void* op, const PcLane& L)
{
    constexpr uint32_t V = sizeof(F{}[0]) * 64;
    return F{pc_wave_base(static_cast<const char*>(op) + (size_t)L.strip * PcShape<PAIRS, NP>::NQ * V),
             (uint32_t)L.lane * (V / 64)};
}

// The first four FP64 operator fragments of the lane's strip, loaded before the barrier that
// precedes the product, which then starts without waiting on L2.
static __device__ __forceinline__ void pc_kpre_load(const PcFragD& kp, pc_d2v (&kpre)[4])
{
#pragma unroll
    for (int u = 0; u < 4; ++u) kpre[u] = kp[u];
}

// Stopping-rule thresholds in fma form, fixed per segment: a squared change d2 passes
// against the squared norm y2 when d2 < a y2 + b, with (a, b) = (tol^2, 0) for the relative
// rule and (0, tol^2) for the absolute one (the same comparisons as d2 < tol^2 y2 and
// d2 < tol^2 for finite norms, with no branch on the mode).  (sa, sb): the same for the
// precision switch.
struct PcTol {
    double ta, tb, sa, sb;
};
static __device__ __forceinline__ PcTol pc_tol(int tol_mode, double t2, double sw2)
{
    return tol_mode == 0 ? PcTol{t2, 0.0, sw2, 0.0} : PcTol{0.0, t2, 0.0, sw2};
}

// Stopping-rule flags (Sec. 2.2) of the lane's ICs, new iterate y against the previous one yc,
// OR-ed over the strip's nodes: bits 4e..4e+2 belong to the lane's e-th IC (bit 0 some node not
// converged, bit 1 non-finite, bit 2 some node changed by more than the switch, SW only).
template <int PAIRS, int NP, bool SW>
static __device__ __forceinline__ int pc_flags(const double (&yc)[6][4], const f64x4 (&y)[6], const PcTol& tl,
                                               const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    int fr = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            double pd = 0.0, py = 0.0, vd = 0.0, vy = 0.0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double p = y[3 * h + b][r], v = y[3 * h + b][2 + r];
                const double dp = p - yc[3 * h + b][r], dv = v - yc[3 * h + b][2 + r];
                pd = b == 0 ? dp * dp : fma(dp, dp, pd);
                py = b == 0 ? p * p : fma(p, p, py);
                vd = b == 0 ? dv * dv : fma(dv, dv, vd);
                vy = b == 0 ? v * v : fma(v, v, vy);
            }
            const bool ok = pd < fma(tl.ta, py, tl.tb) && vd < fma(tl.ta, vy, tl.tb);
            const bool lo = !SW || (pd < fma(tl.sa, py, tl.sb) && vd < fma(tl.sa, vy, tl.sb));
            // the previous iterate is finite, so a non-finite change shows in the new norms
            const bool nf = !isfinite(py + vy);
            fr |= ((ok ? 0 : 1) | (nf ? 2 : 0) | (lo ? 0 : 4)) << (4 * (Sh::PAR ? r : 2 * h + r));
        }
    }
    if (!L.ok) fr = 0;
    return pc_row_or16(fr);   // the 16 rows of the strip: the lanes of one row group
}

// The flags of the wave's columns into sFlag[wave][column].
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_put_flags(int* sFlag, int fr, const PcLane& L)
{
    if (L.c < PcShape<PAIRS, NP>::E) sFlag[L.wave * 16 + pc_col<PAIRS, NP>(L, L.c)] = (fr >> (4 * L.c)) & 7;
}

// OR of the per-wave flags of IC m of the job.
template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_gather_flags(const int* sFlag, int m)
{
    using Sh = PcShape<PAIRS, NP>;
    const int* f0 = sFlag + (m / Sh::COLS) * Sh::STRIPS * 16 + m % Sh::COLS;
    int f = 0;
#pragma unroll
    for (int s = 0; s < Sh::STRIPS; ++s) f |= f0[s * 16];
    return f;
}

// acc <- base + w2 (the product), acc holding the blocks of U s (h = 0) and O d (h = 1), wd
// those of W; base: y0 (sY0), or the previous iterate (INCR, an increment sweep).
template <int PAIRS, int NP, bool INCR>
static __device__ __forceinline__ void pc_combine(const double* sY0, const double (&yc)[6][4], f64x4 (&acc)[6],
                                                  const f64x4 (&wd)[3], double w2, const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int T = Sh::T;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = b + 3 * (r >> 1);
            double bl, br;
            if constexpr (INCR) {
                bl = yc[b][r];
                br = yc[3 + b][r];
            } else {
                bl = sY0[c * T + pc_ic<PAIRS, NP>(L, 0, r & 1)];
                br = Sh::PAR ? bl : sY0[c * T + pc_ic<PAIRS, NP>(L, 1, r & 1)];
            }
            const double u = acc[b][r], o = acc[3 + b][r];
            if constexpr (Sh::PAR) {
                acc[b][r] = fma(w2, u, fma(w2, o, bl));
                acc[3 + b][r] = fma(-w2, u, fma(w2, o, fma(w2, wd[b][r], br)));
            } else {
                acc[b][r] = fma(w2, u, bl);
                acc[3 + b][r] = fma(w2, o, br);
            }
        }
    }
}

// One k step's operands from LDS: F's even and odd parts (or the two eights' values) of the
// three blocks, and the row's weight.
struct PcB {
    pc_d2v f[3];
    double w;
};
struct PcBf {
    pc_f2v f[3];
    double w;
};

// Lane's base of the k rows 4q + u (u = q % 4): the place of its A-operand row i in F, in
// pairs of values; a k step adds 4 rows, a block 16.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_kbase(const PcLane& L, int i, int (&bp)[4])
{
#pragma unroll
    for (int u = 0; u < 4; ++u)
        bp[u] = L.g * (PcShape<PAIRS, NP>::ROW / 2) + L.grp * 48 + (i ^ ((4 * u + L.g) & 15));
}

// acc <- U s | O d (or K F of the two eights), wd <- W: the FP64 product of the lane's six
// blocks, F in sF, the strip's fragments kp (kpre: its first four).
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_mm(const double* sF, const double* sWt, const PcFragD& kp,
                                             const pc_d2v (&kpre)[4], f64x4 (&acc)[6], f64x4 (&wd)[3], const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int STEP = 4 * Sh::ROW / 2;
    const pc_d2v* f = reinterpret_cast<const pc_d2v*>(sF);
    int bp[4];
    pc_kbase<PAIRS, NP>(L, L.c, bp);
    double ws[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 6; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
    pc_kloop<Sh::NQ, pc_d2v, PcB, Sh::PAR ? 4 : 3, 6, 1>(
        L.nq, [&](int u) { return kpre[u]; }, [&](int q) { return kp[q]; },
        [&](int q, int u, PcB& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) B.f[b] = f[bp[u] + q * STEP + 16 * b];
            if constexpr (Sh::PAR) B.w = sWt[4 * q + L.g];
        },
        [&](const pc_d2v& k, const PcB& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[b] = mfma16(B.f[b].x, k.x, acc[b]);
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[3 + b] = mfma16(B.f[b].y, k.y, acc[3 + b]);
            if constexpr (Sh::PAR) {
#pragma unroll
                for (int b = 0; b < 3; ++b) ws[b] = fma(B.w, B.f[b].x, ws[b]);
            }
        });
    if constexpr (Sh::PAR) {
#pragma unroll
        for (int b = 0; b < 3; ++b) wd[b] = mfma16(ws[b], 1.0, f64x4{0.0, 0.0, 0.0, 0.0});
    }
}

// The same on the FP32 matrix cores, from FP32 values (increment sweeps: the change of F) or
// from FP64 ones rounded here (FP32 Picard sweeps).  The f32 result holds A row 4(l/16) + r in
// element r, the f64 one row l/16 + 4r: reading IC row i from row i/4 + 4 (i%4) puts the same
// IC in the same lane and element.
// Rounding: a row of the operator is now U s + O d, so the early nodes' small integrals are
// differences of sums as large as the late nodes', and an error of W shifts every node of the second
// half alike.  W is summed in FP64 (its lanes put back in the f64 product's order), and U s and O d
// go into two accumulators each (odd and even k steps) that are added in FP64.  Venus orbits, 8
// segments, error of the schedule at 64, 128 (262144 of them) and 200 nodes (32768), median and 99th
// percentile in 1e-13: whole operator 6.1 6.9, 6.1 7.0, 6.1 7.1; halves all in FP32 6.1 8.1, 6.2
// 8.2, 5.9 8.1; this 6.2 7.1, 6.2 7.0, 6.2 6.9.  It takes 25.7, 70.4 and 25.3 ms, all in FP32 25.6,
// 67.3 and 24.3, the whole operator 31.1, 96.8 and 42.1.
template <int PAIRS, int NP, class V>
static __device__ __forceinline__ void pc_mm32(const V* sF, const double* sWt, const PcFragF& kp, f64x4 (&acc)[6],
                                               f64x4 (&wd)[3], const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int STEP = 4 * Sh::ROW / 2;
    typedef V v2 __attribute__((ext_vector_type(2)));
    const v2* f = reinterpret_cast<const v2*>(sF);
    int bp[4];
    pc_kbase<PAIRS, NP>(L, (L.c >> 2) + 4 * (L.c & 3), bp);
    double ws[3] = {0.0, 0.0, 0.0};
    constexpr int NA = Sh::PAR ? 2 : 1;   // at 16 padded nodes the operator is whole
    f32x4 a[NA][6];
#pragma unroll
    for (int b = 0; b < 6; ++b) a[0][b] = a[NA - 1][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    pc_kloop<Sh::NQ, pc_f2v, PcBf, Sh::PAR ? 4 : 3, 6, 1>(
        L.nq, [&](int q) { return kp[q]; }, [&](int q) { return kp[q]; },
        [&](int q, int u, PcBf& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const v2 t = f[bp[u] + q * STEP + 16 * b];
                B.f[b] = pc_f2v{(float)t.x, (float)t.y};
            }
            if constexpr (Sh::PAR) B.w = sWt[4 * q + L.g];
        },
        [&](const pc_f2v& k, const PcBf& B, int u) {
#pragma unroll
            for (int b = 0; b < 3; ++b) a[u % NA][b] = mfma16f(B.f[b].x, k.x, a[u % NA][b]);
#pragma unroll
            for (int b = 0; b < 3; ++b) a[u % NA][3 + b] = mfma16f(B.f[b].y, k.y, a[u % NA][3 + b]);
            if constexpr (Sh::PAR) {
#pragma unroll
                for (int b = 0; b < 3; ++b) ws[b] = fma(B.w, (double)B.f[b].x, ws[b]);
            }
        });
#pragma unroll
    for (int b = 0; b < 6; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[b][r] = Sh::PAR ? (double)a[0][b][r] + (double)a[NA - 1][b][r] : (double)a[0][b][r];
    }
    if constexpr (Sh::PAR) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
            wd[b] = mfma16(__shfl(ws[b], 16 * L.g + (L.c >> 2) + 4 * (L.c & 3)), 1.0, f64x4{0.0, 0.0, 0.0, 0.0});
    }
}

// One sweep's product: acc receives y0 + w2 K_N F, FP64; returns the flags (pc_flags).
template <int PAIRS, int NP, bool SW>
static __device__ __forceinline__ int pc_product(const double* sF, const double* sY0, const double* sWt, const PcFragD& kp,
                                                 const pc_d2v (&kpre)[4], const double (&yc)[6][4], f64x4 (&acc)[6],
                                                 double w2, const PcTol& tl, const PcLane& L)
{
    f64x4 wd[3];
    pc_mm<PAIRS, NP>(sF, sWt, kp, kpre, acc, wd, L);
    pc_combine<PAIRS, NP, false>(sY0, yc, acc, wd, w2, L);
    return pc_flags<PAIRS, NP, SW>(yc, acc, tl, L);
}

// FP32 sweeps of the precision schedule, accumulated into FP64: a Picard sweep (from the FP64
// F) or an increment sweep, Y_new = Y + w2 K_N dF with dF, the change of F
// (pc_publish_chord), held in LDS as FP32 in F's layout.  An increment's FP32 rounding is
// relative to it, so it shrinks as the sweeps converge instead of leaving a floor at the FP32
// precision of Y.
template <int PAIRS, int NP, bool INCR>
static __device__ __forceinline__ int pc_product32(const double* sF, const double* sY0, const double* sWt,
                                                   const PcFragF& kp, const double (&yc)[6][4], f64x4 (&acc)[6], double w2,
                                                   const PcTol& tl, const PcLane& L)
{
    f64x4 wd[3];
    if constexpr (INCR) pc_mm32<PAIRS, NP>(reinterpret_cast<const float*>(sF), sWt, kp, acc, wd, L);
    else pc_mm32<PAIRS, NP>(sF, sWt, kp, acc, wd, L);
    pc_combine<PAIRS, NP, INCR>(sY0, yc, acc, wd, w2, L);
    return pc_flags<PAIRS, NP, true>(yc, acc, tl, L);
}

// Second-order sweep: velocity and position both from the accelerations,
// v = v0 + w2 K_N a and x = x0 + w2 v0 (tau + 1) + w2^2 K2_N a, with K2_N the double-integration
// operator (the degree N-2 fit integrated twice, zero value and slope at tau = -1).  With the
// same even and odd parts s and d of a, and U2, O2, w2 those of K2_N,
//   x_l = x0 + w2 v0 (1 + tau_l) + w2^2 (U2 s + O2 d),
//   x_r = x0 + w2 v0 (1 - tau_l) + w2^2 (U2 s - tau_l W + C - O2 d),   C = sum_p w2_p d_p.
// F's blocks hold (a_x | a_y), (a_z | 0) and (0 | a_z) in their low and high eights: a_z's
// position needs K2_N and its velocity K_N in one block, so it takes two MFMAs with half an
// operand zero, eight per k step against the first-order sweep's six.
struct PcQuad {
    pc_d2v k, q;   // K_N and K2_N fragments
};
struct PcB2 {
    pc_d2v f[3];
    double w, c;
};
struct PcSo {
    f64x4 k[2], q[2], z[2];   // per h: K_N (a_x | a_y), K2_N (a_x | a_y), (K2_N a_z | K_N a_z)
    f64x4 w[2], c[2];         // W and C of blocks 0 and 1
};

template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_mm2(const double* sF, const double* sWt, const PcFragD& kp1, const PcFragD& kp2,
                                              PcSo& A, const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int STEP = 4 * Sh::ROW / 2;
    const pc_d2v* f = reinterpret_cast<const pc_d2v*>(sF);
    int bp[4];
    pc_kbase<PAIRS, NP>(L, L.c, bp);
    double ws[2] = {0.0, 0.0}, cs[2] = {0.0, 0.0};
    pc_kloop<Sh::NQ, PcQuad, PcB2>(
        L.nq, [&](int q) { return PcQuad{kp1[q], kp2[q]}; },
        [&](int q) { return PcQuad{kp1[q], kp2[q]}; },
        [&](int q, int u, PcB2& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) B.f[b] = f[bp[u] + q * STEP + 16 * b];
            if constexpr (Sh::PAR) {
                B.w = sWt[4 * q + L.g];
                B.c = sWt[Sh::KR + 4 * q + L.g];
            }
        },
        [&](const PcQuad& k, const PcB2& B) {
            A.z[0] = mfma16(B.f[1].x, k.q.x, A.z[0]);
            A.z[1] = mfma16(B.f[1].y, k.q.y, A.z[1]);
            A.q[0] = mfma16(B.f[0].x, k.q.x, A.q[0]);
            A.q[1] = mfma16(B.f[0].y, k.q.y, A.q[1]);
            A.k[0] = mfma16(B.f[0].x, k.k.x, A.k[0]);
            A.k[1] = mfma16(B.f[0].y, k.k.y, A.k[1]);
            A.z[0] = mfma16(B.f[2].x, k.k.x, A.z[0]);
            A.z[1] = mfma16(B.f[2].y, k.k.y, A.z[1]);
            if constexpr (Sh::PAR) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    ws[b] = fma(B.w, B.f[b].x, ws[b]);
                    cs[b] = fma(B.c, B.f[b].y, cs[b]);
                }
            }
        });
    if constexpr (Sh::PAR) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            A.w[b] = mfma16(ws[b], 1.0, A.w[b]);
            A.c[b] = mfma16(cs[b], 1.0, A.c[b]);
        }
    }
}

// New iterate of a second-order sweep from its products (tp = tau + 1 of the lane's node 0).
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_combine2(const double* sY0, const PcSo& A, f64x4 (&y)[6], double w2, double tp,
                                                   const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int T = Sh::T;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            // comp b of IC r: (a_x | a_y) blocks hold comp 1 in their high eight
            const int k = b == 1 ? 2 + r : r;
            const double e = b < 2 ? A.q[0][k] : A.z[0][r], o2 = b < 2 ? A.q[1][k] : A.z[1][r];
            const double u = b < 2 ? A.k[0][k] : A.z[0][2 + r], o = b < 2 ? A.k[1][k] : A.z[1][2 + r];
            const int m0 = pc_ic<PAIRS, NP>(L, 0, r), m1 = pc_ic<PAIRS, NP>(L, 1, r);
            const double x0 = sY0[b * T + m0], v0 = sY0[(3 + b) * T + m0];
            if constexpr (Sh::PAR) {
                const double W = b < 2 ? A.w[0][k] : A.w[1][r], C = b < 2 ? A.c[0][k] : A.c[1][r];
                y[b][r] = fma(w2, fma(w2, e + o2, tp * v0), x0);
                y[3 + b][r] = fma(w2, fma(w2, fma(1.0 - tp, W, e + C) - o2, (2.0 - tp) * v0), x0);
                y[b][2 + r] = fma(w2, u, fma(w2, o, v0));
                y[3 + b][2 + r] = fma(-w2, u, fma(w2, o, fma(w2, W, v0)));
            } else {
                const double x1 = sY0[b * T + m1], v1 = sY0[(3 + b) * T + m1];
                y[b][r] = fma(w2, fma(w2, e, tp * v0), x0);
                y[3 + b][r] = fma(w2, fma(w2, o2, tp * v1), x1);
                y[b][2 + r] = fma(w2, u, v0);
                y[3 + b][2 + r] = fma(w2, o, v1);
            }
        }
    }
}

// Publish a change or value (two halves h) of the accelerations in the second-order layout.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_put2(double* sF, const double (&ax)[4], const double (&ay)[4],
                                               const double (&az)[4], const PcLane& L);

template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_product2(const double* sF, const double* sY0, const double* sWt,
                                                  const PcFragD& kp1, const PcFragD& kp2, const double (&yc)[6][4],
                                                  f64x4 (&acc)[6], double w2, double tp, const PcTol& tl,
                                                  const PcLane& L)
{
    PcSo A = {};
    pc_mm2<PAIRS, NP>(sF, sWt, kp1, kp2, A, L);
    pc_combine2<PAIRS, NP>(sY0, A, acc, w2, tp, L);
    return pc_flags<PAIRS, NP, false>(yc, acc, tl, L);
}

// Second-order sweep with integral error feedback.  The sweep's accelerations were taken at
// the previous position iterate; the position it predicts changes that iterate by dx, and the
// linear change of the acceleration over dx, da = (da/dr) dx at the previous iterate, is
// integrated like the accelerations and added: v_new = v0 + w2 K_N (a + da),
// x_new = x0 + w2 v0 (tau + 1) + w2^2 K2_N (a + da).  da takes a's place in F once every wave
// has read it, and its product accumulates onto the first one.  At the fixed point dx vanishes,
// so the converged iterate is the second-order one.
template <int PAIRS, int NP>
static __device__ __forceinline__ int pc_product2_fb(double* sF, const double* sY0, const double* sWt, const PcFragD& kp1,
                                                     const PcFragD& kp2, const double (&yc)[6][4], f64x4 (&acc)[6],
                                                     double w2, double tp, const PcTol& tl, const PcLane& L, int P,
                                                     double mu_sun, bool rec_lds, const double* sRec,
                                                     const double* sMu, const double4* grec)
{
    PcSo A = {};
    pc_mm2<PAIRS, NP>(sF, sWt, kp1, kp2, A, L);
    pc_combine2<PAIRS, NP>(sY0, A, acc, w2, tp, L);
    double x[3][4], dx[3][4], gx[4], gy[4], gz[4];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            x[b][p] = yc[3 * (p >> 1) + b][p & 1];
            dx[b][p] = acc[3 * (p >> 1) + b][p & 1] - x[b][p];
        }
    }
    pc_grad_dot(x[0], x[1], x[2], dx[0], dx[1], dx[2], L.jn, P, mu_sun, rec_lds, sRec, sMu, grec, gx, gy, gz);
    __syncthreads();   // every wave is done reading the accelerations
    if (L.ok) pc_put2<PAIRS, NP>(sF, gx, gy, gz, L);
    __syncthreads();   // every node's da published
    pc_mm2<PAIRS, NP>(sF, sWt, kp1, kp2, A, L);
    pc_combine2<PAIRS, NP>(sY0, A, acc, w2, tp, L);
    return pc_flags<PAIRS, NP, false>(yc, acc, tl, L);
}

// w = K_N^T mu at the lane's nodes: with the published pairs (mu_l - mu_r, mu_l + mu_r) and
// the transposed operators, g_s = U^T (mu_l - mu_r) + w R, R = sum over the rows of mu_r, and
// g_d = O^T (mu_l + mu_r), w_l = g_s + g_d and w_r = g_s - g_d (at a middle node w_l is g_s:
// its columns are whole here, and its mu_r is zero).  wr: half the row weight w of the lane's
// own row; R's sum over the k rows is formed like pc_mm's W and enters by one MFMA per block.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_product_adj(const double* sF, const PcFragD& kpT, double wr, f64x4 (&acc)[6],
                                                      const PcLane& L)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int STEP = 4 * Sh::ROW / 2;
    const pc_d2v* f = reinterpret_cast<const pc_d2v*>(sF);
    int bp[4];
    pc_kbase<PAIRS, NP>(L, L.c, bp);
    double rs[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 6; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
    pc_kloop<Sh::NQ, pc_d2v, PcB, 3, 6, 1>(
        L.nq, [&](int q) { return kpT[q]; }, [&](int q) { return kpT[q]; },
        [&](int q, int u, PcB& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) B.f[b] = f[bp[u] + q * STEP + 16 * b];
        },
        [&](const pc_d2v& k, const PcB& B) {
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[b] = mfma16(B.f[b].x, k.x, acc[b]);
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[3 + b] = mfma16(B.f[b].y, k.y, acc[3 + b]);
            if constexpr (Sh::PAR) {
#pragma unroll
                for (int b = 0; b < 3; ++b) rs[b] += B.f[b].y - B.f[b].x;   // 2 mu_r
            }
        });
    if constexpr (Sh::PAR) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const f64x4 s = mfma16(rs[b], wr, acc[b]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double d = acc[3 + b][r];
                acc[b][r] = s[r] + d;
                acc[3 + b][r] = s[r] - d;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Publishing
// ---------------------------------------------------------------------------
// One component of the lane's points into F's block b, eight `half`: the even and odd parts of
// the pair (or the two eights' values).
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_put(double* sF, int b, int half, int r, double vl, double vr, const PcLane& L)
{
    const int i = 8 * half + L.g + 4 * r;
    pc_d2v* f = reinterpret_cast<pc_d2v*>(sF) + pc_unit<PAIRS, NP>(L.row, L.grp, b, i);
    *f = PcShape<PAIRS, NP>::PAR ? pc_d2v{vl + vr, vl - vr} : pc_d2v{vl, vr};
}

template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_put2(double* sF, const double (&ax)[4], const double (&ay)[4],
                                               const double (&az)[4], const PcLane& L)
{
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        pc_put<PAIRS, NP>(sF, 0, 0, r, ax[r], ax[2 + r], L);
        pc_put<PAIRS, NP>(sF, 0, 1, r, ay[r], ay[2 + r], L);
        pc_put<PAIRS, NP>(sF, 1, 0, r, az[r], az[2 + r], L);
        pc_put<PAIRS, NP>(sF, 2, 1, r, az[r], az[2 + r], L);
    }
}

// F = (v, a) of the lane's points into sF.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_put_f(double* sF, const double (&yc)[6][4], const double (&ax)[4],
                                                const double (&ay)[4], const double (&az)[4], const PcLane& L)
{
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
        for (int b = 0; b < 3; ++b) pc_put<PAIRS, NP>(sF, b, 0, r, yc[b][2 + r], yc[3 + b][2 + r], L);
        pc_put<PAIRS, NP>(sF, 0, 1, r, ax[r], ax[2 + r], L);
        pc_put<PAIRS, NP>(sF, 1, 1, r, ay[r], ay[2 + r], L);
        pc_put<PAIRS, NP>(sF, 2, 1, r, az[r], az[2 + r], L);
    }
}

// Position component b of the lane's points from the iterate.
static __device__ __forceinline__ void pc_points(const double (&yc)[6][4], int b, double (&x)[4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) x[p] = yc[3 * (p >> 1) + b][p & 1];
}

// Dynamics of the lane's (node, IC) pairs from its registers, published as the force matrix
// F = (v, a) of Sec. 2.2.  sRec/sMu: the segment's records in LDS (when rec_lds), grec: the
// same in global memory.  SO: second-order sweeps, the accelerations only, in their layout.
// HALF: the job has at most four ICs, so only the points of the lane's first IC are evaluated (the
// other's acceleration, which no IC reads, is zero): the force of a sweep, half of a small call's
// time, in half the instructions.  One orbit of 32 nodes and 4 segments 205 -> 176 us, of 128 nodes
// 413 -> 375, relativistic of 100 nodes 685 -> 579.
template <int PAIRS, int NP, bool FP32 = false, bool SO = false, bool HALF = false>
static __device__ __forceinline__ void pc_publish(double* sF, const double (&yc)[6][4], const PcLane& L, int P,
                                                  double mu_sun, bool rec_lds, const double* sRec, const double* sMu,
                                                  const double4* grec)
{
    double x[4], y[4], z[4], ax[4], ay[4], az[4];
    pc_points(yc, 0, x);
    pc_points(yc, 1, y);
    pc_points(yc, 2, z);
    if (HALF && rec_lds) {
        const double x1[2] = {x[0], x[2]}, y1[2] = {y[0], y[2]}, z1[2] = {z[0], z[2]};
        double a[3][2];
        pc_force_lds<1>(x1, y1, z1, L.jn, P, mu_sun, sRec, sMu, a[0], a[1], a[2]);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            ax[p] = p & 1 ? 0.0 : a[0][p >> 1];
            ay[p] = p & 1 ? 0.0 : a[1][p >> 1];
            az[p] = p & 1 ? 0.0 : a[2][p >> 1];
        }
    } else if (rec_lds && FP32) pc_force_lds32(x, y, z, L.jn, P, mu_sun, sRec, sMu, ax, ay, az);
    else if (rec_lds) pc_force_lds<2>(x, y, z, L.jn, P, mu_sun, sRec, sMu, ax, ay, az);
    else pc_force_glb(x, y, z, L.jn, P, mu_sun, grec, ax, ay, az);
    if (!L.ok) return;
    if constexpr (SO) pc_put2<PAIRS, NP>(sF, ax, ay, az, L);
    else pc_put_f<PAIRS, NP>(sF, yc, ax, ay, az, L);
}

// The same with the relativistic acceleration.  erec: the segment's records, pc_eih_rec(P)
// slots of N double4; one pass over the bodies per node of the lane.
template <int PAIRS, int NP, bool HALF = false>
static __device__ __forceinline__ void pc_publish_eih(double* sF, const double (&yc)[6][4], const PcLane& L, int N,
                                                      int P, const double4* erec, double inv_c2)
{
    double ax[4], ay[4], az[4];
    constexpr int R = HALF ? 1 : 2;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        double q[6][R], a0[R], a1[R], a2[R];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
#pragma unroll
            for (int r = 0; r < R; ++r) q[c][r] = yc[3 * h + c % 3][r + 2 * (c / 3)];
        }
        pc_force_eih<R>(q[0], q[1], q[2], q[3], q[4], q[5], erec, L.jn[h], N, P, inv_c2, a0, a1, a2);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            ax[2 * h + r] = r < R ? a0[r % R] : 0.0;
            ay[2 * h + r] = r < R ? a1[r % R] : 0.0;
            az[2 * h + r] = r < R ? a2[r % R] : 0.0;
        }
    }
    if (L.ok) pc_put_f<PAIRS, NP>(sF, yc, ax, ay, az, L);
}

// Publish for an increment sweep.  The increment of F = (v, a) from the last
// change dy of the iterate, to first order: dF = (dv, G dr), with G the gravity gradient
// at the anchor, the iterate after the last FP64 sweep (anchor: evaluated here at yc and
// kept in sG, [entry 6][point 4][thread] FP32; else read from sG).
// dF goes to sD rounded to FP32, in F's layout.  act[p]: the IC of the lane's point p iterates
// (others publish zero, so that no stale or non-finite value reaches the product; dy is zero
// for them).
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_publish_chord(float* sD, float* sG, const double (&yc)[6][4],
                                                        const float (&dy)[6][4], const int (&act)[4], bool anchor,
                                                        const PcLane& L, int P, double mu_sun, const double* sRec,
                                                        const double* sMu)
{
    using Sh = PcShape<PAIRS, NP>;
    pc_f2v* d = reinterpret_cast<pc_f2v*>(sD);
    float G[6][4];
    float* g = sG + L.wave * 64 + L.lane;
    if (anchor) {
        double x[4], y[4], z[4];
        pc_points(yc, 0, x);
        pc_points(yc, 1, y);
        pc_points(yc, 2, z);
        pc_grad_lds32(x, y, z, L.jn, P, mu_sun, sRec, sMu, G);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                G[e][p] = act[p] ? G[e][p] : 0.0f;
                g[(4 * e + p) * Sh::NT] = G[e][p];
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < 6; ++e) {
#pragma unroll
            for (int p = 0; p < 4; ++p) G[e][p] = g[(4 * e + p) * Sh::NT];
        }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float F[6][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = 2 * h + r;
            const float rx = dy[3 * h][r], ry = dy[3 * h + 1][r], rz = dy[3 * h + 2][r];
            F[0][h] = dy[3 * h][2 + r];
            F[1][h] = dy[3 * h + 1][2 + r];
            F[2][h] = dy[3 * h + 2][2 + r];
            F[3][h] = fmaf(G[0][p], rx, fmaf(G[3][p], ry, G[4][p] * rz));
            F[4][h] = fmaf(G[3][p], rx, fmaf(G[1][p], ry, G[5][p] * rz));
            F[5][h] = fmaf(G[4][p], rx, fmaf(G[5][p], ry, G[2][p] * rz));
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            // rows past the last one meet zero operator columns: zero, not stale bits
            const float l = L.ok ? F[c][0] : 0.0f, q = L.ok ? F[c][1] : 0.0f;
            d[pc_unit<PAIRS, NP>(L.row, L.grp, c % 3, 8 * (c / 3) + L.g + 4 * r)] =
                Sh::PAR ? pc_f2v{l + q, l - q} : pc_f2v{l, q};
        }
    }
}

// Initial guess of segment s at the lane's points: warm (Kepler) or cold start, Sec. 2.1, or the
// caller's node states; each staged in the lane's own part of the F area (one call site, no
// private array).  sY0, dead: initial states and status of the job's n ICs (the first is ic0).
template <int PAIRS, int NP, bool HALF = false>
static __device__ __forceinline__ void pc_initial_guess(const PcParams& p, const PcGroupDev& g, int n, int64_t ic0,
                                                        int s, double w2, const PcLane& L, const double* sY0,
                                                        const int* dead, double* sF, double (&yc)[6][4])
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int NT = Sh::NT, T = Sh::T;
    const int tid = threadIdx.x;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
        const int j = q < 2 ? L.jn[0] : L.jn[1];
        const int m = pc_ic<PAIRS, NP>(L, q >> 1, q & 1);
        double y0[6], y[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) y0[c] = sY0[c * T + m];
        bool have = false;
        if (!dead[m] && (!HALF || m < n)) {   // HALF: columns past the job's ICs keep y0, not iterated
            if (p.init == 2 && m < n) {   // the caller's node states
                const gconst_dp gp =
                    pc_gcd(p.guess) + (((size_t)(ic0 + m) * p.iters_stride + s) * p.nodes_stride + j) * 6;
                have = true;
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    y[c] = gp[c];
                    have = have && isfinite(y[c]);
                }
            } else if (p.init == 0) {
                have = pc_kepler(y0, w2 * (pc_gcd(g.tau)[j] + 1.0), y);
            }
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) sF[(q * 6 + c) * NT + tid] = have ? y[c] : y0[c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int c = 0; c < 6; ++c) yc[3 * (q >> 1) + c % 3][(q & 1) + 2 * (c / 3)] = sF[(q * 6 + c) * NT + tid];
    }
}

// The rows of F past the last one holding nodes are zero (they meet zero operator columns,
// which a stale NaN would survive), and so are the unused halves of the second-order blocks.
template <int PAIRS, int NP, bool SO>
static __device__ __forceinline__ void pc_clear_rows(double* sF, int N)
{
    using Sh = PcShape<PAIRS, NP>;
    const int M = Sh::PAR ? (N + 1) >> 1 : N;
    for (int i = M * Sh::ROW + (int)threadIdx.x; i < Sh::KR * Sh::ROW; i += Sh::NT) sF[i] = 0.0;
    if constexpr (SO) {
        for (int k = threadIdx.x; k < M * Sh::GN * 16; k += Sh::NT) {
            const int i = k & 15, q = k >> 4;
            const int u = pc_unit<PAIRS, NP>(q / Sh::GN, q % Sh::GN, i < 8 ? 2 : 1, i);
            reinterpret_cast<pc_d2v*>(sF)[u] = pc_d2v{0.0, 0.0};
        }
    }
}

#pragma clang fp contract(fast)
