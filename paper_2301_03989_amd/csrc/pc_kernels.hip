// pc_kernels.hip -- gfx950 kernels of the batched Picard-Chebyshev propagator.
//
// Method: arXiv 2301.03989, Sec. 2.2 (matrix form of the Picard-Chebyshev iteration),
// Sec. 3 (augmentation of many trajectories on common nodes), Sec. 5.4 (GPU program:
// dynamics at every node, the fit/integrate/evaluate products, error and its reduction).
//
// The fused kernel gives each workgroup one job (T ICs x NP nodes of one group) and runs
// the whole propagation of those ICs on chip: for every segment it builds the initial
// guess, then repeats {force at all nodes (FP64 VALU), y_new = y0 + w2 K_N F (FP64 MFMA
// 16x16x4), per-IC error and stopping decision} until each IC has converged, chains the
// last node into the next segment and finally writes the end states.  The iterate stays
// in registers and the force matrix in LDS, so HBM traffic is the initial states, the
// ephemeris records, the results and what the bodies spill; K_N fragments are re-read from L2.
#include "pc_device.h"

// ---------------------------------------------------------------------------
// Ephemeris records: one thread per (group, segment, node) and body
// ---------------------------------------------------------------------------
// What bounds it is the chain of one Kepler solve and, relativistic, of the body pairs' roots and
// divisions: a call has few records (128 to some thousands), all in flight at once.  So the W = 8
// or 16 lanes of a record take one body each (8 where the bodies fit: half the lanes would idle),
// and the sums over bodies go over shuffles, in body order.  128 records of 8 bodies take 4.6 us,
// 1024 relativistic ones 9.6; one thread per record with the bodies in turn took 12.2 and 46.6.
static_assert(PC_MAX_PERT_DEV <= 16, "a record's bodies fit 16 lanes");
template <int W>
__global__ __launch_bounds__(256) void pc_ephem_kernel(const PcEphemParams p)
{
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / W;
    if (i >= p.n_recs) return;                   // whole records leave: the shuffles stay within one
    const int P = p.n_pert, b = threadIdx.x % W;
    int lo = 0, hi = p.n_groups - 1;             // last group with rec_offset <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.groups[mid].rec_offset <= i) lo = mid; else hi = mid - 1;
    }
    const PcGroupDev& G = p.groups[lo];
    const int64_t local = i - G.rec_offset;
    const int s = (int)(local / G.N);
    const int j = (int)(local - (int64_t)s * G.N);
    const double Ts = G.t0 + G.h * (s + G.s0), Te = G.t0 + G.h * (s + G.s0 + 1);
    const double t = 0.5 * (Te - Ts) * G.tau[j] + 0.5 * (Te + Ts);   // eq. chnodes1
    double4* rec = reinterpret_cast<double4*>(p.recs) + i * (P + 1);
    const bool on = b < P;
    double r[3] = {1.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, mu = 0.0;   // lanes past the bodies: no mass
    if (on) {
        if (p.recs_eih) pc_body_state(p.bodies[b], t - p.epoch, r, v);
        else pc_body_position(p.bodies[b], t - p.epoch, r);
        mu = p.bodies[b].mu;
        rec[b] = make_double4(r[0], r[1], r[2], mu);
    }
    const double q2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double iq = rsqrt(q2);
    const double sq = mu * (iq * iq * iq);
    double ix = 0.0, iy = 0.0, iz = 0.0;
    for (int k = 0; k < P; ++k) {
        ix += __shfl(sq * r[0], k, W);
        iy += __shfl(sq * r[1], k, W);
        iz += __shfl(sq * r[2], k, W);
    }
    if (b == 0) rec[P] = make_double4(ix, iy, iz, 0.0);
    if (p.recs_eih) {
        // relativistic model: states, accelerations and potentials of the major bodies
        // (pc_eih_rec slots, slot-major within the segment); body 0, the central body,
        // rests at the origin
        const int N = G.N;
        double4* base = reinterpret_cast<double4*>(p.recs_eih) + (i - j) * pc_eih_rec(P) + j;
        auto er = [&](int slot) -> double4& { return base[(size_t)slot * N]; };
        const double q = sqrt(q2);
        const double m = mu / q;
        double u0 = 0.0;
        double u = p.mu_sun / q;   // potential of the central body and the other perturbers
        for (int k = 0; k < P; ++k) {
            u0 += __shfl(m, k, W);
            const double dx = r[0] - __shfl(r[0], k, W), dy = r[1] - __shfl(r[1], k, W), dz = r[2] - __shfl(r[2], k, W);
            const double mk = __shfl(mu, k, W);
            if (k != b) u += mk / sqrt(dx * dx + dy * dy + dz * dz);
        }
        const double iq3 = 1.0 / (q * q * q);   // Keplerian orbit about the central body
        const double v2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        if (on) {
            er(3 * (b + 1)) = make_double4(r[0], r[1], r[2], u - 2.0 * v2);
            er(3 * (b + 1) + 1) = make_double4(4.0 * v[0], 4.0 * v[1], 4.0 * v[2], mu);
            er(3 * (b + 1) + 2) = make_double4(-3.5 * r[0] * iq3, -3.5 * r[1] * iq3, -3.5 * r[2] * iq3, 0.0);
        }
        if (b == 0) {
            er(0) = make_double4(0.0, 0.0, 0.0, u0);
            er(1) = make_double4(0.0, 0.0, 0.0, p.mu_sun);
            er(2) = make_double4(0.0, 0.0, 0.0, 0.0);
            er(3 * (P + 1)) = make_double4(ix, iy, iz, 0.0);
        }
    }
}

int pc_launch_ephem(const PcEphemParams& p, void* stream)
{
    if (p.n_recs <= 0) return hipSuccess;
    const int bs = 256, w = p.n_pert <= 8 ? 8 : 16;
    const int64_t grid = (p.n_recs * w + bs - 1) / bs;
    if (w == 8) hipLaunchKernelGGL(pc_ephem_kernel<8>, dim3((unsigned)grid), dim3(bs), 0, (hipStream_t)stream, p);
    else hipLaunchKernelGGL(pc_ephem_kernel<16>, dim3((unsigned)grid), dim3(bs), 0, (hipStream_t)stream, p);
    return hipGetLastError();
}

// Copies of contiguous runs of 32-bit words, one workgroup per descriptor.
__global__ __launch_bounds__(64) void pc_copy_runs_kernel(const PcCopyDev* __restrict__ list)
{
    const PcCopyDev c = list[blockIdx.x];
    const uint32_t* src = static_cast<const uint32_t*>(c.src);
    uint32_t* dst = static_cast<uint32_t*>(c.dst);
    for (int64_t i = threadIdx.x; i < c.words; i += blockDim.x) dst[i] = src[i];
}

// Flyby screen (the outer-level isolation of flyby sub-groups, Sec. 3.2): one thread per
// (IC, sample point); the thread propagates its IC by two-body motion (mu = 1, the warm
// start's) to its sample point of every segment, t = w2 tau_k + w1 (eq. chnodes1 with
// `samples` CGL points), and keeps the smallest distance to any perturber in units of
// its Hill radius a_p (mu_p/3)^(1/3); the IC's minimum over its threads is taken with an
// atomic minimum on the bit patterns (positive doubles order as unsigned integers).  An
// orbit that is not elliptic gives 0.  ratio must hold +inf for the screened ICs.
__global__ __launch_bounds__(256) void pc_flyby_kernel(PcFlybyParams p)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n_threads) return;
    int lo = 0, hi = p.n_groups - 1;             // last group with thread_offset <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.groups[mid].thread_offset <= i) lo = mid; else hi = mid - 1;
    }
    const PcGroupDev& G = p.groups[lo];
    const int64_t local = i - G.thread_offset;
    const int64_t m = G.ic_offset + local / p.samples;
    const int k = (int)(local % p.samples);
    const double tau = -cos(M_PI * (double)k / (double)(p.samples - 1));
    double y0[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) y0[c] = p.ics[m * 6 + c];
    double best = INFINITY;
    for (int s = 0; s < G.S && best > 0.0; ++s) {
        const double Ts = G.t0 + G.h * s, Te = G.t0 + G.h * (s + 1);
        const double t = 0.5 * (Te - Ts) * tau + 0.5 * (Te + Ts);
        double y[6];
        if (!pc_kepler(y0, t - G.t0, y)) {
            best = 0.0;
            break;
        }
        for (int b = 0; b < p.n_pert; ++b) {
            const PcBodyDev& B = p.bodies[b];
            if (!(B.mu > 0.0)) continue;
            double r[3];
            pc_body_position(B, t - p.epoch, r);
            const double dx = y[0] - r[0], dy = y[1] - r[1], dz = y[2] - r[2];
            const double q = sqrt(dx * dx + dy * dy + dz * dz) / (B.a * cbrt(B.mu / 3.0));
            best = fmin(best, q);
        }
    }
    atomicMin(reinterpret_cast<unsigned long long*>(p.ratio + m), (unsigned long long)__double_as_longlong(best));
}

int pc_launch_flyby(const PcFlybyParams& p, void* stream)
{
    if (p.n_threads <= 0) return hipSuccess;
    const int bs = 256;
    const int64_t grid = (p.n_threads + bs - 1) / bs;
    hipLaunchKernelGGL(pc_flyby_kernel, dim3((unsigned)grid), dim3(bs), 0, (hipStream_t)stream, p);
    return hipGetLastError();
}

int pc_launch_copy_runs(const PcCopyDev* list, int64_t n, void* stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pc_copy_runs_kernel, dim3((unsigned)n), dim3(64), 0, (hipStream_t)stream, list);
    return hipGetLastError();
}

// One job: T = PAIRS/NP ICs of one group, all segments.
//
// Ownership: every wave owns six 16x16 blocks of the iterate (PcShape) for the whole job.  It
// keeps its blocks of the current iterate in registers (in the MFMA result layout), computes
// the dynamics for the (node, IC) pairs it owns straight from them, and publishes only the
// force matrix F = (v, a) to LDS, where the product y_new = y0 + w2 K_N F reads it.
// The workgroup's LDS arena (file scope, so that the non-inlined job bodies below address it as
// LDS), one per kernel and job shape: an arena that two kernels reach, beside another such one,
// has its address looked up in a table in memory by every use.
__shared__ PcSmem<2048> g_smem2048, g_smem2048_adj;
__shared__ PcSmem<1024> g_smem1024, g_smem1024_adj;
template <int PAIRS, bool ADJ = false>
static __device__ __forceinline__ PcSmem<PAIRS>& pc_smem()
{
    if constexpr (PAIRS == 2048) return ADJ ? g_smem2048_adj : g_smem2048;
    else return ADJ ? g_smem1024_adj : g_smem1024;
}

// Segment s's ephemeris records (perturber data per node, Sec. 5.4.1) into LDS: positions
// as [node][body][3] with the indirect term as body P, and per body mu, 3 mu / 2 and
// 15 mu / 8 (the premultiplied series coefficients of pc_mu_r3).
template <int PAIRS>
static __device__ __forceinline__ void pc_stage_records(const double4* grec, int N, int P, PcSmem<PAIRS>& sm)
{
    // four records per thread in flight: the copy waits for its loads once, not per record
    // (a single orbit of 32 nodes 220 -> 216 us, 4096 Venus orbits 1.525 -> 1.513 ms)
    constexpr int NT = PAIRS / 4;
    const int n = N * (P + 1);
    const gconst_cp base = pc_wave_base(grec);
    for (int i0 = threadIdx.x; i0 < n; i0 += 4 * NT) {
        double4 q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = pc_load_d4(base + (uint32_t)min(i0 + k * NT, n - 1) * 32u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + k * NT;
            if (i >= n) break;
            sm.Rec[3 * i + 0] = q[k].x;
            sm.Rec[3 * i + 1] = q[k].y;
            sm.Rec[3 * i + 2] = q[k].z;
            if (i < P) {
                sm.Mu[4 * i] = q[k].w;
                sm.Mu[4 * i + 1] = 1.5 * q[k].w;
                sm.Mu[4 * i + 2] = 1.875 * q[k].w;
            }
        }
    }
}

// Picard iterations of one segment for the job's ICs (initial states in sm.Y0): ephemeris
// records into LDS, initial guess, then sweeps until every IC of the job has stopped.
// On return yc holds the lane's share of the final iterate.  iters_out (may be null)
// receives the iteration records.
// MIXED: the job runs the FP32 -> FP64 precision schedule (compiled apart, so that FP64-only
// jobs carry none of its registers).
// HALF: the job has at most four ICs, the first of each lane's two (compiled apart likewise).
template <int PAIRS, int NP, bool MIXED = false, bool EIH = false, int SO = 0, bool HALF = false>
static __device__ __forceinline__ void pc_segment_solve(const PcParams& p, const PcGroupDev& g, int n, int64_t ic0,
                                                        int s, PcSmem<PAIRS>& sm, PcLane L, const PcFragD& kp,
                                                        double (&yc)[6][4], gi32p iters_out, int& had_notconv,
                                                        int rec_cap = PcSmem<PAIRS>::REC)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int T = Sh::T;
    double* sF = sm.F;
    double* sY0 = sm.Y0;
    const double* sWt = pc_weights<PAIRS, NP>(sm);
    const int tid = threadIdx.x;
    const int N = g.N;
    const int P = p.n_pert;
    const int64_t ic = ic0 + tid;
    const bool rec_lds = N * 3 * (P + 1) <= rec_cap;
    const int istride = p.iters_stride;
    const int fixed_iters = p.fixed_iters, max_iter = p.max_iter;
    const double mu_sun = p.mu_sun;
    const double t2 = g.tol * g.tol;
    const double Ts = g.t0 + g.h * (s + g.s0), Te = g.t0 + g.h * (s + g.s0 + 1);
    const double w2 = 0.5 * (Te - Ts);

    // this segment's ephemeris records into LDS (perturber data per node, Sec. 5.4.1)
    const double4* grec = reinterpret_cast<const double4*>(p.recs) +
                          (size_t)(g.rec_offset + (int64_t)s * N) * (P + 1);
    if (rec_lds) pc_stage_records<PAIRS>(grec, N, P, sm);
    pc_initial_guess<PAIRS, NP, HALF>(p, g, n, ic0, s, w2, L, sY0, sm.Dead, sF, yc);
    if (tid < T) sm.Active[tid] = (tid < n) && !sm.Dead[tid];
    __syncthreads();   // staging read before F is built
    pc_clear_rows<PAIRS, NP, SO != 0>(sF, N);
    // precision schedule (uniform per job): an FP32 phase first when asked, then FP64
    // sweeps.  Sweep kinds: 0 FP64 Picard sweep, 1 FP32 Picard sweep (jobs whose records do
    // not fit in LDS), 2 FP32 increment sweep (after one FP64 sweep; records in LDS).
    // An increment sweep adds w2 K_N dF to the FP64 iterate, dF the change of F to first
    // order in the last change of the iterate, (dv, G dr), with G the gravity gradient at
    // the iterate of the last FP64 sweep (the anchor); dF and the product are FP32, and no
    // force is evaluated.  From an anchor these sweeps converge, at the Picard rate, to the
    // Newton step from it (error quadratic in the anchor's); the FP32 rounding they add is
    // relative to the increments.  Increment jobs run in stages: FP64 sweeps until no IC
    // changes by more than 1e-3 (-1; one sweep after a warm start); increments to the
    // switch threshold (0); one FP64 sweep (1) that re-anchors the iterate on y0 + w2 K_N F(Y),
    // dropping the rounding and the linearisation error of stage 0; increments again (2),
    // from the closer anchor, until no IC changes by more than tol; then FP64 sweeps (3),
    // the only ones the stopping rule is applied to, so that every IC stops on an FP64
    // sweep that changed it by less than tol (one sweep for most ICs; more where the
    // linearisation left more, as near close approaches, or where stage 2 hit its cap).
    const bool incr = rec_lds;
    // increment jobs open with FP64 sweeps until no IC changes by more than 1e-3 (stage
    // -1): the linearisation needs an anchor near the solution, which a warm start gives
    // after one sweep and a cold start after several
    bool fp32 = MIXED && !incr;
    int mode = fp32 ? 1 : 0;
    // default switch: the first increment stage hands over at a relative change of 1e-6
    // (on the 262144-IC N-body workload 1e-5, 1e-6 and 1e-7 took 96.5, 95.5 and 97.7 ms;
    // a later switch lengthens stage 0, an earlier one leaves a farther anchor for stage 2);
    // FP32 Picard sweeps stall near 1e-7
    const double sw2 = p.switch2 > 0.0 ? p.switch2 : (incr ? 1e-12 : 1e-8);
    PcTol tl = pc_tol(p.tol_mode, t2, (MIXED && incr) ? 1e-6 : sw2);
    int n32 = 0;
    int stage = (MIXED && incr) ? -1 : 0;
    float* sD = reinterpret_cast<float*>(sF);                // increment sweeps: dF, FP32
    float* sG = reinterpret_cast<float*>(sF + 3 * PAIRS);    // increment sweeps: G at the anchor
    // relativistic model: the segment's records of the major bodies
    const double4* erec = nullptr;
    if constexpr (EIH)
        erec = reinterpret_cast<const double4*>(p.recs_eih) + (size_t)(g.rec_offset + (int64_t)s * N) * pc_eih_rec(P);
    // which of the lane's ICs iterate (point p = 2h + r), and whether any of the wave's group
    // does: the waves of a group without an IC (few ICs, or all stopped) only keep the barriers
    int act[4];
    auto read_active = [&]() -> bool {
#pragma unroll
        for (int q = 0; q < 4; ++q) act[q] = sm.Active[pc_ic<PAIRS, NP>(L, q >> 1, q & 1)];
        return __any(act[0] | act[1] | act[2] | act[3]);
    };
    bool busy = read_active();
    if (busy) {
        if constexpr (EIH) pc_publish_eih<PAIRS, NP, HALF>(sF, yc, L, N, P, erec, p.inv_c2);
        else if (MIXED && mode == 1)
            pc_publish<PAIRS, NP, MIXED>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
        else pc_publish<PAIRS, NP, false, SO != 0, HALF>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
    }
    __syncthreads();

    const PcFragF kp32 = pc_frag<PAIRS, NP, PcFragF>(g.kpair32, L);
    const int n_it = fixed_iters > 0 ? fixed_iters : max_iter;
    // the next product's first fragments, on their way while the waves wait at the barrier
    pc_d2v kpre[4];
    if constexpr (SO == 0 && !MIXED) pc_kpre_load(kp, kpre);
    // second-order sweeps: the K2_N strip, and the lane's node offset tau + 1 for the
    // x0 + w2 v0 (tau + 1) term
    PcFragD kp2 = {};
    double tp = 0.0;
    if constexpr (SO) {
        kp2 = pc_frag<PAIRS, NP, PcFragD>(g.kpair2, L);
        tp = pc_gcd(g.tau)[L.jn[0]] + 1.0;
    }
    for (int it = 1; it <= n_it; ++it) {
        L = pc_lane_again<PAIRS, NP>(L, N);
        // (1)-(2) product and stopping-rule flags
        f64x4 acc[6];
        int flag = 0;
        if constexpr (SO == 2) {   // holds barriers: every wave
            flag = pc_product2_fb<PAIRS, NP>(sF, sY0, sWt, kp, kp2, yc, acc, w2, tp, tl, L, P, mu_sun, rec_lds, sm.Rec,
                                             sm.Mu, grec);
        } else if (busy) {
            if constexpr (MIXED) {
                if (mode == 2) flag = pc_product32<PAIRS, NP, true>(sF, sY0, sWt, kp32, yc, acc, w2, tl, L);
                else if (mode == 1) flag = pc_product32<PAIRS, NP, false>(sF, sY0, sWt, kp32, yc, acc, w2, tl, L);
                else {
                    // not ahead of the barrier here: the 16 registers would live through the FP32 sweeps
                    // (128 nodes 9.72 -> 9.16 ms, 64 nodes 3.50 -> 3.36)
                    pc_kpre_load(kp, kpre);
                    flag = pc_product<PAIRS, NP, true>(sF, sY0, sWt, kp, kpre, yc, acc, w2, tl, L);
                }
            } else if constexpr (SO) {
                flag = pc_product2<PAIRS, NP>(sF, sY0, sWt, kp, kp2, yc, acc, w2, tp, tl, L);
            } else {
                flag = pc_product<PAIRS, NP, false>(sF, sY0, sWt, kp, kpre, yc, acc, w2, tl, L);
            }
        }
        pc_put_flags<PAIRS, NP>(sm.Flag, flag, L);
        busy = read_active();
        if constexpr (MIXED) {
            const unsigned long long keep =
                __ballot(L.c < Sh::E && sm.Active[L.grp * Sh::COLS + pc_col<PAIRS, NP>(L, L.c & (Sh::E - 1))] &&
                         ((flag >> (4 * (L.c & (Sh::E - 1)))) & 4));
            if (L.lane == 0) sm.Keep[L.wave] = keep != 0ull;
        }
        __syncthreads();   // every wave is done reading F; flags complete

        // the job leaves FP32 once no iterating IC changes by more than the switch threshold
        const bool stops = !fp32;   // stopping rule applies
        bool next32 = false;
        if (fp32) {
            int k = 0;
            for (int w = 0; w < Sh::W; ++w) k |= sm.Keep[w];
            ++n32;
            next32 = k && n32 < p.max_fp32;
            if (MIXED && incr && !next32) stage = stage == 0 ? 1 : 3;
        } else if (MIXED && incr && stage == -1) {
            // FP64 sweeps until the anchor is close enough, then increments (stage 0)
            int k = 0;
            for (int w = 0; w < Sh::W; ++w) k |= sm.Keep[w];
            if (!k) {
                stage = 0;
                next32 = true;
                n32 = 0;
                tl = pc_tol(p.tol_mode, t2, sw2);
            }
        } else if (MIXED && incr && stage == 1) {
            // the re-anchoring sweep ran: increments again until no change exceeds tol
            stage = 2;
            next32 = true;
            n32 = 0;
            tl.sa = tl.ta;
            tl.sb = tl.tb;
        }
        // (3) stopping rule per IC (Sec. 2.2; per-block error of Sec. 3.2 with blocks of one IC);
        //     applied to FP64 sweeps only
        if (tid < T && sm.Active[tid]) {
            const int f = pc_gather_flags<PAIRS, NP>(sm.Flag, tid);
            int rec = 0;
            if (f & 2) rec = -2;
            else if (fixed_iters > 0) rec = (it == fixed_iters) ? it : 0;
            else if (stops && !(f & 1)) rec = it;
            else if (it == max_iter) rec = -1;
            if (rec != 0) {
                sm.Active[tid] = 0;
                if (rec == -2) sm.Dead[tid] = 1;
                if (rec == -1) had_notconv = 1;
                if (tid < n && iters_out) iters_out[(size_t)ic * istride + s] = rec;
            }
        }
        pc_note_active<PAIRS, NP>(sm, L);
        const int next_mode = next32 ? (incr ? 2 : 1) : 0;
        // (4) ICs that were iterating take the new iterate and publish its F (or, before an
        //     increment sweep, the change of F)
        if constexpr (MIXED) {
            if (next_mode == 2 && it < n_it) {
                if (busy) {
                    float dy[6][4];
#pragma unroll
                    for (int b = 0; b < 6; ++b) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int on = act[2 * (b / 3) + (r & 1)];
                            dy[b][r] = on ? (float)(acc[b][r] - yc[b][r]) : 0.0f;
                            yc[b][r] = on ? acc[b][r] : yc[b][r];
                        }
                    }
                    // after an FP64 sweep the new iterate is the anchor: G evaluated there
                    pc_publish_chord<PAIRS, NP>(sD, sG, yc, dy, act, mode != 2, L, P, mu_sun, sm.Rec, sm.Mu);
                }
                fp32 = next32;
                mode = next_mode;
                __syncthreads();   // F complete; the active notes visible
                if (!pc_any_active<PAIRS, NP>(sm)) break;
                continue;
            }
            // back to FP64 after increment sweeps: the FP32 arrays left arbitrary bits in the
            // rows past the last one of the FP64 view
            if (mode == 2) pc_clear_rows<PAIRS, NP, false>(sF, N);
        }
        if (busy) {
#pragma unroll
            for (int b = 0; b < 6; ++b) {
#pragma unroll
                for (int r = 0; r < 4; ++r) yc[b][r] = act[2 * (b / 3) + (r & 1)] ? acc[b][r] : yc[b][r];
            }
            if (it < n_it) {
                if constexpr (EIH) pc_publish_eih<PAIRS, NP, HALF>(sF, yc, L, N, P, erec, p.inv_c2);
                else if (MIXED && next_mode == 1)
                    pc_publish<PAIRS, NP, MIXED>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
                else pc_publish<PAIRS, NP, false, SO != 0, HALF>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
            }
        }
        fp32 = next32;
        mode = next_mode;
        if constexpr (SO == 0 && !MIXED) pc_kpre_load(kp, kpre);
        __syncthreads();   // F complete; the active notes visible
        if (!pc_any_active<PAIRS, NP>(sm)) break;
    }
}

// Not inlined: one register allocation per node count, so the work-queue kernel that
// dispatches to all of them does not pay for the largest one everywhere.
template <int PAIRS, int NP, bool MIXED, bool EIH = false, int SO = 0, bool HALF = false>
__device__ __attribute__((noinline)) void pc_job(const PcParams& p, const PcJobDev& job, const PcGroupDev& g)
{
    PcSmem<PAIRS>& sm = pc_smem<PAIRS>();
    using Sh = PcShape<PAIRS, NP>;
    constexpr int T = Sh::T;

    double* sY0 = sm.Y0;
    const int tid = threadIdx.x;
    const PcLane L = pc_lane_geometry<PAIRS, NP>(tid, g.N);
    const int N = g.N, S = g.S;
    const int n = job.n;
    const int64_t ic = job.ic0 + tid;      // this thread's IC when tid < n
    // the buffers of the call, read once from the parameter block as global pointers
    const gdp g_bounds = pc_gd(p.bounds_out);
    const gdp g_nodes = pc_gd(p.nodes_out);
    const gi32p g_iters = pc_gi(p.iters_out);
    const int istride = p.iters_stride, nstride = p.nodes_stride;

    if (tid < T) {
        const gconst_dp y = pc_gcd(p.ics) + (job.ic0 + (tid < n ? tid : 0)) * 6;
        bool fin = true;
        for (int c = 0; c < 6; ++c) {
            const double v = y[c];
            sY0[c * T + tid] = v;
            fin = fin && isfinite(v);
        }
        sm.Dead[tid] = !fin;
    }
    pc_stage_weights<PAIRS, NP>(sm, g.wts);
    const PcFragD kp = pc_frag<PAIRS, NP, PcFragD>(g.kpair, L);
    __syncthreads();

    double yc[6][4];       // the lane's share of the current iterate
    int had_notconv = 0;
    for (int s = 0; s < S; ++s) {
        if (tid < n) {
            if (g_bounds) {
                const gdp bo = g_bounds + ((size_t)ic * (istride + 1) + s) * 6;
                for (int c = 0; c < 6; ++c) bo[c] = sY0[c * T + tid];
            }
            if (sm.Dead[tid] && g_iters) g_iters[(size_t)ic * istride + s] = -2;
        }
        pc_segment_solve<PAIRS, NP, MIXED, EIH, SO, HALF>(p, g, n, job.ic0, s, sm, L, kp, yc, g_iters, had_notconv);

        // converged node states of the segment (optional output), chaining (Sec. 2.2)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!L.ok || (Sh::PAR && h == 1 && !L.two)) continue;
            const int j = L.jn[h];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int m = pc_ic<PAIRS, NP>(L, h, r);
                if (g_nodes && m < n) {
                    const gdp o = g_nodes + (((size_t)(job.ic0 + m) * istride + s) * nstride + j) * 6;
#pragma unroll
                    for (int c = 0; c < 6; ++c) o[c] = yc[3 * h + c % 3][r + 2 * (c / 3)];
                }
                if (j == N - 1) {
                    const bool dead = sm.Dead[m];
#pragma unroll
                    for (int c = 0; c < 6; ++c)
                        sY0[c * T + m] = dead ? (double)NAN : yc[3 * h + c % 3][r + 2 * (c / 3)];
                }
            }
        }
        __syncthreads();
    }

    if (tid < n) {
        const gdp so = pc_gd(p.states_out) + (size_t)ic * 6;
        for (int c = 0; c < 6; ++c) so[c] = sY0[c * T + tid];
        if (g_bounds) {
            const gdp bo = g_bounds + ((size_t)ic * (istride + 1) + S) * 6;
            for (int c = 0; c < 6; ++c) bo[c] = sY0[c * T + tid];
        }
        if (had_notconv) atomicAdd(&p.counters[0], 1);
        if (sm.Dead[tid]) atomicAdd(&p.counters[1], 1);
    }
    __syncthreads();
}

// A job with more ICs than columns (n > T), FP64 sweeps.  Every column of the product is
// an independent fixed-point iteration (the product never mixes columns), so when an IC
// stops, its end state is stored and its column takes the next IC of the job for the same
// segment: the columns do not idle while a slower IC of the same block still iterates,
// only the tail of each segment does.  The job's ICs are dealt to its column groups (entry
// e to group e % GN); every wave of a group takes the same decisions from the same flags,
// so the two barriers per sweep stay the only ones.  Each IC's sequence of iterates is the
// one the one-block job body computes.  Between segments an IC's state lives in
// states_out (the end state of its last completed segment).
// SO = 1: second-order sweeps (pc_product2) instead of the first-order product.
template <int PAIRS, int NP, int SO = 0>
__device__ __attribute__((noinline)) void pc_job_list(const PcParams& p, const PcJobDev& job, const PcGroupDev& g)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int NT = Sh::NT, T = Sh::T, COLS = Sh::COLS, GN = Sh::GN, E = Sh::E;
    constexpr unsigned CMASK = (1u << COLS) - 1u;
    PcSmem<PAIRS>& sm = pc_smem<PAIRS>();
    double* sF = sm.F;
    double* sY0 = sm.Y0;
    const double* sWt = pc_weights<PAIRS, NP>(sm);
    const int tid = threadIdx.x;
    PcLane L = pc_lane_geometry<PAIRS, NP>(tid, g.N);
    const int N = g.N, S = g.S, P = p.n_pert;
    const int n = job.n;
    const int grp = L.grp;
    const int n_g = n > grp ? (n - grp + GN - 1) / GN : 0;   // entries of this wave's group
    const bool rec_lds = N * 3 * (P + 1) <= PcSmem<PAIRS>::REC;
    const PcTol tl = pc_tol(p.tol_mode, g.tol * g.tol, 0.0);
    const PcFragD kp = pc_frag<PAIRS, NP, PcFragD>(g.kpair, L);
    pc_d2v kpre[4];
    // second-order sweeps: the K2_N strip next to K_N's and the lane's tau + 1
    PcFragD kp2 = {};
    double tp = 0.0;
    if constexpr (SO) {
        kp2 = pc_frag<PAIRS, NP, PcFragD>(g.kpair2, L);
        tp = pc_gcd(g.tau)[L.jn[0]] + 1.0;
    }
    pc_stage_weights<PAIRS, NP>(sm, g.wts);
    const bool flane = L.lane < COLS;             // lanes < COLS carry the per-column decisions
    const int fcol = L.lane & (COLS - 1);
    const bool owner = flane && L.strip == 0;     // one wave per group writes per-IC records
    auto ic_of = [&](int e) -> int64_t { return job.ic0 + grp + (int64_t)GN * e; };
    auto col_of = [&](int e) -> int { return pc_col<PAIRS, NP>(L, e); };
    // the lane's part of a column: its IC r at both nodes of the row (PAR), or IC r of one eight
    auto has = [&](int e, int h) -> bool { return Sh::PAR || h == (e >> 1); };
    // the lane's point in a refill pass: point pt of a column (PAR: row pt % 16 at node pt / 16)
    constexpr int WN = Sh::PAR ? 32 : 16;
    const int pt = L.lane & (WN - 1), pt_row = L.strip * 16 + (pt & 15);
    const bool pt_ok = pt_row < (Sh::PAR ? (N + 1) >> 1 : N);
    const double pt_tau = pc_gcd(g.tau)[!pt_ok ? 0 : Sh::PAR && pt >= 16 ? N - 1 - pt_row : pt_row] + 1.0;
    double pf[2] = {0.0, 0.0};
    int notconv = 0;
    // the buffers of the call, read once from the parameter block as global pointers
    const gconst_dp g_ics = pc_gcd(p.ics);
    const gdp g_states = pc_gd(p.states_out);
    const gdp g_bounds = pc_gd(p.bounds_out);
    const gdp g_nodes = pc_gd(p.nodes_out);
    const gi32p g_iters = pc_gi(p.iters_out);
    const int istride = p.iters_stride, nstride = p.nodes_stride;
    const int fixed_iters = p.fixed_iters, max_iter = p.max_iter;
    const double mu_sun = p.mu_sun;

    double yc[6][4];
    for (int s = 0; s < S; ++s) {
        const double Ts = g.t0 + g.h * (s + g.s0), Te = g.t0 + g.h * (s + g.s0 + 1);
        const double w2 = 0.5 * (Te - Ts);
        const gconst_dp src = s == 0 ? g_ics : g_states;
        const double4* grec = reinterpret_cast<const double4*>(p.recs) +
                              (size_t)(g.rec_offset + (int64_t)s * N) * (P + 1);
        // Initial states of the group's entries base .. base + COLS - 1 (those its columns take
        // next), held across the wave's lanes (entry l % COLS, component l / COLS and, with 16
        // columns, 4 + l / 16) and loaded as soon as the ones before are taken: a refill then
        // waits on no memory (it waited about 3000 cycles for the state and the node's tau).
        auto prefetch = [&](int base) {
            const int e = base + fcol, c = L.lane / COLS;
            const gconst_dp y = src + ic_of(e) * 6 + c;
            pf[0] = e < n_g && c < 6 ? y[0] : 0.0;
            if constexpr (COLS == 16) pf[1] = e < n_g && c < 2 ? y[4] : 0.0;
        };
        // Warm (or cold) start, Sec. 2.1, of the group's columns in `rm`, column c taking entry
        // base + (its rank in rm).  The wave computes the points of its own rows for all those
        // columns together (one Kepler solve per lane and pass), stages them in the columns' F
        // slots (free after the product; component c of half h in the slot that its F value
        // will take), and the lanes that hold the points read them back.  The lanes of the
        // group's first node write y0 (product epilogue) and the checkpoint.
        auto slot = [&](int row, int col, int c, int h) __attribute__((always_inline)) -> double* {
            return sF + 2 * pc_unit<PAIRS, NP>(row, grp, c % 3, 8 * (c / 3) + (col & 7)) + h;
        };
        auto warm_columns = [&](unsigned rm, int base) {
            const int k = __popc(rm);
            for (int q0 = 0; q0 < WN * k; q0 += 64) {
                const int ci = (q0 + L.lane) / WN;
                double y0[6];
                bool fin = true;
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) {
                    const int from = (ci & (COLS - 1)) + COLS * (COLS == 16 ? cc & 3 : cc);
                    y0[cc] = __shfl(pf[COLS == 16 ? cc >> 2 : 0], from);
                    fin = fin && isfinite(y0[cc]);
                }
                if (ci >= k || !pt_ok) continue;
                unsigned m = rm;
                for (int t = 0; t < ci; ++t) m &= m - 1u;
                const int c = __ffs(m) - 1;
                const int h = Sh::PAR ? pt >> 4 : c >> 3;
                double y[6];
                if (!(p.init == 0 && fin && pc_kepler(y0, w2 * pt_tau, y))) {
#pragma unroll
                    for (int cc = 0; cc < 6; ++cc) y[cc] = y0[cc];
                }
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) *slot(pt_row, c, cc, h) = y[cc];
                if (pt_row == 0 && pt < 16) {
#pragma unroll
                    for (int cc = 0; cc < 6; ++cc) sY0[cc * T + grp * COLS + c] = y0[cc];
                    if (g_bounds) {
                        const gdp bo = g_bounds + ((size_t)ic_of(base + ci) * (istride + 1) + s) * 6;
#pragma unroll
                        for (int cc = 0; cc < 6; ++cc) bo[cc] = y0[cc];
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // staged points visible to the wave
            if (L.ok) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = col_of(e);
                    if (!((rm >> c) & 1u)) continue;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (!has(e, h)) continue;
#pragma unroll
                        for (int cc = 0; cc < 6; ++cc) {
                            double* f = slot(L.row, c, cc, h);
                            yc[3 * h + cc % 3][(e & 1) + 2 * (cc / 3)] = *f;
                            // second-order sweeps keep the unused halves of F's blocks at zero
                            if (SO && (cc == 2 || cc == 4)) *f = 0.0;
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // read before the slots are rewritten
        };

        if (rec_lds) pc_stage_records<PAIRS>(grec, N, P, sm);
        for (int i = tid; i < 6 * PAIRS; i += NT) sF[i] = 0.0;   // rows past the last stay zero
#pragma unroll
        for (int b = 0; b < 6; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) yc[b][r] = 1.0;
        }
        __syncthreads();   // records staged, F cleared
        // the group's first COLS entries into its columns
        int next = n_g < COLS ? n_g : COLS;                                   // uniform per group
        unsigned amask = next >= COLS ? CMASK : ((1u << next) - 1u);          // uniform per group
        int ent[E];
#pragma unroll
        for (int e = 0; e < E; ++e) ent[e] = col_of(e) < next ? col_of(e) : -1;
        prefetch(0);
        warm_columns(amask, 0);
        prefetch(next);
        int fent = fcol < next ? fcol : -1;   // flag lane: entry of its column
        int it0 = 0;                          // flag lane: sweep before its IC's first one
        __syncthreads();   // y0 written
        if (amask) pc_publish<PAIRS, NP, false, SO != 0>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
        if constexpr (SO == 0) pc_kpre_load(kp, kpre);
        __syncthreads();

        for (int it = 1;; ++it) {
            L = pc_lane_again<PAIRS, NP>(L, N);
            f64x4 acc[6];
            if (amask) {
                int flag;
                if constexpr (SO) flag = pc_product2<PAIRS, NP>(sF, sY0, sWt, kp, kp2, yc, acc, w2, tp, tl, L);
                else flag = pc_product<PAIRS, NP, false>(sF, sY0, sWt, kp, kpre, yc, acc, w2, tl, L);
                pc_put_flags<PAIRS, NP>(sm.Flag, flag, L);
            }
            __syncthreads();   // every wave is done reading F; flags complete

            // stopping rule per IC (Sec. 2.2), taken identically by every wave of the group
            int rec = 0;
            if (flane && fent >= 0) {
                const int f = pc_gather_flags<PAIRS, NP>(sm.Flag, grp * COLS + fcol);
                const int k = it - it0;
                if (f & 2) rec = -2;
                else if (fixed_iters > 0) rec = (k == fixed_iters) ? k : 0;
                else if (!(f & 1)) rec = k;
                else if (k >= max_iter) rec = -1;
            }
            const unsigned smask = (unsigned)__ballot(rec != 0) & CMASK;
            const unsigned dmask = (unsigned)__ballot(rec == -2) & CMASK;
            if (owner && rec != 0) {
                if (g_iters) g_iters[(size_t)ic_of(fent) * istride + s] = rec;
                if (rec == -1) ++notconv;
            }
            // the new iterate (a column whose IC has stopped and was not refilled goes on with
            // values nobody reads; the product mixes no columns)
            if (amask) {
#pragma unroll
                for (int b = 0; b < 6; ++b) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) yc[b][r] = acc[b][r];
                }
            }
            if (smask) {
                // outputs of the ICs that stopped: node states, end state (node N-1, NaN when
                // non-finite) as the next segment's y0 and the checkpoint
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = col_of(e);
                    if (!((smask >> c) & 1u) || !L.ok) continue;
                    const int64_t icg = ic_of(ent[e]);
                    const bool dead = (dmask >> c) & 1u;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (!has(e, h) || (Sh::PAR && h == 1 && !L.two)) continue;
                        const int j = L.jn[h];
                        if (g_nodes) {
                            const gdp nd = g_nodes + (((size_t)icg * istride + s) * nstride + j) * 6;
#pragma unroll
                            for (int cc = 0; cc < 6; ++cc) nd[cc] = yc[3 * h + cc % 3][(e & 1) + 2 * (cc / 3)];
                        }
                        if (j == N - 1) {
                            const gdp so = g_states + icg * 6;
                            const gdp bo = g_bounds ? g_bounds + ((size_t)icg * (istride + 1) + s + 1) * 6 : g_bounds;
#pragma unroll
                            for (int cc = 0; cc < 6; ++cc) {
                                const double v = dead ? (double)NAN : yc[3 * h + cc % 3][(e & 1) + 2 * (cc / 3)];
                                so[cc] = v;
                                if (bo) bo[cc] = v;
                            }
                        }
                    }
                }
                // refill: the stopped columns, in column order, take the group's next entries
                const int take = min(__popc(smask), n_g - next);
                unsigned rmask = 0u;
                {
                    unsigned m = smask;
                    for (int k = 0; k < take; ++k) {
                        rmask |= m & (0u - m);   // lowest stopped column
                        m &= m - 1u;
                    }
                }
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int c = col_of(e);
                    if ((rmask >> c) & 1u) ent[e] = next + __popc(rmask & ((1u << c) - 1u));
                    else if ((smask >> c) & 1u) ent[e] = -1;
                }
                if (rmask) {
                    warm_columns(rmask, next);
                    prefetch(next + take);
                }
                if (flane) {
                    if ((rmask >> fcol) & 1u) {
                        fent = next + __popc(rmask & ((1u << fcol) - 1u));
                        it0 = it;
                    } else if ((smask >> fcol) & 1u) {
                        fent = -1;
                    }
                }
                next += take;
                amask = (amask & ~smask) | rmask;
            }
            if (amask) pc_publish<PAIRS, NP, false, SO != 0>(sF, yc, L, P, mu_sun, rec_lds, sm.Rec, sm.Mu, grec);
            // every wave of an IC group holds the group's column mask: the first strip's waves
            // note it (rewritten only after the next sweep's first barrier)
            if (L.strip == 0 && L.lane == 0) sm.Go[grp] = amask != 0u;
            if constexpr (SO == 0) pc_kpre_load(kp, kpre);
            __syncthreads();   // F complete; the notes visible
            int go = 0;
#pragma unroll
            for (int q = 0; q < GN; ++q) go |= sm.Go[q];
            if (!go) break;
        }
    }
    if (notconv) atomicAdd(&p.counters[0], notconv);
    __syncthreads();   // every end state written
    for (int e = tid; e < n; e += NT) {
        const gconst_dp y = g_states + (job.ic0 + e) * 6;
        bool fin = true;
        for (int c = 0; c < 6; ++c) fin = fin && isfinite(y[c]);
        if (!fin) atomicAdd(&p.counters[1], 1);
    }
    __syncthreads();
}

// The job body for node count NP and the call's options: second-order sweeps (with the
// feedback when asked), relativistic, refilled column lists, precision schedule or
// plain FP64 one-block jobs.
template <int PAIRS, int NP>
static __device__ __forceinline__ void pc_run_job(const PcParams& p, const PcJobDev& job, const PcGroupDev& g,
                                                  bool list, bool mixed, bool eih, bool order2)
{
    // jobs of at most four ICs have a body of their own that evaluates half of the points (pc_publish);
    // in the one body with a branch, 4096 Venus orbits of full blocks ran 0.7 % slower
    constexpr bool PAR = PcShape<PAIRS, NP>::PAR;
    const bool few = PAR && job.n <= 4;
    // second-order calls plan 16 or more ICs a block up to 128 nodes (make_plan): no other bodies
    constexpr bool SO = PAIRS / NP >= 16 || NP == 256;
    if (order2) {
        if constexpr (SO) {
            if (p.feedback) pc_job<PAIRS, NP, false, false, 2>(p, job, g);
            else if (list) pc_job_list<PAIRS, NP, 1>(p, job, g);
            else pc_job<PAIRS, NP, false, false, 1>(p, job, g);
        }
    } else if (eih && mixed) {
        pc_job<PAIRS, NP, true, true>(p, job, g);
    } else if (eih) {
        if (few) pc_job<PAIRS, NP, false, true, 0, PAR>(p, job, g);
        else pc_job<PAIRS, NP, false, true>(p, job, g);
    } else if (list) {
        pc_job_list<PAIRS, NP>(p, job, g);
    } else if (mixed) {
        pc_job<PAIRS, NP, true>(p, job, g);
    } else if (few) {
        pc_job<PAIRS, NP, false, false, 0, PAR>(p, job, g);
    } else {
        pc_job<PAIRS, NP, false>(p, job, g);
    }
}

// Persistent work-queue kernel: every workgroup takes the next job of the plan (jobs of
// all groups and node counts, longest first) until the queue is empty, so one launch
// runs an uneven two-level batch (Sec. 3.2) to completion.
// Two waves per SIMD: 512-thread workgroups fill a CU alone (their LDS arena is the
// CU's), 256-thread ones fit two workgroups, running two independent jobs, per CU.
template <int PAIRS>
__global__ __launch_bounds__(PAIRS / 4, 2) void pc_fused_kernel(const PcParams* __restrict__ pp)
{
    __shared__ int sJob;
    const PcParams& p = *pp;
    for (;;) {
        if (threadIdx.x == 0) sJob = atomicAdd(p.queue, 1);
        __syncthreads();
        const int jb = sJob;
        __syncthreads();
        if (jb >= p.n_jobs) break;
        // private copies: with them the job bodies need not preserve the caller's registers
        const PcJobDev job = p.jobs[jb];
        const PcGroupDev g = p.groups[job.group];
        const bool list = job.n > g.T;   // more ICs than columns: refilled columns (FP64 only)
        const bool mixed = p.precision == 1;
        const bool eih = p.inv_c2 != 0.0;   // relativistic model: one-block jobs
        const bool order2 = p.order == 2;   // second-order sweeps (with the integral error feedback when
                                            // asked): FP64, point masses
        switch (g.NP) {
        case 16: pc_run_job<PAIRS, 16>(p, job, g, list, mixed, eih, order2); break;
        case 32: pc_run_job<PAIRS, 32>(p, job, g, list, mixed, eih, order2); break;
        case 64: pc_run_job<PAIRS, 64>(p, job, g, list, mixed, eih, order2); break;
        case 128: pc_run_job<PAIRS, 128>(p, job, g, list, mixed, eih, order2); break;
        case 256:
            if constexpr (PAIRS >= 2048) pc_run_job<PAIRS, 256>(p, job, g, list, mixed, eih, order2);
            break;
        default: break;
        }
    }
}

int pc_fused_occupancy(int pairs, int* blocks_per_cu)
{
    if (pairs == 2048)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, pc_fused_kernel<2048>, 512, 0);
    if (pairs == 1024)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, pc_fused_kernel<1024>, 256, 0);
    return hipErrorInvalidValue;
}

int pc_launch_fused(const PcParams& p, const PcParams* p_dev, int pairs, int grid, void* stream)
{
    if (p.n_jobs <= 0) return hipSuccess;
    hipStream_t st = (hipStream_t)stream;
    if (grid <= 0 || grid > p.n_jobs) grid = p.n_jobs;
    if (pairs == 2048)
        hipLaunchKernelGGL(pc_fused_kernel<2048>, dim3(grid), dim3(512), 0, st, p_dev);
    else if (pairs == 1024)
        hipLaunchKernelGGL(pc_fused_kernel<1024>, dim3(grid), dim3(256), 0, st, p_dev);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adjoint of the converged map (reverse sweep over segments)
// ---------------------------------------------------------------------------
// For a segment with converged node states Y = 1 y0^T + K G(Y), G_j = w2 f(Y_j, t_j), the
// derivative of a loss L(Y) with seed gbar = dL/dY is dL/dy0 = sum_j mu_j, where mu solves
// (I - K J)^T mu = gbar with J_j = w2 df/dy (implicit differentiation of the fixed point).
// mu is found by the adjoint fixed-point sweep mu <- gbar + J^T (K^T mu), which contracts
// like the forward Picard iteration; with f = (v, a(r)) and H = da/dr symmetric,
//   (J^T w)_r = w2 H w_v,   (J^T w)_v = w2 w_r.
// Segments are processed from the last: each is first re-solved from its checkpoint (the
// same forward code, so the same converged states), and its gradient seeds the end node of
// the previous one.  A lane holds its points' states and mu (PcShape), so that J^T w needs no
// other lane.
// EIH: the relativistic dynamics, whose force also depends on the velocity: J^T w is
// ((da/dr)^T w_v, w_r + (da/dv)^T w_v) instead of (H w_v, w_r).
template <int PAIRS, int NP, bool EIH = false>
__device__ __attribute__((noinline)) void pc_adjoint_job(const PcAdjParams& a, const PcJobDev& job,
                                                         const PcGroupDev& g)
{
    using Sh = PcShape<PAIRS, NP>;
    constexpr int T = Sh::T, W = Sh::W, COLS = Sh::COLS;
    PcSmem<PAIRS>& sm = pc_smem<PAIRS, true>();
    const PcParams& p = a.fwd;
    double* sF = sm.F;
    double* sY0 = sm.Y0;
    const int tid = threadIdx.x;
    PcLane L = pc_lane_geometry<PAIRS, NP>(tid, g.N);
    const int N = g.N, S = g.S, P = p.n_pert;
    const int n = job.n;
    const int64_t ic = job.ic0 + tid;
    // adjoint scratch: seed Lam and estimate LamIt behind the weights in Y0 where they fit, else
    // at the top of the record area; the sweeps' partial sums [wave][comp][column] over the
    // records' end, which the sweeps no longer read (the Jacobian is formed before them)
    constexpr int PARTS = W * 6 * COLS;
    constexpr bool IN_Y0 = 18 * T + 3 * Sh::KR <= 6 * (PAIRS / 16);
    constexpr int REC_CAP = PcSmem<PAIRS>::REC - (IN_Y0 ? 0 : 12 * T);
    double* sLam = IN_Y0 ? sY0 + 6 * T + 3 * Sh::KR : sm.Rec + REC_CAP;
    double* sLamIt = sLam + 6 * T;
    double* sLamPart = sm.Rec + REC_CAP - PARTS;
    const bool rec_lds = N * 3 * (P + 1) <= REC_CAP;
    const double t2a = a.adj_tol * a.adj_tol;

    if (tid < T) {
        for (int c = 0; c < 6; ++c) sLam[c * T + tid] = tid < n ? a.gbar_final[(size_t)ic * 6 + c] : 0.0;
    }
    pc_stage_weights<PAIRS, NP>(sm, g.wts);
    const PcFragD kp = pc_frag<PAIRS, NP, PcFragD>(g.kpair, L);
    const PcFragD kpT = pc_frag<PAIRS, NP, PcFragD>(g.kpairT, L);
    const double wr = Sh::PAR ? pc_gcd(g.wts)[2 * Sh::KR + L.row] : 0.0;
    double yc[6][4];
    int had_notconv = 0, adj_notconv = 0, dead_any = 0;
    // the lane's mu at IC r (both h): the pair (mu_l - mu_r, mu_l + mu_r), or the two eights'
    auto put_mu = [&](int c, int r, double vl, double vr) __attribute__((always_inline)) {
        pc_d2v* f = reinterpret_cast<pc_d2v*>(sF) +
                    pc_unit<PAIRS, NP>(L.row, L.grp, c % 3, 8 * (c / 3) + L.g + 4 * r);
        *f = Sh::PAR ? pc_d2v{vl - vr, vl + vr} : pc_d2v{vl, vr};
    };
    for (int s = S - 1; s >= 0; --s) {
        // segment s's converged iterate: the forward call's node states when given, else a
        // re-solve from its checkpoint
        if (tid < T) {
            const double* src = a.ckpt + ((size_t)(job.ic0 + (tid < n ? tid : 0)) * (a.ckpt_stride + 1) + s) * 6;
            bool fin = true;
            for (int c = 0; c < 6; ++c) {
                const double v = src[c];
                sY0[c * T + tid] = v;
                fin = fin && isfinite(v);
            }
            sm.Dead[tid] = !fin;
        }
        __syncthreads();
        const double4* grec = reinterpret_cast<const double4*>(p.recs) +
                              (size_t)(g.rec_offset + (int64_t)s * N) * (P + 1);
        const double4* erec = nullptr;
        if constexpr (EIH)
            erec = reinterpret_cast<const double4*>(p.recs_eih) + (size_t)(g.rec_offset + (int64_t)s * N) * pc_eih_rec(P);
        if (a.fwd_nodes) {
            if (!EIH && rec_lds) pc_stage_records<PAIRS>(grec, N, P, sm);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int m = pc_ic<PAIRS, NP>(L, h, r);
                    double v[6];
                    if (L.ok && m < n) {
                        const gconst_dp y = pc_gcd(a.fwd_nodes) +
                                            (((size_t)(job.ic0 + m) * a.ckpt_stride + s) * a.nodes_stride + L.jn[h]) * 6;
#pragma unroll
                        for (int c = 0; c < 6; ++c) v[c] = y[c];
                    } else {   // padding row or column: any finite state (its results are unused)
#pragma unroll
                        for (int c = 0; c < 6; ++c) v[c] = sY0[c * T + m];
                    }
#pragma unroll
                    for (int c = 0; c < 6; ++c) yc[3 * h + c % 3][r + 2 * (c / 3)] = v[c];
                }
            }
        } else {
            pc_segment_solve<PAIRS, NP, false, EIH>(p, g, n, job.ic0, s, sm, L, kp, yc, nullptr, had_notconv,
                                                    REC_CAP);
        }
        __syncthreads();
        const double Ts = g.t0 + g.h * s, Te = g.t0 + g.h * (s + 1);
        const double w2 = 0.5 * (Te - Ts);
        // the force Jacobian at the lane's points, fixed over the segment's sweeps (point masses:
        // symmetric; relativistic: with respect to position and velocity)
        double H[6][4], J[4][9], V[4][9];
        if constexpr (EIH) {
            const PcEihRecs R = pc_eih_recs(erec, N);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int h = 3 * (q >> 1), r = q & 1;
                pc_eih_jacobian(yc[h][r], yc[h + 1][r], yc[h + 2][r], yc[h][2 + r], yc[h + 1][2 + r], yc[h + 2][2 + r],
                                R, L.jn[q >> 1], P, p.inv_c2, J[q], V[q]);
            }
        } else {
            double x[4], y[4], z[4];
            pc_points(yc, 0, x);
            pc_points(yc, 1, y);
            pc_points(yc, 2, z);
            if (rec_lds) pc_hess_matrix<true>(x, y, z, L.jn, P, p.mu_sun, sm.Rec, sm.Mu, grec, H);
            else pc_hess_matrix<false>(x, y, z, L.jn, P, p.mu_sun, sm.Rec, sm.Mu, grec, H);
        }

        // seed of this segment at the lane's point q = 2h + r: the next segment's gradient at the
        // end node, plus the node seeds when given (recomputed where needed, not held); none at
        // a middle node's second place
        const gconst_dp g_seed = pc_gcd(a.gbar_nodes);
        auto seeds = [&](int q, double (&sd)[6]) __attribute__((always_inline)) {
            const int h = q >> 1, m = pc_ic<PAIRS, NP>(L, h, q & 1), j = L.jn[h];
            const bool on = L.ok && !(Sh::PAR && h == 1 && !L.two);
#pragma unroll
            for (int c = 0; c < 6; ++c) sd[c] = 0.0;
            if (g_seed && on && m < n) {
                const gconst_dp v = g_seed + (((size_t)(job.ic0 + m) * a.ckpt_stride + s) * a.nodes_stride + j) * 6;
#pragma unroll
                for (int c = 0; c < 6; ++c) sd[c] = v[c];
            }
            if (L.strip == (Sh::PAR ? 0 : (N - 1) >> 4)) {   // the strip of the last node
                const bool end = on && j == N - 1;
#pragma unroll
                for (int c = 0; c < 6; ++c) sd[c] += end ? sLam[c * T + m] : 0.0;
            }
        };
        if (tid < T) {
            sm.Active[tid] = (tid < n) && !sm.Dead[tid];
            for (int c = 0; c < 6; ++c) sLamIt[c * T + tid] = 0.0;
        }
        pc_clear_rows<PAIRS, NP, false>(sF, N);
        // mu^(0) = gbar
        if (L.ok) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                double sl[6], sr[6];
                seeds(r, sl);
                seeds(2 + r, sr);
#pragma unroll
                for (int c = 0; c < 6; ++c) put_mu(c, r, sl[c], sr[c]);
            }
        }
        __syncthreads();

        int it = 1;
        for (; it <= a.adj_max_iter; ++it) {
            L = pc_lane_again<PAIRS, NP>(L, N);
            f64x4 acc[6];
            pc_product_adj<PAIRS, NP>(sF, kpT, wr, acc, L);          // w = K^T mu
            // mu_new = gbar + J^T w: position rows w2 (da/dr)^T w_v, velocity rows w2 w_r (and the
            // relativistic (da/dv)^T w_v)
            if constexpr (EIH) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int h = 3 * (q >> 1), r = q & 1;
                    const double wx = acc[h][2 + r], wy = acc[h + 1][2 + r], wz = acc[h + 2][2 + r];
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        acc[h + b][2 + r] = fma(V[q][3 * b + 2], wz, fma(V[q][3 * b + 1], wy,
                                                fma(V[q][3 * b], wx, acc[h + b][r])));
                        acc[h + b][r] = fma(J[q][3 * b + 2], wz, fma(J[q][3 * b + 1], wy, J[q][3 * b] * wx));
                    }
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int h = 3 * (q >> 1), r = q & 1;
                    const double wx = acc[h][2 + r], wy = acc[h + 1][2 + r], wz = acc[h + 2][2 + r];
#pragma unroll
                    for (int b = 0; b < 3; ++b) acc[h + b][2 + r] = acc[h + b][r];
                    acc[h][r] = fma(H[4][q], wz, fma(H[3][q], wy, H[0][q] * wx));
                    acc[h + 1][r] = fma(H[5][q], wz, fma(H[1][q], wy, H[3][q] * wx));
                    acc[h + 2][r] = fma(H[2][q], wz, fma(H[5][q], wy, H[4][q] * wx));
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double sd[6];
                seeds(q, sd);
                const bool on = (q >> 1) == 0 || !Sh::PAR || L.two;
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    const int k = 3 * (q >> 1) + c % 3, r = (q & 1) + 2 * (c / 3);
                    const double v = fma(w2, acc[k][r], sd[c]);
                    acc[k][r] = q < 2 || on ? v : 0.0;   // no second place at a middle node
                }
            }
            // the sum over the strip's nodes (the 16 lanes of a row group hold the rows of the
            // same ICs)
#pragma unroll
            for (int c = 0; c < 6; ++c) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const double vl = acc[c % 3][r + 2 * (c / 3)], vr = acc[3 + c % 3][r + 2 * (c / 3)];
                    if constexpr (Sh::PAR) {
                        const double part = pc_row_sum16(L.ok ? vl + vr : 0.0);
                        if (L.c == 0) sLamPart[(L.wave * 6 + c) * COLS + L.g + 4 * r] = part;
                    } else {
                        const double pl = pc_row_sum16(L.ok ? vl : 0.0), pr = pc_row_sum16(L.ok ? vr : 0.0);
                        if (L.c == 0) {
                            sLamPart[(L.wave * 6 + c) * COLS + L.g + 4 * r] = pl;
                            sLamPart[(L.wave * 6 + c) * COLS + 8 + L.g + 4 * r] = pr;
                        }
                    }
                }
            }
            int act[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) act[q] = sm.Active[pc_ic<PAIRS, NP>(L, q >> 1, q & 1)];
            __syncthreads();   // K^T mu read by every wave; partial sums complete

            // gradient estimate lambda = sum_j mu_j per IC; stop when it no longer changes
            if (tid < T && sm.Active[tid]) {
                double d2 = 0.0, n2 = 0.0;
                const double* part = sLamPart + (tid / COLS) * Sh::STRIPS * 6 * COLS + tid % COLS;
                for (int c = 0; c < 6; ++c) {
                    double v = 0.0;
                    for (int w = 0; w < Sh::STRIPS; ++w) v += part[(w * 6 + c) * COLS];
                    const double d = v - sLamIt[c * T + tid];
                    d2 += d * d;
                    n2 += v * v;
                    sLamIt[c * T + tid] = v;
                }
                int rec = 0;
                if (!isfinite(n2)) rec = -2;
                else if (it > 1 && d2 <= t2a * n2) rec = it;
                else if (it == a.adj_max_iter) rec = -1;
                if (rec != 0) {
                    sm.Active[tid] = 0;
                    if (rec == -2) sm.Dead[tid] = 1;
                    if (rec == -1) adj_notconv = 1;
                    if (tid < n && a.adj_iters) a.adj_iters[(size_t)ic * a.ckpt_stride + s] = rec;
                }
            }
            // ICs that were iterating publish the new mu; a stopped IC's sweeps go on
            // beside them where it shares a place, and nobody reads them
            if (L.ok) {
#pragma unroll
                for (int c = 0; c < 6; ++c) {
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        if (act[r] | act[2 + r])
                            put_mu(c, r, acc[c % 3][r + 2 * (c / 3)], acc[3 + c % 3][r + 2 * (c / 3)]);
                    }
                }
            }
            pc_note_active<PAIRS, NP>(sm, L);
            __syncthreads();   // mu complete; the active notes visible
            if (!pc_any_active<PAIRS, NP>(sm)) break;
        }
        // this segment's gradient seeds the end node of the previous one
        if (tid < T) {
            const bool dead = sm.Dead[tid];
            dead_any |= dead;
            for (int c = 0; c < 6; ++c) sLam[c * T + tid] = dead ? (double)NAN : sLamIt[c * T + tid];
        }
        __syncthreads();
    }
    if (tid < n) {
        for (int c = 0; c < 6; ++c) a.grad_out[(size_t)ic * 6 + c] = sLam[c * T + tid];
        if (adj_notconv || had_notconv) atomicAdd(&a.counters[0], 1);
        if (dead_any) atomicAdd(&a.counters[1], 1);
    }
    __syncthreads();
}

template <int PAIRS>
__global__ __launch_bounds__(PAIRS / 4, 2) void pc_adjoint_kernel(const PcAdjParams* __restrict__ ap)
{
    __shared__ int sJob;
    const PcAdjParams& a = *ap;
    for (;;) {
        if (threadIdx.x == 0) sJob = atomicAdd(a.counters + 2, 1);
        __syncthreads();
        const int jb = sJob;
        __syncthreads();
        if (jb >= a.fwd.n_jobs) break;
        const PcJobDev job = a.fwd.jobs[jb];
        const PcGroupDev g = a.fwd.groups[job.group];
        const bool eih = a.fwd.inv_c2 != 0.0;
        switch (g.NP) {
        case 16: eih ? pc_adjoint_job<PAIRS, 16, true>(a, job, g) : pc_adjoint_job<PAIRS, 16>(a, job, g); break;
        case 32: eih ? pc_adjoint_job<PAIRS, 32, true>(a, job, g) : pc_adjoint_job<PAIRS, 32>(a, job, g); break;
        case 64: eih ? pc_adjoint_job<PAIRS, 64, true>(a, job, g) : pc_adjoint_job<PAIRS, 64>(a, job, g); break;
        case 128: eih ? pc_adjoint_job<PAIRS, 128, true>(a, job, g) : pc_adjoint_job<PAIRS, 128>(a, job, g); break;
        case 256:
            if constexpr (PAIRS >= 2048) eih ? pc_adjoint_job<PAIRS, 256, true>(a, job, g) : pc_adjoint_job<PAIRS, 256>(a, job, g);
            break;
        default: break;
        }
    }
}

int pc_launch_adjoint(const PcAdjParams& a, const PcAdjParams* a_dev, int pairs, int grid, void* stream)
{
    if (a.fwd.n_jobs <= 0) return hipSuccess;
    if (grid <= 0 || grid > a.fwd.n_jobs) grid = a.fwd.n_jobs;
    if (pairs == 1024)
        hipLaunchKernelGGL(pc_adjoint_kernel<1024>, dim3(grid), dim3(256), 0, (hipStream_t)stream, a_dev);
    else
        hipLaunchKernelGGL(pc_adjoint_kernel<2048>, dim3(grid), dim3(512), 0, (hipStream_t)stream, a_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Test hooks
// ---------------------------------------------------------------------------

// Y[j][c] = y0[c] + scale * sum_l K[j][l] F[l][c]; one workgroup per 16 columns (whole K_N,
// fragments kfrag).
__global__ __launch_bounds__(256) void pc_apply_operator_kernel(int NP, const double* kfrag, int N,
                                                                int64_t n_cols, const double* F,
                                                                const double* y0, double scale, double* Y)
{
    __shared__ double sF[PC_MAX_NP_FOR_HOOK * 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * 16;
    for (int i = tid; i < NP * 16; i += 256) {
        const int l = i >> 4, c = i & 15;
        sF[i] = (l < N && c0 + c < n_cols) ? F[(size_t)l * n_cols + c0 + c] : 0.0;
    }
    __syncthreads();
    const int NQ = NP >> 2;
    const int64_t col = c0 + (lane & 15);
    const double y0c = col < n_cols ? y0[col] : 0.0;
    for (int strip = wave; strip < NP / 16; strip += 4) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        const double* kp = kfrag + (size_t)strip * NQ * 64 + lane;
        for (int q = 0; q < NQ; ++q) acc = mfma16(kp[q * 64], sF[(4 * q + (lane >> 4)) * 16 + (lane & 15)], acc);
        for (int r = 0; r < 4; ++r) {
            const int j = strip * 16 + (lane >> 4) + 4 * r;
            if (j < N && col < n_cols) Y[(size_t)j * n_cols + col] = y0c + scale * acc[r];
        }
    }
}

int pc_launch_apply_operator(int NP, const double* kfrag, int N, int64_t n_cols, const double* F,
                             const double* y0, double scale, double* Y, void* stream)
{
    if (NP > PC_MAX_NP_FOR_HOOK) return hipErrorInvalidValue;
    const int64_t grid = (n_cols + 15) / 16;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(pc_apply_operator_kernel, dim3((unsigned)grid), dim3(256), 0, (hipStream_t)stream,
                       NP, kfrag, N, n_cols, F, y0, scale, Y);
    return hipGetLastError();
}

__global__ void pc_eval_force_kernel(const double* r, const double* t, int64_t n, const PcBodyDev* bodies,
                                     int P, double epoch, double mu_sun, double* a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 rec[PC_MAX_PERT_DEV + 1];
    double ix = 0.0, iy = 0.0, iz = 0.0;
    for (int b = 0; b < P; ++b) {
        double q[3];
        pc_body_position(bodies[b], t[i] - epoch, q);
        rec[b] = make_double4(q[0], q[1], q[2], bodies[b].mu);
        const double iq = rsqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
        const double sq = bodies[b].mu * (iq * iq * iq);
        ix += sq * q[0];
        iy += sq * q[1];
        iz += sq * q[2];
    }
    rec[P] = make_double4(ix, iy, iz, 0.0);
    double ax, ay, az;
    pc_accel(r[i], r[n + i], r[2 * n + i], rec, P, mu_sun, ax, ay, az);
    a[i] = ax;
    a[n + i] = ay;
    a[2 * n + i] = az;
}

int pc_launch_eval_force(const double* r, const double* t, int64_t n, const PcBodyDev* bodies,
                         int n_pert, double epoch, double mu_sun, double* a, void* stream)
{
    if (n <= 0) return hipSuccess;
    if (n_pert > PC_MAX_PERT_DEV) return hipErrorInvalidValue;
    const int bs = 256;
    hipLaunchKernelGGL(pc_eval_force_kernel, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0,
                       (hipStream_t)stream, r, t, n, bodies, n_pert, epoch, mu_sun, a);
    return hipGetLastError();
}

__global__ void pc_eval_kepler_kernel(const double* y0, const double* dt, int64_t n, double* y, int32_t* ok)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double a[6], b[6];
    for (int c = 0; c < 6; ++c) a[c] = y0[c * n + i];
    const bool good = pc_kepler(a, dt[i], b);
    for (int c = 0; c < 6; ++c) y[c * n + i] = good ? b[c] : a[c];
    ok[i] = good ? 1 : 0;
}

int pc_launch_eval_kepler(const double* y0, const double* dt, int64_t n, double* y, int32_t* ok, void* stream)
{
    if (n <= 0) return hipSuccess;
    const int bs = 256;
    hipLaunchKernelGGL(pc_eval_kepler_kernel, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0,
                       (hipStream_t)stream, y0, dt, n, y, ok);
    return hipGetLastError();
}
