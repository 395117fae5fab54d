// pc_plain.hip -- the "plain" GPU path: one group at a time, a kernel per Picard iteration and
// a host-side loop, the structure of the paper's CUDA program (Sec. 5.4): the iterate lives in
// HBM between the iterations, each of which evaluates the dynamics of all stacked states, takes
// the fit/integrate/evaluate product and the error, reduces it over the group and lets the host
// decide whether another one follows.
//
// Differences from the paper's program: by default the error is per IC (converged ICs are
// frozen and jobs whose ICs have all converged are compacted out of the next launches).
// With PC_CONV_GROUP_MAX the paper's whole-system rule holds per group: no IC stops on
// its own, the sweep kernels count the jobs that still hold a change above tol, and the
// segment ends for the whole group when that count is zero.
//
// One iteration is one kernel (pc_plain_sweep): its last workgroup to finish compacts the job
// list and reduces the group's decision, which the host reads from pinned memory.  Separate
// kernels for the dynamics, the product and the compaction, two copies per iteration and a
// host round trip after each were mostly launches and gaps between kernels of 4 to 15 us: six
// groups of 64 to 256 nodes with 2500 ICs on four streams took 12.0 ms, now 5.0.  The host
// queues several iterations ahead of each read-back (plain_batch); the ones past the end find
// the group's done mark and return.
//
// State in HBM, per job: the register image of the sweep kernel's threads, Y[job][value 24]
// [thread] (value and thread of a node, component and IC: plain_at), so that a wave's loads and
// stores are contiguous.
#include "pcprop.h"
#include "pc_device.h"
#include "pc_plain.h"

namespace {

constexpr int kPlainPairs = 2048;
constexpr int kPlainBs = 256;

// Words of PcPlainArgs::count.
enum { kCountA = 0, kCountB = 1, kOpen = 2, kArrived = 3, kDone = 4 };

// Place of component c of the job's IC k at node j in its job's part of Y.
template <int NP>
__device__ size_t plain_at(int N, int j, int c, int k)
{
    using Sh = PcShape<kPlainPairs, NP>;
    const int M = Sh::PAR ? (N + 1) >> 1 : N;
    const int row = j < M ? j : N - 1 - j;
    const int h = Sh::PAR ? (j < M ? 0 : 1) : (k >> 3) & 1;
    const int m = k & 7, wave = (k / Sh::COLS) * Sh::STRIPS + (row >> 4);
    const int value = (3 * h + c % 3) * 4 + (m >> 2) + 2 * (c / 3);
    return (size_t)value * Sh::NT + wave * 64 + (m & 3) * 16 + (row & 15);
}
__device__ size_t plain_at(int NP, int N, int j, int c, int k)
{
    switch (NP) {
    case 16: return plain_at<16>(N, j, c, k);
    case 32: return plain_at<32>(N, j, c, k);
    case 64: return plain_at<64>(N, j, c, k);
    case 128: return plain_at<128>(N, j, c, k);
    default: return plain_at<256>(N, j, c, k);
    }
}
constexpr size_t kJobValues = (size_t)24 * (kPlainPairs / 4);   // doubles of one job in Y

// Initial states of the group's ICs (padding columns copy the job's first IC), their records,
// the first boundary record and the group's counters.
__global__ void pc_plain_load(PcPlainArgs a)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m < 5) a.count[m] = 0;
    if (m >= a.Mpad) return;
    const PcJobDev job = a.jobs[m / a.T];
    const int i = (int)(m % a.T);
    const double* y = a.p.ics + (job.ic0 + (i < job.n ? i : 0)) * 6;
    bool fin = true;
    for (int c = 0; c < 6; ++c) {
        const double v = y[c];
        a.Y0[c * a.Mpad + m] = v;
        fin = fin && isfinite(v);
        if (i < job.n && a.p.bounds_out) a.p.bounds_out[(size_t)(job.ic0 + i) * (a.p.iters_stride + 1) * 6 + c] = v;
    }
    a.dead[m] = !fin;
    a.notconv[m] = 0;
    a.valid[m] = i < job.n;
}

// Sweep `it` of segment s, one active job per workgroup: the job's iterate (the initial guess
// on the first sweep, which runs every job), its dynamics, the product y_new = y0 + w2 K_N F
// with the error of every IC, the stopping decision, and the new iterate of the ICs that were
// iterating.  Bound by latency: a group rarely fills the chip.
template <int NP, bool EIH>
__global__ __launch_bounds__(kPlainPairs / 4, 2) void pc_plain_sweep(PcPlainArgs a, int s, int it, double w2)
{
    constexpr int PAIRS = kPlainPairs;
    using Sh = PcShape<PAIRS, NP>;
    constexpr int NT = Sh::NT, T = Sh::T, KR = Sh::KR;
    __shared__ alignas(16) double sF[6 * PAIRS];
    __shared__ double sY0[6 * T];
    __shared__ double sWt[2 * KR];
    __shared__ int sFlag[Sh::W * 16];
    __shared__ int sActive[T];
    __shared__ int sDead[T];
    __shared__ int sOpen;   // group-max rule: some IC of the job changed by more than tol
    __shared__ int sLast, sBase;
    __shared__ int sSum[Sh::W];

    const int tid = threadIdx.x;
    const bool first = it == 1;
    if (!first && a.count[kDone]) return;   // queued past the segment's end
    const int n_in = first ? a.n_jobs : a.count[it & 1];
    const int slot = blockIdx.x;
    int job = -1, any = 0, open = 0;
    if (slot < n_in) {
        job = first ? slot : a.job_list[slot];
        const int64_t m0 = (int64_t)job * T;
        const int N = a.N, P = a.p.n_pert;
        const PcLane L = pc_lane_geometry<PAIRS, NP>(tid, N);
        const PcJobDev jd = a.jobs[job];
        for (int i = tid; i < 6 * T; i += NT) sY0[i] = a.Y0[(size_t)(i / T) * a.Mpad + m0 + i % T];
        if constexpr (Sh::PAR) {
            for (int i = tid; i < 2 * KR; i += NT) sWt[i] = pc_gcd(a.g->wts)[i];
        }
        if (tid < T) {
            const int dead = a.dead[m0 + tid];
            sDead[tid] = dead;
            sActive[tid] = first ? a.valid[m0 + tid] && !dead : a.active[m0 + tid];
            if (first) {
                a.active[m0 + tid] = sActive[tid];
                if (dead && tid < jd.n && a.p.iters_out)
                    a.p.iters_out[(size_t)(jd.ic0 + tid) * a.p.iters_stride + s] = -2;
            }
        }
        if (tid == 0) sOpen = 0;
        const PcFragD kp = pc_frag<PAIRS, NP, PcFragD>(a.g->kpair, L);
        pc_d2v kpre[4];
        pc_kpre_load(kp, kpre);
        const gdp Y = pc_gd(a.Y) + (size_t)job * kJobValues + tid;
        double yc[6][4];
        if (!first) {
#pragma unroll
            for (int b = 0; b < 6; ++b) {
#pragma unroll
                for (int r = 0; r < 4; ++r) yc[b][r] = Y[(4 * b + r) * NT];
            }
        }
        __syncthreads();
        if (first) {
            pc_initial_guess<PAIRS, NP>(a.p, *a.g, jd.n, jd.ic0, s, w2, L, sY0, sDead, sF, yc);
            __syncthreads();   // staging read before F is built
        }
        pc_clear_rows<PAIRS, NP, false>(sF, N);
        if constexpr (EIH) {
            const double4* erec = reinterpret_cast<const double4*>(a.p.recs_eih) +
                                  (size_t)(a.g->rec_offset + (int64_t)s * N) * pc_eih_rec(P);
            pc_publish_eih<PAIRS, NP>(sF, yc, L, N, P, erec, a.p.inv_c2);
        } else {
            const double4* grec = reinterpret_cast<const double4*>(a.p.recs) +
                                  (size_t)(a.g->rec_offset + (int64_t)s * N) * (P + 1);
            pc_publish<PAIRS, NP>(sF, yc, L, P, a.p.mu_sun, false, nullptr, nullptr, grec);
        }
        __syncthreads();
        f64x4 acc[6];
        const int flag =
            pc_product<PAIRS, NP, false>(sF, sY0, sWt, kp, kpre, yc, acc, w2, pc_tol(a.p.tol_mode, a.t2, 0.0), L);
        pc_put_flags<PAIRS, NP>(sFlag, flag, L);
        // the new iterate of the ICs that were iterating (on the first sweep the frozen ones
        // keep their guess)
#pragma unroll
        for (int b = 0; b < 6; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int on = sActive[pc_ic<PAIRS, NP>(L, b / 3, r & 1)];
                if (on || first) Y[(4 * b + r) * NT] = on ? acc[b][r] : yc[b][r];
            }
        }
        __syncthreads();   // flags complete
        if (tid < T && sActive[tid]) {
            const int fl = pc_gather_flags<PAIRS, NP>(sFlag, tid);
            int rec = 0;
            if (fl & 2) rec = -2;
            else if (a.p.fixed_iters > 0) rec = (it == a.p.fixed_iters) ? it : 0;
            else if (a.p.conv == PC_CONV_GROUP_MAX) { if (fl & 1) sOpen = 1; }   // decided for the group
            else if (!(fl & 1)) rec = it;
            else if (it == a.p.max_iter) rec = -1;
            if (rec != 0) {
                sActive[tid] = 0;
                a.active[m0 + tid] = 0;
                if (rec == -2) a.dead[m0 + tid] = 1;
                if (rec == -1) a.notconv[m0 + tid] = 1;
                if (tid < jd.n && a.p.iters_out)
                    a.p.iters_out[(size_t)(jd.ic0 + tid) * a.p.iters_stride + s] = rec;
            }
        }
        any = __syncthreads_or(tid < T ? sActive[tid] : 0);
        open = sOpen;
    } else {
        __syncthreads();   // every wave has read the done mark before this workgroup arrives: the last
                           // workgroup to arrive may set it
    }
    // the last workgroup to arrive compacts the jobs that still hold an iterating IC, in list
    // order, and takes the segment's decision (agent scope: the workgroups run on several XCDs)
    if (tid == 0) {
        if (job >= 0) __hip_atomic_store(a.job_flag + job, any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (open) __hip_atomic_fetch_add(a.count + kOpen, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int prev = __hip_atomic_fetch_add(a.count + kArrived, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        sLast = prev == (int)gridDim.x - 1;
        sBase = 0;
    }
    __syncthreads();
    if (!sLast) return;
    for (int c0 = 0; c0 < n_in; c0 += NT) {
        const int i = c0 + tid;
        const int jb = i < n_in ? (first ? i : a.job_list[i]) : -1;
        const bool f = jb >= 0 && __hip_atomic_load(a.job_flag + jb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        const unsigned long long b = __ballot(f);
        if ((tid & 63) == 0) sSum[tid >> 6] = __popcll(b);
        __syncthreads();
        int at = sBase + __popcll(b & ((1ull << (tid & 63)) - 1ull));
        for (int w = 0; w < (tid >> 6); ++w) at += sSum[w];
        if (f) a.job_list_out[at] = jb;
        __syncthreads();
        if (tid == 0) {
            for (int w = 0; w < Sh::W; ++w) sBase += sSum[w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const int op = __hip_atomic_load(a.count + kOpen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.count[(it + 1) & 1] = sBase;
        a.count[kOpen] = 0;
        a.count[kArrived] = 0;
        const bool group = a.p.conv == PC_CONV_GROUP_MAX && a.p.fixed_iters == 0;
        const int n_it = a.p.fixed_iters > 0 ? a.p.fixed_iters : a.p.max_iter;
        const bool settled = group && op == 0;   // no job holds a change above tol
        const int done = settled || sBase == 0 || it >= n_it;
        a.count[kDone] = done;
        // the host reads these once the stream has reached its event
        __hip_atomic_store(a.host + 0, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.host + 1, sBase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.host + 2, settled ? it : -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.host + 3, it, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Segment end: the last node starts the next segment; optional node / boundary outputs.
// Group-max rule: every IC still in the group records the group's status (the sweep count, or
// -1 when max_iter sweeps did not converge).
__global__ void pc_plain_chain(PcPlainArgs a, int s, int last, int group, int status)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m == 0) a.count[kDone] = 0;
    if (m >= a.Mpad) return;
    const PcJobDev job = a.jobs[m / a.T];
    const int i = (int)(m % a.T);
    const bool valid = i < job.n;
    const int64_t ic = job.ic0 + i;
    const double* Y = a.Y + (size_t)(m / a.T) * kJobValues;
    if (group && a.active[m]) {
        a.active[m] = 0;
        if (status == -1) a.notconv[m] = 1;
        if (valid && a.p.iters_out) a.p.iters_out[(size_t)ic * a.p.iters_stride + s] = status;
    }
    if (valid && a.p.nodes_out) {
        for (int j = 0; j < a.N; ++j) {
            double* o = a.p.nodes_out + (((size_t)ic * a.p.iters_stride + s) * a.p.nodes_stride + j) * 6;
            for (int c = 0; c < 6; ++c) o[c] = Y[plain_at(a.NP, a.N, j, c, i)];
        }
    }
    const bool dead = a.dead[m];
    for (int c = 0; c < 6; ++c) {
        const double v = dead ? (double)NAN : Y[plain_at(a.NP, a.N, a.N - 1, c, i)];
        a.Y0[c * a.Mpad + m] = v;
        if (valid && a.p.bounds_out)
            a.p.bounds_out[((size_t)ic * (a.p.iters_stride + 1) + s + 1) * 6 + c] = v;
        if (valid && last) a.p.states_out[(size_t)ic * 6 + c] = v;
    }
    if (valid && last) {
        if (a.notconv[m]) atomicAdd(&a.p.counters[0], 1);
        if (dead) atomicAdd(&a.p.counters[1], 1);
    }
}

template <int NP>
void launch_sweep(const PcPlainArgs& a, int grid, int s, int it, double w2, hipStream_t st)
{
    if (a.p.inv_c2 != 0.0)
        hipLaunchKernelGGL((pc_plain_sweep<NP, true>), dim3(grid), dim3(kPlainPairs / 4), 0, st, a, s, it, w2);
    else
        hipLaunchKernelGGL((pc_plain_sweep<NP, false>), dim3(grid), dim3(kPlainPairs / 4), 0, st, a, s, it, w2);
}

hipError_t launch_sweep_np(const PcPlainArgs& a, int grid, int s, int it, double w2, hipStream_t st)
{
    switch (a.NP) {
    case 16: launch_sweep<16>(a, grid, s, it, w2, st); break;
    case 32: launch_sweep<32>(a, grid, s, it, w2, st); break;
    case 64: launch_sweep<64>(a, grid, s, it, w2, st); break;
    case 128: launch_sweep<128>(a, grid, s, it, w2, st); break;
    case 256: launch_sweep<256>(a, grid, s, it, w2, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

size_t pc_plain_bytes(int, int n_jobs, int T)
{
    const size_t Mpad = (size_t)n_jobs * T;
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    return al((size_t)n_jobs * kJobValues * 8) + al(6 * Mpad * 8) + 4 * al(Mpad * 4) + 3 * al((size_t)n_jobs * 4) + 256;
}

namespace {

// Queue the segment's next sweeps, up to the next read-back: as many as the previous segment of
// the group took but one, then two at a time (a sweep queued past the end costs about 3 us on
// the stream, a read-back and its host round trip about 10 us).
hipError_t plain_batch(PcPlainRun& r)
{
    PcPlainArgs& a = r.a;
    int k = r.it == 0 && r.last > 2 ? r.last - 1 : r.it == 0 ? 4 : 2;
    k = k < r.n_it - r.it ? k : r.n_it - r.it;
    for (; k > 0; --k) {
        ++r.it;
        a.job_list = r.lists[r.it & 1];
        a.job_list_out = r.lists[(r.it + 1) & 1];
        const hipError_t e = launch_sweep_np(a, r.count, r.s, r.it, r.w2, (hipStream_t)r.stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Segment r.s: every job, from the first sweep.
hipError_t plain_begin_segment(PcPlainRun& r)
{
    const double h = r.a.g_host.h;
    const double Ts = r.a.g_host.t0 + h * r.s, Te = r.a.g_host.t0 + h * (r.s + 1);
    r.w2 = 0.5 * (Te - Ts);
    r.last = r.s > 0 ? r.host[3] : 0;
    r.count = r.a.n_jobs;
    r.it = 0;
    return plain_batch(r);
}

}  // namespace

int pc_plain_begin(PcPlainRun& r, const PcPlainArgs& args, void* workspace, int32_t* host, void* stream)
{
    r = PcPlainRun{};
    r.a = args;
    r.host = host;
    r.stream = stream;
    PcPlainArgs& a = r.a;
    a.host = host;
    hipStream_t st = (hipStream_t)stream;
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    char* w = static_cast<char*>(workspace);
    a.Mpad = (int64_t)a.n_jobs * a.T;
    a.Y = reinterpret_cast<double*>(w);                w += al((size_t)a.n_jobs * kJobValues * 8);
    a.Y0 = reinterpret_cast<double*>(w);               w += al(6 * (size_t)a.Mpad * 8);
    a.active = reinterpret_cast<int32_t*>(w);          w += al(a.Mpad * 4);
    a.dead = reinterpret_cast<int32_t*>(w);            w += al(a.Mpad * 4);
    a.notconv = reinterpret_cast<int32_t*>(w);         w += al(a.Mpad * 4);
    a.valid = reinterpret_cast<int32_t*>(w);           w += al(a.Mpad * 4);
    r.lists[0] = reinterpret_cast<int32_t*>(w);        w += al((size_t)a.n_jobs * 4);
    r.lists[1] = reinterpret_cast<int32_t*>(w);        w += al((size_t)a.n_jobs * 4);
    a.job_flag = reinterpret_cast<int32_t*>(w);        w += al((size_t)a.n_jobs * 4);
    a.count = reinterpret_cast<int32_t*>(w);
    r.n_it = a.p.fixed_iters > 0 ? a.p.fixed_iters : a.p.max_iter;
    r.group = a.p.conv == PC_CONV_GROUP_MAX && a.p.fixed_iters == 0;

    const unsigned gm = (unsigned)((a.Mpad + kPlainBs - 1) / kPlainBs);
    hipLaunchKernelGGL(pc_plain_load, dim3(gm), dim3(kPlainBs), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return plain_begin_segment(r);
}

int pc_plain_advance(PcPlainRun& r)
{
    PcPlainArgs& a = r.a;
    hipStream_t st = (hipStream_t)r.stream;
    if (!r.host[0]) {
        r.count = r.host[1];
        return plain_batch(r);
    }
    const unsigned gm = (unsigned)((a.Mpad + kPlainBs - 1) / kPlainBs);
    hipLaunchKernelGGL(pc_plain_chain, dim3(gm), dim3(kPlainBs), 0, st, a, r.s, r.s == a.S - 1 ? 1 : 0,
                       r.group ? 1 : 0, r.host[2]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (++r.s == a.S) {
        r.done = true;
        return hipSuccess;
    }
    return plain_begin_segment(r);
}

int pc_run_plain(PcPlainArgs a, void* workspace, int32_t* host, void* stream)
{
    PcPlainRun r;
    hipError_t e = (hipError_t)pc_plain_begin(r, a, workspace, host, stream);
    while (e == hipSuccess && !r.done) {
        e = hipStreamSynchronize((hipStream_t)stream);
        if (e == hipSuccess) e = (hipError_t)pc_plain_advance(r);
    }
    return e;
}
