// pc_plain.h -- arguments of the per-iteration ("plain") path of pc_plain.hip.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include "pc_internal.h"

struct PcPlainArgs {
    PcParams p;                 // outputs, model and options shared with the fused path
    const PcGroupDev* g;        // device copy of this group's descriptor
    PcGroupDev g_host;          // host copy (interval)
    const PcJobDev* jobs;       // device: this group's jobs in IC order
    int n_jobs, N, NP, T, S;
    double t2;                  // tol^2
    int64_t Mpad;               // n_jobs * T columns
    double* Y;                  // [n_jobs][24][threads]: the jobs' iterates
    double* Y0;                 // [6][Mpad]
    int32_t *active, *dead, *notconv, *valid;   // [Mpad]
    int32_t *job_list, *job_list_out, *job_flag; // [n_jobs]
    int32_t* count;             // [5]: jobs in the lists of odd and even sweeps, jobs with a change
                                //      above tol, workgroups arrived, segment done
    int32_t* host;              // pinned host ints (4): done, jobs left, the group's status, sweeps run
};

// Workspace bytes of one group on the plain path.
size_t pc_plain_bytes(int NP, int n_jobs, int T);

// Host-side state of one group's propagation on the plain path.  The host loop of
// Sec. 5.4 is cut at its read-backs: pc_plain_begin enqueues the group's work up to the
// first read-back, and each pc_plain_advance, called once the stream has run what is queued,
// takes the loop decision from `host` and enqueues the work up to the
// next read-back (or the end of the group, after which `done` is set).  One host thread
// can so drive several groups on several streams, polling each stream's read-back.
struct PcPlainRun {
    PcPlainArgs a;
    int32_t* lists[2];          // device: active-job lists of even and odd sweeps
    int32_t* host;              // pinned host ints (4), written by the sweep kernels
    void* stream;
    int s = 0, it = 0, count = 0, n_it = 0;
    int last = 0;               // sweeps of the group's previous segment
    double w2 = 0.0;            // half-length of the current segment
    bool group = false, done = false;
};

// Lay out the group's state in `workspace` and enqueue its work up to the first read-back
// (returns a hipError_t).  host: pinned host ints (4).
int pc_plain_begin(PcPlainRun& r, const PcPlainArgs& a, void* workspace, int32_t* host, void* stream);
// The read-back enqueued last has completed: decide and enqueue the next part.
int pc_plain_advance(PcPlainRun& r);

// Propagate one group with per-iteration kernels and a host loop that waits on `stream`
// for each read-back (returns a hipError_t).
int pc_run_plain(PcPlainArgs a, void* workspace, int32_t* host, void* stream);
