// sc_gsc_merge_budget: sc_gsc_merge with the similarity threshold chosen for a target cache size.
//
// The paper reports its results at cache budgets (Sec. 3.1: 20 / 35 / 50 % of the entries kept) but does
// not say how a budget becomes the threshold tau of Alg. 1.  The number of rows N'(tau) grows with tau
// (a higher bar merges less), so the largest tau that still meets the budget is found by bisection.
// Every probe is the clustering half of sc_gsc_merge (counts only); the bracket lives in device memory.
// A probe reads the keys once and counts at the seven thresholds that three steps of the bisection may ask for; it ends in the count kernel,
// whose workgroups (one per sequence and head) add up their row counts, and the last of them to arrive moves the bracket three times (where a
// probe is a complete merge, outside the bf16 / d = 128 path, it is at one threshold, and a small kernel after it moves the bracket from the merged lengths).
// Bound by the chain of a probe's windows (its kernel 55 us at 8 heads x 32768 tokens, against 24 for a single threshold) and by launches.  12 iterations,
// us per call, a probe a step / three steps a probe: 8 x 32768 379 / 292, 2 x 2000 163 / 105, 8 x 8 x 16384 1019 / 844; chunks with a long tail, 8 x 32768
// 550 / 420, 8 x 131072 1477 / 1268; all chunks longer than a window, where the thresholds share less: 8 x 32768 in chunks of 200 589 / 524, of 400
// 809 / 793, 8 x 131072 1527 / 1600, 1884 / 1995, 2 x 8000 295 / 175 and 545 / 300.  (Two steps a probe instead of three: 331 and 125 on the first
// two.)  What is left over after threes takes a probe of two steps, or of one threshold (one step in all 79 / 78; by the kernel for several 87).  The
// whole search is a fixed sequence of launches on the caller's stream with no host synchronisation.  The
// last launch runs at the threshold found and leaves its merged cache in the outputs.
#include "sc_device.h"
#include "sc_gsc_params.h"
#include "sc_host.h"

namespace sc {

size_t gsc_budget_state_bytes() { return align_up(sizeof(BudgetState), 256); }

__global__ void budget_init_kernel(BudgetStart start) { budget_begin(start); }

// after a complete merge at st->tau: total rows from the merged lengths (any overflowed head counts as over
// budget), then the same step as after a counting probe
__global__ __launch_bounds__(256) void budget_update_kernel(BudgetState *st, const int32_t *comp_lens, int n_bh) {
    __shared__ long long s_sum[4];
    __shared__ int s_bad[4];
    long long sum = 0;
    int bad = 0;
    for (int i = threadIdx.x; i < n_bh; i += 256) {
        const int v = comp_lens[i];
        if (v < 0) bad = 1; else sum += v;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        sum += __shfl_xor(sum, d, kWave);
        bad |= __shfl_xor(bad, d, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_sum[threadIdx.x / kWave] = sum;
        s_bad[threadIdx.x / kWave] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) budget_bracket_step(st, s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3], (s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]) != 0);
}

hipError_t launch_gsc_budget(GscMergeArgs a, long long budget_rows, float tau_lo, float tau_hi, int iterations,
                             float *tau_out, long long *rows_out, void *state, hipStream_t stream) {
    BudgetState *st = reinterpret_cast<BudgetState *>(state);
    a.tau_dev = &st->tau;
    const bool counting = gsc_merge_takes_fast_path(a);
    const BudgetStart start = {st, tau_lo, tau_hi, iterations, budget_rows, tau_out, rows_out};
    hipError_t e;
    if (!counting || iterations == 0) {      // (the first counting probe's plan starts the search itself)
        hipLaunchKernelGGL(budget_init_kernel, dim3(1), dim3(1), 0, stream, start);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (int it = 0; it <= iterations;) {     // `iterations` probes, then the launch at the result
        // a probe only needs the row counts: clustering without reading the values, without the merge and
        // without writing rows, at all thresholds that the next kProbeLevels steps may ask for, and its count kernel moves the
        // bracket itself (where the fast path runs; elsewhere a probe is a full merge followed by the update kernel, like the final launch)
        const bool probe = it < iterations;
        const int levels = !probe || !counting ? 1 : (iterations - it < kProbeLevels ? iterations - it : kProbeLevels);
        a.count_only = probe;
        a.budget_state = (probe && counting) ? state : nullptr;
        a.probe_levels = levels;
        a.planned = counting && it > 0;      // the windows do not depend on the threshold
        a.budget_start = (probe && counting && it == 0) ? &start : nullptr;
        e = launch_gsc_merge(a, stream);
        if (e != hipSuccess) return e;
        if (!(probe && counting)) {
            hipLaunchKernelGGL(budget_update_kernel, dim3(1), dim3(256), 0, stream, st, a.comp_lens, a.B * a.Hkv);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        it += levels;
    }
    return hipSuccess;
}

}  // namespace sc
