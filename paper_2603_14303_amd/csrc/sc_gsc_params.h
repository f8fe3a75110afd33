// Parameters and constants shared by the sc_gsc_merge kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sc {

constexpr int kGscThreads = 256;
constexpr int kMaxChunksPerItem = 32;
constexpr int kInlinePrefixTokens = 32768;   // up to here the last kernel adds the cluster counts up itself: a launch less
constexpr float kBand = 1e-4f;   // fp32 cosine error for d <= 128 is < 2e-5; inside the band -> fp64

// A counting probe of the budget search counts the rows at every threshold that the next steps of the bisection may ask for: the
// midpoint, the midpoints of its two halves, and so on, kProbeLevels deep.
constexpr int kProbeLevels = 3;
constexpr int kProbeNodes = (1 << kProbeLevels) - 1;
constexpr int kProbeWords = kProbeNodes + 1;      // counts of a window, one unused

// State of the threshold search of sc_gsc_merge_budget (device memory, behind the merge workspace).
struct BudgetState {
    float tau;            // threshold of the next sc_gsc_merge launch
    float lo, hi;         // bracket: lo is assumed to meet the budget, hi not to
    int step;
    long long rows_lo;    // rows at lo (-1 until lo itself has been probed)
    // what the update needs, filed once per call
    long long budget_rows;
    int iterations;
    float *tau_out;
    long long *rows_out;
    // a probe's (sequence, head) workgroups add up their rows here; the last of them moves the bracket
    unsigned int arrived;
    unsigned int bad;                 // bit t: some head overflowed at threshold t
    long long total[kProbeNodes];
};

// What a search starts from, and what starts it: the plan kernel of its first counting probe, or a kernel of its own.  One thread.
struct BudgetStart {
    BudgetState *state;
    float lo, hi;
    int iterations;
    long long budget_rows;
    float *tau_out;
    long long *rows_out;
};
__device__ __forceinline__ void budget_begin(const BudgetStart &b) {
    BudgetState *st = b.state;
    st->lo = b.lo;
    st->hi = b.hi;
    st->step = 0;
    st->rows_lo = -1;
    st->tau = (b.iterations > 0) ? 0.5f * (b.lo + b.hi) : b.lo;   // no probe: the final launch runs at tau_lo
    st->budget_rows = b.budget_rows;
    st->iterations = b.iterations;
    st->tau_out = b.tau_out;
    st->rows_out = b.rows_out;
    st->arrived = 0u;
    st->bad = 0u;
    for (int t = 0; t < kProbeNodes; ++t) st->total[t] = 0;
}

// The threshold of node `node` of the probes' tree (1: the midpoint, 2 j and 2 j + 1: the midpoints of the lower and the upper half that
// node j makes), by the same fp32 midpoints as budget_bracket_step's.
__host__ __device__ __forceinline__ float budget_node_tau(float lo, float hi, int node) {
    int level = 0;
    while ((node >> (level + 1)) != 0) ++level;
    for (; level > 0; --level) {
        const float mid = 0.5f * (lo + hi);
        if ((node >> (level - 1)) & 1) lo = mid; else hi = mid;
    }
    return 0.5f * (lo + hi);
}

// after a probe at st->tau with `sum` rows in all (`bad`: some head overflowed its capacity, which counts
// as over budget): move the bracket and choose the next threshold: another midpoint, or lo itself for the
// final launch.  After the final launch (step == iterations): file the rows it produced.  One thread.
__device__ __forceinline__ void budget_bracket_step(BudgetState *st, long long sum, bool bad) {
    const int step = st->step;
    if (step < st->iterations) {
        const bool fits = !bad && sum <= st->budget_rows;
        if (fits) { st->lo = st->tau; st->rows_lo = sum; } else { st->hi = st->tau; }
        st->step = step + 1;
        st->tau = (step + 1 < st->iterations) ? 0.5f * (st->lo + st->hi) : st->lo;
    } else {
        st->rows_lo = bad ? -1 : sum;   // the final launch ran at lo
    }
    if (st->tau_out) *st->tau_out = st->lo;
    if (st->rows_out) *st->rows_out = st->rows_lo;
}

// A counting probe ends in a kernel that adds up its rows, one workgroup per (sequence, head): each of them adds its row counts (lane t: at
// node t + 1 of the tree; rows < 0: the head overflowed, or has no valid chunking) to the state, and the last one to arrive goes down the tree and
// moves the bracket `levels` times, so no further launch is needed between two probes.  One wavefront.
__device__ __forceinline__ void budget_probe_arrive(BudgetState *st, int rows, int lane, int levels, unsigned int n_heads) {
    const int nodes = (1 << levels) - 1;
    if (lane < nodes) {
        if (rows >= 0) atomicAdd(reinterpret_cast<unsigned long long *>(&st->total[lane]), (unsigned long long)rows);
        else atomicOr(&st->bad, 1u << lane);
    }
    __threadfence();
    unsigned int before = 0u;
    if (lane == 0) before = atomicAdd(&st->arrived, 1u);
    if (__builtin_amdgcn_readfirstlane((int)before) != (int)(n_heads - 1u)) return;
    __threadfence();
    long long total = 0;
    if (lane < nodes) {
        total = (long long)atomicAdd(reinterpret_cast<unsigned long long *>(&st->total[lane]), 0ull);
        st->total[lane] = 0;
    }
    const unsigned int bad = atomicOr(&st->bad, 0u);
    if (lane == 0) {
        st->bad = 0u;
        st->arrived = 0u;
    }
    for (int level = 0, node = 1; level < levels; ++level) {
        const bool over = ((bad >> (node - 1)) & 1u) != 0u;
        const long long sum = (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(total >> 32), node - 1) << 32) |
                                          (unsigned)__builtin_amdgcn_readlane((int)total, node - 1));
        if (lane == 0) budget_bracket_step(st, sum, over);
        node = 2 * node + ((!over && sum <= st->budget_rows) ? 1 : 0);
    }
}

struct GscWindow;
struct GscLongs;
struct GscSegment;

struct GscParams {
    const void *K, *V;
    int64_t stride_b, stride_h, stride_n;
    const int32_t *seq_lens, *offsets;
    int64_t offsets_stride_b;
    const int32_t *num_chunks;
    int B, Hkv, N_max;
    float tau;
    const float *tau_dev;   // if not NULL the threshold is read from device memory instead (budget search)
    BudgetState *budget;    // if not NULL: a counting probe of the budget search, see budget_probe_arrive
    void *Kc, *Vc;
    int out_is_bf16;
    int cap;
    int32_t *counts, *comp_lens;
    const int32_t *base_lens;   // [B, Hkv] rows already in Kc/Vc/counts (append mode), or NULL for none
    int32_t *cid;         // [B, Hkv, N_max]   cluster index of every token (caller's buffer or workspace)
    int32_t *cluster_id;  // the caller's buffer, or NULL if not requested
    int32_t *seedrow;     // [B, Hkv, N_max]   seed positions of a chunk that spans several blocks
    int32_t *pcount;      // [B, Hkv, N_max + 1] generic path: clusters per chunk
    int32_t *rowbase;     // [B, Hkv, N_max + 2] first output row of every chunk; without a scan kernel, generic path: clusters of every item
    int32_t *stmp;        // [B, Hkv, N_max]   fast path: reciprocal norms of the seeds of a chunk that spans several blocks; output row of every row of a window left to others
    void *rows_ws;        // [B, Hkv, N_max, d] twice, in the output type: the fast path lays out the arrays below in it
    GscWindow *windows;   // [B, win_slots]
    uint32_t *published;  // [B, Hkv, win_slots] rows of a window, for the windows behind it
    GscSegment *segments; // [B, Hkv, segments] rows of a segment's windows
    int32_t *win_count;   // [B, Hkv, win_slots, kProbeWords] rows of a window at each threshold of a counting probe
    GscLongs *longs;      // [B, segments] slots of long chunks
    int32_t *long_count;  // [B, segments]
    int ahead_per_head, ahead_wgs;  // workgroups that decide long chunks first: per (sequence, head), in all
    uint32_t *head_state; // [B, Hkv]          whether windows were left to others
    int seg_bits;         // of a segment's word that count windows
    int slots_per_segment, win_slots;   // windows per kSegRows rows / per sequence that there is room for
    int max_chunks;       // chunks per window, <= 0: as many as fit
    int polls;            // looks at the windows before until a workgroup leaves its own to others
    int count_only;       // fast path: cluster and count only, for `budget`; no values are read, no outputs written
    int chunks_per_item;  // generic path
    int probe_levels;     // steps of the search that a counting probe decides
    int short_wgs[2];     // generic path: workgroups per (sequence, head) where short chunks make items of 8 / of 16 or 32, 0: they don't (see gsc_item_shape)
};

// rows already present in the outputs of (sequence, head) bh; an overflowed or impossible state counts as
// a full cache, so that nothing more is written and the new length is filed as -1
template <typename P>
__device__ __forceinline__ int gsc_base_rows(const P &p, int64_t bh, bool &bad) {
    const int raw = p.base_lens ? p.base_lens[bh] : 0;
    bad = raw < 0 || raw > p.cap;
    return bad ? p.cap : raw;
}

bool gsc_fast_holds(int heads, int N_max);   // they fit its words and its launch
// planned: the windows of these offsets are in the workspace already (and nothing has been published since)
hipError_t launch_gsc_fast(const GscParams &p, bool planned, const BudgetStart *start, hipStream_t stream);

}  // namespace sc
