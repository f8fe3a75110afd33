// sc_gsc_merge: Greedy Seed-Based Clustering inside every chunk (paper Sec. 2.3, Alg. 1, Eq. 2)
// followed by mean-pool merging of each cluster (Sec. 2.4, Eq. 3), per (sequence, KV head).
//
// Three kernels:
//   1. gsc_assign  one wavefront per chunk.  The chunk's key rows sit in registers, 8 elements per
//                  lane (d/8 neighbouring lanes cover a row, 64 rows per block).  Seeds are taken in
//                  order; for one seed every lane forms partial dot products for its row pieces, a
//                  transposed DPP reduction hands each lane the full dot product of ONE row, the
//                  cosine is compared with tau and a ballot marks the absorbed rows.  Decisions
//                  inside a +-1e-4 band around tau (and anything involving odd norms) are redone in
//                  fp64 by the whole wave.  Writes the cluster index of every token and the number
//                  of clusters of every chunk.
//   2. gsc_scan    per (sequence, head): exclusive scan over chunks of (clusters + closing
//                  delimiter) -> first output row of every chunk, total rows -> comp_lens.  Sequences of more
//                  than 32k tokens only: shorter ones leave the sum to gsc_merge.
//   3. gsc_merge   one group of d/8 lanes per OUTPUT row: walks the chunk's cluster indices, gathers
//                  the member rows of its cluster (16-byte pieces, coalesced per row), accumulates in
//                  fp32 in member order, divides by the size and writes the core; delimiter rows and
//                  singletons are copied.
#include "sc_device.h"
#include "sc_gsc_params.h"
#include "sc_host.h"

namespace sc {

// ------------------------------------------------------------------------------------------------
// fp64 re-evaluation of one (seed, candidate) pair by the whole wave: Eq. 2 in double precision.
template <typename T, int D>
__device__ bool cosine_exceeds_f64(const T *seed_row, const T *cand_row, float tau, int lane) {
    double dot = 0.0, ss = 0.0, cc = 0.0;
#pragma unroll
    for (int e = lane; e < D; e += kWave) {
        const double s = load1_f64(seed_row + e), c = load1_f64(cand_row + e);
        dot += s * c; ss += s * s; cc += c * c;
    }
    dot = wave_allreduce_sum(dot);
    ss = wave_allreduce_sum(ss);
    cc = wave_allreduce_sum(cc);
    const double sim = dot / (sqrt(ss) * sqrt(cc));
    return sim > (double)tau;   // NaN compares false: a zero-norm key never merges
}

// ------------------------------------------------------------------------------------------------
// Alg. 1 on one chunk by one wavefront.  Returns the number of clusters.
template <typename T, int D>
__device__ int gsc_chunk(const T *__restrict__ Kbh, int64_t stride_n, int start, int l, float tau,
                         int32_t *__restrict__ cid_bh, int32_t *__restrict__ seed_bh, int lane) {
    constexpr int LPR = D / 8;        // lanes per row
    constexpr int RPW = kWave / LPR;  // rows per wave-wide load
    const int g = lane / LPR, c = lane % LPR;
    // lane r of the wave "owns" block row r; the transposed reduction leaves row RPW*c+g in lane (g,c)
    const int owner_of_my_row = (lane % RPW) * LPR + lane / RPW;

    if (l == 1) {
        if (lane == 0) cid_bh[start] = 0;
        return 1;
    }
    int nseeds = 0;
    for (int rb = 0; rb < l; rb += kWave) {
        const int nr = min(kWave, l - rb);
        const int t_eff = (nr + RPW - 1) / RPW;
        float kreg[LPR][8];
        float part[LPR];
#pragma unroll
        for (int t = 0; t < LPR; ++t) {
            const int row = rb + RPW * t + g;
            if (t < t_eff && row < l) {
                load8(Kbh + (int64_t)(start + row) * stride_n + 8 * c, kreg[t]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) kreg[t][e] = 0.f;
            }
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) s = fmaf(kreg[t][e], kreg[t][e], s);
            part[t] = s;
        }
        const float nsq = lane_gather(row_transpose_reduce<LPR>(part, c), owner_of_my_row);
        const float rinv = __frsqrt_rn(nsq);
        const bool odd_norm = !(nsq > 1e-30f && nsq < 1e30f);

        uint64_t todo = (nr == kWave) ? ~0ull : ((1ull << nr) - 1ull);   // unassigned rows of this block
        int my_cid = -1;
        const int seeds_before = nseeds;
        int old = 0;
        while (todo != 0ull) {
            // next seed: first the seeds of earlier blocks (in order), then the first unassigned row
            int srow, cluster;
            float s_nsq;
            float sreg[8];
            if (old < seeds_before) {
                cluster = old;
                srow = __hip_atomic_load(seed_bh + start + old, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                old += 1;
                load8(Kbh + (int64_t)(start + srow) * stride_n + 8 * c, sreg);
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(sreg[e], sreg[e], s);
                s_nsq = row_allreduce_sum<LPR>(s);
            } else {
                const int r = first_bit(todo);
                srow = rb + r;
                cluster = nseeds;
                nseeds += 1;
                if (l > kWave && lane == 0)
                    __hip_atomic_store(seed_bh + start + cluster, srow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lane == r) my_cid = cluster;
                todo &= ~(1ull << r);
                s_nsq = __shfl(nsq, r, kWave);
                if (todo == 0ull) break;
                load8(Kbh + (int64_t)(start + srow) * stride_n + 8 * c, sreg);
            }
            const float s_rinv = __frsqrt_rn(s_nsq);
            const bool s_odd = !(s_nsq > 1e-30f && s_nsq < 1e30f);
#pragma unroll
            for (int t = 0; t < LPR; ++t) {
                float s = 0.f;
                if (t < t_eff) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) s = fmaf(kreg[t][e], sreg[e], s);
                }
                part[t] = s;
            }
            const float dotv = lane_gather(row_transpose_reduce<LPR>(part, c), owner_of_my_row);
            const float sim = dotv * rinv * s_rinv;
            const bool cand = (todo >> lane) & 1ull;
            const bool sure_yes = sim > tau + kBand;
            const bool sure_no = sim < tau - kBand;
            const bool unsure = s_odd || odd_norm || !(sure_yes || sure_no);
            bool yes = cand && !unsure && sure_yes;
            uint64_t recheck = ballot64(cand && unsure);
            while (recheck != 0ull) {
                const int j = first_bit(recheck);
                recheck &= recheck - 1ull;
                const bool res = cosine_exceeds_f64<T, D>(Kbh + (int64_t)(start + srow) * stride_n,
                                                          Kbh + (int64_t)(start + rb + j) * stride_n, tau, lane);
                if (lane == j) yes = res;
            }
            const uint64_t absorbed = ballot64(yes);
            if (yes) my_cid = cluster;
            todo &= ~absorbed;
        }
        if (lane < nr) cid_bh[start + rb + lane] = my_cid;
        if (rb + kWave < l) {
            // the seed positions written above are read back by all lanes for the next block
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
        }
    }
    return nseeds;
}

// Chunks per work item of a sequence of n tokens in M chunks, the same in both kernels.  Short chunks make few rows: an item of
// four or eight of them leaves most groups of gsc_merge without one, and its barriers and trips to memory are for next to
// nothing.  us per call, delimiters at a fixed distance, 8 / 16 / 32 chunks (16 and a scan kernel):
//   distance                  1                     2                     4                     8                    12
//   8 heads x 32768 x 64 f32  265 / 138 / 107 (152) 187 / 104 / 101 (110) 150 / 126 / 129 (128) 118 /  96 /  97 (98)  96 /  92 / 105 (124)
//   64 x 1200 x 64 f32         82 /  56 /  41 (46)   61 /  41 /  39 (40)   53 /  50 /  59 (54)   46 /  45 /  56 (53)  40 /  40 /  65 (65)
// Calls that would take four, 4 / 8 / 16 / 32 chunks, distance 1, 2, 3, 6 (up to four tokens eight, up to two 16 or 32):
//   2 x 32768 x 64 f32 (128 workgroups per head)  123 / 80 / 75 / 56 (99), 85 / 57 / 52 / 50 (65), 79 / 64 / 87 / 80 (95), 52 / 57 / 71 / 87 (76)
// and with an item for every workgroup anyway (2 x 1024 x 64 f32, distance 4) 14.4 / 15.4 / 21.2 / 35.9 (23.9).
//
// Workgroups per (sequence, head): an item per 21 tokens per chunk is what chunks of a few dozen tokens make.  Fewer than 1024 in all
// would leave a short sequence's longest chunks behind one another (128 per head / this: 2 x 32768 x 64 f32, distance 1 55 / 35, 8 42 / 37;
// 4 x 70000 x 64 f32, distance 2 173 / 156), more than 2048 only fill the queue (128 per head / this: 128 x 2000 x 64 f32 83 / 68,
// 16 x 8 x 8192 x 64 bf16 398 / 265; with the item order below).  The grid is for p.chunks_per_item.  (With every workgroup of it on items of
// 16, 8 x 32768 x 64 f32, distance 1, takes 169 instead of 140 us and distance 2 118 instead of 104: not all of them are on the chip
// at once, and the later ones start from the first item again.)
static int gsc_item_workgroups(int heads, int N_max, int C) { return max(heads <= 8 ? 1024 / heads : min(128, 2048 / heads), N_max / (21 * C)); }
__device__ __forceinline__ void gsc_item_shape(const GscParams &p, int M, int n, int launched, int &C, int &wgs) {
    C = p.chunks_per_item;
    wgs = launched;
    if (p.short_wgs[0] == 0) return;
    const int64_t tokens = n, chunks = M;
    const bool dense = 2 * tokens < 5 * chunks;
    if (p.chunks_per_item >= 8) {
        if (tokens < 10 * chunks) C = dense ? 32 : 16;
    } else if (2 * tokens < 9 * chunks && chunks > p.chunks_per_item * wgs) {
        C = dense ? (chunks > 16 * wgs ? 32 : 16) : 8;
    }
    if (C != p.chunks_per_item) wgs = min(wgs, p.short_wgs[C >= 16]);
}

// Grid (sequence and head, first item): workgroup ids go to the eight XCDs in turn, and a short sequence has work for a few of its
// workgroups only.  With the items fastest and a multiple of eight of them, those few were the same XCDs and the same part of
// their compute units for every head (64 heads x 1200 x 64 f32, us per call: 60 with 76 of them, 86 with 128).  (The
// z dimension is for more than 2^23 heads.)
constexpr int kGridHeadsLog2 = 23;
__device__ __forceinline__ int gsc_grid_head() { return (int)(blockIdx.x + (blockIdx.z << kGridHeadsLog2)); }

template <typename T, int D>
__global__ __launch_bounds__(kGscThreads) void gsc_assign_kernel(GscParams p) {
    __shared__ int s_off[kMaxChunksPerItem + 1];
    __shared__ int s_rows[kGscThreads / kWave];
    const int bh_i = gsc_grid_head();
    if (bh_i >= p.B * p.Hkv) return;
    const int b = bh_i / p.Hkv, h = bh_i - b * p.Hkv;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    // wave index as a scalar: everything derived from it (chunk bounds, loop trip counts) stays
    // wave-uniform for the compiler, so the cross-lane operations below always see all 64 lanes
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int M = p.num_chunks[b];
    if (M <= 0) return;
    int n = p.seq_lens ? p.seq_lens[b] : p.N_max;
    n = n < 0 ? 0 : (n > p.N_max ? p.N_max : n);
    int C, wgs;
    gsc_item_shape(p, M, n, (int)gridDim.y, C, wgs);
    if ((int)blockIdx.y >= wgs) return;
    const int items = (M + C - 1) / C;
    const float tau = p.tau_dev ? *p.tau_dev : p.tau;
    const int64_t bh = bh_i;
    const T *Kbh = reinterpret_cast<const T *>(p.K) + b * p.stride_b + h * p.stride_h;
    const int32_t *off = p.offsets + (int64_t)b * p.offsets_stride_b;
    int32_t *cid_bh = p.cid + bh * p.N_max;
    int32_t *seed_bh = p.seedrow + bh * p.N_max;
    int32_t *pcount_bh = p.pcount + bh * ((int64_t)p.N_max + 1);
    int32_t *item_rows_bh = p.rowbase + bh * ((int64_t)p.N_max + 2);   // clusters of every item, see gsc_merge
    auto file_item = [&](int item) {
        int rows = 0;
#pragma unroll
        for (int w = 0; w < kGscThreads / kWave; ++w) rows += s_rows[w];
        item_rows_bh[item] = rows;
    };

    int item = blockIdx.y;
    for (; item < items; item += wgs) {
        const int m0 = item * C;
        const int nch = min(C, M - m0);
        int rows = 0;
        __syncthreads();
        if (tid == 0 && item != (int)blockIdx.y) file_item(item - wgs);
        if (tid <= nch) s_off[tid] = off[m0 + tid];
        __syncthreads();
        for (int idx = wave; idx < nch; idx += kGscThreads / kWave) {
            const int start = __builtin_amdgcn_readfirstlane(s_off[idx]);
            const int l = __builtin_amdgcn_readfirstlane(s_off[idx + 1]) - 1 - start;
            int pc = 0;
            if (l > 0) pc = gsc_chunk<T, D>(Kbh, p.stride_n, start, l, tau, cid_bh, seed_bh, lane);
            rows += pc;
            if (lane == 0) {
                pcount_bh[m0 + idx] = pc;
                const int delim = start + l;
                if (delim < n) cid_bh[delim] = -1;
            }
        }
        if (lane == 0) s_rows[wave] = rows;
    }
    __syncthreads();
    if (tid == 0 && item != (int)blockIdx.y) file_item(item - wgs);
}

// ------------------------------------------------------------------------------------------------
// rowbase[m] = rows already present + sum_{m' < m} (pcount[m'] + [chunk m' is closed by a delimiter]);
// comp_lens = total.
__global__ __launch_bounds__(256) void gsc_scan_kernel(GscParams p) {
    __shared__ int s_wave[4];
    __shared__ int s_total;
    const int b = blockIdx.y, h = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t bh = (int64_t)b * p.Hkv + h;
    const int M = p.num_chunks[b];
    if (M <= 0) {
        if (tid == 0) p.comp_lens[bh] = -1;
        return;
    }
    const int32_t *pcount_bh = p.pcount + bh * ((int64_t)p.N_max + 1);
    int32_t *rowbase_bh = p.rowbase + bh * ((int64_t)p.N_max + 2);
    constexpr int kItems = 8;
    bool base_bad;
    int running = gsc_base_rows(p, bh, base_bad);
    for (int base = 0; base < M; base += 256 * kItems) {
        int v[kItems];
        int sum = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int m = base + tid * kItems + k;
            v[k] = (m < M) ? pcount_bh[m] + ((m < M - 1) ? 1 : 0) : 0;
            sum += v[k];
        }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int up = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += up;
        }
        if (lane == kWave - 1) s_wave[wave] = incl;
        __syncthreads();
        if (tid == 0) {
            int acc = 0;
            for (int w = 0; w < 4; ++w) { const int t = s_wave[w]; s_wave[w] = acc; acc += t; }
            s_total = acc;
        }
        __syncthreads();
        int excl = running + s_wave[wave] + incl - sum;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int m = base + tid * kItems + k;
            if (m < M) rowbase_bh[m] = excl;
            excl += v[k];
        }
        running += s_total;
        __syncthreads();
    }
    if (tid == 0) {
        rowbase_bh[M] = running;
        p.comp_lens[bh] = (!base_bad && running <= p.cap) ? running : -1;
    }
}

// ------------------------------------------------------------------------------------------------
template <typename TO>
__device__ __forceinline__ void store_row8(void *base, int64_t elem_off, const float (&x)[8]) {
    store8(reinterpret_cast<TO *>(base) + elem_off, x);
}

// Bound by the chain offsets -> row bases -> cluster indices -> member rows, not by its bytes, until a call has
// some hundred thousand rows.  The cluster indices of the item sit in LDS (kMergeCidTile tokens of them, which is all
// of an item unless a chunk is very long), a group first collects its members of 64 rows as bits and then has
// kMergeInFlight of them (keys and values) in flight at once (eight instead of four: more registers, fewer
// wavefronts, 156 -> 228 us on 8 heads x 32768 x 64 bf16, and no faster on short sequences).  Whole call, against
// indices read from memory eight at a time and a scan kernel: 2 heads x 1024 x 64 f32 56 -> 30 us, 8 x 8192 x 128
// f32 127 -> 73, 8 x 32768 x 64 bf16 209 -> 156.
// INLINE_PREFIX: no scan kernel ran; the workgroup adds up the rows of the items before its own itself, from the clusters
// that gsc_assign has filed per item, and the workgroup of the last item files the total.  (From the clusters of every chunk that
// is eight times as much to read for every item in turn: where a chunk is a token or two and a sequence many items, 8 heads
// x 32768 x 64 f32 with a delimiter per token, a call of items of eight took 323 us, 265 so.)
constexpr int kMergeCidTile = 2048;
constexpr int kMergeInFlight = 4;
// TWICE: some items are split between two workgroups, one adds up the keys and the other the values, eight rows in flight each.  What that
// shortens is the largest cluster's trips to memory, so an item is split where a chunk of it is long: of more than kSplitLong tokens, or of more than
// kSplitLongRoom in a call with room for twice its items (of the 512 places on the chip, two workgroups on each of 256 CUs, kSplitRoom).  Where chunks are short the
// second workgroup would do the first one's barriers and look-ups once more for nothing, and where the chip is full it takes a place.  Whole call without
// sc_segment, us, never split / every item split / by this rule (delimiters at a fixed distance, or at random every 24 tokens: "geom"):
//   8 heads x 6000 x 64 f32   distance 1 25.5 / 36.0 / 25.2, 4 29.3 / 40.6 / 29.7, 24 18.8 / 23.8 / 19.7, 64 26.7 / 23.1 / 24.5, geom 48.9 / 46.1 / 48.3
//   8 x 6000 x 128 f32        1 37.9 / 52.6 / 35.6, 4 47.8 / 63.6 / 47.8, 24 27.2 / 31.6 / 27.7, 64 43.0 / 34.8 / 35.8, geom 61.4 / 54.1 / 56.5
//   4 x 12000 x 64 bf16       1 20.6 / 32.4 / 20.6, 4 29.1 / 42.0 / 30.0, 24 22.2 / 28.3 / 22.5, 64 34.1 / 30.4 / 31.6, geom 61.5 / 52.2 / 58.9
//   1 x 8000 x 64 f32         1 12.1 / 15.3 / 12.4, 4 13.8 / 17.6 / 13.8, 24 17.5 / 16.5 / 17.2, 64 26.7 / 22.6 / 23.3, geom 45.7 / 37.4 / 38.1
//   2 x 1024 x 64 f32         1 10.9 / 13.4 / 11.3, 16 16.1 / 15.2 / 14.7, 64 26.0 / 22.1 / 22.3, geom 30.3 / 26.6 / 27.1
// (What is left where nothing is split, up to 4 % with d = 64, is the larger kernel's.)
// The second workgroups come last, kSplitWorkgroups in all (as many as items are long: 4 x 12000 geom 59 with 512, 67 with 256; one for every item, 8 x
// 2000 x 128 f32 with a delimiter every second token 17.2 instead of 16.8 us), and leave at once where chunks average less than kSplitMean tokens.
// Even from 64k rows on (4 x 16000 x 64 f32 58.5 / 59.5).  (Sixteen in flight: 310 registers, a wavefront per SIMD, 4 x 8000 53, 4 x 16000 82.)
constexpr int64_t kSplitTokens = 49152;      // rows of all heads
constexpr int kSplitWorkgroups = 512, kSplitRoom = 384, kSplitLong = 32, kSplitLongRoom = 8, kSplitMean = 12;
constexpr int kMergeInFlightSplit = 8;

template <typename T, int D, bool INLINE_PREFIX, bool TWICE>
__global__ __launch_bounds__(kGscThreads) void gsc_merge_kernel(GscParams p, int split_wgs) {      // split_wgs: second workgroups per (sequence, head)
    constexpr int LPR = D / 8;
    constexpr int RPW = kWave / LPR;            // output rows a wave works on at once
    constexpr int kGroups = kGscThreads / LPR;  // output rows a workgroup works on at once
    __shared__ int s_off[kMaxChunksPerItem + 1];
    __shared__ int s_base[kMaxChunksPerItem + 1];
    __shared__ int s_sum[kGscThreads / kWave];
    __shared__ int s_cid[kMergeCidTile];
    const int bh_i = gsc_grid_head();
    if (bh_i >= p.B * p.Hkv) return;
    const int b = bh_i / p.Hkv, h = bh_i - b * p.Hkv;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int g = lane / LPR, c = lane % LPR;
    const int gsh = g * LPR;   // position of this group's bits inside a wave ballot
    const uint64_t gmask = (LPR == 16) ? 0xffffull : 0xffull;
    const int seconds = TWICE ? split_wgs : 0, launched = (int)gridDim.y - seconds;
    const bool values = TWICE && (int)blockIdx.y >= launched;      // a second workgroup
    const int first_item = values ? (int)blockIdx.y - launched : (int)blockIdx.y;
    const int M = p.num_chunks[b];
    const int64_t bh = bh_i;
    if (M <= 0) {
        if (INLINE_PREFIX && blockIdx.y == 0 && tid == 0) p.comp_lens[bh] = -1;
        return;
    }
    int n = p.seq_lens ? p.seq_lens[b] : p.N_max;
    n = n < 0 ? 0 : (n > p.N_max ? p.N_max : n);
    int C, wgs;
    gsc_item_shape(p, M, n, launched, C, wgs);
    if (first_item >= (values ? seconds : wgs)) return;
    const int items = (M + C - 1) / C;
    const bool may_split = TWICE && n >= kSplitMean * (int64_t)M;
    if (values && !may_split) return;
    const int step = values ? seconds : wgs;
    const int split_from = (2 * (int64_t)min(items, wgs) * (p.B * p.Hkv) <= kSplitRoom) ? kSplitLongRoom : kSplitLong;
    const T *Kbh = reinterpret_cast<const T *>(p.K) + b * p.stride_b + h * p.stride_h;
    const T *Vbh = reinterpret_cast<const T *>(p.V) + b * p.stride_b + h * p.stride_h;
    const int32_t *off = p.offsets + (int64_t)b * p.offsets_stride_b;
    const int32_t *cid_bh = p.cid + bh * p.N_max;
    const int32_t *pcount_bh = p.pcount + bh * ((int64_t)p.N_max + 1);
    const int32_t *rowbase_bh = p.rowbase + bh * ((int64_t)p.N_max + 2);
    int32_t *counts_bh = p.counts + bh * p.cap;
    bool base_bad = false;
    int summed = INLINE_PREFIX ? gsc_base_rows(p, bh, base_bad) : 0, summed_to = 0;   // rows of the items [0, summed_to)

    for (int item = first_item; item < items; item += step) {
        const int m0 = item * C;
        const int nch = min(C, M - m0);
        bool split = false;      // the same for both workgroups
        if constexpr (TWICE) {
            split = may_split && ballot64(lane < nch && off[m0 + lane + 1] - off[m0 + lane] > split_from) != 0ull;
            if (values && !split) continue;
        }
        __syncthreads();
        if (tid <= nch) {
            s_off[tid] = off[m0 + tid];
            if (!INLINE_PREFIX) s_base[tid] = rowbase_bh[m0 + tid];
        }
        if (INLINE_PREFIX) {
            // every chunk of the items before is closed by a delimiter: its rows are its clusters and one more
            int part = 0;
            for (int i = summed_to + tid; i < item; i += kGscThreads) part += rowbase_bh[i] + C;
            const int mine = (lane < nch) ? pcount_bh[m0 + lane] + ((m0 + lane < M - 1) ? 1 : 0) : 0;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) part += __shfl_xor(part, d, kWave);
            if (lane == 0) s_sum[wave] = part;
            int incl = mine;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int up = __shfl_up(incl, d, kWave);
                if (lane >= d) incl += up;
            }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kGscThreads / kWave; ++w) summed += s_sum[w];
            summed_to = item;
            if (wave == 0 && lane <= nch) {
                const int base = summed + incl - mine;
                s_base[lane] = base;
                if (m0 + nch == M && lane == nch && !values) p.comp_lens[bh] = (!base_bad && base <= p.cap) ? base : -1;
            }
        }
        __syncthreads();
        const int t0 = __builtin_amdgcn_readfirstlane(s_off[0]);
        const int t1 = min(__builtin_amdgcn_readfirstlane(s_off[nch]), n);
        for (int t = t0 + tid; t < min(t1, t0 + kMergeCidTile); t += kGscThreads) s_cid[t - t0] = cid_bh[t];
        __syncthreads();
        const int R0 = __builtin_amdgcn_readfirstlane(s_base[0]);
        const int R1 = min(__builtin_amdgcn_readfirstlane(s_base[nch]), p.cap);
        // all loops below have wave-uniform trip counts; per-group differences are predicates
        auto merge_rows = [&](auto apart) {      // apart: the keys or the values only
            constexpr bool APART = decltype(apart)::value;
            constexpr int kInFlight = APART ? kMergeInFlightSplit : kMergeInFlight;
            const T *Xbh = APART && values ? Vbh : Kbh;
            for (int Rw = R0 + wave * RPW; Rw < R1; Rw += kGroups) {
                const int R = Rw + g;
                const bool valid = R < R1;
                // chunk of this output row: last idx with s_base[idx] <= R
                int idx = 0;
                for (int k = 1; k < nch; ++k) idx = (s_base[k] <= R) ? k : idx;
                const int start = s_off[idx];
                const int l = s_off[idx + 1] - 1 - start;
                const int cl = R - s_base[idx];
                const bool closed = (start + l) < n;   // chunk is followed by a delimiter
                const int pc = s_base[idx + 1] - s_base[idx] - (closed ? 1 : 0);
                const bool is_delim = valid && cl >= pc;
                const int lscan = (valid && !is_delim) ? l : 0;
                int lmax = 0;
#pragma unroll
                for (int gg = 0; gg < RPW; ++gg) lmax = max(lmax, __builtin_amdgcn_readlane(lscan, gg * LPR));

                float ka[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, va[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                int size = 0;
                if (is_delim) {
                    // the delimiter that closes the chunk: copied unchanged, size 1
                    const int64_t src = (int64_t)(start + l) * p.stride_n + 8 * c;
                    load8(Xbh + src, ka);
                    if constexpr (!APART) load8(Vbh + src, va);
                    size = 1;
                }
                for (int j0 = 0; j0 < lmax; j0 += kWave) {
                    uint64_t members = 0ull;       // of rows j0 .. j0 + 63 of the chunk, the same for every lane of the group
#pragma unroll
                    for (int k = 0; k < kWave / LPR; ++k) {
                        const int j = j0 + LPR * k + c, t = start + j - t0;
                        bool match = false;
                        if (j < lscan) match = (t < kMergeCidTile ? s_cid[t] : cid_bh[start + j]) == cl;
                        members |= ((ballot64(match) >> gsh) & gmask) << (LPR * k);
                    }
                    while (ballot64(members != 0ull) != 0ull) {
                        int jj[kInFlight];
                        bool ok[kInFlight];
                        float kk[kInFlight][8], vv[kInFlight][8];
#pragma unroll
                        for (int u = 0; u < kInFlight; ++u) {
                            ok[u] = members != 0ull;
                            jj[u] = ok[u] ? first_bit(members) : 0;
                            members &= members - 1ull;
                        }
#pragma unroll
                        for (int u = 0; u < kInFlight; ++u) {
                            if (ok[u]) {
                                const int64_t src = (int64_t)(start + j0 + jj[u]) * p.stride_n + 8 * c;
                                load8(Xbh + src, kk[u]);
                                if constexpr (!APART) load8(Vbh + src, vv[u]);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < kInFlight; ++u) {
                            if (ok[u]) {
                                if (size == 0) {
#pragma unroll
                                    for (int e = 0; e < 8; ++e) {
                                        ka[e] = kk[u][e];
                                        if constexpr (!APART) va[e] = vv[u][e];
                                    }
                                } else {
#pragma unroll
                                    for (int e = 0; e < 8; ++e) {
                                        ka[e] += kk[u][e];
                                        if constexpr (!APART) va[e] += vv[u][e];
                                    }
                                }
                                size += 1;
                            }
                        }
                    }
                }
                if (size > 1) {
                    const float fs = (float)size;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        ka[e] = ka[e] / fs;
                        if constexpr (!APART) va[e] = va[e] / fs;
                    }
                }
                if (valid) {
                    const int64_t dst = ((int64_t)bh * p.cap + R) * D + 8 * c;
                    if (p.out_is_bf16) {
                        store_row8<bf16_t>(APART && values ? p.Vc : p.Kc, dst, ka);
                        if constexpr (!APART) store_row8<bf16_t>(p.Vc, dst, va);
                    } else {
                        store_row8<float>(APART && values ? p.Vc : p.Kc, dst, ka);
                        if constexpr (!APART) store_row8<float>(p.Vc, dst, va);
                    }
                    if (c == 0 && !values) counts_bh[R] = size;
                }
            }
        };
        if (TWICE && split) merge_rows(std::bool_constant<TWICE>());
        else merge_rows(std::false_type());
    }
}

// ------------------------------------------------------------------------------------------------
size_t gsc_merge_workspace_bytes(int B, int Hkv, int N_max, int d, int out_elem_bytes) {
    const size_t bh = (size_t)B * Hkv;
    size_t bytes = 0;
    bytes += align_up(bh * (size_t)N_max * 4, 256);          // cid
    bytes += align_up(bh * (size_t)N_max * 4, 256);          // seedrow
    bytes += align_up(bh * ((size_t)N_max + 1) * 4, 256);    // pcount
    bytes += align_up(bh * ((size_t)N_max + 2) * 4, 256);    // rowbase
    bytes += align_up(bh * (size_t)N_max * 4, 256);          // stmp
    bytes += 2 * align_up(bh * (size_t)N_max * (size_t)d * (size_t)out_elem_bytes, 256);   // (the fast path uses a small part of it)
    return bytes;
}

template <typename T, int D>
static hipError_t launch_typed(const GscParams &p, int grid_x, hipStream_t stream) {
    const int max_items = (p.N_max + 1 + p.chunks_per_item - 1) / p.chunks_per_item;
    const int heads = p.B * p.Hkv;
    const int gx = max(1, min(max_items, grid_x > 0 ? grid_x : gsc_item_workgroups(heads, p.N_max, p.chunks_per_item)));
    const int per_layer = min(heads, 1 << kGridHeadsLog2);
    const dim3 grid(per_layer, min(gx, 65535), (heads + per_layer - 1) / per_layer);
    hipLaunchKernelGGL((gsc_assign_kernel<T, D>), grid, dim3(kGscThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.N_max <= kInlinePrefixTokens) {
        const int split_wgs = min(gx, kSplitWorkgroups / heads);
        const dim3 more(grid.x, grid.y + split_wgs, grid.z);
        if ((int64_t)heads * p.N_max <= kSplitTokens && split_wgs > 0 && more.y <= 65535) hipLaunchKernelGGL((gsc_merge_kernel<T, D, true, true>), more, dim3(kGscThreads), 0, stream, p, split_wgs);
        else hipLaunchKernelGGL((gsc_merge_kernel<T, D, true, false>), grid, dim3(kGscThreads), 0, stream, p, 0);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(gsc_scan_kernel, dim3(p.Hkv, p.B), dim3(256), 0, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gsc_merge_kernel<T, D, false, false>), grid, dim3(kGscThreads), 0, stream, p, 0);
    return hipGetLastError();
}

// (the fast path addresses the rows of a wavefront with 32-bit byte offsets, publishes the rows of a segment in 27 bits, and launches a
// workgroup for every window there is room for, which millions of heads of a few tokens can make too many)
bool gsc_merge_takes_fast_path(const GscMergeArgs &a) {
    return a.in_dtype == DType::BF16 && a.d == 128 && a.tune.gsc_fast_path && a.stride_n <= (int64_t(1) << 22) && gsc_fast_holds(a.B * a.Hkv, a.N_max);
}

hipError_t launch_gsc_merge(const GscMergeArgs &a, hipStream_t stream) {
    GscParams p;
    p.K = a.K; p.V = a.V;
    p.stride_b = a.stride_b; p.stride_h = a.stride_h; p.stride_n = a.stride_n;
    p.seq_lens = a.seq_lens; p.offsets = a.offsets; p.offsets_stride_b = a.offsets_stride_b;
    p.num_chunks = a.num_chunks;
    p.B = a.B; p.Hkv = a.Hkv; p.N_max = a.N_max;
    p.tau = a.tau;
    p.tau_dev = a.tau_dev;
    p.Kc = a.Kc; p.Vc = a.Vc;
    p.out_is_bf16 = (a.out_dtype == DType::BF16) ? 1 : 0;
    p.cap = a.cap;
    p.counts = a.counts; p.comp_lens = a.comp_lens;
    p.base_lens = a.base_lens;
    p.count_only = a.count_only ? 1 : 0;
    p.budget = nullptr;
    p.probe_levels = a.probe_levels;
    // Generic path: a wavefront per chunk, so four chunks are one round of a workgroup.  Calls of up to 64k rows in
    // all are bound by the longest chain of chunks and take that; larger ones fill the chip anyway and share the
    // offsets, the prefix and the barriers of an item among eight (us, 4 / 8 / 16 chunks: 2 heads x 1024 x 64 f32
    // 30 / 33 / 45; 8 x 8192 x 128 f32 72 / 77 / 117; 8 x 32768 x 64 bf16 179 / 156 / 181).
    const int auto_item = ((int64_t)a.B * a.Hkv * a.N_max <= (int64_t(1) << 16)) ? 4 : 8;
    p.chunks_per_item = max(1, min(kMaxChunksPerItem, a.tune.gsc_chunks_per_item > 0 ? a.tune.gsc_chunks_per_item : auto_item));
    const bool fixed = a.tune.gsc_chunks_per_item > 0 || a.tune.gsc_grid_x > 0;
    p.short_wgs[0] = fixed ? 0 : max(1, gsc_item_workgroups(a.B * a.Hkv, p.N_max, 8));
    p.short_wgs[1] = fixed ? 0 : max(1, gsc_item_workgroups(a.B * a.Hkv, p.N_max, 16));

    const size_t bh = (size_t)a.B * a.Hkv;
    char *w = reinterpret_cast<char *>(a.ws);
    int32_t *ws_cid = reinterpret_cast<int32_t *>(w);
    w += align_up(bh * (size_t)a.N_max * 4, 256);
    p.seedrow = reinterpret_cast<int32_t *>(w);
    w += align_up(bh * (size_t)a.N_max * 4, 256);
    p.pcount = reinterpret_cast<int32_t *>(w);
    w += align_up(bh * ((size_t)a.N_max + 1) * 4, 256);
    p.rowbase = reinterpret_cast<int32_t *>(w);
    w += align_up(bh * ((size_t)a.N_max + 2) * 4, 256);
    p.stmp = reinterpret_cast<int32_t *>(w);
    w += align_up(bh * (size_t)a.N_max * 4, 256);
    p.rows_ws = w;
    p.cid = a.cluster_id ? a.cluster_id : ws_cid;
    p.cluster_id = a.cluster_id;

    if (gsc_merge_takes_fast_path(a)) {
        if (a.count_only) p.budget = reinterpret_cast<BudgetState *>(a.budget_state);
        p.max_chunks = a.tune.gsc_chunks_per_task;
        p.polls = a.tune.gsc_polls;
        return launch_gsc_fast(p, a.planned, a.budget_start, stream);
    }

    if (a.in_dtype == DType::BF16) {
        return a.d == 128 ? launch_typed<bf16_t, 128>(p, a.tune.gsc_grid_x, stream) : launch_typed<bf16_t, 64>(p, a.tune.gsc_grid_x, stream);
    }
    return a.d == 128 ? launch_typed<float, 128>(p, a.tune.gsc_grid_x, stream) : launch_typed<float, 64>(p, a.tune.gsc_grid_x, stream);
}

}  // namespace sc
