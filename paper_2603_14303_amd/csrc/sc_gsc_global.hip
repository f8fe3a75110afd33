// sc_gsc_merge_global: Alg. 1 / Eq. 2 and Eq. 3 (paper Sec. 2.3, 2.4) when the whole sequence of a
// (sequence, KV head) is ONE chunk -- the "no chunking" variant of the paper's chunking ablation
// (Sec. 3.4) -- for bf16 keys/values with head dim 128 and up to 32768 tokens.
//
// Alg. 1 over one chunk of n rows is sequential in its seeds (a row is a seed iff no earlier seed takes
// it; a row joins the EARLIEST seed it resembles) but every similarity it can ask for is known in
// advance, so the work is split into a dense part and a sparse one:
//   norms    reciprocal norms of all rows.
//   pairs    pairwise comparisons "Sim(i, j) > tau" on the matrix cores
//            (v_mfma_f32_16x16x32_bf16, 64 x 64 rows per product block): one 64-bit word per (row j,
//            block of 64 earlier rows), "surely above" and "inside the +-1e-4 band" (decided later in
//            fp64).  Only blocks that hold such a pair are written; a bit per block says which.
//   decide   which rows are seeds and which seed every row joins, all blocks of 64 rows at once.
//   rank, slots, place   number the clusters and their members in row order (one kernel where a sequence has few rows).
//   sum      one 16-lane group per cluster adds up its members' keys and values in row order (fp32),
//            scales by 1/size and writes the output row: Eq. 3.
// A row needs comparing with SEEDS only, and one row in six is one where merging pays.  Long sequences are therefore taken in stages of 4096 rows
// or a multiple: all pairs inside the stages (one launch), then stage by stage the rows of a stage against the seeds of the stages before, listed without
// gaps, and the decisions of the stage.  8 heads x 32768 tokens, us per call of all pairs and of four stages of 8192 rows: tau 0.7 900 and 555, tau 0.9745
// 908 and 664; where every row is a seed 957 and 1135 (see glob_stage_words).
// Everything else (other element types, head dims, longer sequences) is handed to the ordinary kernels
// of sc_gsc_merge with offsets that describe one chunk per sequence.
#include "sc_device.h"
#include "sc_gsc_params.h"
#include "sc_host.h"

#include <mutex>

namespace sc {

typedef float gl_float4 __attribute__((ext_vector_type(4)));
typedef unsigned int gl_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 gl_bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kGlD = 128;
constexpr int kGlBlock = 64;                    // rows per block
constexpr int kGlTileRowBytes = 272;            // 256 B of keys + 16 B pad: conflict-free operand reads
constexpr int kGlPairWaves = 4;                 // row blocks per workgroup of the pairs kernel
constexpr int kGlSeedUnit = 8, kGlSeedShare = 4;   // with listed seeds: column blocks a work item is rounded up to; work items for a list of one row in so many
constexpr int kGlWordBlocks = 64;               // column blocks per word of tile flags; stages are multiples of this
constexpr int kGlLeader = 1 << 16;              // place of the first row of a cluster in a block

struct GlobParams {
    const bf16_t *K, *V;
    int64_t stride_b, stride_h, stride_n;
    const int32_t *seq_lens;
    int B, Hkv, N_max;
    float tau;
    void *Kc, *Vc;
    int out_is_bf16;
    int cap;
    int32_t *counts, *comp_lens, *cluster_id;
    // workspace, per (sequence, head)
    int nbp;                      // blocks of the longest possible sequence
    long long tri;                // words of one bit array: 64 * nbp * (nbp + 1) / 2
    float *rinv;                  // [nbp * 64]
    unsigned long long *Y, *U;    // [tri]: column block I holds the words of rows 64 I .. 64 nbp - 1
    int nseg;                     // words of a row of tile flags: one per 64 column blocks
    unsigned long long *tany, *tuns;   // [nbp][nseg]: bit I of row J: block (J, I) has any bit set / any unsure bit; Y and U are only written (and read) where it has
    unsigned long long *state;    // [2 nbp]: per 32 rows, low half: decided, high half: is a seed
    int32_t *join;                // [npad]: the seed row that a row belongs to (a seed: itself)
    int32_t *place;               // [npad]: place inside the own block's rows of the cluster, see glob_decide_block
    int32_t *lead, *order;        // [npad]
    int polls;                    // looks at another block's rows before the ordered pass takes over
    int32_t *mbase, *csize;       // [nbp * 64 + 1], the last one: slots given out; [nbp * 64]
    int32_t *nclusters;           // [1]; before the rank kernel: blocks whose wavefronts are through
    int walk;                     // column blocks per work item of the pairs kernel: 8, 16 or 32
    int stage_words, stages, stage;      // words of tile flags of a stage (the last one has the rest); how many; the stage of this launch
    int32_t *seedlist;            // [npad]: the seeds of the stages before, in row order (the memory of `order`)
};
__device__ __forceinline__ int gl_stage_blocks(const GlobParams &p) { return p.stage_words * kGlWordBlocks; }
__device__ __forceinline__ int gl_stage_start(const GlobParams &p, int J) { return min(J / gl_stage_blocks(p), p.stages - 1) * gl_stage_blocks(p); }      // first block of block J's stage

__device__ __forceinline__ long long gl_col_base(int I, int nbp) {   // first word of column block I
    return 64ll * ((long long)I * nbp - (long long)I * (I - 1) / 2);
}
__device__ __forceinline__ uint64_t gl_bits_below(int x) {   // bits [0, x), 0 <= x <= 64
    const uint32_t l = (x >= 32) ? 0xFFFFFFFFu : ((1u << x) - 1u);
    const uint32_t h = (x <= 32) ? 0u : ((x >= 64) ? 0xFFFFFFFFu : ((1u << (x - 32)) - 1u));
    return ((uint64_t)h << 32) | l;
}
__device__ __forceinline__ uint32_t gl_or_rows(uint32_t x) {   // OR over the four 16-lane rows, same lane position
    auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = r[0] | r[1];
    r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return r[0] | r[1];
}
// Eq. 2 in double precision by a whole wavefront (NaN compares false: a zero row resembles nothing)
__device__ __forceinline__ bool gl_cosine_exceeds_f64(const bf16_t *a_row, const bf16_t *b_row, float tau, int lane) {
    double dot = 0.0, aa = 0.0, bb = 0.0;
#pragma unroll
    for (int k = 0; k < kGlD / kWave; ++k) {
        const int e = lane + k * kWave;
        const double a = load1_f64(a_row + e), b = load1_f64(b_row + e);
        dot += a * b; aa += a * a; bb += b * b;
    }
    dot = wave_allreduce_sum(dot);
    aa = wave_allreduce_sum(aa);
    bb = wave_allreduce_sum(bb);
    return dot / (sqrt(aa) * sqrt(bb)) > (double)tau;
}
__device__ __forceinline__ int gl_seq_len(const GlobParams &p, int b) {
    int n = p.seq_lens ? p.seq_lens[b] : p.N_max;
    return n < 0 ? 0 : (n > p.N_max ? p.N_max : n);
}

// ------------------------------------------------------------------------------------------------
// norms: rinv[j] = 1 / |k_j| in fp32 (not a number for rows that do not exist or have an unusable norm:
// every comparison with such a row then lands in the band and is decided in fp64)
__global__ __launch_bounds__(256) void glob_norms_kernel(GlobParams p) {
    const int bh = blockIdx.y, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = gl_seq_len(p, b);
    const int row = blockIdx.x * 16 + threadIdx.x / 16, c = threadIdx.x % 16;
    if (row >= p.nbp * 64) return;
    float nsq = 0.f;
    if (row < n) {
        float x[8];
        load8(p.K + b * p.stride_b + h * p.stride_h + (int64_t)row * p.stride_n + 8 * c, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) nsq = fmaf(x[e], x[e], nsq);
    }
    nsq = row_allreduce_sum<16>(nsq);
    if (row == 0 && c == 0) p.nclusters[bh] = p.mbase[(int64_t)bh * (p.nbp * 64 + 1) + p.nbp * 64] = 0;
    if (c == 0 && (row & 31) == 0) p.state[(int64_t)bh * p.nbp * 2 + row / 32] = 0ull;      // nothing decided yet
    if (c == 0)
        p.rinv[(int64_t)bh * p.nbp * 64 + row] = (row < n && nsq > 1e-30f && nsq < 1e30f) ? __frsqrt_rn(nsq) : __builtin_nanf("");
}

// ------------------------------------------------------------------------------------------------
// pairs: a workgroup owns the row blocks J = 4 JG + wave and walks p.walk of their stage's column blocks up to their own, or (SEEDS) its share of the seeds
// of the stages before, 64 of the list to a column block.
// The rows of block J are the B operand and stay in registers (lane (g, c): row 16 Jt + c, elements
// 32 ks + 8 g .. + 7 -- v_mfma_f32_16x16x32_bf16, the form that runs at the full bf16 rate of this chip);
// the rows of block I pass through an LDS tile shared by the four wavefronts and are the A operand.  The
// product tile leaves lane (g, c) with the dot products of row 16 Jt + c of block J and rows
// 16 It + 4 g + i of block I: four bits of that row's word, completed by an OR over the lane groups.
// Bound by the matrix cores and the threshold step beside them.  Two quarters of a tile in registers at a time, so that three workgroups share a
// compute unit: 8 heads x 32768 rows 606 us a call with all four and two workgroups, 576 so.  A quarter with a pair that comes near is formed again; those of
// a block's own rows, which all have one, are formed that way only (8 x 300 44 us a call with both, 40 so; x 1000 55 and 49).
template <bool SEEDS>
__global__ __launch_bounds__(kGlPairWaves *kWave, 3) void glob_pairs_kernel(GlobParams p) {
    constexpr int kListTiles = kGlSeedUnit * kGlSeedShare;
    __shared__ __attribute__((aligned(16))) char s_tiles[2][kGlBlock * kGlTileRowBytes];      // two tiles: one worked on, one being filled
    __shared__ __attribute__((aligned(16))) float s_rinvs[2][kGlBlock];
    __shared__ int s_odd[2];      // a row of the tile has no usable norm
    [[maybe_unused]] __shared__ unsigned short s_list[SEEDS ? kListTiles * kGlBlock : 1];      // rows of the seeds (n <= 32768)
    [[maybe_unused]] __shared__ int s_part[kGlPairWaves];
    const int bh = (int)blockIdx.x % (p.B * p.Hkv), b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = gl_seq_len(p, b);
    const int nb = (n + kGlBlock - 1) / kGlBlock;
    const int njg = (nb + kGlPairWaves - 1) / kGlPairWaves;
    // Work item = (group JG of four row blocks, segment of p.walk column blocks): short walks of about the same length, so that the
    // triangle of one stage fills the chip.  Within a stage, groups per_seg q .. per_seg (q + 1) - 1 have q + 1 segments each, so
    // per_seg q (q + 1) / 2 items come before them.  With the seeds of the stages before: an equal share of the list for each of `walks` items, as
    // many as give them a unit of eight column blocks if one row in four is a seed.
    const int stage_blocks = gl_stage_blocks(p), x = (int)blockIdx.x / (p.B * p.Hkv);
    [[maybe_unused]] const int walks = p.stage * stage_blocks / kListTiles;
    int JG, seg;
    if constexpr (SEEDS) {
        JG = p.stage * (stage_blocks / kGlPairWaves) + x / walks;
        seg = x % walks;
    } else {
        const int per_seg = p.walk / kGlPairWaves;      // groups of row blocks to a segment
        const int stage_segs = stage_blocks / p.walk, items = per_seg * stage_segs * (stage_segs + 1) / 2, st = min(x / items, p.stages - 1), y = x - st * items;
        int q = 0;
        while (per_seg * (q + 1) * (q + 2) / 2 <= y) ++q;
        const int rem = y - per_seg * q * (q + 1) / 2;
        JG = per_seg * (st * stage_segs + q) + rem / (q + 1);
        seg = st * stage_segs + rem % (q + 1);
    }
    if (JG >= njg) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int g = lane >> 4, c = lane & 15;
    const int J = JG * kGlPairWaves + wave;
    const bool active = J < nb;
    const bf16_t *Kbh = p.K + b * p.stride_b + h * p.stride_h;
    const float *rinv_bh = p.rinv + (int64_t)bh * p.nbp * 64;
    const int sb = (int)p.stride_n * 2;      // bytes between rows
    auto flags8 = [&](unsigned long long *words) { return reinterpret_cast<unsigned char *>(words + ((int64_t)bh * p.nbp + J) * p.nseg); };      // of 8 blocks
    int I_first, I_last;
    [[maybe_unused]] int ns = 0;      // seeds of this walk
    if constexpr (SEEDS) {
        const unsigned long long *st = p.state + (int64_t)bh * p.nbp * 2;
        const int J0 = p.stage * stage_blocks;
        uint64_t mask[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int I = 2 * tid + q;
            const unsigned long long w0 = I < J0 ? st[2 * I] : 0ull, w1 = I < J0 ? st[2 * I + 1] : 0ull;
            mask[q] = (w0 >> 32) | (w1 & 0xFFFFFFFF00000000ull);
        }
        const int mine = __popcll(mask[0]) + __popcll(mask[1]);
        int incl = mine;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += up;
        }
        if (lane == kWave - 1) s_part[wave] = incl;
        __syncthreads();
        int at = incl - mine, total = 0;
#pragma unroll
        for (int w = 0; w < kGlPairWaves; ++w) {
            if (w < wave) at += s_part[w];
            total += s_part[w];
        }
        // units of eight tiles: `units` hold seeds, `per` of them are this walk's; the flags of the others are cleared
        const int units = (total + kGlSeedUnit * kGlBlock - 1) / (kGlSeedUnit * kGlBlock), per = (units + walks - 1) / walks;      // per <= kGlSeedShare
        if (active)
            for (int q = units + seg + walks * lane; q < J0 / kGlSeedUnit; q += walks * kWave) flags8(p.tany)[q] = flags8(p.tuns)[q] = 0;
        const int first = seg * per * kGlSeedUnit * kGlBlock, most = per * kGlSeedUnit * kGlBlock;
        ns = min(total - first, most);
        if (ns <= 0) return;
        at -= first;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (at + 64 <= 0 || at >= most) { at += __popcll(mask[q]); continue; }
            for (uint64_t m = mask[q]; m != 0ull; m &= m - 1ull, ++at)
                if (at >= 0 && at < most) s_list[at] = (unsigned short)((2 * tid + q) * kGlBlock + first_bit(m));
        }
        __syncthreads();
        if (JG == p.stage * (stage_blocks / kGlPairWaves)) {      // for the rows that join one of them
            int32_t *list = p.seedlist + (int64_t)bh * p.nbp * kGlBlock + first;
            for (int i = tid; i < ns; i += kGlPairWaves * kWave) list[i] = s_list[i];
        }
        I_first = seg * per * kGlSeedUnit;
        I_last = I_first + (ns + kGlBlock - 1) / kGlBlock - 1;
    } else {
        I_first = seg * p.walk;
        I_last = min(min(JG * kGlPairWaves + kGlPairWaves - 1, nb - 1), I_first + p.walk - 1);
        if (I_first > I_last) return;
    }
    // rows of block J as B operands, through a descriptor that ends after the sequence's last row
    uint4 bq[4][4];
    float hn[4], wn[4], ln[4];
    bool bad_j = false;      // a row of block J without a usable norm (also: beyond the end of the sequence)
    {
        const int rows_j = active ? min(kGlBlock, n - J * kGlBlock) : 0;
        const auto src = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(Kbh + (int64_t)(active ? J : 0) * kGlBlock * p.stride_n),
                                                           (short)0, rows_j > 0 ? (rows_j - 1) * sb + kGlD * 2 : 0, 0x00020000);
#pragma unroll
        for (int Jt = 0; Jt < 4; ++Jt) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const gl_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(src, (16 * Jt + c) * sb + (32 * ks + 8 * g) * 2, 0, 0);
                bq[Jt][ks] = make_uint4(v.x, v.y, v.z, v.w);
            }
            const float rn = active ? rinv_bh[J * kGlBlock + 16 * Jt + c] : __builtin_nanf("");
            bad_j = bad_j || !(rn == rn);
            const float norm = __builtin_amdgcn_rcpf(rn);
            hn[Jt] = (p.tau + kBand) * norm;
            wn[Jt] = (2.0f * kBand) * norm;
            ln[Jt] = (p.tau - 1.1f * kBand) * norm;      // safely below everything that the band holds
        }
    }
    bad_j = ballot64(bad_j) != 0ull;
    // the tile of block I: thread t brings rows t / 16 + 16 r, piece t % 16
    const int lrow = tid >> 4, lc = tid & 15;
    uint4 pre[4];      // the next tile on its way
    float pre_r = 0.f;
    auto fetch = [&](int I) {
        if (I > I_last) return;
        if constexpr (SEEDS) {
            const int at = (I - I_first) * kGlBlock;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = at + lrow + 16 * r;
                pre[r] = k < ns ? *reinterpret_cast<const uint4 *>(Kbh + (int64_t)s_list[k] * p.stride_n + 8 * lc) : make_uint4(0u, 0u, 0u, 0u);
            }
            if (tid < kGlBlock) pre_r = at + tid < ns ? rinv_bh[s_list[at + tid]] : 0.f;
            return;
        }
        const int rows_i = min(kGlBlock, n - I * kGlBlock);
        const auto src = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(Kbh + (int64_t)I * kGlBlock * p.stride_n), (short)0,
                                                           rows_i > 0 ? (rows_i - 1) * sb + kGlD * 2 : 0, 0x00020000);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const gl_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(src, (lrow + 16 * r) * sb + 16 * lc, 0, 0);
            pre[r] = make_uint4(v.x, v.y, v.z, v.w);
        }
        if (tid < kGlBlock) pre_r = rinv_bh[I * kGlBlock + tid];
    };
    auto park = [&](int I) {
        if (I > I_last) return;
        char *t = s_tiles[I & 1];
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<uint4 *>(t + (lrow + 16 * r) * kGlTileRowBytes + 16 * lc) = pre[r];
        if (wave == 0) {
            s_rinvs[I & 1][lane] = pre_r;
            const bool odd = ballot64(!(pre_r == pre_r)) != 0ull;
            if (lane == 0) s_odd[I & 1] = odd ? 1 : 0;
        }
    };
    uint32_t any_bits = 0u, uns_bits = 0u;      // of this walk's column blocks
    auto work = [&](int I) {
        __syncthreads();          // tile I is complete; everybody is done with tile I - 1, whose buffer takes tile I + 1 now
        park(I + 1);
        fetch(I + 2);      // on its way while this tile is worked on
        const char *s_tile = s_tiles[I & 1];
        const float *s_rinv = s_rinvs[I & 1];
        if (!active || (!SEEDS && I > J)) return;    // wave-uniform
        const bool odd = bad_j || __builtin_amdgcn_readfirstlane(s_odd[I & 1]) != 0;
        uint32_t yl[4], yh[4], ul[4], uh[4];
#pragma unroll
        for (int Jt = 0; Jt < 4; ++Jt) yl[Jt] = yh[Jt] = ul[Jt] = uh[Jt] = 0u;
        // sim(m, n) > t  <=>  dot * rinv_m > t * norm_n.  Hardly any tile holds a pair that comes near: one multiply-add
        // and half a maximum per pair tell, for one quarter of the tile while the products of the next are formed.  A quarter that does is formed again.
        gl_float4 acc[2][4];
        float top[4];
        uint4 a[4];
        gl_float4 rm;
        auto operand = [&](int It, int ks) { return *reinterpret_cast<const uint4 *>(s_tile + (16 * It + c) * kGlTileRowBytes + (32 * ks + 8 * g) * 2); };
        auto product = [&](gl_float4 (&x)[4], const uint4 &rows, int ks) {
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt) {
                if (ks == 0) x[Jt] = gl_float4{0.f, 0.f, 0.f, 0.f};
                x[Jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(gl_bf16x8, rows), __builtin_bit_cast(gl_bf16x8, bq[Jt][ks]), x[Jt], 0, 0, 0);
            }
        };
        auto compare = [&](int It, int Jt) {
            if (Jt == 0) rm = *reinterpret_cast<const gl_float4 *>(s_rinv + 16 * It + 4 * g);
            const gl_float4 &x = acc[It & 1][Jt];
            const float t0 = fmaf(x[0], rm[0], -ln[Jt]), t1 = fmaf(x[1], rm[1], -ln[Jt]), t2 = fmaf(x[2], rm[2], -ln[Jt]), t3 = fmaf(x[3], rm[3], -ln[Jt]);
            top[It] = (Jt == 0) ? fmaxf(t0, t1) : fmaxf(fmaxf(top[It], t0), t1);
            top[It] = fmaxf(fmaxf(top[It], t2), t3);
        };
        int near = 15;      // quarters with a pair that comes near; a block's own rows make one of each (a row and itself), one way is enough for them
        if (!odd && (SEEDS || I != J)) {
#pragma unroll
            for (int step = 0; step < 3; ++step) a[step] = operand(step >> 2, step & 3);
#pragma unroll
            for (int step = 0; step < 16; ++step) {
                if (step + 3 < 16) a[(step + 3) & 3] = operand((step + 3) >> 2, (step + 3) & 3);
                product(acc[(step >> 2) & 1], a[step & 3], step & 3);
                if (step >= 4) compare((step >> 2) - 1, step & 3);
                __builtin_amdgcn_sched_barrier(0);      // the order of issue stays as written
            }
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt) compare(3, Jt);
            near = 0;
#pragma unroll
            for (int It = 0; It < 4; ++It) near |= ballot64(top[It] >= 0.f) != 0ull ? 1 << It : 0;
            if (near == 0) return;
        }
        for (int It = 0; It < 4; ++It) {
            if (((near >> It) & 1) == 0) continue;
            gl_float4 (&x)[4] = acc[0];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) product(x, operand(It, ks), ks);
            rm = *reinterpret_cast<const gl_float4 *>(s_rinv + 16 * It + 4 * g);
            // dd = (tau + band) * norm_n - dot * rinv_m is negative for a sure yes and at most 2 * band * norm_n inside the
            // band: the sign bit of dd is shifted into a nibble, an unsigned minimum over the bit patterns keeps the smallest
            // non-negative dd (negative values compare as huge).  Only if some lane saw a value inside the band, or a row
            // without a usable norm is involved, are the nibbles redone with real comparisons (anything that is not a number
            // is "inside the band" and never a sure yes).
            const int sh = 16 * (It & 1) + 4 * g;
            uint32_t yn[4];
            bool close = odd;
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt) {
                uint32_t nib = 0u, dmin = 0x7F800000u;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const uint32_t dd = __float_as_uint(fmaf(-x[Jt][i], rm[i], hn[Jt]));
                    nib = __builtin_amdgcn_alignbit(nib, dd, 31);      // (nib << 1) | sign bit
                    dmin = min(dmin, dd);
                }
                yn[Jt] = nib;
                close = close || dmin <= __float_as_uint(wn[Jt]);
            }
            if (ballot64(close) != 0ull) {
#pragma unroll
                for (int Jt = 0; Jt < 4; ++Jt) {
                    uint32_t y4 = 0u, u4 = 0u;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float dd = fmaf(-x[Jt][i], rm[i], hn[Jt]);
                        const bool yes = dd < 0.f;
                        const bool unsure = !yes && !(dd > wn[Jt]);
                        y4 |= yes ? (1u << i) : 0u;
                        u4 |= unsure ? (1u << i) : 0u;
                    }
                    yn[Jt] = y4;
                    if (It < 2) ul[Jt] |= u4 << sh; else uh[Jt] |= u4 << sh;
                }
            }
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt) {
                if (It < 2) yl[Jt] |= yn[Jt] << sh; else yh[Jt] |= yn[Jt] << sh;
            }
        }
        // complete the words over the four lane groups; lane 16 Jt + c keeps the words of row 16 Jt + c
        uint32_t myl = 0u, myh = 0u, mul = 0u, muh = 0u;
#pragma unroll
        for (int Jt = 0; Jt < 4; ++Jt) {
            const uint32_t a0 = gl_or_rows(yl[Jt]), a1 = gl_or_rows(yh[Jt]);
            const uint32_t b0 = gl_or_rows(ul[Jt]), b1 = gl_or_rows(uh[Jt]);
            if (g == Jt) { myl = a0; myh = a1; mul = b0; muh = b1; }
        }
        if (J * kGlBlock + lane >= n) myl = myh = mul = muh = 0u;      // no such row
        if constexpr (SEEDS) {      // no such seed
            const uint64_t there = gl_bits_below(min(kGlBlock, ns - (I - I_first) * kGlBlock));
            myl &= (uint32_t)there; mul &= (uint32_t)there;
            myh &= (uint32_t)(there >> 32); muh &= (uint32_t)(there >> 32);
        }
        const long long w = (long long)bh * p.tri + gl_col_base(I, p.nbp) + (long long)(J - I) * kGlBlock + lane;
        const bool any = ballot64((myl | myh | mul | muh) != 0u) != 0ull, any_u = ballot64((mul | muh) != 0u) != 0ull;
        if (any || (!SEEDS && I == J)) p.Y[w] = ((unsigned long long)myh << 32) | myl;      // a block's own words are always read
        if (any_u || (!SEEDS && I == J)) p.U[w] = ((unsigned long long)muh << 32) | mul;
        any_bits |= any ? 1u << (I - I_first) : 0u;
        uns_bits |= any_u ? 1u << (I - I_first) : 0u;
    };
    fetch(I_first);
    park(I_first);
    fetch(I_first + 1);
    for (int I = I_first; I <= I_last; ++I) work(I);
    if (active && lane < kListTiles / 8 && I_first + 8 * lane <= (SEEDS ? I_last : I_first + p.walk - 1)) {
        flags8(p.tany)[I_first / 8 + lane] = (unsigned char)(any_bits >> (8 * lane));
        flags8(p.tuns)[I_first / 8 + lane] = (unsigned char)(uns_bits >> (8 * lane));
    }
}

// ------------------------------------------------------------------------------------------------
// decide: one wavefront per row block J, lane r = row r, all blocks at once.
//
// A row joins the earliest SEED it resembles and is a seed if there is none, so what is known about a row only ever depends
// on earlier rows.  Each row looks at its candidates (set bits of its words) in row order: one that is decided and not a seed is
// passed over, one that is a seed takes the row (an unsure one after a comparison in fp64), one that is undecided is
// waited for.  What has been decided is published at once, 32 rows to a word (decided | seeds, so that one load gives a
// consistent view).  Rows whose candidates all lie in their own block are decided before anything is waited for:
// the members of a cluster mostly sit close together, so a block hardly ever waits for one that waits itself, and
// the rounds are a few microseconds for all blocks instead of 1.4 us for each of them in turn.
//
// Waiting is bounded (p.polls looks in all); blocks that are left undecided are finished in order by the last wavefront of the head.
// Blocks are dispatched in row order, so the ones waited for are running or done, and giving up never pays: with 4096 looks
// (2 ms) the last blocks of a long chain did (8 heads x 32768 rows that drift by 0.4, tau 0.8: 3.6 ms, 3.1 with patience), and all of
// them where many pairs need fp64 (2 heads x 2048 zero rows: 872 ms, 79 with patience).
struct GlobBlock {       // what a wavefront knows about its block
    uint64_t decided, seeds, published;
    int target;          // lane: seed row of the lane's row once decided
};

__device__ __forceinline__ uint64_t gl_uniform64(uint64_t x) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}
__device__ __forceinline__ void gl_load_state(const unsigned long long *st, int I, uint64_t &decided, uint64_t &seeds) {
    const uint64_t w0 = gl_uniform64(__hip_atomic_load(st + 2 * I, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const uint64_t w1 = gl_uniform64(__hip_atomic_load(st + 2 * I + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    decided = (w0 & 0xFFFFFFFFull) | (w1 << 32);
    seeds = (w0 >> 32) | (w1 & 0xFFFFFFFF00000000ull);
}
__device__ __forceinline__ void gl_publish(unsigned long long *st, int J, GlobBlock &k, int lane) {
    if (k.decided == k.published) return;
    if (lane == 0) __hip_atomic_store(st + 2 * J, (k.decided & 0xFFFFFFFFull) | (k.seeds << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane == 1) __hip_atomic_store(st + 2 * J + 1, (k.decided >> 32) | (k.seeds & 0xFFFFFFFF00000000ull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    k.published = k.decided;
}

// One candidate word (64 earlier rows from `first_row` on, or the rows of `list`; decided / seeds: what is known about them) for every lane with
// `open`: follows the candidates as far as they are known.  Lanes that find their seed join k.decided; returns the lanes that
// wait for an undecided row.  uw loses the bits that fp64 has turned down.
__device__ __forceinline__ uint64_t gl_follow(const GlobParams &p, const bf16_t *Kbh, uint64_t yw, uint64_t &uw, int first_row, const int32_t *list, uint64_t decided,
                                              uint64_t seeds, bool open, int j0, int lane, GlobBlock &k) {
    for (;;) {
        const bool undecided = open && ((k.decided >> lane) & 1ull) == 0ull;
        const uint64_t c = undecided ? (yw | uw) & ~(decided & ~seeds) : 0ull;
        const int f = (c != 0ull) ? first_bit(c) : 0;
        const bool known = c != 0ull && ((decided >> f) & 1ull) != 0ull;
        const bool sure = known && ((yw >> f) & 1ull) != 0ull;
        if (sure) k.target = list ? list[f] : first_row + f;
        k.decided |= ballot64(sure);
        uint64_t ask = ballot64(known && !sure);
        if (ask == 0ull) return ballot64(c != 0ull && !known);
        while (ask != 0ull) {
            const int r = __builtin_amdgcn_readfirstlane(first_bit(ask));
            ask &= ask - 1ull;
            const int fr = __builtin_amdgcn_readlane(f, r), row = list ? __builtin_amdgcn_readfirstlane(list[fr]) : first_row + fr;
            const bool ok = gl_cosine_exceeds_f64(Kbh + (int64_t)row * p.stride_n, Kbh + (int64_t)(j0 + r) * p.stride_n, p.tau, lane);
            if (ok) k.decided |= 1ull << r;
            if (lane == r) {
                if (ok) k.target = row;
                else uw &= ~(1ull << fr);
            }
        }
    }
}

// Alg. 1 among the rows of the block as far as it can be told: `cleared` rows have no seed in an earlier block.
// Every row without a candidate left becomes a seed, the rows that resemble one of these first join it: that is all where rows resemble
// few others.  Where each resembles its neighbours it would be one seed and its followers a round; the rows that are left are
// therefore taken in order, a few instructions for a seed and all that join it.  (Rows that drift, 8 heads x 4000, us per call: 0.2 of a
// new direction per row, tau 0.9, 490 in rounds, 410 so; 0.4 and 0.8 600 and 460.)
__device__ __forceinline__ void gl_own_block(const GlobParams &p, const bf16_t *Kbh, uint64_t y, uint64_t &u, uint64_t cleared, int j0, int lane, GlobBlock &k) {
    const bool open = ((cleared >> lane) & 1ull) != 0ull;
    for (;;) {
        const uint64_t before = k.decided;
        if ((cleared & ~before) == 0ull) return;
        gl_follow(p, Kbh, y, u, j0, nullptr, k.decided, k.seeds, open, j0, lane, k);
        auto candidates = [&]() { return (open && ((k.decided >> lane) & 1ull) == 0ull) ? (y | u) & ~(k.decided & ~k.seeds) : 0ull; };
        // no candidate left that is a seed or may become one: a seed itself
        const uint64_t more = ballot64(open && ((k.decided >> lane) & 1ull) == 0ull && candidates() == 0ull);
        if ((more >> lane) & 1ull) k.target = j0 + lane;
        k.seeds |= more;
        k.decided |= more;
        {
            const uint64_t c = candidates();
            const int f = (c != 0ull) ? first_bit(c) : 0;
            const bool joins = c != 0ull && ((k.seeds >> f) & 1ull) != 0ull && ((y >> f) & 1ull) != 0ull;
            if (joins) k.target = j0 + f;
            k.decided |= ballot64(joins);
        }
        // the rest in order, but for rows with a candidate that has just become known, or an unsure one: these are for the next round
        uint64_t ready = cleared & ~k.decided & ~ballot64((candidates() & (k.decided | u)) != 0ull);
        const uint64_t waited = ready;
        while (k.decided != ~0ull) {
            const uint64_t bit = 1ull << first_bit(~k.decided);      // none of its candidates is a seed: a seed itself
            if ((ready & bit) == 0ull) break;
            const uint64_t same = bit | (ballot64((y & bit) != 0ull) & ready);
            k.seeds |= bit;
            k.decided |= same;
            ready &= ~same;
        }
        if (((waited & ~ready) >> lane) & 1ull) k.target = j0 + (((k.seeds >> lane) & 1ull) ? lane : first_bit(y & k.seeds));
        if (k.decided == before) return;
    }
}

// Decides the rows of block J of one (sequence, head); false if it gave up waiting.
__device__ __forceinline__ bool glob_decide_block(const GlobParams &p, int bh, const bf16_t *Kbh, int n, int J, int lane, int polls) {
    const int npad = p.nbp * kGlBlock, j0 = J * kGlBlock;
    const bool valid = j0 + lane < n;
    const uint64_t all = ballot64(valid);
    const unsigned long long *Y = p.Y + (long long)bh * p.tri, *U = p.U + (long long)bh * p.tri;
    const unsigned long long *any_row = p.tany + ((int64_t)bh * p.nbp + J) * p.nseg, *uns_row = p.tuns + ((int64_t)bh * p.nbp + J) * p.nseg;
    unsigned long long *st = p.state + (int64_t)bh * p.nbp * 2;
    // words of tiles before the stage's first block are of 64 seeds each, whose rows are listed
    const int J0 = gl_stage_start(p, J);
    const int32_t *seedlist = p.seedlist + (int64_t)bh * npad;
    int32_t *join = p.join + (int64_t)bh * npad + j0, *place = p.place + (int64_t)bh * npad + j0;
    GlobBlock k;
    gl_load_state(st, J, k.decided, k.seeds);
    k.published = k.decided;
    k.target = ((k.decided >> lane) & 1ull) ? join[lane] : -1;
    const int segs = J >> 6;
    uint64_t y, u;
    {
        const long long w = gl_col_base(J, p.nbp) + lane;
        const uint64_t mine = valid ? gl_bits_below(lane) : 0ull;
        y = Y[w] & mine;
        u = U[w] & mine;
    }
    // the earlier blocks with a bit in any row, in order, up to kBatch at a time
    constexpr int kBatch = 4;
    int seg;
    uint64_t rest_any, rest_uns;
    auto rewind = [&](int s) {
        seg = s;
        rest_any = gl_uniform64(any_row[s]);
        rest_uns = gl_uniform64(uns_row[s]);
        if (s == segs) rest_any &= gl_bits_below(J & 63);      // without the block itself
    };
    int tile[kBatch];
    uint64_t yw[kBatch], uw[kBatch];
    auto next_batch = [&]() {
        int got = 0;
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            while (rest_any == 0ull && seg < segs) rewind(seg + 1);
            tile[q] = -1;
            yw[q] = uw[q] = 0ull;
            if (rest_any != 0ull) {
                const int bit = first_bit(rest_any);
                rest_any &= rest_any - 1ull;
                tile[q] = __builtin_amdgcn_readfirstlane(seg * 64 + bit);
                const long long w = gl_col_base(tile[q], p.nbp) + (long long)(J - tile[q]) * kGlBlock + lane;
                yw[q] = Y[w];
                if ((rest_uns >> bit) & 1ull) uw[q] = U[w];
                got = q + 1;
            }
        }
        return got;
    };
    rewind(0);
    bool has_cross = false, first = true, kept = false;      // kept: the only batch is still in the registers
    while (next_batch() != 0) {
#pragma unroll
        for (int q = 0; q < kBatch; ++q) has_cross = has_cross || (yw[q] | uw[q]) != 0ull;
        kept = first && tile[kBatch - 1] < 0;
        first = false;
        if (tile[kBatch - 1] < 0 || ballot64(valid && !has_cross) == 0ull) break;
    }
    uint64_t cleared = ballot64(valid && !has_cross);
    gl_own_block(p, Kbh, y, u, cleared, j0, lane, k);
    gl_publish(st, J, k, lane);
    bool gave_up = false;
    uint64_t settled = k.decided;      // what the block's own rows have last been followed with
    if (cleared != all) {
        if (!kept) rewind(0);
        while (!gave_up && k.decided != all) {
            if (!kept && next_batch() == 0) break;
            uint64_t dec[kBatch], sds[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                dec[q] = sds[q] = 0ull;
                if (tile[q] >= J0) gl_load_state(st, tile[q], dec[q], sds[q]);
                else if (tile[q] >= 0) dec[q] = sds[q] = ~0ull;
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                if (tile[q] < 0 || gave_up) continue;
                const int32_t *list = tile[q] < J0 ? seedlist + tile[q] * kGlBlock : nullptr;
                uint64_t waiting = gl_follow(p, Kbh, yw[q], uw[q], tile[q] * kGlBlock, list, dec[q], sds[q], valid && has_cross, j0, lane, k);
                while (waiting != 0ull) {
                    // rows that have just joined may settle others of the block, which other blocks may be waiting for
                    if (k.decided != settled) {
                        gl_own_block(p, Kbh, y, u, cleared, j0, lane, k);
                        gl_publish(st, J, k, lane);
                        settled = k.decided;
                    }
                    if (--polls < 0) { gave_up = true; break; }
                    __builtin_amdgcn_s_sleep(4);
                    gl_load_state(st, tile[q], dec[q], sds[q]);
                    waiting = gl_follow(p, Kbh, yw[q], uw[q], tile[q] * kGlBlock, list, dec[q], sds[q], valid && has_cross, j0, lane, k);
                }
            }
            if (kept) break;      // (the block's own rows follow below)
            if (!gave_up && k.decided != settled) {
                gl_own_block(p, Kbh, y, u, cleared, j0, lane, k);
                gl_publish(st, J, k, lane);
                settled = k.decided;
            }
        }
        if (!gave_up) {
            cleared = all;
            gl_own_block(p, Kbh, y, u, cleared, j0, lane, k);
            gl_publish(st, J, k, lane);
        }
    }
    if ((k.decided >> lane) & 1ull) join[lane] = k.target;
    if (k.decided != all) return false;
    // places of the rows inside their clusters as far as this block goes: the first row of a cluster files 64 + the number of its
    // rows here (at most 64), the others file their distance from it and its lane
    int mine = 0;
    uint64_t rem = all;
    while (rem != 0ull) {
        const int l0 = __builtin_amdgcn_readfirstlane(first_bit(rem));
        const uint64_t same = ballot64(valid && k.target == __builtin_amdgcn_readlane(k.target, l0));
        if ((same >> lane) & 1ull) mine = (lane == l0) ? kGlLeader | __popcll(same) : (l0 << 8) | __popcll(same & gl_bits_below(lane));
        rem &= ~same;
    }
    if (valid) place[lane] = mine;
    return true;
}

// Blocks [first, last) that were left undecided, in order; every block before them is decided, so nothing is waited for.  One wavefront.
__device__ __forceinline__ void gl_finish_blocks(const GlobParams &p, int bh, const bf16_t *Kbh, int n, int first, int last, int lane) {
    const unsigned long long *st = p.state + (int64_t)bh * p.nbp * 2;
    for (int J = first; J < last; ++J) {
        uint64_t dec, sds;
        gl_load_state(st, J, dec, sds);
        if (dec == gl_bits_below(min(kGlBlock, n - J * kGlBlock))) continue;
        glob_decide_block(p, bh, Kbh, n, J, lane, 0);
        __threadfence();                                   // the next block's wavefront-wide loads see it
    }
}

__global__ __launch_bounds__(kWave) void glob_decide_kernel(GlobParams p) {
    const int n_bh = p.B * p.Hkv, lane = threadIdx.x;
    const int at = (int)blockIdx.x / n_bh, bh = (int)blockIdx.x - at * n_bh;      // row order; with a multiple of 8 heads a head stays on one XCD
    const int b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = __builtin_amdgcn_readfirstlane(gl_seq_len(p, b));
    const int first = p.stage * gl_stage_blocks(p), J = first + at;
    if (J * kGlBlock >= n) return;
    const bf16_t *Kbh = p.K + b * p.stride_b + h * p.stride_h;
    const bool done = glob_decide_block(p, bh, Kbh, n, J, lane, p.polls);
    // What follows needs all seeds of this stage: the last wavefront to come through decides what others have left undecided.
    const int nb = (n + kGlBlock - 1) / kGlBlock, last = p.stage == p.stages - 1 ? nb : min(first + gl_stage_blocks(p), nb);
    if (!done) __threadfence();      // the seeds that some of its rows have joined
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(p.nclusters + bh, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != last - 1) return;
    bool open = false;
    for (int q = first + lane; q < last; q += kWave) {
        const unsigned long long *st = p.state + (int64_t)bh * p.nbp * 2 + 2 * q;
        const uint32_t d0 = (uint32_t)__hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), d1 = (uint32_t)__hip_atomic_load(st + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t want = gl_bits_below(min(kGlBlock, n - q * kGlBlock));
        open = open || d0 != (uint32_t)want || d1 != (uint32_t)(want >> 32);
    }
    if (ballot64(open) == 0ull) return;
    __threadfence();
    gl_finish_blocks(p, bh, Kbh, n, first, last, lane);
}

// ------------------------------------------------------------------------------------------------
// Clusters are numbered in seed order and their members in row order.
//   rank    a workgroup per kGlRankRows rows: the cluster of every row and its place among the rows of that cluster here; how many rows of these each
//           cluster has.
//   slots   a thread per cluster: sums over the workgroups of rank, the cluster's size and where its members go (space taken in any order).
//   place   a thread per row: its slot.
// (One workgroup per head did all of it before: 86 us for 8 heads x 32768 rows whatever the chip had free.  Up to kGlRankRows rows it does that in less than
// the two launches take: see glob_rank_kernel.)
constexpr int kGlRankRows = 2048, kGlRankThreads = 512;

__device__ __forceinline__ uint64_t gl_seed_mask(const unsigned long long *st, int I) {
    return (st[2 * I] >> 32) | (st[2 * I + 1] & 0xFFFFFFFF00000000ull);
}
// rows of each cluster in every part of kGlRankRows rows, later in the parts before: 16-bit fields, two to a word.  (In the memory of U: nobody reads that
// any more, and its 256 nbp (nbp + 1) bytes per head hold them for every length.)
__device__ __forceinline__ unsigned int *gl_part_sizes(const GlobParams &p, int bh, int part) {
    return reinterpret_cast<unsigned int *>(p.U + (long long)bh * p.tri) + (int64_t)part * (p.nbp * kGlBlock / 2);
}

// ALONE: the sequences have no more rows than that, and the same workgroup finds the clusters' slots and files the rows in them.
template <bool ALONE>
__global__ __launch_bounds__(kGlRankThreads) void glob_rank_kernel(GlobParams p) {
    extern __shared__ unsigned int s_size2[];       // rows filed per cluster, two 16-bit fields a word
    __shared__ unsigned long long s_mask[512];      // seeds of every block
    __shared__ int s_pref[512];                     // clusters before block J
    __shared__ int s_scan[kGlRankThreads / kWave];
    __shared__ int s_lead[kGlRankRows];
    const int bh = (int)blockIdx.x % (p.B * p.Hkv), part = ALONE ? 0 : (int)blockIdx.x / (p.B * p.Hkv);
    const int n = __builtin_amdgcn_readfirstlane(gl_seq_len(p, bh / p.Hkv));
    const int first = part * kGlRankRows;
    if (first >= n && part > 0) return;      // (the first one reports, too)
    const int nb = (n + kGlBlock - 1) / kGlBlock, npad = p.nbp * kGlBlock;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int32_t *join = p.join + (int64_t)bh * npad, *place = p.place + (int64_t)bh * npad;
    constexpr int kPer = kGlRankRows / kGlRankThreads;
    int t[kPer], pl[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int j = first + q * kGlRankThreads + tid;
        t[q] = j < n ? join[j] : 0;
        pl[q] = j < n ? place[j] : 0;
    }
    // ---- clusters before every block (512 at most)
    const uint64_t m = tid < nb ? gl_seed_mask(p.state + (int64_t)bh * p.nbp * 2, tid) : 0ull;
    const int mine = __popcll(m);
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) s_scan[wave] = incl;
    s_mask[tid] = m;
    __syncthreads();
    int before = 0, P = 0;
#pragma unroll
    for (int w = 0; w < kGlRankThreads / kWave; ++w) {
        if (w < wave) before += s_scan[w];
        P += s_scan[w];
    }
    s_pref[tid] = before + incl - mine;
    for (int i = tid; i < (P + 1) / 2; i += kGlRankThreads) s_size2[i] = 0u;
    if (part == 0 && tid == 0) {
        p.nclusters[bh] = P;
        p.comp_lens[bh] = (P <= p.cap) ? P : -1;
    }
    __syncthreads();
    // ---- the cluster of every row; the first rows of a cluster in a block file all its rows there
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int j = first + q * kGlRankThreads + tid;
        t[q] = s_pref[t[q] >> 6] + (int)__popcll(s_mask[t[q] >> 6] & gl_bits_below(t[q] & 63));
        if (p.cluster_id && j < n) p.cluster_id[(int64_t)bh * p.N_max + j] = t[q];
        s_lead[q * kGlRankThreads + tid] = (j < n && (pl[q] & kGlLeader)) ? t[q] | ((pl[q] & 0x7F) << 16) : -1;
    }
    __syncthreads();
    // ---- places in row order: one wavefront, block by block (LDS additions of one wavefront execute in order)
    if (wave == 0) {
        constexpr int kAhead = 8;
        for (int J0 = 0; J0 < kGlRankRows / kGlBlock && first + J0 * kGlBlock < n; J0 += kAhead) {
            int v[kAhead];
            unsigned int old[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) v[q] = s_lead[(J0 + q) * kGlBlock + lane];
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (v[q] >= 0) old[q] = atomicAdd(&s_size2[(v[q] & 0xFFFF) >> 1], (unsigned)(v[q] >> 16) << (16 * (v[q] & 1)));
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (v[q] >= 0) s_lead[(J0 + q) * kGlBlock + lane] = (int)((old[q] >> (16 * (v[q] & 1))) & 0xFFFFu);
        }
    }
    __syncthreads();
    auto place_of = [&](int q) {      // among the rows of its cluster here
        const int i = q * kGlRankThreads + tid;
        return (pl[q] & kGlLeader) ? s_lead[i] : s_lead[(i & ~63) + (pl[q] >> 8)] + (pl[q] & 0x7F);
    };
    if constexpr (ALONE) {
        // first slots of four clusters a thread, in place of their sizes (kGlRankRows rows at most: 16 bits hold them)
        static_assert(kGlRankRows <= 4 * kGlRankThreads, "a look each");
        unsigned short *size = reinterpret_cast<unsigned short *>(s_size2);
        int mine4[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            mine4[q] = 4 * tid + q < P ? (int)size[4 * tid + q] : 0;
            sum += mine4[q];
        }
        int upto = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(upto, off, kWave);
            if (lane >= off) upto += up;
        }
        if (lane == kWave - 1) s_scan[wave] = upto;      // (everybody is done with the sums over the blocks)
        __syncthreads();
        int at = upto - sum;
        for (int w = 0; w < wave; ++w) at += s_scan[w];
        int32_t *mbase = p.mbase + (int64_t)bh * (npad + 1), *csize = p.csize + (int64_t)bh * npad, *counts = p.counts + (int64_t)bh * p.cap;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = 4 * tid + q;
            if (c < P) {
                mbase[c] = at;
                csize[c] = mine4[q];
                if (c < p.cap) counts[c] = mine4[q];
                size[c] = (unsigned short)at;
            }
            at += mine4[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int j = q * kGlRankThreads + tid;
            if (j < n) p.order[(int64_t)bh * npad + (int)size[t[q]] + place_of(q)] = j;
        }
    } else {
        int32_t *lead = p.lead + (int64_t)bh * npad;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int at = place_of(q), j = first + q * kGlRankThreads + tid;
            if (j < n) lead[j] = t[q] | (at << 16);
        }
        unsigned int *sizes = gl_part_sizes(p, bh, part);
        for (int i = tid; i < (P + 1) / 2; i += kGlRankThreads) sizes[i] = s_size2[i];
    }
}

__global__ __launch_bounds__(256) void glob_slots_kernel(GlobParams p) {
    __shared__ int s_scan[4];
    __shared__ int s_base;
    const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int n = gl_seq_len(p, bh / p.Hkv), P = p.nclusters[bh], npad = p.nbp * kGlBlock;
    if ((int)blockIdx.x * 512 >= P) return;
    const int c = ((int)blockIdx.x * 256 + tid) * 2;      // two clusters a thread
    unsigned int sum = 0u;      // (n <= 32768: the fields do not spill over)
    if (c < P)
        for (int part = 0; part * kGlRankRows < n; part += 4) {
            unsigned int x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = (part + q) * kGlRankRows < n ? gl_part_sizes(p, bh, part + q)[c / 2] : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if ((part + q) * kGlRankRows < n) gl_part_sizes(p, bh, part + q)[c / 2] = sum;
                sum += x[q];
            }
        }
    const int s0 = (int)(sum & 0xFFFFu), s1 = (int)(sum >> 16);
    int incl = s0 + s1;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) s_scan[wave] = incl;
    __syncthreads();
    int32_t *mbase = p.mbase + (int64_t)bh * (npad + 1);
    if (tid == 0) s_base = atomicAdd(mbase + npad, s_scan[0] + s_scan[1] + s_scan[2] + s_scan[3]);
    __syncthreads();
    int at = s_base + incl - s0 - s1;
    for (int w = 0; w < wave; ++w) at += s_scan[w];
    int32_t *csize = p.csize + (int64_t)bh * npad, *counts = p.counts + (int64_t)bh * p.cap;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (c + q < P) {
            mbase[c + q] = at;
            csize[c + q] = q ? s1 : s0;
            if (c + q < p.cap) counts[c + q] = q ? s1 : s0;
        }
        at += s0;
    }
}

__global__ __launch_bounds__(256) void glob_place_kernel(GlobParams p) {
    const int bh = blockIdx.y, j = (int)blockIdx.x * 256 + (int)threadIdx.x, npad = p.nbp * kGlBlock;
    if (j >= gl_seq_len(p, bh / p.Hkv)) return;
    const int v = p.lead[(int64_t)bh * npad + j], c = v & 0xFFFF;
    const unsigned int before = gl_part_sizes(p, bh, j / kGlRankRows)[c / 2];
    p.order[(int64_t)bh * npad + p.mbase[(int64_t)bh * (npad + 1) + c] + (int)((c & 1) ? before >> 16 : before & 0xFFFFu) + (v >> 16)] = j;
}

// ------------------------------------------------------------------------------------------------
// sum: Eq. 3.  16 lanes per cluster, members in row order; keys and values in workgroups of their own, sixteen rows in flight: a cluster of a hundred
// rows is the kernel's tail, its trips to memory are what that costs.  (Both in one, eight of each: 98 registers; 8 heads x 32768 44 us, 38 so;
// the call at 8 x 5000 107 and 99, at 2 x 5000 79 and 72.)
template <typename TO>
__global__ __launch_bounds__(256) void glob_sum_kernel(GlobParams p) {
    const int bh = blockIdx.y, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int npad = p.nbp * kGlBlock;
    const int P = min(p.nclusters[bh], p.cap);
    const int cl = blockIdx.x * 16 + threadIdx.x / 16, c = threadIdx.x % 16;
    if (cl >= P) return;
    const bool values = blockIdx.z != 0;
    const bf16_t *X = (values ? p.V : p.K) + b * p.stride_b + h * p.stride_h + 8 * c;
    const int32_t *order = p.order + (int64_t)bh * npad + p.mbase[(int64_t)bh * (npad + 1) + cl];
    const int size = p.csize[(int64_t)bh * npad + cl];
    float sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = 0.f;
    const int first_lane = (threadIdx.x & (kWave - 1)) & ~15;
    for (int t0 = 0; t0 < size; t0 += 16) {
        const int members = min(16, size - t0);
        const int mine = (c < members) ? order[t0 + c] : 0;      // sixteen members in one load
        uint4 x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t row = __shfl(mine, first_lane + u, kWave);
            if (u < members) x[u] = *reinterpret_cast<const uint4 *>(X + row * p.stride_n);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (u < members) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sum[2 * e] += bf16_lo(dword_of(x[u], e));
                    sum[2 * e + 1] += bf16_hi(dword_of(x[u], e));
                }
            }
        }
    }
    // 1/size: a row of size 1 is passed on unchanged
    const float inv = (size > 1) ? 1.0f / (float)size : 1.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] *= inv;
    store8(reinterpret_cast<TO *>(values ? p.Vc : p.Kc) + ((int64_t)bh * p.cap + cl) * kGlD + 8 * c, sum);
}

// one chunk per sequence in the offsets format of sc_segment: off = {0, n + 1}, one chunk
__global__ void glob_one_chunk_kernel(const int32_t *seq_lens, int B, int N_max, int32_t *offsets, int32_t *num_chunks) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int n = seq_lens ? seq_lens[b] : N_max;
    n = n < 0 ? 0 : (n > N_max ? N_max : n);
    offsets[2 * b] = 0;
    offsets[2 * b + 1] = n + 1;
    num_chunks[b] = 1;
}

// ------------------------------------------------------------------------------------------------
static bool glob_fast_ok(const GscMergeArgs &a) {
    return a.in_dtype == DType::BF16 && a.d == kGlD && a.N_max <= 32768 && a.stride_n % 8 == 0 && a.stride_n * 2 * kGlBlock < (1ll << 31) &&
           a.tune.gsc_fast_path != 0;
}
static size_t glob_head_bytes(int N_max) {   // upper bound of what launch_gsc_global lays out per (sequence, head)
    const size_t nbp = (size_t)(N_max + kGlBlock - 1) / kGlBlock, npad = nbp * kGlBlock, nseg = (nbp + kGlWordBlocks - 1) / kGlWordBlocks;
    const size_t tri = 64 * nbp * (nbp + 1) / 2;
    return 6 * align_up(npad * 4, 256) + 2 * align_up(tri * 8, 256) + align_up((npad + 1) * 4, 256) + 2 * align_up(nbp * nseg * 8, 256) +
           align_up(nbp * 16, 256);
}
// workspace: [one-chunk offsets and counts | the larger of (ordinary sc_gsc_merge workspace, arrays of this path)]
static size_t glob_prefix_bytes(int B) { return align_up((size_t)B * 3 * 4, 256); }

size_t gsc_global_workspace_bytes(int B, int Hkv, int N_max, int d) {
    const size_t ordinary = gsc_merge_workspace_bytes(B, Hkv, N_max, d);
    size_t fast = 0;
    if (d == kGlD && N_max <= 32768) {
        fast = glob_head_bytes(N_max) * (size_t)B * Hkv + align_up((size_t)B * Hkv * 4, 256);
    }
    return glob_prefix_bytes(B) + (ordinary > fast ? ordinary : fast);
}

// Stages of `m` words of flags (of 64 column blocks); the last one has what is left, half as much again or less.
static int glob_stages(int nbp, int m) { return max(1, (2 * nbp + m * kGlWordBlocks) / (2 * m * kGlWordBlocks)); }
// Words of a stage.  In us: all pairs at 1.25 PFLOP/s; with the seeds of the stages before 0.45 of that, which is a seed in four or five rows, and half as fast for
// short lists of unequal length; and what a further stage's two launches and the chain of its decisions cost.  Us per call, stages of 4096 /
// 8192 / 16384 rows / one, tau 0.7 and 0.9745 (a seed in six and in four rows) and where every row is a seed:
//   8 heads x 32768   544 / 555 / 651 / 900    691 / 664 / 736 / 908    1279 / 1135 / 1034 / 957
//   16 x 32768        918 / 987 / 1219 / 1813  1129 / 1165 / 1341 / 1797  2272 / 2108 / 1993 / 1878
//   1 x 32768         261 / 173 / 139 / 158    373 / 231 / 167 / 164    563 / 318 / 205 / 172
//   16 x 16384        371 / 403 / - / 524      446 / 455 / - / 538      719 / 635 / - / 581
//   8 x 12365         212 / 207 / - / 207      285 / 251 / - / 213      436 / 348 / - / 226
// So a call in stages in which next to nothing merges takes up to a fifth longer than one of all pairs would (with all pairs, and the kernels of the time before
// stages, 8 x 32768 took 990 / 1003 / 1079); a threshold that nothing can exceed is known here, and is not taken in stages.
static int glob_stage_words(size_t heads, int n, int nbp, float tau) {
    const int nseg = (nbp + kGlWordBlocks - 1) / kGlWordBlocks;
    if (tau >= 1.0f) return nseg;
    const double all = (double)heads * n * n * 128 / 1.25e9, stage_cost = 25.0 + 0.8 * (double)heads, seeds = 0.45;
    int best = nseg;
    double least = all;
    for (int m = nseg - 1; m >= 1; --m) {
        const int stages = glob_stages(nbp, m), first = m * kGlWordBlocks, last = nbp - (stages - 1) * first;
        const double own = ((double)(stages - 1) * first * first + (double)last * last) / ((double)nbp * nbp);      // share of the pairs that lie within a stage
        const double cost = all * (own + seeds * (1.0 - own)) + stage_cost * (stages - 1);
        if (cost < least) { least = cost; best = m; }
    }
    return best;
}

hipError_t launch_gsc_global(const GscMergeArgs &a, hipStream_t stream) {
    char *ws = reinterpret_cast<char *>(a.ws);
    int32_t *offsets = reinterpret_cast<int32_t *>(ws), *num_chunks = offsets + 2 * a.B;
    char *rest = ws + glob_prefix_bytes(a.B);
    if (!glob_fast_ok(a)) {
        hipLaunchKernelGGL(glob_one_chunk_kernel, dim3((a.B + 255) / 256), dim3(256), 0, stream, a.seq_lens, a.B, a.N_max, offsets, num_chunks);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        GscMergeArgs o = a;
        o.offsets = offsets; o.offsets_stride_b = 2; o.num_chunks = num_chunks; o.ws = rest;
        return launch_gsc_merge(o, stream);
    }
    GlobParams p;
    p.K = reinterpret_cast<const bf16_t *>(a.K); p.V = reinterpret_cast<const bf16_t *>(a.V);
    p.stride_b = a.stride_b; p.stride_h = a.stride_h; p.stride_n = a.stride_n;
    p.seq_lens = a.seq_lens; p.B = a.B; p.Hkv = a.Hkv; p.N_max = a.N_max; p.tau = a.tau;
    p.Kc = a.Kc; p.Vc = a.Vc; p.out_is_bf16 = a.out_dtype == DType::BF16; p.cap = a.cap;
    p.counts = a.counts; p.comp_lens = a.comp_lens; p.cluster_id = a.cluster_id;
    p.nbp = (a.N_max + kGlBlock - 1) / kGlBlock;
    p.tri = 64ll * p.nbp * (p.nbp + 1) / 2;
    const size_t BH = (size_t)a.B * a.Hkv;
    const size_t npad = (size_t)p.nbp * kGlBlock;
    // array by array, each holding all (sequence, head) pairs back to back
    size_t o = 0;
    p.rinv = reinterpret_cast<float *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.Y = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.tri * 8 * BH, 256);
    p.U = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.tri * 8 * BH, 256);
    p.join = reinterpret_cast<int32_t *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.place = reinterpret_cast<int32_t *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.lead = reinterpret_cast<int32_t *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.order = reinterpret_cast<int32_t *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.mbase = reinterpret_cast<int32_t *>(rest + o); o += align_up((npad + 1) * 4 * BH, 256);
    p.csize = reinterpret_cast<int32_t *>(rest + o); o += align_up(npad * 4 * BH, 256);
    p.nclusters = reinterpret_cast<int32_t *>(rest + o); o += align_up(4 * BH, 256);
    p.nseg = (p.nbp + kGlWordBlocks - 1) / kGlWordBlocks;
    p.tany = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * p.nseg * 8 * BH, 256);
    p.tuns = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * p.nseg * 8 * BH, 256);
    p.state = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * 16 * BH, 256);
    p.polls = a.tune.global_polls;

    hipLaunchKernelGGL(glob_norms_kernel, dim3((unsigned)(npad / 16), (unsigned)BH), dim3(256), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.seedlist = p.order;
    p.stage_words = glob_stage_words(BH, a.N_max, p.nbp, a.tau);
    p.stage = 0;
    const int M = p.stage_words, stages = p.stages = glob_stages(p.nbp, M);
    // Length of a walk: the longest that leaves some five items for each of the 768 places (three workgroups on each of 256 CUs), so that the last ones do not
    // matter.  (Us per call with 8 / 16 / 32 blocks: 8 heads x 32768 619 / 600 / 599; x 20000 367 / 372 / 411; x 3000 79 / 97 / 143.)
    // Items are those of the blocks that the longest sequence has.
    const int last_groups = (p.nbp - (stages - 1) * M * kGlWordBlocks + kGlPairWaves - 1) / kGlPairWaves;      // of row blocks
    size_t items = 0;
    for (p.walk = 32;; p.walk /= 2) {
        const int stage_segs = M * kGlWordBlocks / p.walk, per_seg = p.walk / kGlPairWaves;
        items = (size_t)(stages - 1) * per_seg * stage_segs * (stage_segs + 1) / 2;
        for (int jg = 0; jg < last_groups; ++jg) items += jg / per_seg + 1;
        if (items * BH >= 4096 || p.walk == 8) break;
    }
    hipLaunchKernelGGL((glob_pairs_kernel<false>), dim3((unsigned)(items * BH)), dim3(kGlPairWaves * kWave), 0, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (p.stage = 0; p.stage < stages; ++p.stage) {
        const int first = p.stage * M * kGlWordBlocks, blocks = p.stage == stages - 1 ? p.nbp - first : M * kGlWordBlocks;
        if (p.stage > 0) {
            const int groups = (blocks + kGlPairWaves - 1) / kGlPairWaves;
            hipLaunchKernelGGL((glob_pairs_kernel<true>), dim3((unsigned)(groups * (first / (kGlSeedUnit * kGlSeedShare)) * BH)), dim3(kGlPairWaves * kWave), 0, stream, p);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(glob_decide_kernel, dim3((unsigned)(blocks * BH)), dim3(kWave), 0, stream, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const size_t dyn = npad * sizeof(unsigned short);
    if (a.N_max <= kGlRankRows) {
        hipLaunchKernelGGL((glob_rank_kernel<true>), dim3((unsigned)BH), dim3(kGlRankThreads), dyn, stream, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else {
        if (dyn > 48 * 1024) {   // a host-side setting of the kernel (per device), not a stream operation
            int dev = 0;
            e = hipGetDevice(&dev);
            if (e != hipSuccess) return e;
            static std::mutex mu;
            static bool raised[64];
            if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
            std::lock_guard<std::mutex> lock(mu);
            if (!raised[dev]) {
                e = hipFuncSetAttribute(reinterpret_cast<const void *>(glob_rank_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
                if (e != hipSuccess) return e;
                raised[dev] = true;
            }
        }
        hipLaunchKernelGGL((glob_rank_kernel<false>), dim3((unsigned)((a.N_max + kGlRankRows - 1) / kGlRankRows * BH)), dim3(kGlRankThreads), dyn, stream, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(glob_slots_kernel, dim3((unsigned)((a.N_max + 511) / 512), (unsigned)BH), dim3(256), 0, stream, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(glob_place_kernel, dim3((unsigned)((a.N_max + 255) / 256), (unsigned)BH), dim3(256), 0, stream, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int max_clusters = a.N_max < a.cap ? a.N_max : a.cap;
    const dim3 grid_sum((unsigned)((max_clusters + 15) / 16), (unsigned)BH, 2);
    if (p.out_is_bf16) hipLaunchKernelGGL((glob_sum_kernel<bf16_t>), grid_sum, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((glob_sum_kernel<float>), grid_sum, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace sc
