// sc_gsc_merge_global: Alg. 1 / Eq. 2 and Eq. 3 (paper Sec. 2.3, 2.4) when the whole sequence of a
// (sequence, KV head) is ONE chunk -- the "no chunking" variant of the paper's chunking ablation
// (Sec. 3.4) -- for bf16 keys/values with head dim 128 and up to 32768 tokens.
//
// Alg. 1 over one chunk of n rows is sequential in its seeds (a row is a seed iff no earlier seed takes
// it; a row joins the EARLIEST seed it resembles) but every similarity it can ask for is known in
// advance, so the work is split into a dense part and a sparse one:
//   norms    reciprocal norms of all rows.
//   pairs    all pairwise comparisons "Sim(i, j) > tau" for i < j on the matrix cores
//            (v_mfma_f32_16x16x32_bf16, 64 x 64 rows per product block): one 64-bit word per (row j,
//            block of 64 earlier rows), "surely above" and "inside the +-1e-4 band" (decided later in
//            fp64).  Only blocks that hold such a pair are written; a bit per block says which.
//   decide   which rows are seeds and which seed every row joins, all blocks of 64 rows at once.
//   number   one workgroup per (sequence, head) numbers the clusters and their members in row order.
//   sum      one 16-lane group per cluster adds up its members' keys and values in row order (fp32),
//            scales by 1/size and writes the output row: Eq. 3.
// 8 heads x 32768 tokens, tau 0.7, us per call: 2550 with every word written, read back into candidate lists and resolved
// block by block in order (pairs 1370, lists 307, resolve 762, sum 107); now 1060 (pairs 948, decide 14, number 92, sum 42).
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
constexpr int kGlNumberThreads = 1024;
constexpr int kGlSegment = 64;                  // column blocks per work item of the pairs kernel
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
    int polls;                    // looks at another block's rows before the number kernel takes over
    int32_t *mbase, *csize;       // [nbp * 64 + 1], [nbp * 64]
    int32_t *nclusters;           // [1]
};

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
    if (c == 0 && (row & 31) == 0) p.state[(int64_t)bh * p.nbp * 2 + row / 32] = 0ull;      // nothing decided yet
    if (c == 0)
        p.rinv[(int64_t)bh * p.nbp * 64 + row] = (row < n && nsq > 1e-30f && nsq < 1e30f) ? __frsqrt_rn(nsq) : __builtin_nanf("");
}

// ------------------------------------------------------------------------------------------------
// pairs: workgroup (JG, bh) owns the row blocks J = 4 JG + wave and walks the column blocks I = 0 .. max J.
// The rows of block J are the B operand and stay in registers (lane (g, c): row 16 Jt + c, elements
// 32 ks + 8 g .. + 7 -- v_mfma_f32_16x16x32_bf16, the form that runs at the full bf16 rate of this chip);
// the rows of block I pass through an LDS tile shared by the four wavefronts and are the A operand.  The
// product tile leaves lane (g, c) with the dot products of row 16 Jt + c of block J and rows
// 16 It + 4 g + i of block I: four bits of that row's word, completed by an OR over the lane groups.
__global__ __launch_bounds__(kGlPairWaves *kWave, 2) void glob_pairs_kernel(GlobParams p) {
    __shared__ __attribute__((aligned(16))) char s_tiles[2][kGlBlock * kGlTileRowBytes];      // two tiles: one worked on, one being filled
    __shared__ __attribute__((aligned(16))) float s_rinvs[2][kGlBlock];
    __shared__ int s_odd[2];      // a row of the tile has no usable norm
    const int bh = blockIdx.y, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = gl_seq_len(p, b);
    const int nb = (n + kGlBlock - 1) / kGlBlock;
    const int njg = (nb + kGlPairWaves - 1) / kGlPairWaves;
    // Work item = (group JG of four row blocks, segment of kGlSegment column blocks): the walks over the column
    // blocks have about the same length whatever the row.  Groups 16 q .. 16 q + 15 have q + 1 segments each
    // (kGlSegment = 64 column blocks = 16 groups), so 8 q (q + 1) items come before group 16 q.
    int JG, seg;
    {
        const int x = (int)gridDim.x - 1 - (int)blockIdx.x;      // the longest rows first
        int q = 0;
        while (8 * (q + 1) * (q + 2) <= x) ++q;
        const int rem = x - 8 * q * (q + 1);
        JG = 16 * q + rem / (q + 1);
        seg = rem % (q + 1);
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
    const int I_first = seg * kGlSegment;
    const int I_last = min(min(JG * kGlPairWaves + kGlPairWaves - 1, nb - 1), I_first + kGlSegment - 1);
    if (I_first > I_last) return;
    // the tile of block I: thread t brings rows t / 16 + 16 r, piece t % 16
    const int lrow = tid >> 4, lc = tid & 15;
    uint4 pre[4];
    float pre_r = 0.f;
    auto fetch = [&](int I) {
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
        char *t = s_tiles[I & 1];
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<uint4 *>(t + (lrow + 16 * r) * kGlTileRowBytes + 16 * lc) = pre[r];
        if (wave == 0) {
            s_rinvs[I & 1][lane] = pre_r;
            const bool odd = ballot64(!(pre_r == pre_r)) != 0ull;
            if (lane == 0) s_odd[I & 1] = odd ? 1 : 0;
        }
    };
    uint64_t any_bits = 0ull, uns_bits = 0ull;      // of this segment's column blocks
    fetch(I_first);
    park(I_first);
    if (I_first < I_last) fetch(I_first + 1);
    for (int I = I_first; I <= I_last; ++I) {
        __syncthreads();          // tile I is complete; everybody is done with tile I - 1, whose buffer takes tile I + 1 now
        if (I < I_last) {
            park(I + 1);
            if (I + 1 < I_last) fetch(I + 2);      // on its way while this tile is worked on
        }
        const char *s_tile = s_tiles[I & 1];
        const float *s_rinv = s_rinvs[I & 1];
        if (!active || I > J) continue;    // wave-uniform
        const bool odd = bad_j || __builtin_amdgcn_readfirstlane(s_odd[I & 1]) != 0;
        uint32_t yl[4], yh[4], ul[4], uh[4];
#pragma unroll
        for (int Jt = 0; Jt < 4; ++Jt) yl[Jt] = yh[Jt] = ul[Jt] = uh[Jt] = 0u;
        bool touched = odd;
#pragma unroll
        for (int It = 0; It < 4; ++It) {
            gl_float4 acc[4];
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt) acc[Jt] = gl_float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const uint4 a = *reinterpret_cast<const uint4 *>(s_tile + (16 * It + c) * kGlTileRowBytes + (32 * ks + 8 * g) * 2);
#pragma unroll
                for (int Jt = 0; Jt < 4; ++Jt)
                    acc[Jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(gl_bf16x8, a),
                                                                      __builtin_bit_cast(gl_bf16x8, bq[Jt][ks]), acc[Jt], 0, 0, 0);
            }
            const gl_float4 rm = *reinterpret_cast<const gl_float4 *>(s_rinv + 16 * It + 4 * g);
            // sim(m, n) > t  <=>  dot * rinv_m > t * norm_n.  Hardly any tile holds a pair that comes near: one multiply-add
            // and half a maximum per pair tell.
            float top = fmaf(acc[0][0], rm[0], -ln[0]);
#pragma unroll
            for (int Jt = 0; Jt < 4; ++Jt)
#pragma unroll
                for (int i = (Jt == 0) ? 1 : 0; i < 4; ++i) top = fmaxf(top, fmaf(acc[Jt][i], rm[i], -ln[Jt]));
            if (!odd && ballot64(top >= 0.f) == 0ull) continue;
            touched = true;
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
                    const uint32_t dd = __float_as_uint(fmaf(-acc[Jt][i], rm[i], hn[Jt]));
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
                        const float dd = fmaf(-acc[Jt][i], rm[i], hn[Jt]);
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
        if (!touched && I != J) continue;
        // complete the words over the four lane groups; lane 16 Jt + c keeps the words of row 16 Jt + c
        uint32_t myl = 0u, myh = 0u, mul = 0u, muh = 0u;
#pragma unroll
        for (int Jt = 0; Jt < 4; ++Jt) {
            const uint32_t a0 = gl_or_rows(yl[Jt]), a1 = gl_or_rows(yh[Jt]);
            const uint32_t b0 = gl_or_rows(ul[Jt]), b1 = gl_or_rows(uh[Jt]);
            if (g == Jt) { myl = a0; myh = a1; mul = b0; muh = b1; }
        }
        if (J * kGlBlock + lane >= n) myl = myh = mul = muh = 0u;      // no such row
        const long long w = (long long)bh * p.tri + gl_col_base(I, p.nbp) + (long long)(J - I) * kGlBlock + lane;
        const bool any = ballot64((myl | myh | mul | muh) != 0u) != 0ull, any_u = ballot64((mul | muh) != 0u) != 0ull;
        if (any || I == J) p.Y[w] = ((unsigned long long)myh << 32) | myl;      // a block's own words are always read
        if (any_u || I == J) p.U[w] = ((unsigned long long)muh << 32) | mul;
        any_bits |= any ? 1ull << (I & 63) : 0ull;
        uns_bits |= any_u ? 1ull << (I & 63) : 0ull;
    }
    if (active && lane == 0) {      // (a segment is the 64 column blocks of one word)
        const int64_t at = ((int64_t)bh * p.nbp + J) * p.nseg + seg;
        p.tany[at] = any_bits;
        p.tuns[at] = uns_bits;
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
// Waiting is bounded (p.polls looks in all); blocks that are left undecided are finished in order by one wavefront of the number kernel.
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

// One candidate word (64 earlier rows from `first_row` on; decided / seeds: what is known about them) for every lane with
// `open`: follows the candidates as far as they are known.  Lanes that find their seed join k.decided; returns the lanes that
// wait for an undecided row.  uw loses the bits that fp64 has turned down.
__device__ __forceinline__ uint64_t gl_follow(const GlobParams &p, const bf16_t *Kbh, uint64_t yw, uint64_t &uw, int first_row, uint64_t decided,
                                              uint64_t seeds, bool open, int j0, int lane, GlobBlock &k) {
    for (;;) {
        const bool undecided = open && ((k.decided >> lane) & 1ull) == 0ull;
        const uint64_t c = undecided ? (yw | uw) & ~(decided & ~seeds) : 0ull;
        const int f = (c != 0ull) ? first_bit(c) : 0;
        const bool known = c != 0ull && ((decided >> f) & 1ull) != 0ull;
        const bool sure = known && ((yw >> f) & 1ull) != 0ull;
        if (sure) k.target = first_row + f;
        k.decided |= ballot64(sure);
        uint64_t ask = ballot64(known && !sure);
        if (ask == 0ull) return ballot64(c != 0ull && !known);
        while (ask != 0ull) {
            const int r = __builtin_amdgcn_readfirstlane(first_bit(ask));
            ask &= ask - 1ull;
            const int fr = __builtin_amdgcn_readlane(f, r);
            const bool ok = gl_cosine_exceeds_f64(Kbh + (int64_t)(first_row + fr) * p.stride_n, Kbh + (int64_t)(j0 + r) * p.stride_n, p.tau, lane);
            if (ok) k.decided |= 1ull << r;
            if (lane == r) {
                if (ok) k.target = first_row + fr;
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
        gl_follow(p, Kbh, y, u, j0, k.decided, k.seeds, open, j0, lane, k);
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
                if (tile[q] >= 0) gl_load_state(st, tile[q], dec[q], sds[q]);
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                if (tile[q] < 0 || gave_up) continue;
                uint64_t waiting = gl_follow(p, Kbh, yw[q], uw[q], tile[q] * kGlBlock, dec[q], sds[q], valid && has_cross, j0, lane, k);
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
                    waiting = gl_follow(p, Kbh, yw[q], uw[q], tile[q] * kGlBlock, dec[q], sds[q], valid && has_cross, j0, lane, k);
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

__global__ __launch_bounds__(kWave) void glob_decide_kernel(GlobParams p) {
    const int n_bh = p.B * p.Hkv;
    const int J = (int)blockIdx.x / n_bh, bh = (int)blockIdx.x - J * n_bh;      // row order; with a multiple of 8 heads a head stays on one XCD
    const int b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = __builtin_amdgcn_readfirstlane(gl_seq_len(p, b));
    if (J * kGlBlock >= n) return;
    glob_decide_block(p, bh, p.K + b * p.stride_b + h * p.stride_h, n, J, threadIdx.x, p.polls);
}

// ------------------------------------------------------------------------------------------------
// number: one workgroup per (sequence, head).  Clusters are numbered in seed order and their members in row order: every row gets
// its cluster, the first row of a cluster in a block takes the next slots of that cluster for all its rows there (one
// wavefront, in block order: LDS additions of one wavefront execute in order and nothing waits for their results but
// the stores), sizes become first slots, rows go to their slots.
__global__ __launch_bounds__(kGlNumberThreads) void glob_number_kernel(GlobParams p) {
    extern __shared__ unsigned int s_size2[];       // members filed per cluster, two 16-bit fields a word (n <= 32768); later first slots
    __shared__ unsigned long long s_mask[512];      // seeds of every block
    __shared__ int s_pref[512];                     // clusters before block J
    __shared__ int s_scan[kGlNumberThreads];
    __shared__ int s_undecided;
    const int bh = blockIdx.x, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int n = __builtin_amdgcn_readfirstlane(gl_seq_len(p, b));
    const int nb = (n + kGlBlock - 1) / kGlBlock;
    const int npad = p.nbp * kGlBlock;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const unsigned long long *st = p.state + (int64_t)bh * p.nbp * 2;
    const int32_t *join = p.join + (int64_t)bh * npad, *place = p.place + (int64_t)bh * npad;
    int32_t *lead = p.lead + (int64_t)bh * npad, *order = p.order + (int64_t)bh * npad;
    int32_t *cid_out = p.cluster_id ? p.cluster_id + (int64_t)bh * p.N_max : nullptr;
    unsigned short *s_size = reinterpret_cast<unsigned short *>(s_size2);
    if (tid == 0) s_undecided = 0;
    for (int i = tid; i < npad / 2; i += kGlNumberThreads) s_size2[i] = 0u;
    __syncthreads();
    {
        bool open = false;
        if (tid < 2 * nb) {
            const int rows = n - tid * 32;
            const uint32_t want = rows <= 0 ? 0u : (rows >= 32 ? 0xFFFFFFFFu : (1u << rows) - 1u);
            open = ((uint32_t)st[tid] & want) != want;
        }
        if (open) s_undecided = 1;
    }
    __syncthreads();
    if (s_undecided != 0) {      // (2 * nb <= 1024 words: one look each)
        if (wave == 0) {
            const bf16_t *Kbh = p.K + b * p.stride_b + h * p.stride_h;
            for (int J = 0; J < nb; ++J) {
                uint64_t dec, sds;
                gl_load_state(st, J, dec, sds);
                const uint64_t all = gl_bits_below(min(kGlBlock, n - J * kGlBlock));
                if (dec == all) continue;
                glob_decide_block(p, bh, Kbh, n, J, lane, 0);      // every earlier row is decided: nothing to wait for
                __threadfence();                                   // the next block's wavefront-wide loads see it
            }
        }
        __threadfence();
        __syncthreads();
    }
    // ---- clusters before every block
    int mine = 0;
    if (tid < 512) {
        uint64_t m = 0ull;
        if (tid < nb) {
            const unsigned long long w0 = __hip_atomic_load(st + 2 * tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long w1 = __hip_atomic_load(st + 2 * tid + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            m = (w0 >> 32) | (w1 & 0xFFFFFFFF00000000ull);
        }
        s_mask[tid] = m;
        mine = __popcll(m);
    }
    // exclusive sum over the workgroup; total in the last entry
    auto scan = [&](int x) {
        int incl = x;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += up;
        }
        if (lane == kWave - 1) s_scan[wave] = incl;
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wave; ++w) before += s_scan[w];
        return before + incl - x;
    };
    const int pref = scan(mine);
    if (tid < 512) s_pref[tid] = pref;
    int P = 0;
    for (int w = 0; w < kGlNumberThreads / kWave; ++w) P += s_scan[w];
    __syncthreads();
    // ---- the cluster of every row
    constexpr int kPer = 32;             // 1024 threads x 32 = 32768 clusters at most
    auto cluster_of = [&](int seed_row) { return s_pref[seed_row >> 6] + (int)__popcll(s_mask[seed_row >> 6] & gl_bits_below(seed_row & 63)); };
    for (int j0 = tid; j0 < n; j0 += 8 * kGlNumberThreads) {
        int t[8], pl[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + q * kGlNumberThreads;
            t[q] = j < n ? join[j] : 0;
            pl[q] = j < n ? place[j] : 0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + q * kGlNumberThreads;
            if (j < n) {
                const int c = cluster_of(t[q]);
                if (cid_out) cid_out[j] = c;
                lead[j] = (pl[q] & kGlLeader) ? c | ((pl[q] & 0x7F) << 16) : -1;
            }
        }
    }
    __syncthreads();
    // ---- slots inside the clusters, in row order
    if (wave == 0) {
        constexpr int kAhead = 8;
        int v[kAhead], w[kAhead];
        auto get = [&](int J0, int (&x)[kAhead]) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int j = (J0 + q) * kGlBlock + lane;
                x[q] = j < n ? lead[j] : -1;
            }
        };
        get(0, v);
        for (int J0 = 0; J0 < nb; J0 += kAhead) {
            get(J0 + kAhead, w);
            unsigned int old[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (v[q] >= 0) old[q] = atomicAdd(&s_size2[(v[q] & 0xFFFF) >> 1], (unsigned)(v[q] >> 16) << (16 * (v[q] & 1)));
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (v[q] >= 0) lead[(J0 + q) * kGlBlock + lane] = (int)((old[q] >> (16 * (v[q] & 1))) & 0xFFFFu);
#pragma unroll
            for (int q = 0; q < kAhead; ++q) v[q] = w[q];
        }
    }
    __syncthreads();
    // ---- cluster sizes -> first slot of every cluster; sizes and length to the outputs
    {
        const int per = (P + kGlNumberThreads - 1) / kGlNumberThreads;
        int local[kPer];
        int sum = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int c = tid * per + q;
            local[q] = (q < per && c < P) ? (int)s_size[c] : 0;
            sum += local[q];
        }
        int run = scan(sum);
        int32_t *mbase = p.mbase + (int64_t)bh * (npad + 1), *csize = p.csize + (int64_t)bh * npad;
        int32_t *counts_bh = p.counts + (int64_t)bh * p.cap;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int c = tid * per + q;
            if (q < per && c < P) {
                mbase[c] = run;
                csize[c] = local[q];
                if (c < p.cap) counts_bh[c] = local[q];
                s_size[c] = (unsigned short)run;      // n <= 32768: a slot index fits 16 bits
                run += local[q];
            }
        }
        if (tid == 0) {
            p.nclusters[bh] = P;
            p.comp_lens[bh] = (P <= p.cap) ? P : -1;
        }
    }
    __syncthreads();
    for (int j0 = tid; j0 < n; j0 += 8 * kGlNumberThreads) {
        int t[8], pl[8], at[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + q * kGlNumberThreads;
            t[q] = j < n ? join[j] : 0;
            pl[q] = j < n ? place[j] : kGlLeader;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + q * kGlNumberThreads;
            at[q] = j < n ? lead[(pl[q] & kGlLeader) ? j : (j & ~63) + (pl[q] >> 8)] + ((pl[q] & kGlLeader) ? 0 : (pl[q] & 0x7F)) : 0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + q * kGlNumberThreads;
            if (j < n) order[(int)s_size[cluster_of(t[q])] + at[q]] = j;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// sum: Eq. 3.  16 lanes per cluster, members in row order.
template <typename TO>
__global__ __launch_bounds__(256) void glob_sum_kernel(GlobParams p) {
    const int bh = blockIdx.y, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int npad = p.nbp * kGlBlock;
    const int P = min(p.nclusters[bh], p.cap);
    const int cl = blockIdx.x * 16 + threadIdx.x / 16, c = threadIdx.x % 16;
    if (cl >= P) return;
    const bf16_t *Kbh = p.K + b * p.stride_b + h * p.stride_h + 8 * c;
    const bf16_t *Vbh = p.V + b * p.stride_b + h * p.stride_h + 8 * c;
    const int32_t *order = p.order + (int64_t)bh * npad + p.mbase[(int64_t)bh * (npad + 1) + cl];
    const int size = p.csize[(int64_t)bh * npad + cl];
    float ka[8], va[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) ka[e] = va[e] = 0.f;
    const int first_lane = (threadIdx.x & (kWave - 1)) & ~15;
    constexpr int kRows = 8;      // in flight: a cluster of a hundred rows is the kernel's tail, its trips to memory are what that costs
    for (int t0 = 0; t0 < size; t0 += 16) {
        const int members = min(16, size - t0);
        const int mine = (c < members) ? order[t0 + c] : 0;      // sixteen members in one load
        for (int u0 = 0; u0 < members; u0 += kRows) {
            uint4 kk[kRows], vv[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int64_t row = __shfl(mine, first_lane + u0 + u, kWave);
                if (u0 + u < members) {
                    kk[u] = *reinterpret_cast<const uint4 *>(Kbh + row * p.stride_n);
                    vv[u] = *reinterpret_cast<const uint4 *>(Vbh + row * p.stride_n);
                }
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                if (u0 + u < members) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        ka[2 * e] += bf16_lo(dword_of(kk[u], e)); ka[2 * e + 1] += bf16_hi(dword_of(kk[u], e));
                        va[2 * e] += bf16_lo(dword_of(vv[u], e)); va[2 * e + 1] += bf16_hi(dword_of(vv[u], e));
                    }
                }
            }
        }
    }
    // 1/size: a row of size 1 is passed on unchanged
    const float inv = (size > 1) ? 1.0f / (float)size : 1.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) { ka[e] *= inv; va[e] *= inv; }
    TO *Kc = reinterpret_cast<TO *>(p.Kc) + ((int64_t)bh * p.cap + cl) * kGlD + 8 * c;
    TO *Vc = reinterpret_cast<TO *>(p.Vc) + ((int64_t)bh * p.cap + cl) * kGlD + 8 * c;
    store8(Kc, ka);
    store8(Vc, va);
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
    const size_t nbp = (size_t)(N_max + kGlBlock - 1) / kGlBlock, npad = nbp * kGlBlock, nseg = (nbp + kGlSegment - 1) / kGlSegment;
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
    p.nseg = (p.nbp + kGlSegment - 1) / kGlSegment;
    p.tany = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * p.nseg * 8 * BH, 256);
    p.tuns = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * p.nseg * 8 * BH, 256);
    p.state = reinterpret_cast<unsigned long long *>(rest + o); o += align_up((size_t)p.nbp * 16 * BH, 256);
    p.polls = a.tune.global_polls;

    hipLaunchKernelGGL(glob_norms_kernel, dim3((unsigned)(npad / 16), (unsigned)BH), dim3(256), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int njg = (p.nbp + kGlPairWaves - 1) / kGlPairWaves;
    int items = 0;      // see the kernel: group JG has JG / 16 + 1 segments
    for (int jg = 0; jg < njg; ++jg) items += jg / 16 + 1;
    hipLaunchKernelGGL(glob_pairs_kernel, dim3((unsigned)items, (unsigned)BH), dim3(kGlPairWaves * kWave), 0, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(glob_decide_kernel, dim3((unsigned)(p.nbp * BH)), dim3(kWave), 0, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t dyn = npad * sizeof(unsigned short);
    if (dyn > 48 * 1024) {   // a host-side setting of the kernel (per device), not a stream operation
        int dev = 0;
        e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        static std::mutex mu;
        static bool raised[64];
        if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lock(mu);
        if (!raised[dev]) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(glob_number_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    hipLaunchKernelGGL(glob_number_kernel, dim3((unsigned)BH), dim3(kGlNumberThreads), dyn, stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int max_clusters = a.N_max < a.cap ? a.N_max : a.cap;
    const dim3 grid_sum((unsigned)((max_clusters + 15) / 16), (unsigned)BH);
    if (p.out_is_bf16) hipLaunchKernelGGL((glob_sum_kernel<bf16_t>), grid_sum, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((glob_sum_kernel<float>), grid_sum, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace sc
