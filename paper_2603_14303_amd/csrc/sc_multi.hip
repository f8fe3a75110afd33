// sc_multi_attn: Proportional Attention for a block of query rows (paper Sec. 2.4, Eq. 4 with
// Q in R^{n x d}):   O[j] = softmax(Q[j] K_c^T * scale + ln s) V_c   for every query row j, no mask
// (sc_multi_attn_tail: over cache and tail, optionally with the causal mask of the rows' own tokens).
//
// Fast path (bf16 queries and cache, d = 128) on the matrix cores.  The query rows that share a KV head -- (query j, head g of
// the group), nq * G of them -- are the columns of 32 x 32 product tiles, the cache rows are cut into splits:
//   multi_wave_kernel   few query rows: every wavefront of a workgroup holds the same 32 and takes cache rows of its own;
//   multi_block_kernel  more: the wavefronts of a workgroup hold 32 query rows each and share tiles of cache rows in LDS.
// Both form S^T = K Q^T and O^T += V^T P^T, so that a query row stays on one lane pair from the logits to the output, and
// write one partial (sums, maximum, denominator) per query row and split; multi_attn_combine_kernel folds them.  Two launches instead of a
// hand-over inside the kernel: the call is for several rows at once, a few microseconds of launch matter less than for
// single-row decode.  With one split the first kernel writes the outputs itself.
//
// Everything else (fp32, d = 64) goes row by row through the decode kernels.
#include "sc_device.h"
#include "sc_host.h"

namespace sc {

constexpr int kMqD = 128;
constexpr int kMqWaves = 4;
constexpr int kMqMaxSplits = 64;
constexpr int kMqPart = kMqD + 4;                 // floats per partial row: acc[128], m, l, pad
constexpr float kMqLog2e = 1.4426950408889634f;
constexpr float kMqLn2 = 0.6931471805599453f;

struct MqParams {
    const bf16_t *Q;          // [nq, B, Hq, 128]
    const bf16_t *Kc, *Vc;    // [B, Hkv, cap, 128]
    const int32_t *counts, *comp_lens;
    const bf16_t *Kt, *Vt;    // uncompressed tail [B, Hkv, tail_cap, 128], or NULL
    const int32_t *tail_lens; // [B]
    int tail_cap, causal;     // causal: the last nq tail rows are the query rows' own tokens
    int nq, cap, B, Hq, Hkv, G;
    float scale_log2;
    float *part;              // [B*Hkv*row_blocks][max_splits][part_rows][kMqPart]
    int row_blocks, max_splits, min_rows;
    int block_rows;           // query rows per workgroup: 32 (multi_wave_kernel) or 128 (multi_block_kernel)
    int part_rows;            // rows of a partial: as many as the workgroups have query rows, block_rows at most
    void *O;                  // [nq, B, Hq, 128]
    int o_is_bf16;
    float *lse;               // [nq, B, Hq] or NULL
};

__device__ __forceinline__ int mq_splits_for(int rows, int max_splits, int min_rows) {
    const int s = (rows + min_rows - 1) / min_rows;
    return s < 1 ? 1 : (s > max_splits ? max_splits : s);
}
typedef __bf16 mq_bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ mq_bf16x8 mq_op8(const uint4 &u) { return __builtin_bit_cast(mq_bf16x8, u); }
__device__ __forceinline__ float mq_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ------------------------------------------------------------------------------------------------
typedef float mb_float16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ void mq_wave_handover() {   // LDS traffic of one wavefront executes in order: only the compiler must not reorder
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
typedef unsigned int mq_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 mq_load16(__amdgpu_buffer_rsrc_t src, int off) {
    const mq_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(src, off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float mq_halves_sum(float x) {      // over lane and lane ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float mq_halves_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Softmax of T tiles of 32 x 32 logits in units of log 2: lane l holds query row l % 32 and, of a tile, the cache rows
// 8 (i / 4) + 4 (l / 32) + i % 4.
// The reference follows the maximum at once.  A weight enters the second product as two bf16 parts, which round it at about
// 2^-18 unless it is a power of two: relative to the true maximum the largest weight is 1 and costs nothing.  (A reference
// that moves only when the maximum has grown 2^8-fold saves most of the rescaling, 4 % of the block kernel's time, and
// rounds the largest weights as well: rms error with fp32 outputs, 5 900 rows, scale 0.3, 8.8e-7 -> 1.9e-6.)
template <int T>
__device__ __forceinline__ void block_grow(const mb_float16 (&s)[T], float &m_run, float &l_run, mb_float16 (&o)[4]) {
    float mx = s[0][0];
#pragma unroll
    for (int i = 1; i < 16 * T; ++i) mx = fmaxf(mx, s[i >> 4][i & 15]);
    mx = mq_halves_max(mx);
    if (ballot64(mx > m_run) != 0ull) {
        const float m_new = fmaxf(m_run, mx);
        const float alpha = (m_new == -INFINITY) ? 1.0f : mq_exp2(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
    }
}
// Dot products of one tile -> logits; bias: log2 of the sizes of the tile's rows in LDS, -inf for a row that does not exist.  (Added
// here and not started from in the accumulator: there every one of the eight steps of the product would round a larger sum.)
__device__ __forceinline__ void block_logits(mb_float16 &s, float scale_log2, const float *bias, int half) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 bb = *reinterpret_cast<const float4 *>(bias + 8 * k + 4 * half);
        s[4 * k] = fmaf(s[4 * k], scale_log2, bb.x); s[4 * k + 1] = fmaf(s[4 * k + 1], scale_log2, bb.y);
        s[4 * k + 2] = fmaf(s[4 * k + 2], scale_log2, bb.z); s[4 * k + 3] = fmaf(s[4 * k + 3], scale_log2, bb.w);
    }
}
// The probabilities of one tile as B operands of the second product: leading parts and remainders, a pair per 16 cache rows.
__device__ __forceinline__ void block_probabilities(const mb_float16 &s, float m_run, float &l_run, uint4 (&ph)[2], uint4 (&pl)[2]) {
    const float shift = (m_run == -INFINITY) ? 0.f : m_run;
    uint32_t h[8], l[8];
    float psum = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float e0 = mq_exp2(s[2 * k] - shift), e1 = mq_exp2(s[2 * k + 1] - shift);
        h[k] = pack_bf16x2(e0, e1);
        l[k] = pack_bf16x2(e0 - bf16_lo(h[k]), e1 - bf16_hi(h[k]));
        psum += e0 + e1;
    }
    l_run += psum;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ph[u] = make_uint4(h[4 * u], h[4 * u + 1], h[4 * u + 2], h[4 * u + 3]);
        pl[u] = make_uint4(l[4 * u], l[4 * u + 1], l[4 * u + 2], l[4 * u + 3]);
    }
}
// four columns of a finished query row: sums x over the denominator l
__device__ __forceinline__ void mq_store_row4(const MqParams &p, int64_t orow, int col, const float4 &x, float m_log2, float l, bool write_lse) {
    const float inv = (l > 0.f) ? 1.0f / l : 0.f;
    store_row4(p.O, p.o_is_bf16, orow * kMqD + col, make_float4(x.x * inv, x.y * inv, x.z * inv, x.w * inv));
    if (write_lse && p.lse) p.lse[orow] = (l > 0.f) ? (m_log2 + __log2f(l)) * kMqLn2 : -INFINITY;
}

// ------------------------------------------------------------------------------------------------
// A few query rows (nq * G <= 32 per KV head, more in small calls): multi_wave_kernel.
//
// The four wavefronts of a workgroup hold the same 32 query rows and take alternate steps of 32 cache rows, each in an
// LDS area of its own: no barrier until the end, and a wavefront's 16 KB of loads for the next step fly while it works on
// this one (64 KB in flight per workgroup; what bounds the kernel is the trip to memory and the chain after it).
// Arithmetic and operand layouts are those of multi_block_kernel below; the wavefronts fold through LDS at the end.
// 8 heads x 32 query rows behind 5 385 + 108 rows (22.5 MB): 15.4 us per call with the second kernel, 24.0 with 16 query rows per
// workgroup in registers only, whose 256 vector registers left nothing in flight while a step was worked on; 5 400 rows without
// a tail 14.5 / 14.7.
constexpr int kMwThreads = kMqWaves * kWave;
constexpr int kMwRows = 32;                       // query rows per workgroup
constexpr int kMwStep = 32;                       // cache rows per wavefront and step
constexpr int kMwKRowBytes = 2 * kMqD + 16;
constexpr int kMwAccStride = kMqD + 4;            // floats per query row when the wavefronts fold
constexpr int kMwKBytes = kMwStep * kMwKRowBytes, kMwVBytes = kMqD * kMwStep * 2;
static_assert(kMwRows * kMwAccStride * 4 <= kMwKBytes + kMwVBytes, "the fold reuses the tiles");

// 16-byte slot of LDS row d (= column d of V, 32 cache rows in four slots) that holds slot s: the sixteen rows of an
// operand read then cover all banks
__device__ __forceinline__ int vt_slot32(int d, int s) { return (s ^ ((d >> 2) ^ (d >> 4))) & 3; }

template <bool TAIL>
__global__ __launch_bounds__(kMwThreads, 2) void multi_wave_kernel(MqParams p) {
    __shared__ __attribute__((aligned(16))) char s_tiles[kMqWaves][kMwKBytes + kMwVBytes];
    __shared__ __attribute__((aligned(16))) float s_bias[kMqWaves][kMwStep];
    __shared__ float s_m[kMqWaves][kMwRows], s_l[kMqWaves][kMwRows];

    const int n_bh = p.B * p.Hkv;
    const int bh_i = (int)blockIdx.x % n_bh, rest = (int)blockIdx.x / n_bh;
    const int rb = rest % p.row_blocks, split = rest / p.row_blocks;
    const int b = bh_i / p.Hkv, h = bh_i - b * p.Hkv;
    const int64_t bh = bh_i;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = lane & 31, half = lane >> 5;
    const int rows_c = __builtin_amdgcn_readfirstlane(min(max(p.comp_lens[bh], 0), p.cap));
    const int rows_t = TAIL ? __builtin_amdgcn_readfirstlane(min(max(p.tail_lens[b], 0), p.tail_cap)) : 0;
    const int rows_total = rows_c + rows_t;
    const int S = mq_splits_for(rows_total, p.max_splits, p.min_rows);
    if (split >= S) return;
    int per = (rows_total + S - 1) / S;
    per = (per + kMwStep - 1) / kMwStep * kMwStep;
    const int r0 = min(split * per, rows_total), r1 = min(r0 + per, rows_total);

    const bf16_t *Kbh = p.Kc + bh * (int64_t)p.cap * kMqD;
    const bf16_t *Vbh = p.Vc + bh * (int64_t)p.cap * kMqD;
    const int32_t *cnt_bh = p.counts + bh * (int64_t)p.cap;
    const bf16_t *Ktbh = TAIL ? p.Kt + bh * (int64_t)p.tail_cap * kMqD : nullptr;
    const bf16_t *Vtbh = TAIL ? p.Vt + bh * (int64_t)p.tail_cap * kMqD : nullptr;

    // ---- a step's loads: lane (g4, c4) brings piece c4 of the K rows 4 r + g4 and of the V rows 16 (r / 4) + 4 g4 + r % 4
    const int c4 = lane & 15, g4 = lane >> 4;
    uint4 kx[8], vx[8];
    int cx = 0;
    auto fetch = [&](int base) {      // (base and the bounds are the same for the whole wavefront)
        const bool plain = base + kMwStep <= min(r1, rows_c);
        if (plain) {
            const bf16_t *k0 = Kbh + ((int64_t)base + g4) * kMqD + 8 * c4, *v0 = Vbh + ((int64_t)base + 4 * g4) * kMqD + 8 * c4;
#pragma unroll
            for (int r = 0; r < 8; ++r) kx[r] = load16_stream(k0 + 4 * r * kMqD);
            if (lane < kMwStep) cx = cnt_bh[base + lane];
#pragma unroll
            for (int r = 0; r < 8; ++r) vx[r] = load16_stream(v0 + (16 * (r >> 2) + (r & 3)) * kMqD);
        } else {
            auto piece = [&](const bf16_t *main, const bf16_t *tail, int row) {
                if (row >= r1) return make_uint4(0, 0, 0, 0);
                return load16_stream(((TAIL && row >= rows_c) ? tail + (int64_t)(row - rows_c) * kMqD : main + (int64_t)row * kMqD) + 8 * c4);
            };
#pragma unroll
            for (int r = 0; r < 8; ++r) kx[r] = piece(Kbh, Ktbh, base + 4 * r + g4);
            const int row = base + c;
            cx = (row >= r1) ? 0 : ((TAIL && row >= rows_c) ? 1 : cnt_bh[row]);
#pragma unroll
            for (int r = 0; r < 8; ++r) vx[r] = piece(Vbh, Vtbh, base + 16 * (r >> 2) + 4 * g4 + (r & 3));
        }
    };
    int base = r0 + wave * kMwStep;
    if (base < r1) fetch(base);

    const int R = rb * kMwRows + c;
    const bool valid = R < p.nq * p.G;
    const int j = valid ? R / p.G : 0, g = valid ? R - j * p.G : 0;
    uint4 q[8];
    {
        const bf16_t *qp = p.Q + (((int64_t)j * p.B + b) * p.Hq + (int64_t)h * p.G + g) * kMqD + 8 * half;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) q[ks] = valid ? *reinterpret_cast<const uint4 *>(qp + 16 * ks) : make_uint4(0, 0, 0, 0);
    }
    const bool masked = TAIL && p.causal;
    const int limit = masked ? rows_c + max(0, rows_t - p.nq + 1 + j) : rows_total;   // rows [0, limit) are visible

    float m_run = -INFINITY, l_run = 0.f;      // of the lane's query row; l: this half's share
    mb_float16 o[4];                           // o[dt][i]: column 32 dt + 8 (i / 4) + 4 half + i % 4 of the lane's query row
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;

    char *kt = s_tiles[wave], *vt = kt + kMwKBytes;
    while (base < r1) {
#pragma unroll
        for (int r = 0; r < 8; ++r) *reinterpret_cast<uint4 *>(kt + (4 * r + g4) * kMwKRowBytes + 16 * c4) = kx[r];
        if (lane < kMwStep) s_bias[wave][lane] = (cx > 0) ? __log2f((float)cx) : -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t d0 = dword_of(vx[4 * u], e >> 1), d1 = dword_of(vx[4 * u + 1], e >> 1);
                const uint32_t d2 = dword_of(vx[4 * u + 2], e >> 1), d3 = dword_of(vx[4 * u + 3], e >> 1);
                const uint2 w = (e & 1) ? make_uint2(pack_hi(d0, d1), pack_hi(d2, d3)) : make_uint2(pack_lo(d0, d1), pack_lo(d2, d3));
                const int d = 8 * c4 + e;      // rows 4 g4 .. + 3 of group u: operand half g4 % 2, first or second four of it g4 / 2
                *reinterpret_cast<uint2 *>(vt + d * (kMwStep * 2) + 16 * vt_slot32(d, 2 * u + (g4 & 1)) + 8 * (g4 >> 1)) = w;
            }
        mq_wave_handover();
        const int next = base + kMqWaves * kMwStep;
        if (next < r1) fetch(next);
        mb_float16 s[1] = {};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const uint4 a = *reinterpret_cast<const uint4 *>(kt + c * kMwKRowBytes + 32 * ks + 16 * half);
            s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(q[ks]), s[0], 0, 0, 0);
        }
        block_logits(s[0], p.scale_log2, s_bias[wave], half);
        if (masked && base + kMwStep > rows_c) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[0][i] = (base + 8 * (i >> 2) + 4 * half + (i & 3) < limit) ? s[0][i] : -INFINITY;
        }
        uint4 ph[2], pl[2];
        block_grow<1>(s, m_run, l_run, o);
        block_probabilities(s[0], m_run, l_run, ph, pl);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const int d = 32 * dt + c;
                const uint4 a = *reinterpret_cast<const uint4 *>(vt + d * (kMwStep * 2) + 16 * vt_slot32(d, 2 * u + half));
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(ph[u]), o[dt], 0, 0, 0);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(pl[u]), o[dt], 0, 0, 0);
            }
        mq_wave_handover();     // the tiles are rewritten in the next step
        base = next;
    }

    // ---- fold the wavefronts
    l_run = mq_halves_sum(l_run);
    if (half == 0) { s_m[wave][c] = m_run; s_l[wave][c] = l_run; }
    float *acc = reinterpret_cast<float *>(s_tiles[wave]);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<float4 *>(acc + c * kMwAccStride + 32 * dt + 8 * k + 4 * half) =
                make_float4(o[dt][4 * k], o[dt][4 * k + 1], o[dt][4 * k + 2], o[dt][4 * k + 3]);
    __syncthreads();
    // thread: piece tid % 32 of the query rows tid / 32 + 8 r
    const int q4 = tid & 31;
    float *part = p.part + (((bh * p.row_blocks + rb) * (int64_t)p.max_splits + split) * p.part_rows) * kMqPart;
#pragma unroll
    for (int r = 0; r < kMwRows / 8; ++r) {
        const int row = (tid >> 5) + 8 * r, Rr = rb * kMwRows + row;
        float mw = -INFINITY;
#pragma unroll
        for (int w = 0; w < kMqWaves; ++w) mw = fmaxf(mw, s_m[w][row]);
        const float m_safe = (mw == -INFINITY) ? 0.f : mw;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < kMqWaves; ++w) {
            const float f = mq_exp2(s_m[w][row] - m_safe);
            const float4 t = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(s_tiles[w]) + row * kMwAccStride + 4 * q4);
            x.x = fmaf(t.x, f, x.x); x.y = fmaf(t.y, f, x.y); x.z = fmaf(t.z, f, x.z); x.w = fmaf(t.w, f, x.w);
            l = fmaf(s_l[w][row], f, l);
        }
        if (Rr >= p.nq * p.G) continue;
        if (p.max_splits == 1) {
            const int jr = Rr / p.G, gr = Rr - jr * p.G;
            mq_store_row4(p, ((int64_t)jr * p.B + b) * p.Hq + (int64_t)h * p.G + gr, 4 * q4, x, mw, l, q4 == 0);
        } else {
            *reinterpret_cast<float4 *>(part + (int64_t)row * kMqPart + 4 * q4) = x;
            if (q4 == 0) *reinterpret_cast<float2 *>(part + (int64_t)row * kMqPart + kMqD) = make_float2(mw, l);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Many query rows (a chunk of prompt behind a compressed cache): multi_block_kernel.
//
// The four wavefronts of a workgroup own 32 query rows EACH and share
// tiles of 64 cache rows in LDS, double-buffered (the next tile's loads fly while this one is worked on):
//   * S^T = K Q^T with v_mfma_f32_32x32x16_bf16: cache rows are the A operand (LDS rows of 256 + 16 bytes, free of bank
//     conflicts), query rows the B operand, which stays in registers.
//   * the result has the query row on the lane (l % 32) and sixteen cache rows in its registers: the running maximum and sum
//     are one value per lane, a rescale is a multiplication by a lane's own factor, and the probabilities already are
//     the B operand of  O^T += V^T P^T  (index (l / 32, j) of both operands stands for cache row 16 u + 8 (j / 4) + 4 (l / 32) + j % 4).
//   * V^T comes from an LDS tile that is transposed while it is parked: a thread brings sixteen bytes of four
//     neighbouring rows, regroups them with byte permutes and stores eight pieces of four cache rows.  The 16-byte slots of an
//     LDS row are XORed with a function of the row (vt_slot) that keeps operand reads free of conflicts.
// P enters as two bf16 parts (leading part and remainder), i.e. with 16 bits of every weight but the largest of a stretch, which
// is 1.  A stretch (the rows of one split) is one sum in row order: level with four wavefronts that take a quarter each at
// 1 500 rows (rms error with fp32 outputs 2.07e-6 / 2.05e-6 at scale 1/sqrt(d), 8.4e-7 / 8.2e-7 at 0.3), above it where one
// split takes 8 192 (2.4e-6 / 2.1e-6 and 1.3e-6 / 8.7e-7): fewer largest weights, longer sums.
// Bound by the overlap of two wavefronts per SIMD: per 64 cache rows a wavefront spends 48 matrix instructions of 32 cycles and as many cycles
// of vector work on the logits of its lanes, and a third of its time it waits for loads and at barriers (counters: 46 % of the
// time matrix, 50 % vector).  8 heads x 2048 query rows (nq = 512, G = 4) x 5 900 cache rows, 49 GFLOP: 238 us with 32 rows
// per workgroup and no sharing of tiles (208 TFLOP/s), now 100 us with the second kernel (496 TFLOP/s).
constexpr int kMbWaves = 4;
constexpr int kMbThreads = kMbWaves * kWave;
constexpr int kMbRows = 32 * kMbWaves;            // query rows per workgroup
constexpr int kMbTile = 64;                       // cache rows per LDS tile
constexpr int kMbKRowBytes = 2 * kMqD + 16;

// 16-byte slot of LDS row d (= column d of V) that holds slot s of the row: rows 0..15 of an operand read fall on different
// banks (bits 1..3 of d), and so do the pieces that the sixteen lanes of a row write (bits 4..6)
__device__ __forceinline__ int vt_slot(int d, int s) { return (s ^ ((d >> 1) ^ (d >> 4))) & 7; }

template <bool TAIL>
__global__ __launch_bounds__(kMbThreads, 2) void multi_block_kernel(MqParams p) {
    __shared__ __attribute__((aligned(16))) char s_k[2][kMbTile * kMbKRowBytes];
    __shared__ __attribute__((aligned(16))) char s_v[2][kMqD * kMbTile * 2];
    __shared__ __attribute__((aligned(16))) float s_bias[2][kMbTile];

    // one-dimensional grid, (sequence, head) fastest: with a multiple of 8 of them a head stays on one XCD and its cache
    // rows in that XCD's L2
    const int n_bh = p.B * p.Hkv;
    const int bh_i = (int)blockIdx.x % n_bh, rest = (int)blockIdx.x / n_bh;
    const int rb = rest % p.row_blocks, split = rest / p.row_blocks;
    const int b = bh_i / p.Hkv, h = bh_i - b * p.Hkv;
    const int64_t bh = bh_i;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = lane & 31, half = lane >> 5;
    const int rows_c = __builtin_amdgcn_readfirstlane(min(max(p.comp_lens[bh], 0), p.cap));
    const int rows_t = TAIL ? __builtin_amdgcn_readfirstlane(min(max(p.tail_lens[b], 0), p.tail_cap)) : 0;
    const int rows_total = rows_c + rows_t;
    const int S = mq_splits_for(rows_total, p.max_splits, p.min_rows);
    if (split >= S) return;
    int per = (rows_total + S - 1) / S;
    per = (per + kMbTile - 1) / kMbTile * kMbTile;
    // (the divisions above leave the bounds in vector registers: back to scalars, the descriptors below need them there)
    const int r0 = __builtin_amdgcn_readfirstlane(min(split * per, rows_total));
    // cache rows beyond the last query row's own token are masked for the whole workgroup
    const int n_rows_q = p.nq * p.G;
    const bool masked = TAIL && p.causal;
    const int j_last = (min((rb + 1) * kMbRows, n_rows_q) - 1) / p.G;
    const int seen = masked ? rows_c + max(0, rows_t - p.nq + 1 + j_last) : rows_total;
    const int r1 = __builtin_amdgcn_readfirstlane(min(min(r0 + per, rows_total), seen));

    const bf16_t *Kbh = p.Kc + bh * (int64_t)p.cap * kMqD;
    const bf16_t *Vbh = p.Vc + bh * (int64_t)p.cap * kMqD;
    const int32_t *cnt_bh = p.counts + bh * (int64_t)p.cap;
    const bf16_t *Ktbh = TAIL ? p.Kt + bh * (int64_t)p.tail_cap * kMqD : nullptr;
    const bf16_t *Vtbh = TAIL ? p.Vt + bh * (int64_t)p.tail_cap * kMqD : nullptr;

    const int R = rb * kMbRows + wave * 32 + c;
    const bool valid = R < n_rows_q;
    const int j = valid ? R / p.G : 0, g = valid ? R - j * p.G : 0;
    const bool wave_live = rb * kMbRows + wave * 32 < n_rows_q;
    uint4 q[8];
    {
        const bf16_t *qp = p.Q + (((int64_t)j * p.B + b) * p.Hq + (int64_t)h * p.G + g) * kMqD + 8 * half;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) q[ks] = valid ? *reinterpret_cast<const uint4 *>(qp + 16 * ks) : make_uint4(0, 0, 0, 0);
    }
    const int limit = (masked && valid) ? rows_c + max(0, rows_t - p.nq + 1 + j) : rows_total;   // rows [0, limit) are visible
    int limit_min = limit;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) limit_min = min(limit_min, __shfl_xor(limit_min, off, kWave));
    limit_min = __builtin_amdgcn_readfirstlane(limit_min);

    // ---- tiles: a thread brings one 16-byte piece of the rows 4 lr .. 4 lr + 3 of K and of V.  A tile of merged rows or of tail
    // rows comes through descriptors that end at its last row (zeros beyond: no predicates, no 64-bit addresses per
    // lane); only the one tile that holds both picks its rows one by one.
    const int lc = tid & 15, lr = tid >> 4;
    const int voff = lr * (4 * 2 * kMqD) + 16 * lc;
    uint4 kx[4], vx[4];
    float bx = 0.f;
    auto row_piece = [&](const bf16_t *main, const bf16_t *tail, int row) {
        if (row >= r1) return make_uint4(0, 0, 0, 0);
        const bf16_t *src = (TAIL && row >= rows_c) ? tail + (int64_t)(row - rows_c) * kMqD : main + (int64_t)row * kMqD;
        return *reinterpret_cast<const uint4 *>(src + 8 * lc);
    };
    auto fetch = [&](int base) {
        const int end = min(base + kMbTile, r1);
        const bool in_tail = TAIL && base >= rows_c;
        if (TAIL && !in_tail && end > rows_c) {
#pragma unroll
            for (int r = 0; r < 4; ++r) kx[r] = row_piece(Kbh, Ktbh, base + 4 * lr + r);
#pragma unroll
            for (int r = 0; r < 4; ++r) vx[r] = row_piece(Vbh, Vtbh, base + 4 * lr + r);
        } else {
            const int64_t first = (int64_t)(in_tail ? base - rows_c : base) * kMqD;
            const auto k_src = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((in_tail ? Ktbh : Kbh) + first), (short)0, (end - base) * 2 * kMqD, 0x00020000);
            const auto v_src = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((in_tail ? Vtbh : Vbh) + first), (short)0, (end - base) * 2 * kMqD, 0x00020000);
#pragma unroll
            for (int r = 0; r < 4; ++r) kx[r] = mq_load16(k_src, voff + 2 * kMqD * r);
#pragma unroll
            for (int r = 0; r < 4; ++r) vx[r] = mq_load16(v_src, voff + 2 * kMqD * r);
        }
        if (tid < kMbTile) {
            const int row = base + tid;
            const int cnt = (row >= r1) ? 0 : ((TAIL && row >= rows_c) ? 1 : cnt_bh[row]);
            bx = (cnt > 0) ? __log2f((float)cnt) : -INFINITY;
        }
    };
    auto park = [&](int buf) {
        char *kt = s_k[buf], *vt = s_v[buf];
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<uint4 *>(kt + (4 * lr + r) * kMbKRowBytes + 16 * lc) = kx[r];
        // cache rows 4 lr .. 4 lr + 3 = rows 4 qq .. of group tg: operand half qq % 2, first or second four of it qq / 2
        const int tg = lr >> 2, qq = lr & 3;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t d0 = dword_of(vx[0], e >> 1), d1 = dword_of(vx[1], e >> 1);
            const uint32_t d2 = dword_of(vx[2], e >> 1), d3 = dword_of(vx[3], e >> 1);
            const uint2 w = (e & 1) ? make_uint2(pack_hi(d0, d1), pack_hi(d2, d3)) : make_uint2(pack_lo(d0, d1), pack_lo(d2, d3));
            const int d = 8 * lc + e;
            *reinterpret_cast<uint2 *>(vt + d * (kMbTile * 2) + 16 * vt_slot(d, 2 * tg + (qq & 1)) + 8 * (qq >> 1)) = w;
        }
        if (tid < kMbTile) s_bias[buf][tid] = bx;
    };

    float m_run = -INFINITY, l_run = 0.f;      // of the lane's query row; l: this half's share
    mb_float16 o[4];                           // o[dt][i]: column 32 dt + 8 (i / 4) + 4 half + i % 4 of the lane's query row
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;

    if (r0 < r1) {
        fetch(r0);
        park(0);
    }
    __syncthreads();
    int buf = 0;
    for (int base = r0; base < r1; base += kMbTile, buf ^= 1) {
        const bool more = base + kMbTile < r1;
        if (more) fetch(base + kMbTile);
        if (wave_live) {
            const char *kt = s_k[buf], *vt = s_v[buf];
            __builtin_amdgcn_s_setprio(1);      // products first: 752 -> 729 us for eight calls of the shape above
            mb_float16 s[2] = {};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const uint4 a = *reinterpret_cast<const uint4 *>(kt + (32 * tt + c) * kMbKRowBytes + 32 * ks + 16 * half);
                    s[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(q[ks]), s[tt], 0, 0, 0);
                }
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) block_logits(s[tt], p.scale_log2, s_bias[buf] + 32 * tt, half);
            if (masked && base + kMbTile > limit_min) {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[tt][i] = (base + 32 * tt + 8 * (i >> 2) + 4 * half + (i & 3) < limit) ? s[tt][i] : -INFINITY;
            }
            __builtin_amdgcn_s_setprio(0);
            block_grow<2>(s, m_run, l_run, o);
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                uint4 ph[2], pl[2];
                block_probabilities(s[tt], m_run, l_run, ph, pl);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        const int d = 32 * dt + c;
                        const uint4 a = *reinterpret_cast<const uint4 *>(vt + d * (kMbTile * 2) + 16 * vt_slot(d, 2 * (2 * tt + u) + half));
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(ph[u]), o[dt], 0, 0, 0);
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mq_op8(a), mq_op8(pl[u]), o[dt], 0, 0, 0);
                    }
            }
        }
        if (more) park(buf ^ 1);      // (everybody left that buffer at the barrier that ended the previous tile)
        __syncthreads();
    }

    l_run = mq_halves_sum(l_run);
    if (!valid) return;
    if (p.max_splits == 1) {      // nothing to fold: the outputs themselves
        const int64_t orow = ((int64_t)j * p.B + b) * p.Hq + (int64_t)h * p.G + g;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                mq_store_row4(p, orow, 32 * dt + 8 * k + 4 * half, make_float4(o[dt][4 * k], o[dt][4 * k + 1], o[dt][4 * k + 2], o[dt][4 * k + 3]),
                              m_run, l_run, half == 0 && dt == 0 && k == 0);
        return;
    }
    float *part = p.part + (((bh * p.row_blocks + rb) * (int64_t)p.max_splits + split) * p.part_rows + wave * 32 + c) * kMqPart;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<float4 *>(part + 32 * dt + 8 * k + 4 * half) =
                make_float4(o[dt][4 * k], o[dt][4 * k + 1], o[dt][4 * k + 2], o[dt][4 * k + 3]);
    if (half == 0) { part[kMqD] = m_run; part[kMqD + 1] = l_run; }
}

// One wavefront per query row of a (sequence, KV head), four of them per workgroup.  The (m, l) of all splits are fetched
// in one trip (one split per lane) and turned into weights; a lane owns four output columns of the even or of the odd
// splits, and the first sixteen splits' pieces are requested together with the pairs, not after the weights are known.
constexpr int kMqCombineRows = 4;
__global__ __launch_bounds__(kMqCombineRows *kWave) void multi_attn_combine_kernel(MqParams p) {
    static_assert(kMqMaxSplits <= kWave, "one split per lane");
    const int lane = threadIdx.x & (kWave - 1);
    const int R = (int)blockIdx.x * kMqCombineRows + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);   // row inside the (sequence, KV head): j * G + g
    if (R >= p.nq * p.G) return;
    const int h = blockIdx.y, b = blockIdx.z;
    const int q4 = lane & 31, half = lane >> 5;
    const int64_t bh = (int64_t)b * p.Hkv + h;
    const int rows_total = min(max(p.comp_lens[bh], 0), p.cap) + (p.Kt ? min(max(p.tail_lens[b], 0), p.tail_cap) : 0);
    const int S = mq_splits_for(rows_total, p.max_splits, p.min_rows);
    const int rb = R / p.block_rows, row = R - rb * p.block_rows;
    const float *part = p.part + (((bh * p.row_blocks + rb) * (int64_t)p.max_splits) * p.part_rows + row) * kMqPart;
    const int64_t split_stride = (int64_t)p.part_rows * kMqPart;
    constexpr int kPass = 8;
    float4 v[kPass];
    auto load_pass = [&](int s0) {
#pragma unroll
        for (int k = 0; k < kPass; ++k) {
            const int s = s0 + 2 * k + half;
            v[k] = (s < S) ? *reinterpret_cast<const float4 *>(part + s * split_stride + 4 * q4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    const float2 ml = (lane < S) ? *reinterpret_cast<const float2 *>(part + lane * split_stride + kMqD) : make_float2(-INFINITY, 0.f);
    load_pass(0);
    float mx = ml.x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
    const float wgt = mq_exp2(ml.x - ((mx == -INFINITY) ? 0.f : mx));
    float l = ml.y * wgt;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off, kWave);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < S; s0 += 2 * kPass) {
        if (s0 != 0) load_pass(s0);
#pragma unroll
        for (int k = 0; k < kPass; ++k) {
            const float w = __shfl(wgt, (s0 + 2 * k + half) & (kWave - 1), kWave);      // beyond S: the weight of an empty split, times zeros
            acc.x = fmaf(v[k].x, w, acc.x); acc.y = fmaf(v[k].y, w, acc.y);
            acc.z = fmaf(v[k].z, w, acc.z); acc.w = fmaf(v[k].w, w, acc.w);
        }
    }
    acc.x += __shfl_xor(acc.x, 32, kWave); acc.y += __shfl_xor(acc.y, 32, kWave);
    acc.z += __shfl_xor(acc.z, 32, kWave); acc.w += __shfl_xor(acc.w, 32, kWave);
    if (half != 0) return;
    const int j = R / p.G, g = R - j * p.G;
    const int64_t orow = ((int64_t)j * p.B + b) * p.Hq + (int64_t)h * p.G + g;
    mq_store_row4(p, orow, 4 * q4, acc, mx, l, q4 == 0);
}

// ------------------------------------------------------------------------------------------------
constexpr int kMbMostRounds = 4;      // multi_block_kernel: splits end at this many workgroups per compute unit
static void mq_shape(int B, int Hq, int Hkv, int nq, int cap /* merged + tail rows */, int &row_blocks, int &max_splits, int &min_rows, int &block_rows) {
    const int G = Hq / Hkv;
    // Up to 32 query rows per KV head fit the lanes of every wavefront, and the wavefronts share out the cache rows.  More of
    // them are shared out themselves, 32 to a wavefront, so that a cache row is fetched once per 128 of them: that pays once
    // the products do, and not while a call waits for its cache rows on chains that are longer with fewer rows per workgroup and step.
    // us per call, first / second kernel / 16 or 32 rows per workgroup in registers, rows of a KV head x cache rows:
    //   8 heads   64 x 5 400  15.8 / 20.6 / 19.5   128  20.8 / 24.2 / 27.5   256  30.3 / 30.2 / 40.9   384  39.6 / 34.4 / 83.4
    //   8 heads, masked tail  64  17.4 / 21.1 / 27.3   128  24.0 / 24.7 / 42.7   160  30.0 / 28.9 / 48.6
    //   2 heads  160 x 5 400  15.7 / 18.7 / 17.3   256  16.2 / 21.6 / 19.1;  1 head  64 x 30 000  18.2 / 28.1 / 22.3   256  30.8 / 31.8 / 31.8
    //   32 heads  96 x 2 000  22.1 / 24.8 / 41.0   128  28.4 / 26.7 / 35.8;  64 heads  64 x 4 000  48.5 / 43.3 / 61.2
    //   128 heads  64 x 500  14.1 / 24.0 / 27.8 (one split, all workgroups at once, four steps)
    const int blocks = (nq * G + kMwRows - 1) / kMwRows;
    const int64_t groups = (int64_t)B * Hkv * blocks, steps = 3 * (int64_t)cap / (4 * kMqWaves * kMwStep);
    const bool wave = blocks <= 1 || (blocks <= 4 && (groups <= 96 || (groups <= 256 && steps <= 8))) || (blocks <= 8 && groups <= 16);
    block_rows = wave ? kMwRows : kMbRows;
    // (a single query row always takes the first kernel: sc_decode_attn's workspace has room for that route, whatever the knob says)
    if (nq > 1 && (tuning().multi_block_rows == kMwRows || tuning().multi_block_rows == kMbRows)) block_rows = tuning().multi_block_rows;
    row_blocks = (nq * G + block_rows - 1) / block_rows;
    min_rows = 128;
    const int by_cap = (int)(((int64_t)cap + min_rows - 1) / min_rows);      // never more splits than the capacity can feed
    const int most = max(1, min(kMqMaxSplits, by_cap));
    const int base = B * Hkv * row_blocks;
    if (block_rows == kMwRows) {
        // Bound by the trip to memory: three workgroups on four compute units have enough in flight, and every further split
        // only adds partials for the second kernel (32 rows, 8 heads x 5 500 cache rows: 14.7 us with 24 splits, 19.2 with 42).
        // From 97 (sequence, KV head, row block) groups on that is one split: 128 x 2 000 cache rows 29.9 us, 30.0 with three,
        // 192 x 500 14.8 / 20.5, 192 x 2 000 35.3 / 41.8, but 104 x 2 000 28.8 / 27.4 and 128 x 4 000 53.3 / 49.0.
        max_splits = max(1, min(most, max(1, tuning().multi_target_wgs) * 3 / 4 / base));
        return;
    }
    // A tile takes a workgroup alone on its compute unit 3.0 us, a pair of them 4.3 (see multi_block_kernel); a second
    // round of pairs takes as long as the first; partials cost the second kernel 3 us and 20 ns per workgroup
    // (1400 rows, 4 heads, 5 200 cache rows: 57 us with 12 splits = 1.03 rounds, 46 us with 11).  In units of 0.1 us:
    const int64_t units = max(1, tuning().multi_target_wgs);
    const int64_t tiles = max((int64_t)1, 3 * (int64_t)cap / (4 * kMbTile));       // the caches are hardly ever full
    int64_t best = INT64_MAX;
    max_splits = 1;
    for (int s = 1; s <= most; ++s) {
        const int64_t wgs = (int64_t)base * s;
        if (s > 1 && wgs > kMbMostRounds * units) break;         // what the workspace is sized for
        const int64_t per_tile = wgs <= units ? 30 : 43 * ((wgs + 2 * units - 1) / (2 * units));
        const int64_t cost = per_tile * ((tiles + s - 1) / s) + (s > 1 ? 30 + wgs / 5 : 0);
        if (cost < best) { best = cost; max_splits = s; }
    }
}

static int mq_part_rows(int nq, int G, int block_rows) { return min(nq * G, block_rows); }

static bool mq_fast(const MultiArgs &a) {
    return a.d == kMqD && a.q_dtype == DType::BF16 && a.kv_dtype == DType::BF16;
}

// Partials of the largest split count that mq_shape may choose, not of the one it does choose: the choice falls and rises with
// the shape, and a workspace sized for the longest chunk and the fullest cache has to serve every shorter one.  One split
// writes no partials.
size_t multi_fast_workspace_bytes(int B, int Hq, int Hkv, int nq, int cap) {
    int rb, ms, mr, br;
    mq_shape(B, Hq, Hkv, nq, cap, rb, ms, mr, br);
    const int64_t most = min((int64_t)kMqMaxSplits, ((int64_t)cap + mr - 1) / mr), units = max(1, tuning().multi_target_wgs);
    if (most <= 1) return 0;
    const int64_t wgs = min((int64_t)B * Hkv * rb * most, br == kMwRows ? units * 3 / 4 : kMbMostRounds * units);
    return align_up((size_t)wgs * mq_part_rows(nq, Hq / Hkv, br) * kMqPart * 4, 256);
}

size_t multi_workspace_bytes(int B, int Hq, int Hkv, int nq, int cap, int d) {
    const size_t fast = multi_fast_workspace_bytes(B, Hq, Hkv, nq, cap);
    const size_t generic = decode_workspace_bytes(B, Hq, Hkv, cap, d);   // (covers any cap)
    return fast > generic ? fast : generic;
}

hipError_t launch_multi(const MultiArgs &a, hipStream_t stream) {
    if (!mq_fast(a)) {
        // row by row through the decode kernels; their workspace starts with flags that must be zero
        hipError_t e = launch_decode_init_workspace(a.ws, decode_workspace_state_bytes(a.B, a.Hkv), stream);
        if (e != hipSuccess) return e;
        const size_t q_es = a.q_dtype == DType::BF16 ? 2 : 4, o_es = a.o_dtype == DType::BF16 ? 2 : 4;
        const size_t per = (size_t)a.B * a.Hq * a.d;
        for (int j = 0; j < a.nq; ++j) {
            DecodeArgs d;
            d.Q = reinterpret_cast<const char *>(a.Q) + j * per * q_es;
            d.q_dtype = a.q_dtype;
            d.Kc = a.Kc; d.Vc = a.Vc; d.kv_dtype = a.kv_dtype; d.cap = a.cap;
            d.counts = a.counts; d.comp_lens = a.comp_lens;
            d.Kt = a.Kt; d.Vt = a.Vt; d.tail_lens = a.tail_lens; d.tail_cap = a.tail_cap;   // (no mask: checked by the caller)
            d.B = a.B; d.Hq = a.Hq; d.Hkv = a.Hkv; d.d = a.d;
            d.scale = a.scale;
            d.O = reinterpret_cast<char *>(a.O) + j * per * o_es;
            d.o_dtype = a.o_dtype;
            d.lse = a.lse ? a.lse + (size_t)j * a.B * a.Hq : nullptr;
            d.ws = a.ws;
            e = launch_decode(d, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    return launch_multi_fast(a, stream);
}

hipError_t launch_multi_fast(const MultiArgs &a, hipStream_t stream) {
    MqParams p;
    p.Q = reinterpret_cast<const bf16_t *>(a.Q);
    p.Kc = reinterpret_cast<const bf16_t *>(a.Kc);
    p.Vc = reinterpret_cast<const bf16_t *>(a.Vc);
    p.counts = a.counts; p.comp_lens = a.comp_lens;
    p.Kt = reinterpret_cast<const bf16_t *>(a.Kt);
    p.Vt = reinterpret_cast<const bf16_t *>(a.Vt);
    p.tail_lens = a.tail_lens; p.tail_cap = a.Kt ? a.tail_cap : 0; p.causal = a.causal;
    p.nq = a.nq; p.cap = a.cap; p.B = a.B; p.Hq = a.Hq; p.Hkv = a.Hkv; p.G = a.Hq / a.Hkv;
    p.scale_log2 = a.scale * kMqLog2e;
    p.part = reinterpret_cast<float *>(a.ws);
    mq_shape(a.B, a.Hq, a.Hkv, a.nq, a.cap + p.tail_cap, p.row_blocks, p.max_splits, p.min_rows, p.block_rows);
    p.part_rows = mq_part_rows(a.nq, p.G, p.block_rows);
    p.O = a.O; p.o_is_bf16 = a.o_dtype == DType::BF16; p.lse = a.lse;
    const dim3 grid((unsigned)(p.max_splits * p.row_blocks * a.Hkv * a.B));
    if (p.block_rows == kMbRows) {
        if (p.Kt) hipLaunchKernelGGL((multi_block_kernel<true>), grid, dim3(kMbThreads), 0, stream, p);
        else hipLaunchKernelGGL((multi_block_kernel<false>), grid, dim3(kMbThreads), 0, stream, p);
    } else {
        if (p.Kt) hipLaunchKernelGGL((multi_wave_kernel<true>), grid, dim3(kMwThreads), 0, stream, p);
        else hipLaunchKernelGGL((multi_wave_kernel<false>), grid, dim3(kMwThreads), 0, stream, p);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.max_splits == 1) return e;      // one split: the outputs are written already
    hipLaunchKernelGGL(multi_attn_combine_kernel, dim3((a.nq * p.G + kMqCombineRows - 1) / kMqCombineRows, a.Hkv, a.B),
                       dim3(kMqCombineRows * kWave), 0, stream, p);
    return hipGetLastError();
}

}  // namespace sc
