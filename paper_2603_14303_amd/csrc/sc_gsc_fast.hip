// Fast path of sc_gsc_merge for bf16 keys/values with head dim 128 (paper Sec. 2.3 Alg. 1 / Eq. 2 and
// Sec. 2.4 Eq. 3).
//
// Two launches:
//   plan      cuts every sequence into windows: whole chunks (each with its closing delimiter) of at most 128 rows in all, or one
//             chunk that is longer.  Independent per 1024 rows of a sequence, shared by the heads.
//   compress  reads K and V once and writes the merged rows to their final place.  One workgroup of four wavefronts per window and
//             head.  The keys are parked in LDS, the values wait in registers.  All pairwise cosines inside the chunks come from a
//             Gram matrix on the matrix cores, are compared with tau (decisions inside +-1e-4 of tau are redone in fp64 where
//             they matter) and filed as a bit matrix, on which the seed set of Alg. 1 is found as the fixed point of the
//             first-fit rule (a few bit operations per application; seed by seed as the fallback).  A delimiter is a
//             one-row chunk, so the seeds in row order ARE the output rows of the window.  Their number is published at once,
//             and the number of rows before the window is put together from what the windows before it have published
//             while the cluster means are formed: a second matrix product, (128 columns x window rows) keys or values times
//             (window row x output row) 0/1 membership, fp32 accumulate.
// A chunk longer than a window runs over several 128-row blocks, its seeds re-read through L2, and its values are read once more for
// the means.
//
// Bounds: a window's chain (rows in, Gram product, decisions, the rows before, means, rows out), some 13 us with all places of the chip
// taken, and the bytes of K, V and the merged rows next (8 heads x 131072 tokens, bf16: 537 MB in, a tenth of it out); fp64
// pairs where tau lies inside the band of the similarities, the chain of blocks in long chunks.  Up to a few hundred workgroups it is one
// window's chain alone.
// Merged rows that are written once, to their final place, and a decision by one wavefront with the pairs shared by four, against
// provisional rows that a second launch moves, and one wavefront per 64-row task (us per call with its sc_segment): 8 heads x 32768
// 54.5 -> 49.5, 8 x 131072 178 -> 168, 32 sequences of 8192 to 16384 x 4 heads, tau inside the band, 326 -> 267, 4 x 8 x 32768, tau
// inside the band, 290 -> 196.
#include "sc_device.h"
#include "sc_gsc_params.h"
#include "sc_gsc_words.h"
#include "sc_host.h"

namespace sc {

typedef __bf16 bf16x8f_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kFastD = 128;
constexpr int kWinWaves = 4;
constexpr int kWinThreads = kWinWaves * kWave;
constexpr int kWinRows = 128;            // rows of a window
constexpr int kAheadWgs = 512;           // workgroups that decide long chunks ahead of the windows (one per head if there are more heads)
constexpr int kAheadProbes = 1536;       // the same in a counting probe, where nobody waits for anybody (512: long-tailed chunks 558 us instead of 514, 768 to 3072 within 2 %)
constexpr int kTogetherFrom = 3;         // see gsc_compress_kernel
constexpr int kSegRows = 1024;           // rows of a sequence whose chunks one wavefront of the plan kernel packs
constexpr float kFastBand = 1e-4f;       // fp32 cosine error for d = 128 is < 2e-5; inside the band -> fp64

// A window of one sequence, filed by the plan kernel.  rows == 0: the slot is not used.
struct __attribute__((aligned(32))) GscWindow {
    int32_t first;            // first row
    int32_t rows;             // its rows (kWinLong: the rows of the chunk without its closing delimiter)
    int32_t flags;
    int32_t pad;
    uint64_t delim[2];        // bit r: row r closes a chunk
};
// The windows of a segment that are one long chunk: its first kMaxLongs slots of them (it has no more).
// The means of its first sixteen clusters over the keys wait in the workspace, at the chunk's own rows from kMeansAt on, for the workgroup of its slot.
constexpr int kMeansAt = 64;
constexpr int kMaxLongs = kSegRows / (kWinRows + 1) + 1;
struct GscLongs {
    int16_t slot[kMaxLongs];
};
constexpr int kWinLong = 1;      // one chunk with more than kWinRows rows
constexpr int kWinLast = 2;      // the last window of its sequence
constexpr int kWinClosed = 4;    // kWinLong: a delimiter follows

// What a window's workgroup publishes as soon as it knows it: its rows, in its own word and added to those of its segment (sc_gsc_words.h).
constexpr int kSegFront = 8;                   // room before the segments' words: those of eight are read at a time, down to the first

// Windows that can start in `rows` consecutive rows: two neighbours hold more than kWinRows rows together.  An odd number: the last slots of
// every segment stay empty, and workgroups go to the shader engines in turn (with sixteen slots two of four engines got half
// as much again as the others, and all waited for them: 8 heads x 32768 tokens 60 us, with seventeen 55).
__host__ __device__ inline int gsc_slots_per_segment(int n_max, int max_chunks) {
    const int rows = n_max < kSegRows ? n_max : kSegRows;
    int slots = 2 * ((rows - 1) / (kWinRows + 1)) + 2;
    if (max_chunks > 0) slots += rows / max_chunks + 1;
    return (slots < rows ? slots : rows) | 1;
}

__device__ __forceinline__ uint64_t bits_below(int x) {   // bits [0, x), 0 <= x <= 64, from 32-bit operations
    const uint32_t l = (x >= 32) ? 0xFFFFFFFFu : ((1u << x) - 1u);
    const uint32_t h = (x <= 32) ? 0u : ((x >= 64) ? 0xFFFFFFFFu : ((1u << (x - 32)) - 1u));
    return ((uint64_t)h << 32) | l;
}
__device__ __forceinline__ int last_bit(uint64_t m) { return 63 - __clzll((long long)m); }      // m != 0
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int nth_set_bit(uint64_t m, int k) {   // position of the k-th set bit, 0 <= k < popcount(m)
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const uint64_t part = (m >> pos) & ((1ull << w) - 1ull);
        const int cnt = __popcll(part);
        if (k >= cnt) { k -= cnt; pos += w; }
    }
    return pos;
}

// ------------------------------------------------------------------------------------------------
// plan: one wavefront per (kSegRows rows, sequence) packs the chunks that start there into windows, greedily and in order.  Windows of
// neighbouring wavefronts meet at the first chunk that starts in the later one's rows.  Slots that are left over are
// filed as empty, and what the windows' workgroups will publish is cleared: the workspace may hold anything.
// Bound by its chain: two trips to memory and the walk.
// start: the budget search that begins with this plan, if any.
template <typename... Start>
__global__ __launch_bounds__(kWave) void gsc_plan_kernel(GscParams p, Start... start) {
    constexpr int kSpan = kSegRows + kWinRows;       // rows whose delimiters the walk can ask for
    constexpr int kLook = 8;
    __shared__ uint32_t s_bits[kWave];               // (kSpan / 32 + 5 <= 64 words)
    __shared__ int s_off[kLook * kWave + 1];         // the offsets looked at
    const int seg = (int)blockIdx.x / p.B, b = (int)blockIdx.x - seg * p.B;
    const int lane = threadIdx.x;
    const int M = uniform(p.num_chunks[b]);
    int n = p.seq_lens ? uniform(p.seq_lens[b]) : p.N_max;
    n = n < 0 ? 0 : (n > p.N_max ? p.N_max : n);
    const int32_t *off = p.offsets + (int64_t)b * p.offsets_stride_b;
    const int S = p.slots_per_segment, slots = p.win_slots;
    GscWindow *win = p.windows + (int64_t)b * slots + (int64_t)seg * S;
    const int seg0 = seg * kSegRows;
    s_bits[lane] = 0u;
    if constexpr (sizeof...(Start) != 0) {
        if (blockIdx.x == 0 && lane == 0) budget_begin(start...);
    }
    if (lane == 0) s_off[kLook * kWave] = 0x7FFFFFFF;
    int used = 0, n_long = 0;
    GscLongs *longs = p.longs + (int64_t)b * (slots / S) + seg;
    if (M > 0) {
        const int n_rows = min(uniform(off[M]) - 1, n);      // rows of the sequence
        // m_lo, m_hi: first chunks that start at or behind seg0, seg0 + kSegRows (M if none).  Their places are guessed from the mean
        // chunk length; kLook * 64 offsets around the guess are looked at together.
        int m_lo = 0, m_hi = 0, first_hi = 0;      // and where the latter starts
        bool found;
        int look_base = 0;
        {
            const int guess = n > 0 ? (int)((int64_t)M * seg0 / n) : 0;
            const int base = max(0, min(guess - kLook * kWave / 2 + (int)((int64_t)M * kSegRows / (2 * (int64_t)max(n, 1))), M - kLook * kWave));
            int v[kLook];
#pragma unroll
            for (int q = 0; q < kLook; ++q) {
                const int m = base + q * kWave + lane;
                v[q] = m < M ? off[m] : 0x7FFFFFFF;
            }
#pragma unroll
            for (int q = 0; q < kLook; ++q) {
                if (base + q * kWave >= M) break;
                m_lo += __popcll(ballot64(v[q] < seg0));
                m_hi += __popcll(ballot64(v[q] < seg0 + kSegRows));
            }
            const int last = __builtin_amdgcn_readlane(v[kLook - 1], kWave - 1);
            found = (base == 0 || m_lo > 0) && (base + kLook * kWave >= M || last >= seg0 + kSpan + 1);
#pragma unroll
            for (int q = 0; q < kLook; ++q) {
                if ((m_hi >> 6) == q) first_hi = __builtin_amdgcn_readlane(v[q], m_hi & 63);
            }
            m_lo += base;
            m_hi += base;
            look_base = base;
            if (found) {
#pragma unroll
                for (int q = 0; q < kLook; ++q) {
                    if (base + q * kWave > M) break;      // (the first offset behind the last chunk's is looked at, too)
                    const int m = base + q * kWave + lane, rel = v[q] - 1 - seg0;
                    s_off[q * kWave + lane] = v[q];
                    if (m > m_lo && m < M && rel >= 0 && rel < kSpan) atomicOr(&s_bits[rel >> 5], 1u << (rel & 31));
                }
            }
        }
        if (!found) {
            int lo = 0, hi = M;       // off[m] < seg0 for m < lo, off[m] >= seg0 for m >= hi
            while (hi > lo) {
                const int step = (hi - lo + kWave - 1) / kWave;
                const int m = lo + lane * step;
                const int below = __popcll(ballot64(m < hi && off[min(m, M - 1)] < seg0));      // (the first `below` probes: offsets ascend)
                if (below == 0) { hi = lo; break; }
                const int l2 = lo + (below - 1) * step + 1;
                hi = min(hi, lo + below * step);
                lo = l2;
            }
            m_lo = m_hi = lo;
            for (int m0 = lo; m0 < M; m0 += kWave) {
                const int m = m0 + lane;
                const int v = m < M ? off[m] : 0x7FFFFFFF;
                const int rel = v - 1 - seg0;
                if (m > m_lo && m < M && rel >= 0 && rel < kSpan) atomicOr(&s_bits[rel >> 5], 1u << (rel & 31));
                m_hi += __popcll(ballot64(v < seg0 + kSegRows));
                if (__builtin_amdgcn_readlane(v, kWave - 1) >= seg0 + kSpan + 1) break;
            }
            first_hi = (m_hi < M) ? uniform(off[m_hi]) : 0;
        }
        __syncthreads();
        // The chunks m_lo .. m_hi - 1, 64 at a time: every lane works out the window that would start with its chunk, then the
        // greedy walk only hops from lane to lane.  Rows relative to seg0.
        const int end_rel = n_rows - seg0;
        const int stop = (m_hi < M) ? min(first_hi - seg0, end_rel) : end_rel;
        int m = m_lo;
        while (m < m_hi && used < S) {
            const int count = min(kWave, m_hi - m);
            const int at = min(m + lane, m_hi - 1);
            // (where the chunks were found among the offsets looked at, so were the next chunk's; there is nothing behind the last of all)
            const int from = found ? s_off[at - look_base] : off[at], to = found ? s_off[at + 1 - look_base] : off[at + 1];
            const int pos = from - seg0, chunk_end = min(to - 1, n_rows) - seg0;      // its closing delimiter, or the end of the sequence
            const bool valid = lane < count && pos >= 0 && pos < min(stop, kSegRows);
            // delimiters among the 128 rows from its start on
            const int w = valid ? pos >> 5 : 0, sh = pos & 31;
            uint32_t x[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) x[i] = s_bits[w + i];
            uint64_t d0 = (((uint64_t)x[1] << 32) | x[0]) >> sh, d1 = (((uint64_t)x[3] << 32) | x[2]) >> sh;
            if (sh != 0) {
                d0 |= (uint64_t)x[2] << (64 - sh);
                d1 |= (uint64_t)x[4] << (64 - sh);
            }
            const int lim = max(0, min(kWinRows, stop - pos));
            d0 &= bits_below(min(lim, 64));
            d1 &= bits_below(max(lim - 64, 0));
            int rows = 0, flags = 0;
            if (stop - pos <= kWinRows) rows = stop - pos;      // (ends with a delimiter or with the sequence)
            else if (d1 != 0ull) rows = 65 + last_bit(d1);
            else if (d0 != 0ull) rows = 1 + last_bit(d0);
            if (p.max_chunks > 0 && rows > 0) {
                const int c0 = __popcll(d0), c1 = __popcll(d1), k = p.max_chunks - 1;
                if (c0 + c1 > k) rows = 1 + (k < c0 ? nth_set_bit(d0, k) : 64 + nth_set_bit(d1, k - c0));
            }
            int chunks = 1, next_pos;
            if (rows > 0) {
                d0 &= bits_below(min(rows, 64));
                d1 &= bits_below(max(rows - 64, 0));
                next_pos = pos + rows;
                chunks = max(1, __popcll(d0) + __popcll(d1));
                if (next_pos >= end_rel) chunks = M - at;      // the last window
            } else {
                rows = chunk_end - pos;
                flags = kWinLong | ((at < M - 1) ? kWinClosed : 0);
                next_pos = chunk_end + ((at < M - 1) ? 1 : 0);
            }
            if (next_pos >= end_rel) flags |= kWinLast;
            const uint64_t usable = ballot64(valid && rows > 0);
            const int hop = lane + chunks;
            uint64_t starts = 0ull;
            int cur = 0;
            while (cur < count && ((usable >> cur) & 1ull) != 0ull) {
                starts |= 1ull << cur;
                cur = __builtin_amdgcn_readlane(hop, cur);
            }
            const int slot = used + __popcll(starts & bits_below(lane));
            if (((starts >> lane) & 1ull) != 0ull && slot < S) {
                GscWindow o;
                o.first = seg0 + pos; o.rows = rows; o.flags = flags; o.pad = 0;
                o.delim[0] = d0; o.delim[1] = d1;
                win[slot] = o;
            }
            const uint64_t is_long = starts & ballot64((flags & kWinLong) != 0);
            const int at_long = n_long + __popcll(is_long & bits_below(lane));
            if (((is_long >> lane) & 1ull) != 0ull && slot < S && at_long < kMaxLongs) longs->slot[at_long] = (int16_t)slot;
            n_long = min(kMaxLongs, n_long + (int)__popcll(is_long));
            used = min(S, used + (int)__popcll(starts));
            if (cur < count) break;      // the end of the sequence, or offsets that do not ascend
            m += cur;
        }
        if (seg == 0 && n_rows <= 0) {       // nothing to do
            for (int h = lane; h < p.Hkv; h += kWave) {
                bool bad;
                const int base = gsc_base_rows(p, (int64_t)b * p.Hkv + h, bad);
                p.comp_lens[(int64_t)b * p.Hkv + h] = bad ? -1 : base;
            }
        }
    } else if (seg == 0) {
        for (int h = lane; h < p.Hkv; h += kWave) p.comp_lens[(int64_t)b * p.Hkv + h] = -1;
    }
    for (int k = used + lane; k < S; k += kWave) win[k].rows = 0;
    if (lane == 0) p.long_count[(int64_t)b * (slots / S) + seg] = n_long;
    // four heads at a time: a segment has seventeen slots
    const int64_t bh0 = (int64_t)b * p.Hkv;
    const int segments = slots / S;
    for (int h = lane >> 4; h < p.Hkv; h += 4) {
        const int64_t at = (bh0 + h) * slots + (int64_t)seg * S;
        for (int k = lane & 15; k < S; k += 16) {
            p.published[at + k] = k < used ? 0u : kPubRows;
            if (p.count_only && k >= used) {
                uint4 *none = reinterpret_cast<uint4 *>(p.win_count + (at + k) * kProbeWords);
                none[0] = none[1] = make_uint4(0u, 0u, 0u, 0u);
            }
        }
        if ((lane & 15) == 0) p.segments[(bh0 + h) * segments + seg] = GscSegment{segment_start(used), 0u};
    }
    if (seg == 0)
        for (int h = lane; h < p.Hkv; h += kWave) p.head_state[bh0 + h] = 0u;
}

// ------------------------------------------------------------------------------------------------
// LDS of the compress kernel.  Four workgroups share a compute unit up to 39 680 bytes (31 pieces of 1280: with 32, which would fill it to the
// last byte, three did).
constexpr int kKeyRowBytes = 272;        // 256 B of keys + 16 B pad: conflict-free operand reads in both products
struct CompressLds {
    char rows[kWinRows * kKeyRowBytes];  // keys, later values
    union {
        uint32_t yes[kWinRows][4];       // bit m of row r: Sim(m, r) is surely above tau (m < r, same chunk)
        uint16_t hot[kWinRows / 16][kWinRows];      // once decided: bit c of row r in tile t: r belongs to output row 16 t + c
    };
    union {
        uint32_t unsure[kWinRows][4];    // bit m of row r: within the band, or a norm is unusable
        struct {                         // once the deciding wavefront has read them: pairs to be settled in fp64, and their outcome
            uint32_t list[kWinRows], above[kWinRows];
        };
    };
    float rinv[kWinRows];
    union {
        struct {                         // a long chunk's first sixteen seeds: reciprocal norms, rows of the chunk
            float seed_rinv[16];
            int seed_row[16];
        };
        uint64_t sets[kProbeWords][2];   // a long chunk at all thresholds of a probe: rows of the block that are open, then the seeds among them
    };
    int tile_steps[kWinRows / 16];       // bit ks of tile t: one of the rows 32 ks .. 32 ks + 31 belongs to it
    int any_unsure, base_lo, base_ok;
    unsigned char odd_norms[kWinWaves];  // wavefront w's rows hold one without a usable norm
    int pairs, first_seed;               // pairs the deciding wavefront wants settled (0: it has decided); seed that the list counts from
    int nseed, open;                     // outcome: seeds; a long chunk: rows still open
    int any_left, left_from, left_slot;  // windows of the head were left; where the search for them goes on, and the one found
};
static_assert(sizeof(CompressLds) <= 39680, "four workgroups per compute unit");

// cache policy of the key/value row loads: nt = read once by this launch
constexpr int kAuxReadOnce = 2;

// A wavefront's 32 rows as loaded: lane (g = lane / 16, c = lane % 16) holds elements 8c .. 8c + 7 of rows 4t + g
struct RowRegs {
    uint4 r[8];
};
// Rows [first_row, first_row + nrows) through a buffer descriptor that ends after the last wanted row: the hardware returns zeros
// for every access beyond it, so no lane needs a predicate or a 64-bit address.  row_stride_bytes * 32 must fit in 31
// bits (checked by the launcher).
template <int AUX = kAuxReadOnce>
__device__ __forceinline__ void load_rows(RowRegs &x, const bf16_t *base, int64_t stride_n, int first_row, int nrows, int g, int c) {
    const int sb = (int)stride_n * 2;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(base + (int64_t)first_row * stride_n), (short)0,
                                                                        nrows > 0 ? (nrows - 1) * sb + kFastD * 2 : 0, 0x00020000);
    const int voff = g * sb + 16 * c;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 4 * t * sb, 0, AUX);
        x.r[t] = make_uint4(v.x, v.y, v.z, v.w);
    }
}
__device__ __forceinline__ void park_rows(CompressLds &s, const RowRegs &x, int wave, int g, int c) {
#pragma unroll
    for (int t = 0; t < 8; ++t) *reinterpret_cast<uint4 *>(s.rows + (32 * wave + 4 * t + g) * kKeyRowBytes + 16 * c) = x.r[t];
}
__device__ __forceinline__ float safe_rinv(float nsq) {
    // a norm that is zero, denormal, huge or not a number makes every cosine with that row "unsure"
    return (nsq > 1e-30f && nsq < 1e30f) ? __frsqrt_rn(nsq) : __builtin_nanf("");
}
// reciprocal norms of the wavefront's rows, 0 for rows that do not exist; whether one of them is unusable
__device__ __forceinline__ void file_norms(CompressLds &s, const RowRegs &x, int nrows, int wave, int g, int c) {
    float nsq[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bf16x2_t w = __builtin_bit_cast(bf16x2_t, dword_of(x.r[t], k));
            a = __builtin_amdgcn_fdot2_f32_bf16(w, w, a, false);
        }
        nsq[t] = a;
    }
    float mine = row_transpose_reduce<8>(nsq, c);      // lane c: row 4 (c % 8) + g, over eight of the sixteen lanes
    mine += dpp<kDppRor8>(mine);
    const float ri = (4 * c + g < nrows) ? safe_rinv(mine) : 0.f;      // (c < 8)
    if (c < 8) s.rinv[32 * wave + 4 * c + g] = ri;
    const bool odd = ballot64(c < 8 && !(ri == ri)) != 0ull;
    if (c == 0 && g == 0) s.odd_norms[wave] = odd ? 1 : 0;
}

// eight elements of two rows into the sums of Eq. 2 in double precision (products of bf16 values are exact there)
__device__ __forceinline__ void cosine_sums_f64(const uint4 &a, const uint4 &b, double &dot, double &aa, double &bb) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t wa = dword_of(a, k), wb = dword_of(b, k);
        const double a0 = (double)__uint_as_float(wa << 16), a1 = (double)__uint_as_float(wa & 0xFFFF0000u);
        const double b0 = (double)__uint_as_float(wb << 16), b1 = (double)__uint_as_float(wb & 0xFFFF0000u);
        dot += a0 * b0; aa += a0 * a0; bb += b0 * b0;
        dot += a1 * b1; aa += a1 * a1; bb += b1 * b1;
    }
}
// Eq. 2 against tau, NaN compares false.  The roots and the division (half of a comparison's instructions) are left out where the squares
// differ by more than all their roundings can add up to (a few 2^-53 of either side).
__device__ __forceinline__ bool cosine_exceeds_f64(double dot, double aa, double bb, float tau) {
    const double t = (double)tau, q = dot * dot, r = (t * t) * (aa * bb), margin = r * 0x1p-44;
    const bool above = q - r > margin, below = r - q > margin;
    bool yes = above && dot > 0.0;
    if (ballot64(!(tau > 0.f) || !(above || below)) != 0ull) yes = dot / (sqrt(aa) * sqrt(bb)) > t;
    return yes;
}
__device__ __forceinline__ uint32_t or_rows(uint32_t x) {   // OR over the four 16-lane rows, same lane position
    auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = r[0] | r[1];
    r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return r[0] | r[1];
}

// sim(m, n) > t  <=>  dot * rinv_m > t * norm_n.  Per pair one fused multiply-add gives
//     dd = (tau + band) * norm_n - dot * rinv_m :   dd < 0  the pair is above the band (a sure yes),
//     0 <= dd <= 2 * band * norm_n  inside the band (unsure),  beyond that a sure no.
// Its sign bit is shifted into a nibble (v_alignbit), and an unsigned minimum over the bit patterns keeps the smallest
// non-negative dd (negative values compare as huge).  Only if some lane saw a pair inside the band, or a norm is unusable
// (then dd is not a number and counts as unsure), are the unsure bits made, from the same dd: yes, no and unsure partition the pairs.
struct Nibbles {
    uint32_t yes, least;
    float dd[4];
};
__device__ __forceinline__ Nibbles threshold_nibbles(const floatx4_t &acc, const floatx4_t &rm, float hn) {
    Nibbles r;
    r.yes = 0u;
    r.least = 0x7F800000u;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
        r.dd[i] = fmaf(-acc[i], rm[i], hn);
        r.yes = __builtin_amdgcn_alignbit(r.yes, __float_as_uint(r.dd[i]), 31);     // (yes << 1) | sign bit
        r.least = min(r.least, __float_as_uint(r.dd[i]));
    }
    return r;
}
__device__ __forceinline__ uint32_t unsure_nibble(Nibbles &r, float wn) {
    uint32_t unsure = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (!(r.dd[i] < 0.f) && !(r.dd[i] > wn)) unsure |= 1u << i;
    r.yes &= ~unsure;
    return unsure;
}

// bounds of a column's row; one that does not exist resembles nothing
__device__ __forceinline__ void column_bounds(float rn, bool exists, float tau, float &hn, float &wn) {
    const float norm = __builtin_amdgcn_rcpf(rn);
    hn = exists ? (tau + kFastBand) * norm : 1.0f;
    wn = exists ? (2.0f * kFastBand) * norm : 0.0f;
}

// Gram tiles of column tile J (rows 16 J .. 16 J + 15 of the window as columns) with row tiles I_first .. J.  The parked rows are
// both operands of v_mfma_f32_16x16x32_bf16 (lane l: row l % 16 of a tile, elements 8 (l / 16) .. + 7 of a 32-element slice); lane
// (g, c) gets the products of rows 16 I + 4 g + i with row 16 J + c: four bits of that row's word, completed by an OR over the lane
// groups.  Two row tiles are one word.
// odd: a row of the window has no usable norm
__device__ __forceinline__ void gram_column(CompressLds &s, int J, int I_first, int R, float tau, bool odd, int g, int c) {
    bf16x8f_t bq[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        bq[ks] = __builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(s.rows + (16 * J + c) * kKeyRowBytes + (32 * ks + 8 * g) * 2));
    float hn, wn;
    column_bounds(s.rinv[16 * J + c], 16 * J + c < R, tau, hn, wn);
    for (int I2 = I_first >> 1; I2 <= J >> 1; ++I2) {
        floatx4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const char *at = s.rows + (32 * I2 + c) * kKeyRowBytes + (32 * ks + 8 * g) * 2;
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(at)), bq[ks], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(at + 16 * kKeyRowBytes)), bq[ks], acc1, 0, 0, 0);
        }
        const floatx4_t rm0 = *reinterpret_cast<const floatx4_t *>(s.rinv + 32 * I2 + 4 * g), rm1 = *reinterpret_cast<const floatx4_t *>(s.rinv + 32 * I2 + 16 + 4 * g);
        Nibbles n0 = threshold_nibbles(acc0, rm0, hn), n1 = threshold_nibbles(acc1, rm1, hn);
        uint32_t u = 0u;
        if (odd || ballot64(min(n0.least, n1.least) <= __float_as_uint(wn)) != 0ull) {
            const uint32_t u0 = unsure_nibble(n0, wn), u1 = unsure_nibble(n1, wn);
            u = or_rows((u0 << (4 * g)) | (u1 << (16 + 4 * g)));
            if (ballot64(u != 0u) != 0ull) s.any_unsure = 1;
        }
        const uint32_t y = or_rows((n0.yes << (4 * g)) | (n1.yes << (16 + 4 * g)));
        if (g == 0) {
            s.yes[16 * J + c][I2] = y;
            s.unsure[16 * J + c][I2] = u;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Decisions.  One wavefront of the workgroup takes them (which one differs from window to window: the wavefronts of a place share a
// SIMD); lane l has rows l ("A") and 64 + l ("B").  The others wait and share in comparisons in fp64.
struct Words {      // candidates of the lane's two rows: rows 0..63, and for row B rows 64..127
    uint64_t a, b0, b1;
};
struct Pair64 {     // a set of rows
    uint64_t a, b;
};
__device__ __forceinline__ uint64_t row_word(const uint32_t (*words)[4], int row, int half) {
    return *reinterpret_cast<const uint64_t *>(&words[row][2 * half]);
}

__device__ __forceinline__ void wave_handover() {   // LDS traffic of one wavefront executes in order: only the compiler must not reorder
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// a pair of rows, one sixteenth of either in each lane of sixteen
__device__ __forceinline__ bool settle_one(const uint4 &a, const uint4 &b, float tau) {
    double dot = 0.0, sa = 0.0, sb = 0.0;
    cosine_sums_f64(a, b, dot, sa, sb);
    dot = row_allreduce_sum(dot);
    sa = row_allreduce_sum(sa);
    sb = row_allreduce_sum(sb);
    return cosine_exceeds_f64(dot, sa, sb, tau);
}
// Pairs of s.list, `n` of them, by the whole workgroup: row, and partner (another row of the window, or with a chunk's seed rows given the
// number of a carried seed, whose key is fetched from memory).  A pair takes the 16 lanes of a row, so sixteen are settled
// at once: the chain of a pair is long, and a threshold inside the band of the similarities asks for many.
__device__ __forceinline__ void settle_share(CompressLds &s, int n, float tau, int lane, int wave, const bf16_t *Kchunk, int64_t stride_n, const int32_t *seed_rows) {
    const int g = lane >> 4, c = lane & 15;
    for (int e0 = 4 * wave; e0 < n; e0 += 4 * kWinWaves) {
        const int e = e0 + g;
        const uint32_t w = s.list[min(e, n - 1)];
        const int i = (int)(w >> 8), j = (int)(w & 0xFFu);
        uint4 a;
        if (seed_rows) {
            const int at = s.first_seed + i;
            const int row = at < 16 ? s.seed_row[at] : __hip_atomic_load(seed_rows + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a = *reinterpret_cast<const uint4 *>(Kchunk + (int64_t)row * stride_n + 8 * c);
        } else {
            a = *reinterpret_cast<const uint4 *>(s.rows + i * kKeyRowBytes + 16 * c);
        }
        const bool above = settle_one(a, *reinterpret_cast<const uint4 *>(s.rows + j * kKeyRowBytes + 16 * c), tau);
        if (c == 0 && e < n) s.above[e] = above ? 1u : 0u;
    }
}
// The deciding wavefront asks for pairs, one for every row of `todo` (other_a, other_b: the partner of the lane's own rows), takes its share and
// returns the rows whose pair is above tau.
__device__ __forceinline__ Pair64 settle_pairs(CompressLds &s, const Pair64 &todo, int other_a, int other_b, float tau, int lane, int wave,
                                               const bf16_t *Kchunk, int64_t stride_n, const int32_t *seed_rows) {
    const int n_a = __popcll(todo.a), n = n_a + __popcll(todo.b);
    const bool in_a = (todo.a >> lane) & 1ull, in_b = (todo.b >> lane) & 1ull;
    const int at_a = __popcll(todo.a & bits_below(lane)), at_b = n_a + __popcll(todo.b & bits_below(lane));
    if (in_a) s.list[at_a] = ((uint32_t)other_a << 8) | (uint32_t)lane;
    if (in_b) s.list[at_b] = ((uint32_t)other_b << 8) | (uint32_t)(64 + lane);
    if (lane == 0) s.pairs = n;
    __syncthreads();
    settle_share(s, n, tau, lane, wave, Kchunk, stride_n, seed_rows);
    __syncthreads();
    Pair64 r;
    r.a = ballot64(in_a && s.above[min(at_a, kWinRows - 1)] != 0u);
    r.b = ballot64(in_b && s.above[min(at_b, kWinRows - 1)] != 0u);
    return r;
}
// The same by one wavefront for itself (a probe's four wavefronts decide at thresholds of their own), with the rows from memory: the window's
// keys are at Kwin.  list: room for 2 * kWinRows words in LDS.
__device__ __forceinline__ Pair64 settle_alone(uint32_t *list, const bf16_t *Kwin, int64_t stride_n, const Pair64 &todo, int other_a, int other_b, float tau, int lane) {
    const int g = lane >> 4, c = lane & 15;
    uint32_t *above = list + kWinRows;
    const int n_a = __popcll(todo.a), n = n_a + __popcll(todo.b);
    const bool in_a = (todo.a >> lane) & 1ull, in_b = (todo.b >> lane) & 1ull;
    const int at_a = __popcll(todo.a & bits_below(lane)), at_b = n_a + __popcll(todo.b & bits_below(lane));
    if (in_a) list[at_a] = ((uint32_t)other_a << 8) | (uint32_t)lane;
    if (in_b) list[at_b] = ((uint32_t)other_b << 8) | (uint32_t)(64 + lane);
    wave_handover();
    for (int e0 = 0; e0 < n; e0 += 4) {
        const int e = e0 + g;
        const uint32_t w = list[min(e, n - 1)];
        const bool yes = settle_one(*reinterpret_cast<const uint4 *>(Kwin + (int64_t)(w >> 8) * stride_n + 8 * c),
                                    *reinterpret_cast<const uint4 *>(Kwin + (int64_t)(w & 0xFFu) * stride_n + 8 * c), tau);
        if (c == 0 && e < n) above[e] = yes ? 1u : 0u;
    }
    wave_handover();
    Pair64 r;
    r.a = ballot64(in_a && above[min(at_a, kWinRows - 1)] != 0u);
    r.b = ballot64(in_b && above[min(at_b, kWinRows - 1)] != 0u);
    wave_handover();
    return r;
}
// the other wavefronts, until the deciding one is done
__device__ __forceinline__ void settle_until_decided(CompressLds &s, float tau, int lane, int wave, const bf16_t *Kchunk, int64_t stride_n, const int32_t *seed_rows) {
    for (;;) {
        __syncthreads();
        const int n = uniform(s.pairs);
        if (n == 0) return;
        settle_share(s, n, tau, lane, wave, Kchunk, stride_n, seed_rows);
        __syncthreads();
    }
}
__device__ __forceinline__ void decided(CompressLds &s, int lane) {
    if (lane == 0) s.pairs = 0;
    __syncthreads();
}

struct Decision {
    Pair64 seeds;
    int seed_a, seed_b;      // seed row of the lane's rows (-1: not an open row)
};

// Alg. 1 over the open rows of a window or block without walking the seeds one by one.  Seeds are taken in row
// order and a seed absorbs every open row of its chunk that resembles it, so a row joins the FIRST seed before
// it that it resembles and is a seed itself iff there is none: the seed set T is the one set with
//     r in T  <=>  no row of T before r (in r's chunk) resembles r            (induction over r: unique).
// With F(S) = { r : no row of S before r resembles r }, T is the only fixed point of F.  Starting from the rows
// that nothing earlier resembles (all of them seeds), F is applied until the set stops changing; when
// "resembles" is transitive inside the chunks, the usual case, that is the first application.  The words hold, restricted to
// the open rows before r in its own chunk, the rows it surely resembles (y) and those inside the band around tau (u).  A pair inside the band can
// change the outcome only if its earlier row is a seed that the later row, a seed itself, might resemble after all, or one before the seed
// the later row joins: the first such pair of every row is settled in fp64 and the fixed point is taken
// again.  Returns false, with nothing decided but the settled pairs, if the set has not settled after a few applications of F or
// pairs keep turning up: the caller then takes the seeds one at a time.
// settle(set, other_a, other_b): for every row of the set the pair with the partner given for it; the rows whose pair is above tau.
template <typename Settle>
__device__ __forceinline__ bool first_fit_fixed_point(Settle settle, Words &y, Words &u, bool open_a, bool open_b, int lane, Decision &d) {
    for (int pass = 0; pass < 8; ++pass) {
        Pair64 S;
        S.a = ballot64(open_a && y.a == 0ull);
        S.b = ballot64(open_b && (y.b0 | y.b1) == 0ull);
        bool settled = false;
        for (int it = 0; it < 8 && !settled; ++it) {
            const uint64_t na = ballot64(open_a && (y.a & S.a) == 0ull);
            const uint64_t nb = ballot64(open_b && ((y.b0 & S.a) | (y.b1 & S.b)) == 0ull);
            settled = na == S.a && nb == S.b;
            S.a = na;
            S.b = nb;
        }
        if (!settled) return false;
        const uint64_t ma = y.a & S.a, mb0 = y.b0 & S.a, mb1 = y.b1 & S.b;
        const bool is_seed_a = ma == 0ull, is_seed_b = (mb0 | mb1) == 0ull;
        const int first_a = is_seed_a ? lane : first_bit(ma);
        const int first_b = is_seed_b ? 64 + lane : (mb0 != 0ull ? first_bit(mb0) : 64 + first_bit(mb1));
        const uint64_t doubt_a = u.a & S.a & (is_seed_a ? ~0ull : bits_below(first_a));
        const uint64_t doubt_b0 = u.b0 & S.a & bits_below(min(first_b, 64));
        const uint64_t doubt_b1 = u.b1 & S.b & bits_below(max(first_b - 64, 0));
        Pair64 doubtful;
        doubtful.a = ballot64(open_a && doubt_a != 0ull);
        doubtful.b = ballot64(open_b && (doubt_b0 | doubt_b1) != 0ull);
        if ((doubtful.a | doubtful.b) == 0ull) {
            d.seeds = S;
            d.seed_a = open_a ? first_a : -1;
            d.seed_b = open_b ? first_b : -1;
            return true;
        }
        const int oa = doubt_a != 0ull ? first_bit(doubt_a) : 0;
        const int ob = doubt_b0 != 0ull ? first_bit(doubt_b0) : (doubt_b1 != 0ull ? 64 + first_bit(doubt_b1) : 0);
        const Pair64 above = settle(doubtful, oa, ob);
        if ((doubtful.a >> lane) & 1ull) {
            u.a &= ~(1ull << oa);
            if ((above.a >> lane) & 1ull) y.a |= 1ull << oa;
        }
        if ((doubtful.b >> lane) & 1ull) {
            const uint64_t bit = 1ull << (ob & 63);
            const bool yes = (above.b >> lane) & 1ull;
            if (ob < 64) { u.b0 &= ~bit; y.b0 |= yes ? bit : 0ull; }
            else { u.b1 &= ~bit; y.b1 |= yes ? bit : 0ull; }
        }
    }
    return false;
}

// The literal loop: per round every chunk takes its first open row as its next seed, and the open rows with that bit set join it
// (chunks never interact, so their loops run side by side; inside a chunk the order is exactly Alg. 1's).  ra, rb: the chunk's rows for the lane's rows.
template <typename Settle>
__device__ __forceinline__ void first_fit_by_seed(Settle settle, Words &y, Words &u, Pair64 todo, const Pair64 &ra, const Pair64 &rb, int lane, Decision &d) {
    d.seeds.a = d.seeds.b = 0ull;
    d.seed_a = d.seed_b = -1;
    while ((todo.a | todo.b) != 0ull) {
        const uint64_t a0 = todo.a & ra.a, a1 = todo.b & ra.b, b0 = todo.a & rb.a, b1 = todo.b & rb.b;
        const int sa = a0 != 0ull ? first_bit(a0) : (a1 != 0ull ? 64 + first_bit(a1) : 128);
        const int sb = b0 != 0ull ? first_bit(b0) : (b1 != 0ull ? 64 + first_bit(b1) : 128);
        const bool open_a = (todo.a >> lane) & 1ull, open_b = (todo.b >> lane) & 1ull;
        const bool seed_a = open_a && sa == lane, seed_b = open_b && sb == 64 + lane;
        // (an open row's chunk has an open row, the row itself if no other: sa <= lane, sb <= 64 + lane)
        const bool cand_a = open_a && sa < lane, cand_b = open_b && sb < 64 + lane;
        bool yes_a = cand_a && ((y.a >> (sa & 63)) & 1ull);
        bool yes_b = cand_b && (((sb < 64 ? y.b0 : y.b1) >> (sb & 63)) & 1ull);
        Pair64 ask;
        ask.a = ballot64(cand_a && ((u.a >> (sa & 63)) & 1ull));
        ask.b = ballot64(cand_b && (((sb < 64 ? u.b0 : u.b1) >> (sb & 63)) & 1ull));
        if ((ask.a | ask.b) != 0ull) {
            const Pair64 above = settle(ask, sa & 127, sb & 127);
            yes_a = yes_a || ((above.a >> lane) & 1ull);
            yes_b = yes_b || ((above.b >> lane) & 1ull);
        }
        if (seed_a || yes_a) d.seed_a = sa;
        if (seed_b || yes_b) d.seed_b = sb;
        const uint64_t new_a = ballot64(seed_a), new_b = ballot64(seed_b);
        const uint64_t got_a = ballot64(yes_a), got_b = ballot64(yes_b);
        d.seeds.a |= new_a;
        d.seeds.b |= new_b;
        todo.a &= ~(new_a | got_a);
        todo.b &= ~(new_b | got_b);
    }
}
// Where the chunks of the lane's two rows of a window of whole chunks start.
struct RowChunks {
    int lo_a, lo_b;
    __device__ __forceinline__ RowChunks(const Pair64 &D, int lane) {
        const uint64_t below = bits_below(lane), da = D.a & below, db = D.b & below;
        lo_a = da != 0ull ? 1 + last_bit(da) : 0;
        lo_b = db != 0ull ? 65 + last_bit(db) : (D.a != 0ull ? 1 + last_bit(D.a) : 0);
    }
};
// Alg. 1 in a window of whole chunks (delimiters D, R rows) from its bit matrices
template <typename Settle>
__device__ __forceinline__ void decide_window(const RowChunks &r, const uint32_t (*yes)[4], const uint32_t (*unsure)[4], const int &any_unsure, const Pair64 &D, int R,
                                              int lane, Settle settle, Decision &d) {
    const uint64_t below = bits_below(lane);
    const bool delim_a = (D.a >> lane) & 1ull, delim_b = (D.b >> lane) & 1ull;      // a delimiter is a chunk of its own
    const bool open_a = lane < R, open_b = 64 + lane < R;
    const uint64_t before_a = (delim_a || !open_a) ? 0ull : below & ~bits_below(r.lo_a);
    const uint64_t before_b0 = (delim_b || !open_b) ? 0ull : ~bits_below(min(r.lo_b, 64));
    const uint64_t before_b1 = (delim_b || !open_b) ? 0ull : below & ~bits_below(max(r.lo_b - 64, 0));
    Words y, u;
    y.a = row_word(yes, lane, 0) & before_a;
    y.b0 = row_word(yes, 64 + lane, 0) & before_b0;
    y.b1 = row_word(yes, 64 + lane, 1) & before_b1;
    u.a = u.b0 = u.b1 = 0ull;
    if (uniform(any_unsure) != 0) {
        u.a = row_word(unsure, lane, 0) & before_a;
        u.b0 = row_word(unsure, 64 + lane, 0) & before_b0;
        u.b1 = row_word(unsure, 64 + lane, 1) & before_b1;
    }
    if (first_fit_fixed_point(settle, y, u, open_a, open_b, lane, d)) return;
    // chunk ranges: up to the first delimiter from the row on
    const uint64_t ea = D.a & ~below, eb = D.b & ~below;
    const int hi_a = ea != 0ull ? first_bit(ea) : (D.b != 0ull ? 64 + first_bit(D.b) : R);
    const int hi_b = eb != 0ull ? 64 + first_bit(eb) : R;
    const int la = delim_a ? lane : r.lo_a, ha = delim_a ? lane + 1 : hi_a;
    const int lb = delim_b ? 64 + lane : r.lo_b, hb = delim_b ? 65 + lane : hi_b;
    const Pair64 ra = {bits_below(min(ha, 64)) & ~bits_below(min(la, 64)), bits_below(max(ha - 64, 0)) & ~bits_below(max(la - 64, 0))};
    const Pair64 rb = {bits_below(min(hb, 64)) & ~bits_below(min(lb, 64)), bits_below(max(hb - 64, 0)) & ~bits_below(max(lb - 64, 0))};
    const Pair64 all = {bits_below(min(R, 64)), bits_below(max(R - 64, 0))};
    first_fit_by_seed(settle, y, u, all, ra, rb, lane, d);
}
__device__ __forceinline__ int rows_below(const Pair64 &set, int row) {      // rows of the set before `row` (0..128)
    return __popcll(set.a & bits_below(min(row, 64))) + __popcll(set.b & bits_below(max(row - 64, 0)));
}

// ------------------------------------------------------------------------------------------------
// Rows before a window: those of the windows before it in its segment, and of the segments before.  Workgroups are dispatched in slot order, so the
// ones waited for are running or done, but for other calls: every XCD dispatches for itself, and with the heads of two calls spread over XCDs
// each call's next window can find an XCD full of the other's that wait.  A long chunk can take seconds to decide, too.  So the wait is
// bounded, and a window whose workgroup stops waiting is left to others (next_left).
// One wavefront asks through the scalar cache (glc: past it, from L2): a vector load would queue behind the rows that the compute unit's other
// wavefronts have asked for, 3 us where this takes less than one.  Where the windows of a head are spread over XCDs (their number is no multiple
// of eight), and every kVectorEvery-th time elsewhere, the look goes the other way, for words that another XCD's stores have changed in memory.
constexpr int kVectorEvery = 8;
constexpr int kSettledPolls = 1 << 20;       // where everything that is asked for has been published already
typedef uint32_t u32x16_t __attribute__((ext_vector_type(16)));
__device__ __forceinline__ void load_words(u32x16_t &w, const void *at, bool scalar, int lane) {      // `at`: uniform
    if (scalar) {
        asm volatile("s_load_dwordx16 %0, %1, 0x0 glc\n\ts_waitcnt lgkmcnt(0)" : "=&s"(w) : "s"(at) : "memory");
    } else {
        const uint32_t v = __hip_atomic_load(static_cast<const uint32_t *>(at) + (lane & 15), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = (uint32_t)__builtin_amdgcn_readlane((int)v, k);
    }
}
__device__ __forceinline__ bool rows_before(const uint32_t *published, GscSegment *segments, int bits, int S, int slot, bool one_xcd, int &polls, int lane, int &rows) {
    const int seg = slot / S, own = slot - seg * S;
    int sum = 0, look = 0;
    auto again = [&]() {
        if (--polls < 0) return false;
        look += 1;
        __builtin_amdgcn_s_sleep(1);
        return true;
    };
    // (sixteen words from the first on: of a segment's slots, the last is never anybody's predecessor; what lies behind the array is workspace)
    for (int k0 = 0; k0 < own; k0 += 16) {
        u32x16_t w;
        for (;;) {
            load_words(w, published + (int64_t)seg * S + k0, one_xcd && look % kVectorEvery != kVectorEvery - 1, lane);
            bool there = true;
            int part = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                if (k0 + k < own) {
                    there = there && (w[k] & kPubRows) != 0u;
                    part += (int)(w[k] & kPubValue);
                }
            }
            if (there) { sum += part; break; }
            if (!again()) return false;
        }
    }
    int before = 0;
    bool known = seg == 0;
    for (int top = seg; !known && top > 0; top -= 8) {      // segments top - 8 .. top - 1
        u32x16_t w;
        for (;;) {
            load_words(w, segments + top - 8, one_xcd && look % kVectorEvery != kVectorEvery - 1, lane);
            bool there = true;
            int part = 0;
            known = false;
#pragma unroll
            for (int k = 7; k >= 0; --k) {
                if (!known && top - 8 + k >= 0) {
                    known = (w[2 * k + 1] & kPubRows) != 0u;
                    there = there && (known || segment_complete(w[2 * k], bits));
                    part += known ? (int)(w[2 * k + 1] & kPubValue) : segment_rows(w[2 * k], bits);
                }
            }
            if (there) { before += part; break; }
            if (!again()) return false;
        }
    }
    // the end of the segment before is known now
    if (own == 0 && seg > 0 && lane == 0)
        __hip_atomic_store(&segments[seg - 1].upto, kPubRows | (uint32_t)before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    rows = before + sum;
    return true;
}

// ------------------------------------------------------------------------------------------------
// Means.  The product is formed transposed, columns x output rows: A holds 16 columns of the rows (lane (g, c): column 32 w + 2 c + parity,
// contraction index (g, i) = row 32 ks + 16 (i / 4) + 4 g + i % 4 of the window), B the 0/1 membership of the same rows (column c: output row 16 ot + c).
// Wavefront w takes columns 32 w .. 32 w + 31 in two tiles, even and odd: a lane ends up with eight neighbouring columns of one output row.
struct ColumnOps {
    bf16x8f_t x[4][2];
};
__device__ __forceinline__ void column_step(const CompressLds &s, int wave, int g, int c, int ks, bf16x8f_t &even, bf16x8f_t &odd) {
    uint32_t d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        d[i] = *reinterpret_cast<const uint32_t *>(s.rows + (32 * ks + 16 * (i >> 2) + 4 * g + (i & 3)) * kKeyRowBytes + 64 * wave + 4 * c);
    even = __builtin_bit_cast(bf16x8f_t, make_uint4(pack_lo(d[0], d[1]), pack_lo(d[2], d[3]), pack_lo(d[4], d[5]), pack_lo(d[6], d[7])));
    odd = __builtin_bit_cast(bf16x8f_t, make_uint4(pack_hi(d[0], d[1]), pack_hi(d[2], d[3]), pack_hi(d[4], d[5]), pack_hi(d[6], d[7])));
}
__device__ __forceinline__ void column_operands(const CompressLds &s, int wave, int g, int c, int nks, ColumnOps &o) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        if (ks < nks) column_step(s, wave, g, c, ks, o.x[ks][0], o.x[ks][1]);
}
// out_a, out_b: output row of the lane's rows, -1 for none, counted from the first of `tiles` tiles
__device__ __forceinline__ void file_membership(CompressLds &s, int out_a, int out_b, int tiles, int lane) {
    for (int t = 0; t < tiles; ++t) {
        const bool a = out_a >= 0 && (out_a >> 4) == t, b = out_b >= 0 && (out_b >> 4) == t;
        s.hot[t][lane] = a ? (uint16_t)(1u << (out_a & 15)) : (uint16_t)0;
        s.hot[t][64 + lane] = b ? (uint16_t)(1u << (out_b & 15)) : (uint16_t)0;
        const uint64_t ma = ballot64(a), mb = ballot64(b);
        if (lane == 0)
            s.tile_steps[t] = (((uint32_t)ma != 0u) ? 1 : 0) | (((ma >> 32) != 0ull) ? 2 : 0) | (((uint32_t)mb != 0u) ? 4 : 0) | (((mb >> 32) != 0ull) ? 8 : 0);
    }
}
// the lane's bit of its rows, turned to bit 14 of either half of a word: bf16 2.0.  (The sums are twice what they stand for, exactly, as long as
// they are finite; see all_finite.)
__device__ __forceinline__ bf16x8f_t membership_operand(const uint16_t *hot, int ks, int c, int g) {
    uint32_t aw[4];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
        const uint2 w = *reinterpret_cast<const uint2 *>(hot + 32 * ks + 16 * h2 + 4 * g);
        aw[2 * h2] = __builtin_amdgcn_alignbit(w.x, w.x, (uint32_t)(c + 18)) & 0x40004000u;
        aw[2 * h2 + 1] = __builtin_amdgcn_alignbit(w.y, w.y, (uint32_t)(c + 18)) & 0x40004000u;
    }
    return __builtin_bit_cast(bf16x8f_t, make_uint4(aw[0], aw[1], aw[2], aw[3]));
}
__device__ __forceinline__ bf16x8f_t ones_operand() {
    return __builtin_bit_cast(bf16x8f_t, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
}
// A zero row times an infinity is not a number, and twice a sum of 2^127 or more is an infinity: sums that are not finite are taken again,
// once instead of twice and without the other clusters' rows.
__device__ __forceinline__ bool all_finite(const floatx4_t &a, const floatx4_t &b) {
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) z = fmaf(a[i], 0.f, fmaf(b[i], 0.f, z));
    return z == 0.f;
}
// what twice the sums are multiplied with, from twice the size: 1/size is exact for powers of two, 1 ulp otherwise; a row of size 1 is passed
// on unchanged.  (Sums taken once: twice that.)
__device__ __forceinline__ float mean_scale(float size2) { return (size2 > 3.f) ? __builtin_amdgcn_rcpf(size2) : 0.5f; }
__device__ __forceinline__ void scale_mean(float (&v)[8], const floatx4_t &even, const floatx4_t &odd, float scale) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = even[i] * scale; v[2 * i + 1] = odd[i] * scale; }
}
template <typename TO>
__device__ __forceinline__ void store_mean(TO *row, const floatx4_t &even, const floatx4_t &odd, float scale, int wave, int g) {
    float v[8];
    scale_mean(v, even, odd, scale);
    TO *at = row + 32 * wave + 8 * g;
    if constexpr (sizeof(TO) == 2) {
        store16_stream(at, make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])));
    } else {
        store16_stream(at, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])));
        store16_stream(at + 4, make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])));
    }
}
// to row c of sixteen at `rows` (uniform), written through (sc1) to where another XCD's loads find it
template <typename TO>
__device__ __forceinline__ void store_mean_through(TO *rows, int c, const floatx4_t &even, const floatx4_t &odd, float scale, int wave, int g) {
    constexpr int kThrough = 16;
    float v[8];
    scale_mean(v, even, odd, scale);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(rows, (short)0, 16 * kFastD * (int)sizeof(TO), 0x00020000);
    const int off = (c * kFastD + 32 * wave + 8 * g) * (int)sizeof(TO);
    if constexpr (sizeof(TO) == 2) {
        const u32x4_t t = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
        __builtin_amdgcn_raw_buffer_store_b128(t, rs, off, 0, kThrough);
    } else {
        const u32x4_t t0 = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
        const u32x4_t t1 = {__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])};
        __builtin_amdgcn_raw_buffer_store_b128(t0, rs, off, 0, kThrough);
        __builtin_amdgcn_raw_buffer_store_b128(t1, rs, off + 16, 0, kThrough);
    }
}
// the sums, once, member by member from memory, rows [0, rows) at X with output rows given by `member` (rare: see all_finite)
template <typename F>
__device__ __forceinline__ void sums_by_member(const bf16_t *X, int64_t stride_n, int rows, F member, int wave, int g, floatx4_t &even, floatx4_t &odd) {
    even = odd = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int r = 0; r < rows; ++r) {
        if (member(r)) {
            float x[8];
            load8(X + (int64_t)r * stride_n + 32 * wave + 8 * g, x);
#pragma unroll
            for (int i = 0; i < 4; ++i) { even[i] += x[2 * i]; odd[i] += x[2 * i + 1]; }
        }
    }
}

// Everything derived from the lane number is recomputed from phase to phase instead of being carried in registers across the kernel (they
// spilled): the optimiser cannot see through the empty asm statement.
__device__ __forceinline__ int fresh_lane() {
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));
    return lane;
}
// The same for the kernel's arguments: read again where a phase needs them, instead of being held in a hundred scalar registers (and their spills).
typedef const __attribute__((address_space(4))) GscParams ConstParams;
__device__ __forceinline__ ConstParams *fresh_params() {
    ConstParams *p = (ConstParams *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
#define SC_FRESH_PARAMS ConstParams &p = *fresh_params()
#define SC_FRESH_LANE                     \
    const int lane = fresh_lane();        \
    [[maybe_unused]] const int g = lane >> 4, c = lane & 15

// ------------------------------------------------------------------------------------------------
// A probe of the budget search: the rows of a window at up to seven thresholds from one reading of its keys.  The cosines of its Gram
// matrix stay in registers (five pairs of tiles per wavefront); once all are there, bit matrices of all thresholds take the place of the
// keys in LDS, and every wavefront decides at one or two of them by itself.
struct ProbeWords {
    uint32_t yes[kProbeWords][kWinRows][4], unsure[kProbeWords][kWinRows][4];
};
static_assert(sizeof(ProbeWords) <= kWinRows * kKeyRowBytes, "in place of the keys");

// OR over the four 16-lane rows, same lane position, of four values: row g gets the one of v[g]
__device__ __forceinline__ uint32_t or_rows_transposed(const uint32_t (&v)[4]) {
    auto r = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const uint32_t x = r[0] | r[1];
    r = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const uint32_t z = r[0] | r[1];
    r = __builtin_amdgcn_permlane16_swap(x, z, false, false);
    return r[0] | r[1];
}
constexpr int kProbePairs = 5;      // pairs of row tiles of a wavefront's two column tiles, 7 - wave and wave: (9 - wave) / 2 and wave / 2 + 1
struct ProbeTiles {
    floatx4_t cosine[kProbePairs][2];
    uint32_t live;                  // bit q: pair q lies in the window and holds pairs of one chunk
};
__device__ __forceinline__ void probe_pair(int q, int wave, int &J, int &I2) {      // column tile and pair of row tiles
    const int n0 = (9 - wave) >> 1;
    J = q < n0 ? 7 - wave : wave;
    I2 = q < n0 ? q : q - n0;
}
__device__ __forceinline__ void probe_products(const CompressLds &s, const Pair64 &D, int R, int wave, int g, int c, ProbeTiles &t) {
    t.live = 0u;
#pragma unroll
    for (int q = 0; q < kProbePairs; ++q) {
        int J, I2;
        probe_pair(q, wave, J, I2);
        const uint64_t da = D.a & bits_below(min(16 * J, 64)), db = D.b & bits_below(max(16 * J - 64, 0));
        const int lo = db != 0ull ? 65 + last_bit(db) : (da != 0ull ? 1 + last_bit(da) : 0);      // first row of the chunk of row 16 J
        if (16 * J >= R || I2 < (lo >> 5)) continue;
        t.live |= 1u << q;
        floatx4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int col = (32 * ks + 8 * g) * 2;
            const bf16x8f_t b = __builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(s.rows + (16 * J + c) * kKeyRowBytes + col));
            const char *at = s.rows + (32 * I2 + c) * kKeyRowBytes + col;
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(at)), b, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8f_t, *reinterpret_cast<const uint4 *>(at + 16 * kKeyRowBytes)), b, acc1, 0, 0, 0);
        }
        // (two roundings more than the band's other users have: a few 2^-24 of a cosine, the band is 1e-4.)  Rows that do not exist have a
        // reciprocal norm of zero; a norm that is not usable makes all its cosines not a number.
        const floatx4_t rm0 = *reinterpret_cast<const floatx4_t *>(s.rinv + 32 * I2 + 4 * g), rm1 = *reinterpret_cast<const floatx4_t *>(s.rinv + 32 * I2 + 16 + 4 * g);
        const float rn = s.rinv[16 * J + c];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            t.cosine[q][0][i] = acc0[i] * (rm0[i] * rn);
            t.cosine[q][1][i] = acc1[i] * (rm1[i] * rn);
        }
    }
}
// The wavefront's tiles at four thresholds: words of threshold k to yes[k] and unsure[k], all four at once.  A subtraction and a shift of
// its sign bit (v_alignbit) per pair and threshold, and half a minimum that tells whether any pair came near.
__device__ __forceinline__ void probe_words(const ProbeTiles &t, const float (&tau)[kWinWaves], bool odd, int wave, int g, int c, uint32_t (*yes)[4], uint32_t (*unsure)[4]) {
#pragma unroll
    for (int q = 0; q < kProbePairs; ++q) {
        if (((t.live >> q) & 1u) == 0u) continue;
        int J, I2;
        probe_pair(q, wave, J, I2);
        uint32_t y[kWinWaves], u[kWinWaves];
        bool any = false;
#pragma unroll
        for (int k = 0; k < kWinWaves; ++k) {
            float diff[8], least = 1.f;
            uint32_t n0 = 0u, n1 = 0u;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                diff[i] = tau[k] - t.cosine[q][0][i];
                diff[4 + i] = tau[k] - t.cosine[q][1][i];
                n0 = __builtin_amdgcn_alignbit(n0, __float_as_uint(diff[i]), 31);      // (n0 << 1) | sign bit
                n1 = __builtin_amdgcn_alignbit(n1, __float_as_uint(diff[4 + i]), 31);
                least = fminf(least, fminf(fabsf(diff[i]), fabsf(diff[4 + i])));
            }
            u[k] = 0u;
            y[k] = (n0 | (n1 << 16)) << (4 * g);
            if (odd || ballot64(least <= kFastBand) != 0ull) {      // (a minimum passes over what is not a number)
                uint32_t near = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    near |= !(fabsf(diff[i]) > kFastBand) ? 1u << i : 0u;
                    near |= !(fabsf(diff[4 + i]) > kFastBand) ? 65536u << i : 0u;
                }
                u[k] = near << (4 * g);
                any = true;
            }
        }
        const uint32_t yy = or_rows_transposed(y), uu = any ? or_rows_transposed(u) : 0u;
        yes[16 * J + c][I2] = yy & ~uu;
        unsure[16 * J + c][I2] = uu;
    }
}

// ------------------------------------------------------------------------------------------------
// A chunk longer than a window at all thresholds of a probe, by one workgroup: its blocks' keys are read, and the products of a block's rows formed, once
// for all of them.  Seeds of the blocks before are listed in the workspace, those of any threshold once: row, reciprocal norm, and a bit per
// threshold that it is a seed at.  Whether a row joins one of them, and not which, is all that counts.
// Bound by instructions, words and decisions of seven thresholds where three steps of a search one by one need three: 8 heads x 131072 tokens in chunks of 200, 12
// steps, 1600 us a call, 1527 with a probe a step, 3037 with a workgroup per chunk and threshold; 8 x 32768 in chunks of 200 524, 589 and 840.
// (With the listed seeds taken by all wavefronts in turn instead of sixteen by each: chunks of 400 1010 us, 793 so; every pair inside the band settled before
// the decisions instead of when one needs it: chunks of 200 613, 580.)
struct ProbeSeeds {
    int32_t *row, *rinv, *at;      // (rinv: the bits of a float)
    int n;
};
__device__ __forceinline__ float max_rows(float x) {   // maximum over the four 16-lane rows, same lane position
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// sixteen listed seeds from the s0-th on: the keys as an operand (row c), reciprocal norms and thresholds of seeds 4 g + i
struct ProbeGroup {
    bf16x8f_t keys[4];
    float rinv[4];
    uint32_t at[4];
    int row;      // of seed c
    __device__ __forceinline__ static int row_of(const ProbeSeeds &u, int s0, int c) {
        return c < u.n - s0 ? __hip_atomic_load(u.row + s0 + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
    __device__ __forceinline__ ProbeGroup(const ProbeSeeds &u, int s0, int row_c, const bf16_t *Kch, int64_t stride_n, int g, int c) : row(row_c) {
        const int ns = u.n - s0;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            keys[ks] = __builtin_bit_cast(bf16x8f_t, c < ns ? *reinterpret_cast<const uint4 *>(Kch + (int64_t)row * stride_n + 32 * ks + 8 * g) : make_uint4(0u, 0u, 0u, 0u));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool there = 4 * g + i < ns;
            rinv[i] = there ? __int_as_float(__hip_atomic_load(u.rinv + s0 + 4 * g + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0.f;
            at[i] = there ? (uint32_t)__hip_atomic_load(u.at + s0 + 4 * g + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        }
    }
    // cosines of seeds 4 g + i with row 16 J + c of the block
    __device__ __forceinline__ floatx4_t cosines(const CompressLds &s, int J, int g, int c) const {
        floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint4 v = *reinterpret_cast<const uint4 *>(s.rows + (16 * J + c) * kKeyRowBytes + (32 * ks + 8 * g) * 2);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(keys[ks], __builtin_bit_cast(bf16x8f_t, v), acc, 0, 0, 0);
        }
        const float rn = s.rinv[16 * J + c];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] *= rinv[i] * rn;
        return acc;
    }
};
// floats as integers of the same order
__device__ __forceinline__ int ordered(float x) { const int b = __float_as_int(x); return b ^ ((b >> 31) & 0x7FFFFFFF); }
__device__ __forceinline__ float unordered(int b) { return __int_as_float(b ^ ((b >> 31) & 0x7FFFFFFF)); }
struct ProbeTops {      // (in place of the words of single thresholds)
    int top[kProbeNodes][kWinRows];          // the largest cosine of a row with a listed seed of the threshold, ordered
    uint64_t doubt[kProbeNodes][2];          // rows that fp64 decides
    int odd_seed;                            // a listed seed has no usable norm
};
static_assert(sizeof(ProbeTops) <= sizeof(CompressLds::yes) + sizeof(CompressLds::unsure), "in their place");
// The rows of a block (R of them) that resemble no listed seed of threshold t: s.sets[t].  Sixteen seeds at a time and wavefront, against all rows (one group
// in all: its row tiles are shared out).  Per pair a choice, which takes the seed out where it is none, and a maximum for each threshold; rows
// whose nearest seed is inside the band, or that have no usable norm, are settled in fp64.  For all wavefronts.
__device__ __forceinline__ void probe_open_rows(CompressLds &s, const ProbeSeeds &u, const bf16_t *Kch, int64_t stride_n, int rb, int R, float tau_lo, float tau_hi, int nodes,
                                                int wave, int lane) {
    const int g = lane >> 4, c = lane & 15;
    ProbeTops &tops = *reinterpret_cast<ProbeTops *>(&s.yes[0][0]);
    for (int i = threadIdx.x; i < kProbeNodes * kWinRows; i += kWinThreads) (&tops.top[0][0])[i] = ordered(-INFINITY);
    if (threadIdx.x == 0) tops.odd_seed = 0;
    __syncthreads();
    const bool shared = u.n <= 16;
    const int own = shared ? 0 : 16 * wave;
    if (own < u.n) {
        float top[8][kProbeNodes];
#pragma unroll
        for (int J = 0; J < 8; ++J)
#pragma unroll
            for (int t = 0; t < kProbeNodes; ++t) top[J][t] = -INFINITY;
        bool odd = false;
        int row = ProbeGroup::row_of(u, own, c);
#pragma unroll 1
        for (int s0 = own; s0 < u.n; s0 += 16 * kWinWaves) {
            const ProbeGroup seeds(u, s0, row, Kch, stride_n, g, c);
            row = ProbeGroup::row_of(u, s0 + 16 * kWinWaves, c);
            const float sum = (seeds.rinv[0] + seeds.rinv[1]) + (seeds.rinv[2] + seeds.rinv[3]);      // not a number if one of them is
            odd = odd || !(sum == sum);
#pragma unroll
            for (int J = 0; J < 8; ++J) {
                if (16 * J >= R || (shared && (J & 3) != wave)) continue;
                const floatx4_t x = seeds.cosines(s, J, g, c);
#pragma unroll
                for (int t = 0; t < kProbeNodes; ++t) {
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = ((seeds.at[i] >> t) & 1u) != 0u ? x[i] : -INFINITY;
                    top[J][t] = fmaxf(fmaxf(top[J][t], y[0]), y[1]);
                    top[J][t] = fmaxf(fmaxf(top[J][t], y[2]), y[3]);
                }
            }
        }
        if (ballot64(odd) != 0ull && lane == 0) tops.odd_seed = 1;
#pragma unroll
        for (int t = 0; t < kProbeNodes; ++t) {
#pragma unroll
            for (int J = 0; J < 8; J += 4) {      // lane group g files tile J + g
                const float a = max_rows(top[J][t]), b = max_rows(top[J + 1][t]), d = max_rows(top[J + 2][t]), e = max_rows(top[J + 3][t]);
                const float x = g < 2 ? (g == 0 ? a : b) : (g == 2 ? d : e);
                if (t < nodes) atomicMax(&tops.top[t][16 * (J + g) + c], ordered(x));
            }
        }
    }
    __syncthreads();
    const bool odd_seed = uniform(tops.odd_seed) != 0;
    for (int t = wave; t < nodes; t += kWinWaves) {
        const float tau = budget_node_tau(tau_lo, tau_hi, t + 1);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int r = 64 * half + lane;
            const float x = unordered(tops.top[t][r]) - tau, rn = s.rinv[r];
            const uint64_t left = ballot64(r < R && !(x > kFastBand)), near = ballot64(!(x < -kFastBand) || odd_seed || !(rn == rn));
            if (lane == 0) {
                s.sets[t][half] = left;
                tops.doubt[t][half] = left & near;
            }
        }
    }
    __syncthreads();
    // in fp64: listed seeds inside the band, four pairs at a time.  Lane 8 t + J has the doubtful rows of threshold t in tile J.
    int doubt = lane < 8 * nodes ? (int)reinterpret_cast<const uint16_t *>(tops.doubt)[lane] : 0;
    if (ballot64(doubt != 0) == 0ull || own >= u.n) return;
    uint32_t *open = reinterpret_cast<uint32_t *>(s.sets);      // [threshold][32 rows]
    int row = ProbeGroup::row_of(u, own, c);
#pragma unroll 1
    for (int s0 = own; s0 < u.n; s0 += 16 * kWinWaves) {
        const ProbeGroup seeds(u, s0, row, Kch, stride_n, g, c);
        row = ProbeGroup::row_of(u, s0 + 16 * kWinWaves, c);
#pragma unroll 1
        for (int J = 0; J < 8; ++J) {
            const uint64_t asked = ballot64(doubt != 0 && (lane & 7) == J);      // bit 8 t + J
            if (asked == 0ull || (shared && (J & 3) != wave)) continue;
            const floatx4_t x = seeds.cosines(s, J, g, c);
#pragma unroll 1
            for (uint64_t left = asked; left != 0ull; left &= left - 1ull) {
                const int from = uniform(first_bit(left)), t = from >> 3;
                int unsure = __builtin_amdgcn_readlane(doubt, from);
                const float tau = budget_node_tau(tau_lo, tau_hi, t + 1);
                uint32_t mine = 0u;      // the lane's pairs
#pragma unroll
                for (int i = 0; i < 4; ++i) mine |= (((seeds.at[i] >> t) & 1u) != 0u && ((unsure >> c) & 1) != 0 && !(fabsf(x[i] - tau) > kFastBand)) ? 1u << i : 0u;
                while (true) {
                    const uint64_t ask = ballot64(mine != 0u && ((unsure >> c) & 1) != 0);
                    if (ask == 0ull) break;
                    const int n = min(__popcll(ask), 4), at = nth_set_bit(ask, min(g, n - 1));      // group g takes the g-th lane's next pair, or the last one's
                    const int i = __shfl(__ffs((int)mine) - 1, at, kWave), r = 16 * J + (at & 15), seed = __shfl(seeds.row, 4 * (at >> 4) + i, kWave);
                    const bool yes = settle_one(*reinterpret_cast<const uint4 *>(Kch + (int64_t)seed * stride_n + 8 * c),
                                                *reinterpret_cast<const uint4 *>(Kch + (int64_t)(rb + r) * stride_n + 8 * c), tau);
                    unsure &= ~uniform((int)or_rows(yes ? 1u << (at & 15) : 0u));
                    uint64_t done = 0ull;
                    for (int k = 0, m = n; k < m; ++k) done |= 1ull << nth_set_bit(ask, k);
                    if ((done >> lane) & 1ull) mine &= mine - 1u;
                    if (yes && c == 0) atomicAnd(open + 4 * t + (r >> 5), ~(1u << (r & 31)));
                }
                if (lane == from) doubt = unsure;
            }
        }
    }
}
// One block of the chunk: rows [rb, rb + R), keys in s.rows.  Between two barriers the caller's; `fetch` asks for the next rows.  counts: seeds so far
// at thresholds wave and wave + 4.
template <typename Fetch>
__device__ __forceinline__ void probe_block(CompressLds &s, ProbeSeeds &u, const bf16_t *Kch, int64_t stride_n, int rb, int R, bool last, float tau_lo, float tau_hi, int nodes,
                                            int wave, Fetch fetch, int (&counts)[2]) {
    SC_FRESH_LANE;
    const bool odd = uniform(*reinterpret_cast<const int *>(s.odd_norms)) != 0;
    if (u.n > 0) probe_open_rows(s, u, Kch, stride_n, rb, R, tau_lo, tau_hi, nodes, wave, lane);
    else if (wave == 0 && lane < 2 * kProbeWords) s.sets[lane >> 1][lane & 1] = bits_below(max(min(R - 64 * (lane & 1), 64), 0));
    const Pair64 none = {0ull, 0ull};
    ProbeTiles tiles;
    probe_products(s, none, R, wave, g, c, tiles);
    const float rinv_a = s.rinv[lane], rinv_b = s.rinv[64 + lane];
    __syncthreads();      // the keys have been read, the open rows are known
    const uint64_t mine = lane < 2 * nodes ? s.sets[lane >> 1][lane & 1] : 0ull;
    const bool any_open = ballot64(mine != 0ull) != 0ull;
    ProbeWords &words = *reinterpret_cast<ProbeWords *>(s.rows);
    if (any_open) {
        for (int t0 = 0; t0 < nodes; t0 += kWinWaves) {
            float taus[kWinWaves];
#pragma unroll
            for (int k = 0; k < kWinWaves; ++k) taus[k] = budget_node_tau(tau_lo, tau_hi, min(t0 + k, nodes - 1) + 1);
            probe_words(tiles, taus, odd, wave, g, c, words.yes[t0 + g], words.unsure[t0 + g]);
        }
        __syncthreads();
    }
    if (!any_open) {
        fetch();
        return;
    }
    const uint64_t below = bits_below(lane);
    for (int t = wave; t < nodes; t += kWinWaves) {
        const float tau = budget_node_tau(tau_lo, tau_hi, t + 1);
        uint32_t *list = (wave < 2 ? &s.yes[0][0] : &s.unsure[0][0]) + (wave & 1) * 2 * kWinRows;
        const Pair64 open = {s.sets[t][0], s.sets[t][1]};
        const bool open_a = (open.a >> lane) & 1ull, open_b = (open.b >> lane) & 1ull;
        Words y, n;
        y.a = open_a ? row_word(words.yes[t], lane, 0) & below & open.a : 0ull;
        y.b0 = open_b ? row_word(words.yes[t], 64 + lane, 0) & open.a : 0ull;
        y.b1 = open_b ? row_word(words.yes[t], 64 + lane, 1) & below & open.b : 0ull;
        n.a = open_a ? row_word(words.unsure[t], lane, 0) & below & open.a : 0ull;
        n.b0 = open_b ? row_word(words.unsure[t], 64 + lane, 0) & open.a : 0ull;
        n.b1 = open_b ? row_word(words.unsure[t], 64 + lane, 1) & below & open.b : 0ull;
        Decision d;
        auto settle = [&](const Pair64 &ask, int oa, int ob) { return settle_alone(list, Kch + (int64_t)rb * stride_n, stride_n, ask, oa, ob, tau, lane); };
        if (!first_fit_fixed_point(settle, y, n, open_a, open_b, lane, d)) {
            const Pair64 all = {~0ull, ~0ull};
            first_fit_by_seed(settle, y, n, open, all, all, lane, d);
        }
        const int found = __popcll(d.seeds.a) + __popcll(d.seeds.b);
        counts[0] += t < kWinWaves ? found : 0;
        counts[1] += t < kWinWaves ? 0 : found;
        if (lane == 0) {
            s.sets[t][0] = d.seeds.a;
            s.sets[t][1] = d.seeds.b;
        }
    }
    fetch();
    __syncthreads();      // (the next rows may take the words' place)
    if (last) return;
    // the list grows by the rows that are seeds at any threshold
    uint32_t at_a = 0u, at_b = 0u;
    for (int t = 0; t < nodes; ++t) {
        at_a |= (uint32_t)((s.sets[t][0] >> lane) & 1ull) << t;
        at_b |= (uint32_t)((s.sets[t][1] >> lane) & 1ull) << t;
    }
    const uint64_t new_a = ballot64(at_a != 0u), new_b = ballot64(at_b != 0u);
    if (wave == 0) {
        const int to_a = u.n + __popcll(new_a & below), to_b = u.n + __popcll(new_a) + __popcll(new_b & below);
        if (at_a != 0u) {
            __hip_atomic_store(u.row + to_a, rb + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(u.rinv + to_a, __float_as_int(rinv_a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(u.at + to_a, (int)at_a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (at_b != 0u) {
            __hip_atomic_store(u.row + to_b, rb + 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(u.rinv + to_b, __float_as_int(rinv_b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(u.at + to_b, (int)at_b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    u.n += __popcll(new_a) + __popcll(new_b);
}

// PROBE: a probe of the budget search, at one threshold or at several.  Only the numbers of rows are wanted: no values are read and nothing is merged.
constexpr int kNoProbe = 0, kProbeOne = 1, kProbeSeveral = 2;
template <typename TO, int PROBE>
__global__ __launch_bounds__(kWinThreads, 4) void gsc_compress_kernel(GscParams p) {
    constexpr bool COUNT = PROBE != kNoProbe;
    __shared__ __attribute__((aligned(16))) CompressLds s;
    // Slots in order, (sequence, head) fastest: every workgroup waits for earlier ones only, and with a multiple of eight
    // heads the windows of a head stay on one XCD.  Long chunks are decided ahead of everything else, by ahead_per_head workgroups per
    // head that wait for nothing: a window waits for the rows of all before it, and a long chunk in between, which takes twice as long, would hold up
    // those of half the chip (8 heads x 131072, a quarter of the windows long: 225 us, decided ahead 165).
    const int n_bh = p.B * p.Hkv;
    const int ahead_wgs = p.ahead_wgs;
    [[maybe_unused]] const int nodes = PROBE == kProbeSeveral ? (1 << p.probe_levels) - 1 : 1;
    const bool ahead = (int)blockIdx.x < ahead_wgs;
    const unsigned id = ahead ? blockIdx.x : blockIdx.x - (unsigned)ahead_wgs;
    const int place = (int)(id / (unsigned)n_bh), bh_i = (int)(id - (unsigned)place * (unsigned)n_bh);
    const int b = bh_i / p.Hkv, h = bh_i - b * p.Hkv;
    const int64_t bh = bh_i;
    // (through the constant address space: scalar loads, which do not queue behind the vector loads of other wavefronts)
    typedef int i32x8_t __attribute__((ext_vector_type(8)));
    struct Window { int slot, first, rows, flags; };
    auto take_window = [&](int at, Pair64 *delim) {
        SC_FRESH_PARAMS;
        const i32x8_t wd = *reinterpret_cast<const __attribute__((address_space(4))) i32x8_t *>((uintptr_t)(p.windows + (int64_t)b * p.win_slots + at));
        if (delim) {
            delim->a = ((uint64_t)(uint32_t)wd[5] << 32) | (uint32_t)wd[4];
            delim->b = ((uint64_t)(uint32_t)wd[7] << 32) | (uint32_t)wd[6];
        }
        return Window{at, wd[0], wd[1], wd[2]};
    };
    // the `at`-th long chunk of the sequence, if it has as many
    auto take_long = [&](int at, Window &w) {
        SC_FRESH_PARAMS;
        const int lane = fresh_lane(), S = p.slots_per_segment, segments = p.win_slots / S;
        const int32_t *count = p.long_count + (int64_t)b * segments;
        for (int s0 = 0; s0 < segments; s0 += kWave) {
            const int mine = s0 + lane < segments ? count[s0 + lane] : 0;
            int incl = mine;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int up = __shfl_up(incl, d, kWave);
                if (lane >= d) incl += up;
            }
            const uint64_t behind = ballot64(incl > at);
            if (behind != 0ull) {
                const int l = first_bit(behind), k = at - __builtin_amdgcn_readlane(incl - mine, l);
                w = take_window((s0 + l) * S + uniform((int)p.longs[(int64_t)b * segments + s0 + l].slot[k]), nullptr);
                return true;
            }
            at -= __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        return false;
    };
    // A probe's work ahead is a long chunk at one threshold; or at all of them, where that many items would be kTogetherFrom / 2 times the workgroups
    // (2 heads x 8000 tokens, us per call of 12 steps: chunks of 200 174 the first way and 261 the second, of 1000 885 and 1729; 8 x 32768:
    // of 200 840 and 524, of 700, twice the workgroups, 1389 and 1481, of 850 1549 and 1907).
    [[maybe_unused]] bool together = false;
    if constexpr (PROBE == kProbeSeveral) {
        if (ahead) {
            SC_FRESH_PARAMS;
            const int lane = fresh_lane(), segments = p.win_slots / p.slots_per_segment;
            int all = 0;
            for (int q = lane; q < segments; q += kWave) all += p.long_count[(int64_t)b * segments + q];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) all += __shfl_xor(all, d, kWave);
            all = uniform(all);
            together = 2 * (int64_t)all * nodes > (int64_t)kTogetherFrom * p.ahead_per_head;
            if (place >= (together ? all : all * nodes)) return;
        }
    }
    int next_long = place;
    Window win, next;
    Pair64 D = {0ull, 0ull};
    if (!ahead) {
        win = take_window(place, &D);
        if (win.rows <= 0 || (COUNT && (win.flags & kWinLong) != 0)) return;
    } else if (!together) {
        if (!take_long(next_long / nodes, win)) return;
        D.a = D.b = 0ull;
    }
    const int &slot = win.slot, &w0 = win.first, &R = win.rows, &flags = win.flags;
    const int tid = threadIdx.x, wave = uniform(tid / kWave);
    const bf16_t *Kbh = reinterpret_cast<const bf16_t *>(p.K) + b * p.stride_b + h * p.stride_h;
    const bf16_t *Vbh = reinterpret_cast<const bf16_t *>(p.V) + b * p.stride_b + h * p.stride_h;
    float tau = p.tau_dev ? *p.tau_dev : p.tau;
    [[maybe_unused]] float tau_lo = 0.f, tau_hi = 0.f;      // the search's bracket
    if constexpr (COUNT) {
        tau_lo = p.budget->lo;
        tau_hi = p.budget->hi;
        if (ahead) tau = budget_node_tau(tau_lo, tau_hi, 1 + next_long % nodes);
    }
    if constexpr (PROBE == kProbeSeveral) {
        if (together) {
            int at = place;
            Window now, then;
            if (!take_long(at, now)) return;
            RowRegs x;
            {
                SC_FRESH_LANE;
                load_rows<0>(x, Kbh, p.stride_n, now.first + 32 * wave, min(32, now.rows - 32 * wave), g, c);
            }
            for (;;) {
                SC_FRESH_PARAMS;
                at += p.ahead_per_head;
                const bool more = take_long(at, then);
                const int start = now.first, l = now.rows;
                const bf16_t *Kch = Kbh + (int64_t)start * p.stride_n;
                int32_t *list = reinterpret_cast<int32_t *>(p.rows_ws) + bh * kProbeWords * p.N_max + start;      // (where the means of a merge would go)
                ProbeSeeds seeds = {list, list + p.N_max, list + 2 * (int64_t)p.N_max, 0};
                int counts[2] = {0, 0};
#pragma unroll 1
                for (int rb = 0; rb < l; rb += kWinRows) {
                    const int Rb = min(kWinRows, l - rb), nx = rb + kWinRows;
                    {
                        SC_FRESH_LANE;
                        file_norms(s, x, Rb - 32 * wave, wave, g, c);
                        park_rows(s, x, wave, g, c);
                    }
                    __syncthreads();
                    auto fetch = [&]() {
                        SC_FRESH_LANE;
                        const int first = nx < l ? start + nx : (more ? then.first : start), rows = nx < l ? l - nx : (more ? then.rows : 0);
                        load_rows<0>(x, Kbh, p.stride_n, first + 32 * wave, min(32, rows - 32 * wave), g, c);
                    };
                    probe_block(s, seeds, Kch, p.stride_n, rb, Rb, nx >= l, tau_lo, tau_hi, nodes, wave, fetch, counts);
                }
                if (fresh_lane() == 0) {
                    int32_t *count = p.win_count + (bh * p.win_slots + now.slot) * kProbeWords;
                    const int closes = (now.flags & kWinClosed) != 0 ? 1 : 0;
                    if (wave < nodes) count[wave] = counts[0] + closes;
                    if (wave + kWinWaves < nodes) count[wave + kWinWaves] = counts[1] + closes;
                }
                if (!uniform(more ? 1 : 0)) return;
                now = Window{uniform(then.slot), uniform(then.first), uniform(then.rows), uniform(then.flags)};
            }
        }
    }
    // the window's rows are known: tell the windows behind it
    auto publish = [&](int rows, bool is_long, int lane) {      // one wavefront
        SC_FRESH_PARAMS;
        if (lane == 0) {
            if constexpr (COUNT) p.win_count[(bh * p.win_slots + slot) * kProbeWords + next_long % nodes] = rows;
            else {
                const int S = p.slots_per_segment;
                uint32_t *pub = p.published + bh * p.win_slots;
                GscSegment *segments = p.segments + bh * (p.win_slots / S);
                if (is_long) __hip_atomic_fetch_or(pub + slot, kPubRows | (uint32_t)rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (its slot's workgroup may have left it)
                else __hip_atomic_store(pub + slot, kPubRows | (uint32_t)rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(&segments[slot / S].part, segment_added(rows, p.seg_bits), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    };
    // First output row of the window, for all wavefronts (between two barriers).  left: somebody else's window, the rows before are published; should
    // they not arrive all the same, the head ends with a length of -1.
    auto find_base = [&](int rows, bool left) {      // one wavefront
        SC_FRESH_LANE;
        SC_FRESH_PARAMS;
        const int S = p.slots_per_segment;
        const int64_t cap = p.cap;
        uint32_t *pub = p.published + bh * p.win_slots;
        GscSegment *segments = p.segments + bh * (p.win_slots / S);
        int before = 0, polls = left ? kSettledPolls : p.polls;
        const bool ok = polls >= -1 && rows_before(pub, segments, p.seg_bits, S, slot, ((p.B * p.Hkv) & 7) == 0, polls, lane, before);
        bool bad;
        const int held = gsc_base_rows(p, bh, bad);
        if (lane == 0) {
            const int64_t total = (int64_t)held + before + rows;
            if (ok && (flags & kWinLast)) {
                // (-1 in the end if the rows before any window of the head did not arrive, whatever the order)
                __hip_atomic_store(p.comp_lens + bh, (!bad && total <= cap) ? (int32_t)total : -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if ((__hip_atomic_load(p.head_state + bh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kHeadFailed) != 0u)
                    __hip_atomic_store(p.comp_lens + bh, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!ok && left) {
                __hip_atomic_fetch_or(p.head_state + bh, kHeadFailed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __hip_atomic_store(p.comp_lens + bh, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s.base_ok = ok ? 1 : 0;
            s.base_lo = (int)min((int64_t)held + before, (int64_t)0x7FFFFFFF);      // (beyond any capacity: nothing is written)
        }
    };

    // Windows that were left.  Their workgroups have filed what the merged rows need (whole chunks: the output row of every row, in the workspace),
    // marked them in their words and set kHeadLeft; then they search, and so does every workgroup of the head that finds kHeadLeft set after
    // what it has published has arrived.  A search takes the slots in order up to the first whose rows are not published, clears the marks that it finds
    // (a long chunk's not before its clusters have arrived, too) and finishes those windows.  So the last of the windows before a left one to publish
    // finds it, if no other has, and every window is finished once, by a workgroup that finds the rows of all before it published.  (The look costs
    // 0.4 to 1 %: 8 heads x 32768 49.3 us and 49.5, x 131072 166.5 and 168.3.  The value that the addition to the segment's rows can return
    // would say the same, but its returning form costs 1.5 to 2 %.)
    // The next window to finish goes to `win`, its rows to s.nseed; false: none.  For all wavefronts.
    [[maybe_unused]] auto next_left = [&](bool mark) {
        __syncthreads();
        if (threadIdx.x < kWave) {
            SC_FRESH_PARAMS;
            const int lane = fresh_lane(), slots = p.win_slots;
            uint32_t *pub = p.published + bh * slots;
            if (mark) {
                if (lane == 0) __hip_atomic_fetch_or(pub + win.slot, kPubLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (lane == 0) __hip_atomic_fetch_or(p.head_state + bh, kHeadLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            int found = -1, k0 = uniform(s.left_from);
            uint32_t word = 0u;
            for (; k0 < slots; k0 += kWave) {
                uint32_t w = kPubRows;
                bool mine = false;
                if (k0 + lane < slots) {
                    w = __hip_atomic_load(pub + k0 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    mine = (w & kPubLeft) != 0u && ((w & kPubReady) != 0u || (p.windows[(int64_t)b * slots + k0 + lane].flags & kWinLong) == 0);
                }
                const uint64_t missing = ballot64((w & kPubRows) == 0u);
                uint64_t marked = ballot64(mine);
                if (missing != 0ull) marked &= bits_below(first_bit(missing));
                for (; marked != 0ull && found < 0; marked &= marked - 1ull) {
                    const int at = k0 + first_bit(marked);
                    if (lane == 0) word = __hip_atomic_fetch_and(pub + at, ~kPubLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    word = (uint32_t)uniform((int)word);
                    if ((word & kPubLeft) != 0u) found = at;
                }
                if (found >= 0 || missing != 0ull) break;
            }
            if (lane == 0) {
                s.left_slot = found;
                s.left_from = k0;
                s.nseed = (int)(word & kPubValue);
            }
        }
        __syncthreads();
        const int at = uniform(s.left_slot);
        if (at >= 0) win = take_window(at, nullptr);
        return at >= 0;
    };
    // Last of all: were windows of the head left?  The wavefront that has published looks, once that has arrived.  For all wavefronts.
    [[maybe_unused]] auto any_left = [&](bool looks) {
        if (looks) {
            SC_FRESH_PARAMS;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const uint32_t state = __hip_atomic_load(p.head_state + bh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (fresh_lane() == 0) {
                s.any_left = (state & kHeadLeft) != 0u ? 1 : 0;
                s.left_from = 0;
            }
        }
        __syncthreads();
        return uniform(s.any_left) != 0;
    };

    const int decider = (place + bh_i) & (kWinWaves - 1);
    [[maybe_unused]] bool own = true;      // the merged rows of a long chunk: of this slot's; else of windows that were left
    [[maybe_unused]] bool mark = false;    // and this one is the first of them
    if (!ahead && !(flags & kWinLong)) {
        {
            SC_FRESH_LANE;
            RowRegs xk;
            load_rows(xk, Kbh, p.stride_n, w0 + 32 * wave, min(32, R - 32 * wave), g, c);
            if (tid == 0) s.any_unsure = 0;
            file_norms(s, xk, R - 32 * wave, wave, g, c);
            park_rows(s, xk, wave, g, c);
        }
        __syncthreads();
        const bool odd = uniform(*reinterpret_cast<const int *>(s.odd_norms)) != 0;
        if constexpr (PROBE == kProbeSeveral) {
            SC_FRESH_LANE;
            ProbeTiles tiles;
            probe_products(s, D, R, wave, g, c, tiles);
            const RowChunks rows(D, lane);
            __syncthreads();      // the keys have been read
            ProbeWords &words = *reinterpret_cast<ProbeWords *>(s.rows);
            for (int t0 = 0; t0 < nodes; t0 += kWinWaves) {
                float taus[kWinWaves];
#pragma unroll
                for (int k = 0; k < kWinWaves; ++k) taus[k] = budget_node_tau(tau_lo, tau_hi, min(t0 + k, nodes - 1) + 1);
                // (lane group g files the words of threshold t0 + g)
                probe_words(tiles, taus, odd, wave, g, c, words.yes[t0 + g], words.unsure[t0 + g]);
            }
            __syncthreads();
            for (int t = wave; t < nodes; t += kWinWaves) {
                const float mine = budget_node_tau(tau_lo, tau_hi, t + 1);
                uint32_t *list = (wave < 2 ? &s.yes[0][0] : &s.unsure[0][0]) + (wave & 1) * 2 * kWinRows;
                Decision d;
                decide_window(rows, words.yes[t], words.unsure[t], 1, D, R, lane,
                              [&](const Pair64 &ask, int oa, int ob) { return settle_alone(list, Kbh + (int64_t)w0 * p.stride_n, p.stride_n, ask, oa, ob, mine, lane); }, d);
                if (lane == 0) p.win_count[(bh * p.win_slots + slot) * kProbeWords + t] = __popcll(d.seeds.a) + __popcll(d.seeds.b);
            }
            return;
        } else {
        // the values, on their way while the rows are decided.  (Requested with the keys they delay those of the windows behind, and with
        // them everything that waits for those windows' rows.)
        [[maybe_unused]] RowRegs xv;
        if constexpr (!COUNT) {
            SC_FRESH_LANE;
            load_rows(xv, Vbh, p.stride_n, w0 + 32 * wave, min(32, R - 32 * wave), g, c);
        }
        // wavefront w: column tiles 7 - w and w, nine tiles of the upper triangle; those of other chunks are left out
#pragma unroll 1
        for (int jj = 0; jj < 2; ++jj) {
            const int J = jj == 0 ? 7 - wave : wave;
            if (16 * J < R) {
                SC_FRESH_LANE;
                const uint64_t da = D.a & bits_below(min(16 * J, 64)), db = D.b & bits_below(max(16 * J - 64, 0));
                const int lo = db != 0ull ? 65 + last_bit(db) : (da != 0ull ? 1 + last_bit(da) : 0);      // first row of the chunk of row 16 J
                gram_column(s, J, lo >> 4, R, tau, odd, g, c);
            }
        }
        __syncthreads();
        [[maybe_unused]] ColumnOps kk;
        const int nks = (R + 31) >> 5;
        if (wave == decider) {
            SC_FRESH_LANE;
            const RowChunks rows(D, lane);
            const bool delim_a = (D.a >> lane) & 1ull, delim_b = (D.b >> lane) & 1ull;
            const bool open_a = lane < R, open_b = 64 + lane < R;
            Decision d;
            decide_window(rows, s.yes, s.unsure, s.any_unsure, D, R, lane,
                          [&](const Pair64 &ask, int oa, int ob) { return settle_pairs(s, ask, oa, ob, tau, lane, wave, nullptr, 0, nullptr); }, d);
            const int nseed = __popcll(d.seeds.a) + __popcll(d.seeds.b);
            publish(nseed, false, lane);
            if constexpr (!COUNT) {
                const int out_a = open_a ? rows_below(d.seeds, d.seed_a) : -1, out_b = open_b ? rows_below(d.seeds, d.seed_b) : -1;
                SC_FRESH_PARAMS;
                if (p.cluster_id) {
                    int32_t *cid = p.cluster_id + bh * p.N_max + w0;
                    if (open_a) cid[lane] = delim_a ? -1 : out_a - rows_below(d.seeds, rows.lo_a);
                    if (open_b) cid[64 + lane] = delim_b ? -1 : out_b - rows_below(d.seeds, rows.lo_b);
                }
                file_membership(s, out_a, out_b, (nseed + 15) >> 4, lane);
                if (lane == 0) s.nseed = nseed;
                column_operands(s, wave, g, c, nks, kk);
            }
            decided(s, lane);
        } else {
            SC_FRESH_LANE;
            if constexpr (!COUNT) column_operands(s, wave, g, c, nks, kk);
            settle_until_decided(s, tau, lane, wave, nullptr, 0, nullptr);
        }
        if constexpr (COUNT) return;
        else {
            // everybody has the keys: the values take their place
            SC_FRESH_LANE;
            const int nseed = uniform(s.nseed);
            park_rows(s, xv, wave, g, c);
            if (wave == ((decider + 1) & (kWinWaves - 1))) find_base(nseed, false);
            __syncthreads();
            if (uniform(s.base_ok) != 0) {
                ColumnOps vv;
                column_operands(s, wave, g, c, nks, vv);
                const int64_t base = uniform(s.base_lo);
                const bool odd_keys = uniform(s.any_unsure) != 0;      // (a key that is not finite has no usable norm)
                SC_FRESH_PARAMS;
                const int64_t cap = p.cap;
                TO *Kat = reinterpret_cast<TO *>(p.Kc) + (bh * cap + base) * kFastD, *Vat = reinterpret_cast<TO *>(p.Vc) + (bh * cap + base) * kFastD;
                int32_t *counts = p.counts + bh * cap;
                for (int ot = 0; 16 * ot < nseed; ++ot) {
                    floatx4_t ke = {0.f, 0.f, 0.f, 0.f}, ko = ke, ve = ke, vo = ke, cn = ke;
                    const int steps = uniform(s.tile_steps[ot]);
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        if ((steps >> ks) & 1) {
                            const bf16x8f_t mem = membership_operand(s.hot[ot], ks, c, g);
                            ke = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk.x[ks][0], mem, ke, 0, 0, 0);
                            ko = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk.x[ks][1], mem, ko, 0, 0, 0);
                            ve = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv.x[ks][0], mem, ve, 0, 0, 0);
                            vo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv.x[ks][1], mem, vo, 0, 0, 0);
                            cn = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_operand(), mem, cn, 0, 0, 0);
                        }
                    }
                    const int o = 16 * ot + c;
                    float scale = mean_scale(cn[0]);
                    if (ballot64(!all_finite(ve, vo) || (odd_keys && !all_finite(ke, ko))) != 0ull) {
                        scale *= 2.f;
                        auto member = [&](int r) { return ((s.hot[ot][r] >> c) & 1) != 0; };
                        sums_by_member(Kbh + (int64_t)w0 * p.stride_n, p.stride_n, R, member, wave, g, ke, ko);
                        sums_by_member(Vbh + (int64_t)w0 * p.stride_n, p.stride_n, R, member, wave, g, ve, vo);
                    }
                    if (o < nseed && base + o < cap) {
                        store_mean<TO>(Kat + o * kFastD, ke, ko, scale, wave, g);
                        store_mean<TO>(Vat + o * kFastD, ve, vo, scale, wave, g);
                        if (wave == 0 && g == 0) counts[base + o] = (int)(0.5f * cn[0] + 0.5f);
                    }
                }
                if ((flags & kWinLast) || !any_left(wave == decider)) return;      // (nobody waits for the last one's rows)
            } else {
                // left to others, who need the output row of every row
                SC_FRESH_PARAMS;
                if (tid < R) {
                    int out = -1;
                    for (int t = 0; 16 * t < nseed; ++t)
                        if (s.hot[t][tid] != 0) out = 16 * t + __ffs((int)s.hot[t][tid]) - 1;
                    __hip_atomic_store(p.stmp + bh * p.N_max + w0 + tid, out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (tid == 0) s.left_from = 0;
                mark = true;
            }
            own = false;
        }
        }
    }

    // ---------------- one chunk longer than a window: blocks of 128 rows.  Seeds are listed in the workspace (row and reciprocal norm); a block's rows
    // are first compared with the seeds of the blocks before, 64 at a time, sixteen per wavefront, then among themselves.
    else if (ahead) {
    own = false;
    RowRegs x;
    {
        SC_FRESH_LANE;
        load_rows<0>(x, Kbh, p.stride_n, w0 + 32 * wave, min(32, R - 32 * wave), g, c);
    }
    for (;;) {
    SC_FRESH_PARAMS;
    // (the next one is looked up and its first rows are requested while this one is worked on)
    const int after = next_long + p.ahead_per_head;
    const bool more = take_long(after / nodes, next);
    const int start = w0, l = R;
    const bool closed = (flags & kWinClosed) != 0;
    int32_t *seed_rows = p.seedrow + bh * p.N_max + start;
    int32_t *seed_rinv = p.stmp + bh * p.N_max + start;
    if constexpr (COUNT) {      // the chunk is decided at several thresholds at once: a list for each, where the means of a merge would go
        const int64_t lists = (int64_t)n_bh * kProbeWords * p.N_max;
        seed_rows = reinterpret_cast<int32_t *>(p.rows_ws) + (bh * kProbeWords + next_long % nodes) * p.N_max + start;
        seed_rinv = seed_rows + lists;
    }
    int32_t *cid = p.cid + bh * p.N_max + start;
    const bf16_t *Kch = Kbh + (int64_t)start * p.stride_n;
    // The first sixteen stay at hand: their keys in registers (the A operand of the comparison), their sums over the keys in accumulators.  If there are
    // no more, their means wait in the workspace, and the keys need not be read again.
    int nseeds = 0;
    bf16x8f_t carried[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) carried[ks] = __builtin_bit_cast(bf16x8f_t, make_uint4(0u, 0u, 0u, 0u));
    [[maybe_unused]] floatx4_t ke = {0.f, 0.f, 0.f, 0.f}, ko = ke;
    [[maybe_unused]] int members = 0;      // rows of cluster c among those that the lane's operands have held
#pragma unroll 1
    for (int rb = 0; rb < l; rb += kWinRows) {
        const int Rb = min(kWinRows, l - rb), nx = rb + kWinRows;
        {
            SC_FRESH_LANE;
            if (tid == 0) s.any_unsure = 0;
            file_norms(s, x, Rb - 32 * wave, wave, g, c);
            park_rows(s, x, wave, g, c);
            // on its way while this block is worked on
            if (nx < l) load_rows<0>(x, Kch, p.stride_n, nx + 32 * wave, min(32, l - nx - 32 * wave), g, c);
            else if (more) load_rows<0>(x, Kbh, p.stride_n, next.first + 32 * wave, min(32, next.rows - 32 * wave), g, c);
        }
        __syncthreads();
        const bool odd = uniform(*reinterpret_cast<const int *>(s.odd_norms)) != 0;
        Pair64 open = {bits_below(min(Rb, 64)), bits_below(max(Rb - 64, 0))};      // (the deciding wavefront's)
        int my_a = -1, my_b = -1;      // cluster of the lane's rows
        bool any_open = true;
#pragma unroll 1
        for (int s0 = 0; s0 < nseeds && any_open; s0 += 16 * kWinWaves) {
            SC_FRESH_LANE;
            // (one group of sixteen: its row tiles are shared out)
            const bool shared = nseeds - s0 <= 16;
            const int first = s0 + (shared ? 0 : 16 * wave), ns = min(16, nseeds - first);
            if (ns > 0) {
                bf16x8f_t a[4];
                floatx4_t rs;
                if (first == 0) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) a[ks] = carried[ks];
                    rs = *reinterpret_cast<const floatx4_t *>(s.seed_rinv + 4 * g);
                } else {
                    const int srow = (c < ns) ? __hip_atomic_load(seed_rows + first + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                    const bf16_t *sp = Kch + (int64_t)srow * p.stride_n + 8 * g;
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        a[ks] = __builtin_bit_cast(bf16x8f_t, (c < ns) ? *reinterpret_cast<const uint4 *>(sp + 32 * ks) : make_uint4(0u, 0u, 0u, 0u));
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        rs[i] = (4 * g + i < ns) ? __int_as_float(__hip_atomic_load(seed_rinv + first + 4 * g + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0.f;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) rs[i] = (4 * g + i < ns) ? rs[i] : 0.f;
                const float rsum = (rs[0] + rs[1]) + (rs[2] + rs[3]);      // not a number if one of them is
                const bool odd_seed = ballot64(!(rsum == rsum)) != 0ull;
                const int J_step = shared ? kWinWaves : 1;
                for (int J = shared ? wave : 0; 16 * J < Rb; J += J_step) {
                    floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        const uint4 v = *reinterpret_cast<const uint4 *>(s.rows + (16 * J + c) * kKeyRowBytes + (32 * ks + 8 * g) * 2);
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], __builtin_bit_cast(bf16x8f_t, v), acc, 0, 0, 0);
                    }
                    float hn, wn;
                    column_bounds(s.rinv[16 * J + c], 16 * J + c < Rb, tau, hn, wn);
                    Nibbles n = threshold_nibbles(acc, rs, hn);
                    uint32_t ub = 0u;
                    if (odd_seed || odd || ballot64(n.least <= __float_as_uint(wn)) != 0ull) ub = unsure_nibble(n, wn);
                    const uint32_t yb = n.yes;
                    const uint32_t both = or_rows((yb << (4 * g)) | (ub << (16 + 4 * g)));
                    const uint32_t valid = (1u << ns) - 1u;
                    if (g == 0) {
                        reinterpret_cast<uint16_t *>(s.yes[16 * J + c])[shared ? 0 : wave] = (uint16_t)(both & valid);
                        reinterpret_cast<uint16_t *>(s.unsure[16 * J + c])[shared ? 0 : wave] = (uint16_t)((both >> 16) & valid);
                    }
                }
            }
            __syncthreads();
            if (wave == decider) {
                const bool open_a = (open.a >> lane) & 1ull, open_b = (open.b >> lane) & 1ull;
                const uint64_t there = bits_below(min(64, nseeds - s0));      // (groups that do not exist have filed nothing)
                uint64_t ya = open_a ? row_word(s.yes, lane, 0) & there : 0ull, ua = open_a ? row_word(s.unsure, lane, 0) & there : 0ull;
                uint64_t yb = open_b ? row_word(s.yes, 64 + lane, 0) & there : 0ull, ub = open_b ? row_word(s.unsure, 64 + lane, 0) & there : 0ull;
                if (lane == 0) s.first_seed = s0;
                // first fit over these seeds; a pair inside the band is settled in fp64 when it is the first candidate of its row
                for (;;) {
                    const int fa = (ya | ua) != 0ull ? first_bit(ya | ua) : 0, fb = (yb | ub) != 0ull ? first_bit(yb | ub) : 0;
                    Pair64 ask;
                    ask.a = ballot64((ua >> fa) & 1ull);
                    ask.b = ballot64((ub >> fb) & 1ull);
                    if ((ask.a | ask.b) == 0ull) break;
                    const Pair64 above = settle_pairs(s, ask, fa, fb, tau, lane, wave, Kch, p.stride_n, seed_rows);
                    if ((ask.a >> lane) & 1ull) {
                        ua &= ~(1ull << fa);
                        if ((above.a >> lane) & 1ull) ya |= 1ull << fa;
                    }
                    if ((ask.b >> lane) & 1ull) {
                        ub &= ~(1ull << fb);
                        if ((above.b >> lane) & 1ull) yb |= 1ull << fb;
                    }
                }
                if (ya != 0ull) my_a = s0 + first_bit(ya);
                if (yb != 0ull) my_b = s0 + first_bit(yb);
                open.a &= ~ballot64(ya != 0ull);
                open.b &= ~ballot64(yb != 0ull);
                if (lane == 0) s.open = (open.a | open.b) != 0ull ? 1 : 0;
                decided(s, lane);
            } else {
                settle_until_decided(s, tau, lane, wave, Kch, p.stride_n, seed_rows);
            }
            any_open = uniform(s.open) != 0;      // (the words are read: the next seeds' may come)
        }
        if (any_open) {
#pragma unroll 1
            for (int jj = 0; jj < 2; ++jj) {
                const int J = jj == 0 ? 7 - wave : wave;
                SC_FRESH_LANE;
                if (16 * J < Rb) gram_column(s, J, 0, Rb, tau, odd, g, c);
            }
            __syncthreads();
        }
        if (wave == decider) {
            SC_FRESH_LANE;
            int now = nseeds;
            if (any_open) {
                // the rows still open are decided among themselves; the new seeds continue the chunk's numbering
                const bool open_a = (open.a >> lane) & 1ull, open_b = (open.b >> lane) & 1ull;
                const uint64_t below = bits_below(lane);
                Words y, u;
                y.a = open_a ? row_word(s.yes, lane, 0) & below & open.a : 0ull;
                y.b0 = open_b ? row_word(s.yes, 64 + lane, 0) & open.a : 0ull;
                y.b1 = open_b ? row_word(s.yes, 64 + lane, 1) & below & open.b : 0ull;
                u.a = u.b0 = u.b1 = 0ull;
                if (uniform(s.any_unsure) != 0) {
                    u.a = open_a ? row_word(s.unsure, lane, 0) & below & open.a : 0ull;
                    u.b0 = open_b ? row_word(s.unsure, 64 + lane, 0) & open.a : 0ull;
                    u.b1 = open_b ? row_word(s.unsure, 64 + lane, 1) & below & open.b : 0ull;
                }
                Decision d;
                auto settle = [&](const Pair64 &ask, int oa, int ob) { return settle_pairs(s, ask, oa, ob, tau, lane, wave, nullptr, 0, nullptr); };
                if (!first_fit_fixed_point(settle, y, u, open_a, open_b, lane, d)) {
                    const Pair64 all = {~0ull, ~0ull};
                    first_fit_by_seed(settle, y, u, open, all, all, lane, d);
                }
                if (open_a) my_a = nseeds + rows_below(d.seeds, d.seed_a);
                if (open_b) my_b = nseeds + rows_below(d.seeds, d.seed_b);
                // seed list of the chunk, filed by the new seeds themselves
                if ((d.seeds.a >> lane) & 1ull) {
                    __hip_atomic_store(seed_rows + my_a, rb + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(seed_rinv + my_a, __float_as_int(s.rinv[lane]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (my_a < 16) {
                        s.seed_rinv[my_a] = s.rinv[lane];
                        s.seed_row[my_a] = rb + lane;
                    }
                }
                if ((d.seeds.b >> lane) & 1ull) {
                    __hip_atomic_store(seed_rows + my_b, rb + 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(seed_rinv + my_b, __float_as_int(s.rinv[64 + lane]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (my_b < 16) {
                        s.seed_rinv[my_b] = s.rinv[64 + lane];
                        s.seed_row[my_b] = rb + 64 + lane;
                    }
                }
                now = nseeds + __popcll(d.seeds.a) + __popcll(d.seeds.b);
            }
            // cluster of every row: the caller's output, and what the sweeps for the means read back
            if (!COUNT && lane < Rb) __hip_atomic_store(cid + rb + lane, my_a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!COUNT && 64 + lane < Rb) __hip_atomic_store(cid + rb + 64 + lane, my_b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) s.nseed = now;
            if constexpr (!COUNT) file_membership(s, (lane < Rb) ? my_a : -1, (64 + lane < Rb) ? my_b : -1, 1, lane);
            if (nx >= l) publish(now + (closed ? 1 : 0), true, lane);
            // seeds and clusters are where others read them: seeds beyond the sixteenth in the next block, clusters in the workgroup of the window's slot
            if (now > 16 || nx >= l) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            decided(s, lane);
        } else {
            settle_until_decided(s, tau, fresh_lane(), wave, nullptr, 0, nullptr);
        }
        const int known = nseeds;
        nseeds = uniform(s.nseed);
        SC_FRESH_LANE;
        if (known < 16 && nseeds > known) {
            const bool fresh = c >= known && c < nseeds;
            const int row = fresh ? s.seed_row[c] - rb : 0;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const uint4 v = *reinterpret_cast<const uint4 *>(s.rows + row * kKeyRowBytes + (32 * ks + 8 * g) * 2);
                if (fresh) carried[ks] = __builtin_bit_cast(bf16x8f_t, v);
            }
        }
        if constexpr (!COUNT) {
            const int steps = uniform(s.tile_steps[0]);
#pragma unroll 1
            for (int ks = 0; ks < 4; ++ks) {
                if ((steps >> ks) & 1) {
                    bf16x8f_t even, odds;
                    column_step(s, wave, g, c, ks, even, odds);
                    const bf16x8f_t mem = membership_operand(s.hot[0], ks, c, g);
                    ke = __builtin_amdgcn_mfma_f32_16x16x32_bf16(even, mem, ke, 0, 0, 0);
                    ko = __builtin_amdgcn_mfma_f32_16x16x32_bf16(odds, mem, ko, 0, 0, 0);
                    const uint4 bits = __builtin_bit_cast(uint4, mem);
                    members += __popc(bits.x) + __popc(bits.y) + __popc(bits.z) + __popc(bits.w);
                }
            }
        }
        __syncthreads();      // the next block overwrites the parked keys and the words
    }
    if constexpr (!COUNT) {
        uint32_t *pub = p.published + bh * p.win_slots;
        if (nseeds <= 16) {
            SC_FRESH_LANE;
            TO *key_means = reinterpret_cast<TO *>(p.rows_ws) + bh * p.N_max * kFastD;
            members += __shfl_xor(members, 16, kWave);
            members += __shfl_xor(members, 32, kWave);
            float scale = mean_scale(2.f * (float)members);
            if (ballot64(!all_finite(ke, ko)) != 0ull) {
                scale *= 2.f;
                sums_by_member(Kch, p.stride_n, l, [&](int r) { return __hip_atomic_load(cid + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == c; }, wave, g, ke, ko);
            }
            if (c < nseeds) store_mean_through<TO>(key_means + (int64_t)(start + kMeansAt) * kFastD, c, ke, ko, scale, wave, g);
        }
        if (closed && tid == 0 && p.cluster_id) p.cluster_id[bh * p.N_max + start + l] = -1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_or(pub + slot, kPubReady, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!uniform(more ? 1 : 0)) break;
    win = Window{uniform(next.slot), uniform(next.first), uniform(next.rows), uniform(next.flags)};
    next_long = after;
    if constexpr (COUNT) tau = budget_node_tau(tau_lo, tau_hi, 1 + next_long % nodes);
    }
    if constexpr (!COUNT) {
        if (!any_left(wave == 0)) return;      // (the rows arrived before the clusters were announced)
    }
    }

    // ---------------- means of a long chunk, and of windows that were left
    if constexpr (!COUNT) {
    for (;;) {
        if (!own && !next_left(mark)) return;
        mark = false;
        win = Window{uniform(win.slot), uniform(win.first), uniform(win.rows), uniform(win.flags)};
        own = uniform(own ? 1 : 0) != 0;
        SC_FRESH_PARAMS;
        const int64_t cap = p.cap;
        TO *Kout = reinterpret_cast<TO *>(p.Kc) + bh * cap * kFastD, *Vout = reinterpret_cast<TO *>(p.Vc) + bh * cap * kFastD;
        int32_t *counts = p.counts + bh * cap;
        TO *key_means = reinterpret_cast<TO *>(p.rows_ws) + bh * p.N_max * kFastD;
        const int start = w0, l = R;
        const bool closed = (flags & kWinClosed) != 0;
        // (cluster of every row; a window of whole chunks: the output row)
        const int32_t *cid = ((flags & kWinLong) ? p.cid : p.stmp) + bh * p.N_max + start;
        const bf16_t *Kch = Kbh + (int64_t)start * p.stride_n;
        // the values of the first block are on their way while the place is looked up
        const bf16_t *Vch = Vbh + (int64_t)start * p.stride_n;
        SC_FRESH_LANE;
        RowRegs x;
        load_rows(x, Vch, p.stride_n, 32 * wave, min(32, l - 32 * wave), g, c);
        if (own && wave == decider) {      // what the workgroup that has decided the chunk has left
            const bool one_xcd = ((p.B * p.Hkv) & 7) == 0;
            u32x16_t w;
            int polls = p.polls;
            w[0] = 0u;
            for (int look = 0; polls >= -1; ++look) {
                load_words(w, p.published + bh * p.win_slots + slot, one_xcd && look % kVectorEvery != kVectorEvery - 1, lane);
                if ((w[0] & kPubReady) != 0u || --polls < 0) break;
                __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0) s.nseed = (w[0] & kPubReady) != 0u ? (int)(w[0] & kPubValue) : -1;
        }
        int oa = -1, ob = -1;      // clusters of the block's rows
        auto request_clusters = [&](int rb) {
            oa = ob = -1;
            if (wave == decider) {
                if (rb + lane < l) oa = __hip_atomic_load(cid + rb + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (rb + 64 + lane < l) ob = __hip_atomic_load(cid + rb + 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        request_clusters(0);
        __syncthreads();
        const int rows = uniform(s.nseed), nseeds = rows - (closed ? 1 : 0);
        // The place is looked up when the first sums are there: the windows just before are being decided meanwhile.
        int64_t base = -1;
        auto look_up = [&]() {
            if (wave == decider) find_base(rows, !own);
            __syncthreads();
            base = uniform(s.base_lo);
            return uniform(s.base_ok) != 0;
        };
        bool ok = rows >= 0;
        // kTiles tiles of sixteen clusters per sweep over the chunk: values, then keys
        constexpr int kTiles = 2;
        auto finish = [&](const bf16_t *X, TO *out, int o0, floatx4_t even, floatx4_t odd, const floatx4_t &n, bool sizes) {
            const int o = o0 + c;
            float scale = mean_scale(n[0]);
            if (ballot64(!all_finite(even, odd)) != 0ull) {
                scale *= 2.f;
                auto member = [&](int r) { return __hip_atomic_load(cid + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == o; };
                sums_by_member(X, p.stride_n, l, member, wave, g, even, odd);
            }
            if (o < nseeds && base + o < cap) {
                store_mean<TO>(out + (base + o) * kFastD, even, odd, scale, wave, g);
                if (sizes && wave == 0 && g == 0) counts[base + o] = (int)(0.5f * n[0] + 0.5f);
            }
        };
        const bool keys_done = (flags & kWinLong) != 0 && nseeds <= 16;
        bool first = true;
#pragma unroll 1
        for (int src = 0; ok && src < (keys_done ? 1 : 2); ++src) {
            const bf16_t *Xch = src == 0 ? Vch : Kch;
#pragma unroll 1
            for (int o0 = 0; o0 < nseeds; o0 += 16 * kTiles) {
                floatx4_t ev[kTiles], od[kTiles], sz[kTiles];
#pragma unroll
                for (int t = 0; t < kTiles; ++t) ev[t] = od[t] = sz[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
                if (!first) {
                    load_rows(x, Xch, p.stride_n, 32 * wave, min(32, l - 32 * wave), g, c);
                    request_clusters(0);
                }
                first = false;
#pragma unroll 1
                for (int rb = 0; rb < l; rb += kWinRows) {
                    const int Rb = min(kWinRows, l - rb);
                    __syncthreads();      // the block before has been read
                    park_rows(s, x, wave, g, c);
                    if (wave == decider) file_membership(s, oa - o0, ob - o0, kTiles, lane);
                    const int nx = rb + kWinRows;
                    if (nx < l) {      // on their way while this block is worked on
                        load_rows(x, Xch, p.stride_n, nx + 32 * wave, min(32, l - nx - 32 * wave), g, c);
                        request_clusters(nx);
                    }
                    __syncthreads();
                    int steps[kTiles];
#pragma unroll
                    for (int t = 0; t < kTiles; ++t) steps[t] = uniform(s.tile_steps[t]);
#pragma unroll 1
                    for (int ks = 0; 32 * ks < Rb; ++ks) {
                        bf16x8f_t even, odd;
                        column_step(s, wave, g, c, ks, even, odd);
#pragma unroll
                        for (int t = 0; t < kTiles; ++t) {
                            if ((steps[t] >> ks) & 1) {
                                const bf16x8f_t mem = membership_operand(s.hot[t], ks, c, g);
                                ev[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(even, mem, ev[t], 0, 0, 0);
                                od[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(odd, mem, od[t], 0, 0, 0);
                                sz[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_operand(), mem, sz[t], 0, 0, 0);
                            }
                        }
                    }
                }
                if (base < 0) {
                    ok = look_up();
                    if (!ok) break;
                    if (keys_done) {
                        // sixteen lanes a row
                        constexpr int kPieces = (int)sizeof(TO) * kFastD / 256;
                        const int o = tid >> 4;
                        if (o < nseeds && base + o < cap) {
                            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(key_means + (int64_t)(start + kMeansAt) * kFastD, (short)0, 16 * kFastD * (int)sizeof(TO), 0x00020000);
#pragma unroll
                            for (int e = 0; e < kPieces; ++e) {
                                const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, o * kFastD * (int)sizeof(TO) + 16 * (16 * e + (tid & 15)), 0, 16);
                                store16_stream(reinterpret_cast<char *>(Kout + (base + o) * kFastD) + 16 * (16 * e + (tid & 15)), make_uint4(v.x, v.y, v.z, v.w));
                            }
                        }
                    }
                }
#pragma unroll
                for (int t = 0; t < kTiles; ++t)
                    if (o0 + 16 * t < nseeds) finish(Xch, src == 0 ? Vout : Kout, o0 + 16 * t, ev[t], od[t], sz[t], src == 0);
            }
        }
        if (ok && closed && base + nseeds < cap && tid < 16) {
            // the closing delimiter is the output row behind: a copy with size 1
            float kv[8], vv[8];
            load8(Kbh + (int64_t)(start + l) * p.stride_n + 8 * c, kv);
            load8(Vbh + (int64_t)(start + l) * p.stride_n + 8 * c, vv);
            store8(Kout + (base + nseeds) * kFastD + 8 * c, kv);
            store8(Vout + (base + nseeds) * kFastD + 8 * c, vv);
            if (tid == 0) counts[base + nseeds] = 1;
        }
        if (own) {
            if (ok) return;
            // left to others; its clusters are, or will be, in the workspace
            own = false;
            mark = true;
            if (tid == 0) s.left_from = 0;
        }
    }
    }
}

// ------------------------------------------------------------------------------------------------
// count: rows of every (sequence, head) at each threshold of a counting probe, and what the budget search does with them.  Two threads a window,
// 512 windows at a time: one trip to memory for a sequence of 32768 tokens, and a kernel of little else.
constexpr int kCountThreads = 1024;
__global__ __launch_bounds__(kCountThreads) void gsc_count_kernel(GscParams p) {
    constexpr int kWaves = kCountThreads / kWave;
    static_assert(kProbeWords == 8 && kWaves == 16, "two threads a window; two wavefronts a lane in the last sum");
    __shared__ __attribute__((aligned(16))) int s_sum[kWaves][kProbeWords];
    const int64_t bh = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid / kWave), half = tid & 1;
    const int4 *cnt = reinterpret_cast<const int4 *>(p.win_count + bh * p.win_slots * kProbeWords) + half;
    int4 sum = make_int4(0, 0, 0, 0);
    for (int i = tid >> 1; i < p.win_slots; i += 2 * (kCountThreads / 2)) {
        const int j = i + kCountThreads / 2;
        const int4 x = cnt[2 * (int64_t)i], y = j < p.win_slots ? cnt[2 * (int64_t)j] : make_int4(0, 0, 0, 0);
        sum.x += x.x + y.x; sum.y += x.y + y.y; sum.z += x.z + y.z; sum.w += x.w + y.w;
    }
#pragma unroll
    for (int d = 32; d >= 2; d >>= 1) {
        sum.x += __shfl_xor(sum.x, d, kWave); sum.y += __shfl_xor(sum.y, d, kWave);
        sum.z += __shfl_xor(sum.z, d, kWave); sum.w += __shfl_xor(sum.w, d, kWave);
    }
    if (lane < 2) *reinterpret_cast<int4 *>(&s_sum[wave][4 * half]) = sum;
    __syncthreads();
    if (wave == 0) {
        int at = s_sum[lane / kProbeWords][lane & (kProbeWords - 1)] + s_sum[lane / kProbeWords + 8][lane & (kProbeWords - 1)];
#pragma unroll
        for (int d = 32; d >= kProbeWords; d >>= 1) at += __shfl_xor(at, d, kWave);
        bool bad;
        const int64_t total = (int64_t)gsc_base_rows(p, bh, bad) + at;
        const int rows = (p.num_chunks[bh / p.Hkv] > 0 && !bad && total <= p.cap) ? (int)total : -1;
        budget_probe_arrive(p.budget, rows, lane, p.probe_levels, (unsigned int)(p.B * p.Hkv));      // (lane t: threshold t; the eighth sum is of words that nobody asks for)
    }
}

// ------------------------------------------------------------------------------------------------
static int segments_of(int n_max) { return (n_max + kSegRows - 1) / kSegRows; }
// a workgroup of the compress kernel for every slot and those ahead (a probe's, which are more than a merge's): fewer than 2^32 threads in a launch, and
// the rows of a segment in its word
static bool fast_holds(int heads, int n_max, int max_chunks) {
    const int S = gsc_slots_per_segment(n_max, max_chunks);
    return segment_holds(S, n_max) && ((int64_t)segments_of(n_max) * S * heads + max(heads, max(kAheadWgs, kAheadProbes))) * kWinThreads < (int64_t(1) << 32);
}
bool gsc_fast_holds(int heads, int N_max) { return fast_holds(heads, N_max, 0); }

hipError_t launch_gsc_fast(const GscParams &p0, bool planned, const BudgetStart *start, hipStream_t stream) {
    GscParams p = p0;
    const int segments = segments_of(p.N_max);
    if (!fast_holds(p.B * p.Hkv, p.N_max, p.max_chunks)) p.max_chunks = 0;
    p.slots_per_segment = gsc_slots_per_segment(p.N_max, p.max_chunks);
    p.seg_bits = segment_bits(p.slots_per_segment);
    p.win_slots = segments * p.slots_per_segment;
    // the workspace has two arrays of rows, 256 bytes or more per token and head each: means of long chunks at rows of their own in the one, everything
    // else in the other (at most 1024 + 16 slots per 1024 tokens)
    const size_t bh = (size_t)p.B * p.Hkv;
    p.segments = reinterpret_cast<GscSegment *>(reinterpret_cast<char *>(p.rows_ws) + align_up(bh * (size_t)p.N_max * kFastD * (p.out_is_bf16 ? 2 : 4), 256)) + kSegFront;
    p.windows = reinterpret_cast<GscWindow *>(reinterpret_cast<char *>(p.segments - kSegFront) + align_up((bh * (size_t)segments + kSegFront) * sizeof(GscSegment), sizeof(GscWindow)));
    p.published = reinterpret_cast<uint32_t *>(p.windows + (size_t)p.B * p.win_slots);
    p.win_count = reinterpret_cast<int32_t *>(p.published + align_up(bh * (size_t)p.win_slots, 8));
    p.longs = reinterpret_cast<GscLongs *>(p.win_count + bh * (size_t)p.win_slots * kProbeWords);
    p.head_state = reinterpret_cast<uint32_t *>(p.rowbase);
    p.long_count = reinterpret_cast<int32_t *>(p.longs + (size_t)segments * p.B);
    // Half of what is resident together, the rest goes to windows (a quarter or three quarters: the same within 1 %); where there are no long
    // chunks, all of them leave within a microsecond.  (One for every 512 tokens instead: a long-tailed call of 8 heads x 4000 took
    // 41 us against 32.)
    const size_t longest = ((size_t)p.N_max / (kWinRows + 1) + 1) * (p.count_only ? (size_t(1) << p.probe_levels) - 1 : 1);
    p.ahead_per_head = p.N_max < kWinRows ? 0 : (int)max((size_t)1, min(longest, (size_t)(p.count_only ? kAheadProbes : kAheadWgs) / bh));
    p.ahead_wgs = (int)(bh * p.ahead_per_head);
    if (!planned) {
        const dim3 grid((unsigned)(segments * p.B));
        if (start) hipLaunchKernelGGL((gsc_plan_kernel<BudgetStart>), grid, dim3(kWave), 0, stream, p, *start);
        else hipLaunchKernelGGL((gsc_plan_kernel<>), grid, dim3(kWave), 0, stream, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((size_t)p.win_slots * bh + p.ahead_wgs));
    if (p.count_only && p.probe_levels == 1) hipLaunchKernelGGL((gsc_compress_kernel<bf16_t, kProbeOne>), grid, dim3(kWinThreads), 0, stream, p);
    else if (p.count_only) hipLaunchKernelGGL((gsc_compress_kernel<bf16_t, kProbeSeveral>), grid, dim3(kWinThreads), 0, stream, p);
    else if (p.out_is_bf16) hipLaunchKernelGGL((gsc_compress_kernel<bf16_t, kNoProbe>), grid, dim3(kWinThreads), 0, stream, p);
    else hipLaunchKernelGGL((gsc_compress_kernel<float, kNoProbe>), grid, dim3(kWinThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p.count_only) return e;
    hipLaunchKernelGGL(gsc_count_kernel, dim3((unsigned)bh), dim3(kCountThreads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace sc
