// Paged attention over fp32 pools on the double-precision matrix cores (gfx950), head_dim 64 and 128, pages of 16 tokens
// and more, no hooks: decode (one query per sequence, with or without the step's append) and ragged prefill.
//
// fp32 results are held to about 2e-7, so every product and every sum runs in fp64 (v_mfma_f64_16x16x4_f64, 64 cycles,
// the same 78 TFLOP/s as the vector unit's fp64 but with 16 x 16 reuse of its operands); only the exponential is taken in
// fp32, of an argument reduced in fp64.  A workgroup of 8 waves owns 16 rows -- (query, head) pairs of one KV head, row =
// query * G + head -- and its waves take every eighth tile of 16 keys, each with its own softmax state; the 8 partials are
// merged through LDS.  16 rows rather than 32 or 64: a prompt of a few hundred tokens is all an fp32 call sees in earnest,
// and 8 heads x 777 tokens are then 392 workgroups instead of 200.  No LDS in the loop: both operands come from global
// memory in whole 16-byte pieces, because a contraction may run over its index in any order --
//   S^T[key, row] = K[key, :] . Q[row, :]^T   A: lane%16 = key, lane/16 picks elements 16*i + 4*(lane/16) + e of step (i, e)
//   O^T[col, row] += V^T[col, key] P^T        A: lane%16 = column 4*(lane%16) + e, lane/16 = key 4*r + lane/16 of step r
// and the accumulator of S^T (lane%16 = row, register r = key 4*r + lane/16) is the B operand of the second product as it
// stands.  Bound by the matrix pipe: 32 instructions of 64 cycles per 16 x 16 tile at head_dim 64, 8 us of a 777-token
// prompt over 8 heads if every SIMD had its share; the last row tile's 6 tiles a wave, two waves a SIMD, are 10.5.
// Append + prefill, portable kernel / this one: 1 x 777, 8 / 8 heads, head_dim 64 178 / 28.9 us, head_dim 128 367 / 49;
// 1 x 400 49.0 / 18.2; 1 x 64 10.4 / 8.4; error against 64 bits 1.1e-7 / 4.1e-8.  4 or 16 waves instead of 8: 36, 39 us
// at 1 x 777; registers held to 128 for two workgroups a compute unit: 41 us (spills).
#include "common.h"

namespace pa {

namespace {

typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kWaves = 8;
constexpr int kRows = 16;                // rows of a workgroup
constexpr int kKeys = 16;                // keys of a tile
constexpr double kLog2e = 1.44269504088896340736;
constexpr double kLn2 = 0.69314718055994530942;

// 2^y rounded to fp32: the fraction in [-1/2, 1/2] is exact in fp32 to 2^-26, so only the exponential itself rounds.
// NaN stays NaN; -inf (a key without weight, the reference of a row that has seen no key) gives 0.
__device__ __forceinline__ float exp2_of(double y)
{
    y = y < -200.0 ? -200.0 : y;
    const double n = __builtin_rint(y);
    return __builtin_ldexpf(__builtin_amdgcn_exp2f((float)(y - n)), (int)n);
}

// Lanes that hold the same r16 combined, by register swaps between rows of 16 lanes instead of LDS permutes (about 10
// cycles instead of 60 a step, in the middle of every tile's chain).  a = the value of rows 0, 2 (0, 1), b = of 1, 3 (2, 3).
struct DoublePair {
    double a, b;
};
__device__ __forceinline__ DoublePair swap16(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return {__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]), __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1])};
}
__device__ __forceinline__ DoublePair swap32(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return {__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]), __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1])};
}
__device__ __forceinline__ double quad_max(double v)
{
    const DoublePair p = swap16(v);
    const DoublePair r = swap32(__builtin_fmax(p.a, p.b));
    return __builtin_fmax(r.a, r.b);
}
__device__ __forceinline__ double quad_sum(double v)
{
    const DoublePair p = swap16(v);
    const DoublePair r = swap32(p.a + p.b);
    return r.a + r.b;
}
// v of the lane CTRL (row_ror) positions further in the row of 16
template <int CTRL>
__device__ __forceinline__ double rotate16(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double row_sum(double v)
{
    v += rotate16<0x128>(v);
    v += rotate16<0x124>(v);
    v += rotate16<0x122>(v);
    return v + rotate16<0x121>(v);
}
__device__ __forceinline__ double row_max(double v)
{
    v = __builtin_fmax(v, rotate16<0x128>(v));
    v = __builtin_fmax(v, rotate16<0x124>(v));
    v = __builtin_fmax(v, rotate16<0x122>(v));
    return __builtin_fmax(v, rotate16<0x121>(v));
}

template <int D>
struct TileRegs {
    float4 k[D / 16];        // row lane%16 of the tile: elements 16*i + 4*(lane/16) ..+3
    float4 v[D / 64][4];     // row 4*r + lane/16: elements 64*c + 4*(lane%16) ..+3
};

struct Rows {
    const char* k;           // pools at this KV head
    const char* v;
    const int32_t* table;
    int64_t page_bytes, token_bytes;
    int32_t log2_page, pmask;
    const char* knew;        // decode step: rows of the token at position new_pos
    const char* vnew;
    int32_t new_pos;
};

template <int D>
__device__ __forceinline__ void load_k(TileRegs<D>& t, const Rows& a, int64_t page, int32_t t0, int32_t last, int r16, int quad)
{
    const int32_t key = min(t0 + r16, last);
    const char* p = a.k + page * a.page_bytes + (int64_t)(key & a.pmask) * a.token_bytes;
    if (key == a.new_pos) p = a.knew;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) t.k[i] = *reinterpret_cast<const float4*>(p + 64 * i + 16 * quad);
}

template <int D>
__device__ __forceinline__ void load_v(TileRegs<D>& t, const Rows& a, int64_t page, int32_t t0, int32_t last, int r16, int quad)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int32_t key = min(t0 + 4 * r + quad, last);
        const char* p = a.v + page * a.page_bytes + (int64_t)(key & a.pmask) * a.token_bytes;
        if (key == a.new_pos) p = a.vnew;
#pragma unroll
        for (int c = 0; c < D / 64; ++c) t.v[c][r] = *reinterpret_cast<const float4*>(p + 256 * c + 16 * r16);
    }
}

// The compact grid's numbering of row tiles: sequence s has tiles first_tile(s) .. first_tile(s + 1) - 1, at most one more
// than its rows fill.  Returns the sequence of tile t (64 candidates a step: one round trip up to 64 sequences).
__device__ __forceinline__ int64_t first_tile(const int32_t* __restrict__ cu_q_lens, int32_t s, int32_t G)
{
    return (int64_t)cu_q_lens[s] * G / kRows + s;
}
__device__ __forceinline__ int32_t tile_sequence(const int32_t* __restrict__ cu_q_lens, int32_t batch, int32_t G, int64_t t,
                                                 int lane)
{
    int32_t lo = 0, hi = batch;
    while (hi - lo > 1) {
        const int32_t step = (hi - lo + 63) / 64, i = lo + lane * step;
        const uint64_t below = __ballot(i < hi && first_tile(cu_q_lens, min(i, batch - 1), G) <= t);
        lo += (__popcll((unsigned long long)below) - 1) * step;            // (lane 0 always is)
        hi = min(lo + step, hi);
    }
    return lo;
}

__device__ __forceinline__ float elem(const float4& v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; }

template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void paged_attention_f32_kernel(
    CacheView cache, const float* __restrict__ q, float* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_q_heads, int32_t max_blocks, float scale,
    int32_t causal, float* __restrict__ part_o, float* __restrict__ part_lse, int32_t chunk, int32_t nsplit,
    int32_t row_tiles, const float* __restrict__ k_new, const float* __restrict__ v_new)
{
    constexpr int kPad = D + 4;          // rows padded by 16 bytes: the 16 rows of a store land on distinct banks
    __shared__ __attribute__((aligned(16))) float sm_o[NW * kRows * kPad];
    __shared__ double sm_m[NW * kRows];
    __shared__ double sm_l[NW * kRows];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r16 = lane & 15, quad = lane >> 4;
    const int32_t G = num_q_heads / cache.num_kv_heads;
    // last row tiles (the heaviest under a causal bound) first
    int32_t b = blockIdx.x;
    const int32_t split = b % nsplit;
    b /= nsplit;
    const int32_t kvh = b % cache.num_kv_heads;
    b /= cache.num_kv_heads;
    int32_t s, m0;
    if (row_tiles > 0) {
        s = b % batch;
        m0 = (row_tiles - 1 - b / batch) * kRows;
    } else {                                                 // compact grid (see launch_attention_f32)
        s = tile_sequence(cu_q_lens, batch, G, b, lane);
        const int32_t rows = (cu_q_lens[s + 1] - cu_q_lens[s]) * G;
        m0 = ((rows + kRows - 1) / kRows - 1 - (int32_t)(b - first_tile(cu_q_lens, s, G))) * kRows;
        if (m0 < 0) return;
    }
    const int32_t c0 = split * chunk;

    Rows a;
    a.table = block_table + (int64_t)s * max_blocks;
    a.log2_page = cache.log2_page;
    a.pmask = cache.page_size - 1;
    // the page of this wave's first tile is requested along with the lengths (inside the table whatever the length is)
    const int32_t first = c0 + wave * kKeys;
    int32_t page = a.table[min(first >> a.log2_page, max_blocks - 1)];

    const int32_t len = seq_lens[s];
    int32_t q_begin = s, q_len = 1;
    if (cu_q_lens) {
        q_begin = cu_q_lens[s];
        q_len = cu_q_lens[s + 1] - q_begin;
    }
    const int32_t n_rows = q_len * G;
    if (m0 >= n_rows) return;
    const int32_t row = m0 + r16;
    const int32_t row_c = min(row, n_rows - 1);
    const int32_t qi = row_c / G;
    const int64_t o_row = (int64_t)(q_begin + qi) * num_q_heads + kvh * G + (row_c - qi * G);
    int32_t nk = len, nk_wg = len;                           // keys this lane's row sees; keys any row sees
    if (causal) {
        nk = max(min(len, len - q_len + qi + 1), 0);
        nk_wg = max(min(len, len - q_len + (min(m0 + kRows, n_rows) - 1) / G + 1), 0);
    }
    const int32_t c1 = min(nk_wg, c0 + chunk);
    if (c0 >= c1 && nsplit > 1) return;                      // (the merge reads only chunks that hold keys of a row)

    a.k = reinterpret_cast<const char*>(cache.k) + (int64_t)kvh * cache.head_stride * 4;
    a.v = reinterpret_cast<const char*>(cache.v) + (int64_t)kvh * cache.head_stride * 4;
    a.page_bytes = cache.page_stride * 4;
    a.token_bytes = cache.token_stride * 4;
    a.knew = a.vnew = nullptr;
    a.new_pos = -1;
    const int32_t last = len - 1;
    if (k_new) {                                             // decode step: the token at position len - 1 comes along
        const int64_t off = ((int64_t)s * cache.num_kv_heads + kvh) * D;
        a.knew = reinterpret_cast<const char*>(k_new + off);
        a.vnew = reinterpret_cast<const char*>(v_new + off);
        a.new_pos = last;
        // the wave whose tile holds it stores its rows (Algorithm 1, Assign); the tile reads k_new / v_new
        if (m0 == 0 && last >= c0 && last < c1 && ((last - c0) / kKeys) % NW == wave && lane < D / 2) {
            const bool is_v = lane >= D / 4;
            const int piece = lane - (is_v ? D / 4 : 0);
            const int64_t slot = (int64_t)a.table[last >> a.log2_page] * a.page_bytes + (int64_t)(last & a.pmask) * a.token_bytes;
            *reinterpret_cast<float4*>(const_cast<char*>(is_v ? a.v : a.k) + slot + 16 * piece) =
                *reinterpret_cast<const float4*>((is_v ? a.vnew : a.knew) + 16 * piece);
        }
    }

    f64x4 o[D / 64][4];
#pragma unroll
    for (int c = 0; c < D / 64; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c][e] = f64x4{0.0, 0.0, 0.0, 0.0};
    double m = -INFINITY, l = 0.0;

    if (first < c1) {
        TileRegs<D> t;
        load_k<D>(t, a, page, first, last, r16, quad);
        // (fp32 in registers: held as fp64 it spills at head_dim 128)
        float4 qf[D / 16];
#pragma unroll
        for (int i = 0; i < D / 16; ++i) qf[i] = *reinterpret_cast<const float4*>(q + o_row * D + 16 * i + 4 * quad);
        load_v<D>(t, a, page, first, last, r16, quad);
#pragma unroll 1
        for (int32_t t0 = first; t0 < c1; t0 += NW * kKeys) {
#pragma unroll
            for (int i = 0; i < D / 16; ++i)                         // (or they are converted once, in front of the loop)
                asm volatile("" : "+v"(qf[i].x), "+v"(qf[i].y), "+v"(qf[i].z), "+v"(qf[i].w));
            const int32_t next = t0 + NW * kKeys;
            if (next < c1) page = a.table[next >> a.log2_page];
            f64x4 sc = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < D / 16; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)elem(t.k[i], e), (double)elem(qf[i], e), sc, 0, 0, 0);
                if (D > 64) __builtin_amdgcn_sched_barrier(0);       // conversions stay with their products (registers)
            }
            if (next < c1) load_k<D>(t, a, page, next, last, r16, quad);   // under the softmax and the value product
            double x[4], top = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[r] = sc[r] * (double)scale;
                if (t0 + 4 * r + quad >= nk) x[r] = -INFINITY;       // mask by selection
                top = __builtin_fmax(top, x[r]);
            }
            const double m_new = __builtin_fmax(m, quad_max(top));
            const double m_use = m_new == -INFINITY ? 0.0 : m_new;   // a row without a key so far
            const double alpha = exp2_of((m - m_use) * kLog2e);
            double p[4];
            l *= alpha;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = exp2_of((x[r] - m_use) * kLog2e);
                l += p[r];
            }
            m = m_new;
            if (__any(alpha != 1.0)) {
#pragma unroll
                for (int c = 0; c < D / 64; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[c][e] *= alpha;
            }
            // Weights of masked keys are exact zeros, but a live key that some row does not see (or that stands in for the
            // keys behind the end) can hold values that are not finite: those must not reach the rows that do not see it.
            bool odd = false;
            if (t0 + kKeys > (causal ? nk_wg - kRows : c1)) {        // (only tiles at the edge; wave-uniform)
#pragma unroll
                for (int c = 0; c < D / 64; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e) odd |= !(__builtin_fabsf(elem(t.v[c][r], e)) <= 3.402823466e38f);
            }
            if (__any(odd)) {
                // one key at a time, kept by the rows that see it
#pragma unroll
                for (int c = 0; c < D / 64; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll 1
                        for (int kq = 0; kq < 4; ++kq) {
                            const bool seen = t0 + 4 * r + kq < nk;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                float ve = elem(t.v[c][r], e);
                                asm volatile("" : "+v"(ve));         // (converted here, not once for both paths above them)
                                const f64x4 one = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    quad == kq ? (double)ve : 0.0, quad == kq ? p[r] : 0.0,
                                    f64x4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
#pragma unroll
                                for (int g = 0; g < 4; ++g) o[c][e][g] = seen ? o[c][e][g] + one[g] : o[c][e][g];
                            }
                        }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (D > 64) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < D / 64; ++c)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            o[c][e] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)elem(t.v[c][r], e), p[r], o[c][e], 0, 0, 0);
                }
            }
            if (next < c1) load_v<D>(t, a, page, next, last, r16, quad);   // under the next score product
        }
    }

    // publish the wave's partial: unnormalised accumulator, reference, sum
    l = quad_sum(l);
    float* po = sm_o + (wave * kRows + r16) * kPad;
#pragma unroll
    for (int c = 0; c < D / 64; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)      // rows 4*g + quad of the four accumulators: columns 64*c + 4*(4*g + quad) ..+3
            *reinterpret_cast<float4*>(po + 64 * c + 16 * g + 4 * quad) =
                float4{(float)o[c][0][g], (float)o[c][1][g], (float)o[c][2][g], (float)o[c][3][g]};
    if (quad == 0) {
        sm_m[wave * kRows + r16] = m;
        sm_l[wave * kRows + r16] = l;
    }
    __syncthreads();                                         // every wave arrives once, with or without tiles

    // merge: thread -> (row, 4 columns)
    for (int it = threadIdx.x; it < kRows * (D / 4); it += NW * 64) {
        const int mrow = it / (D / 4), c4 = it % (D / 4);
        if (m0 + mrow >= n_rows) continue;
        double M = -INFINITY;
#pragma unroll
        for (int p = 0; p < NW; ++p) M = __builtin_fmax(M, sm_m[p * kRows + mrow]);
        double sum = 0.0, acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < NW; ++p) {
            const double mp = sm_m[p * kRows + mrow];
            // a wave without tiles weighs nothing; one whose sum is NaN hands that on
            const double w = mp == -INFINITY ? 0.0 : (double)exp2_of((mp - M) * kLog2e);
            const float4 v = *reinterpret_cast<const float4*>(sm_o + (p * kRows + mrow) * kPad + 4 * c4);
            sum += mp == -INFINITY ? sm_l[p * kRows + mrow] : w * sm_l[p * kRows + mrow];
            acc[0] += w * v.x;
            acc[1] += w * v.y;
            acc[2] += w * v.z;
            acc[3] += w * v.w;
        }
        const int32_t mq = (m0 + mrow) / G;
        const bool none = min(c1, causal ? len - q_len + mq + 1 : len) <= c0;   // no key at all
        const double inv = none ? 0.0 : 1.0 / sum;
        const float4 r = float4{(float)(acc[0] * inv), (float)(acc[1] * inv), (float)(acc[2] * inv), (float)(acc[3] * inv)};
        const float r_lse = none ? -INFINITY : (float)(M + log(sum));
        const int64_t o_idx = (int64_t)(q_begin + mq) * num_q_heads + kvh * G + (m0 + mrow - mq * G);
        if (nsplit == 1) {
            *reinterpret_cast<float4*>(out + o_idx * D + 4 * c4) = r;
            if (lse && c4 == 0) lse[o_idx] = r_lse;
        } else {
            *reinterpret_cast<float4*>(part_o + (o_idx * nsplit + split) * D + 4 * c4) = r;
            if (c4 == 0) part_lse[o_idx * nsplit + split] = r_lse;
        }
    }
}

// Decode with few query heads per KV head (G <= 4): 16 x 16 matrix tiles would be 1/16 to 1/4 full, and the vector unit has
// the same fp64 rate, so the products run there: a lane's piece of a K row against rows of q (held in LDS, one address per
// quad), a 4-lane sum, and for P.V four keys times a lane's columns per row.  A wave holds R rows (two
// at head_dim 64, one at 128: more spill); the `groups` (a power of two) waves that share a tile take other rows each and read it through the cache.
// Everything else -- tiles, loads, LDS merge -- is as above, plus the context split: several workgroups share a (sequence,
// KV head), as many as its length asks for, leave their merged partial in `part`, and the one that arrives last merges them
// in split order (the scheme of the one-launch decode kernel of the
// 16-bit pools).  One launch, whatever the context; bound by launch and memory
// round trips while a wave has a tile or two, by the stream of K and V beyond.
// Portable kernel / this one, us: 1 x 16 tokens 8 / 8 heads, head_dim 64 6.0 / 4.7; 1 x 128 7.9 / 5.5; 1 x 2048 16.6 / 10.5;
// 8 x 2048 at head_dim 128 50 / 26 (134 MB), with 32 / 8 heads 99 / 45; 8 x 100 with 32 / 8 heads, head_dim 64 7.7 / 7.7.  With
// more than 4 heads a group the matrix kernel above is the better one (8 x 2048, 64 / 8 heads: 91 here, 44 there).
//     part: per workgroup 4 rows of D normalised accumulators, then 4 x (reference, sum) as doubles (G = 1: one row).
template <int D, int R, int HEADS>
__global__ __launch_bounds__(kWaves * 64) void paged_decode_f32_kernel(
    CacheView cache, const float* __restrict__ q, float* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens, int32_t num_q_heads,
    int32_t max_blocks, float scale, int32_t log2_groups, int32_t max_split, int32_t fill, int32_t chunk, float* __restrict__ part,
    uint64_t* __restrict__ arrive, uint64_t arrive_step, const float* __restrict__ k_new, const float* __restrict__ v_new)
{
    constexpr int kHeads = HEADS;                            // rows a workgroup has room for
    constexpr int kParts = kHeads * (D + 4);
    __shared__ __attribute__((aligned(16))) double sm_q[kHeads * D];
    __shared__ __attribute__((aligned(16))) float sm_o[kWaves * R * D];
    __shared__ double sm_m[kWaves * R];
    __shared__ double sm_l[kWaves * R];
    __shared__ uint32_t sm_last;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r16 = lane & 15, quad = lane >> 4;
    const int32_t s = (int32_t)blockIdx.x / max_split;
    const int32_t split = (int32_t)blockIdx.x - s * max_split;
    const int32_t kvh = blockIdx.y;
    const int32_t G = num_q_heads / cache.num_kv_heads;
    const int64_t row0 = (int64_t)s * num_q_heads + (int64_t)kvh * G;

    // lengths and queries are requested together
    const int64_t unit = (int64_t)s * gridDim.y + kvh;
    uint64_t* const counter = arrive + unit * kArrivalStride;
    uint64_t seen = 0;
    const int32_t len = seq_lens[s];
    const int32_t nt = (len + kKeys - 1) / kKeys;
    const int group = kHeads == 1 ? 0 : wave & ((1 << log2_groups) - 1);          // this wave's rows: R * group ..
    const int slot = kHeads == 1 ? wave : wave >> log2_groups, slots = kHeads == 1 ? kWaves : kWaves >> log2_groups;
    for (int i = threadIdx.x; i < kHeads * D; i += kWaves * 64)
        sm_q[i] = i < G * D ? (double)q[row0 * D + i] * ((double)scale * kLog2e) : 0.0;
    // the workgroups of this sequence: a round of tiles for each up to `fill`, more where they would get beyond `chunk`
    const uint32_t rounds = (uint32_t)nt >> (kHeads == 1 ? 3 : 3 - log2_groups), shares = (uint32_t)(nt + chunk - 1) / (uint32_t)chunk;
    const int32_t nsplit = (int32_t)min(max(min((uint32_t)fill, rounds), max(shares, 1u)), (uint32_t)max_split);
    if (split >= nsplit) return;

    Rows a;
    a.table = block_table + (int64_t)s * max_blocks;
    a.log2_page = cache.log2_page;
    a.pmask = cache.page_size - 1;
    a.k = reinterpret_cast<const char*>(cache.k) + (int64_t)kvh * cache.head_stride * 4;
    a.v = reinterpret_cast<const char*>(cache.v) + (int64_t)kvh * cache.head_stride * 4;
    a.page_bytes = cache.page_stride * 4;
    a.token_bytes = cache.token_stride * 4;
    a.knew = a.vnew = nullptr;
    a.new_pos = -1;
    const int32_t last = len - 1;
    // this workgroup's tiles, dealt to its waves in turn
    const int32_t each = (int32_t)((uint32_t)nt / (uint32_t)nsplit), more = nt - each * nsplit;   // the first `more` take one more
    const int32_t tb = split * each + min(split, more), te = tb + each + (split < more ? 1 : 0);
    if (k_new) {
        const int64_t off = ((int64_t)s * cache.num_kv_heads + kvh) * D;
        a.knew = reinterpret_cast<const char*>(k_new + off);
        a.vnew = reinterpret_cast<const char*>(v_new + off);
        a.new_pos = last;
        if (len > 0 && split == nsplit - 1 && wave == kWaves - 1 && lane < D / 2) {
            const bool is_v = lane >= D / 4;
            const int piece = lane - (is_v ? D / 4 : 0);
            const int64_t slot = (int64_t)a.table[last >> a.log2_page] * a.page_bytes + (int64_t)(last & a.pmask) * a.token_bytes;
            *reinterpret_cast<float4*>(const_cast<char*>(is_v ? a.v : a.k) + slot + 16 * piece) =
                *reinterpret_cast<const float4*>((is_v ? a.vnew : a.knew) + 16 * piece);
        }
    }

    double o[R][D / 64][4], m[R], l[R];
#pragma unroll
    for (int g = 0; g < R; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.0;
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[g][c][e] = 0.0;
    }

    auto fetch = [&](TileRegs<D>& t, int32_t tile) {
        const int64_t page = a.table[tile * kKeys >> a.log2_page];
        load_k<D>(t, a, page, tile * kKeys, last, r16, quad);
        load_v<D>(t, a, page, tile * kKeys, last, r16, quad);
    };
    auto attend = [&](const TileRegs<D>& t, int32_t tile) {
        const bool live = tile * kKeys + r16 < len;
        asm volatile("" ::: "memory");                       // (q is read for each tile: held across tiles it does not fit)
        double x[R];                                         // log2-domain scores of key r16
        bool raise = false;
#pragma unroll
        for (int g = 0; g < R; ++g) {
            double x4[4] = {0.0, 0.0, 0.0, 0.0};             // (four chains: an fp64 fma is waited for twice as long as it issues)
            const double2* qs = reinterpret_cast<const double2*>(sm_q + (R * group + g) * D + 4 * quad);
#pragma unroll
            for (int i = 0; i < D / 16; ++i) {
                const double2 q0 = qs[8 * i], q1 = qs[8 * i + 1];
                x4[0] = __builtin_fma((double)t.k[i].x, q0.x, x4[0]);
                x4[1] = __builtin_fma((double)t.k[i].y, q0.y, x4[1]);
                x4[2] = __builtin_fma((double)t.k[i].z, q1.x, x4[2]);
                x4[3] = __builtin_fma((double)t.k[i].w, q1.y, x4[3]);
            }
            x[g] = quad_sum((x4[0] + x4[1]) + (x4[2] + x4[3]));
            x[g] = live ? x[g] : -INFINITY;
            // The reference may trail the largest score by 2^16: weights stay far inside fp32, and out = O / l does not
            // depend on it.  A fresh one is the score of the tile's first key.
            const uint64_t u = __builtin_bit_cast(uint64_t, x[g]);
            const double first = __builtin_bit_cast(double, (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32 |
                                                                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u));
            m[g] = m[g] == -INFINITY && first == first ? first : m[g];
            raise |= x[g] > m[g] + 16.0;
        }
        if (__any(raise)) {
#pragma unroll
            for (int g = 0; g < R; ++g) {
                const double top = __builtin_fmax(m[g], row_max(x[g]));
                const double alpha = top == m[g] ? 1.0 : (double)exp2_of(m[g] - top);
                m[g] = top;
                l[g] *= alpha;
#pragma unroll
                for (int c = 0; c < D / 64; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[g][c][e] *= alpha;
            }
        }
        float p[R];
#pragma unroll
        for (int g = 0; g < R; ++g) {
            p[g] = m[g] == -INFINITY && !(x[g] != x[g]) ? 0.f : exp2_of(x[g] - m[g]);
            l[g] += p[g];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool in = tile * kKeys + 4 * r + quad < len;   // (a key behind the end repeats the last row: no part in it)
            double pk[R];
#pragma unroll
            for (int g = 0; g < R; ++g) pk[g] = __shfl(p[g], 4 * r + quad, 64);
            if (!in) continue;
#pragma unroll
            for (int g = 0; g < R; ++g)
#pragma unroll
                for (int c = 0; c < D / 64; ++c) {
                    o[g][c][0] = __builtin_fma(pk[g], (double)t.v[c][r].x, o[g][c][0]);
                    o[g][c][1] = __builtin_fma(pk[g], (double)t.v[c][r].y, o[g][c][1]);
                    o[g][c][2] = __builtin_fma(pk[g], (double)t.v[c][r].z, o[g][c][2]);
                    o[g][c][3] = __builtin_fma(pk[g], (double)t.v[c][r].w, o[g][c][3]);
                }
        }
    };
    TileRegs<D> ta, tc;
    if (tb + slot < te) fetch(ta, tb + slot);
    __syncthreads();                                         // q is in LDS
    // (looked at behind the first tile's loads, so that nothing waits for it; opened when the loop is done)
    if (nsplit > 1 && threadIdx.x == 0) seen = arrival_peek(counter);
    for (int32_t t = tb + slot; t < te; t += 2 * slots) {
        if (t + slots < te) fetch(tc, t + slots);
        attend(ta, t);
        if (t + slots >= te) break;
        if (t + 2 * slots < te) fetch(ta, t + 2 * slots);
        attend(tc, t + slots);
    }
    if (nsplit > 1 && threadIdx.x == 0) arrival_open(counter, seen, arrive_step, nsplit);

    // the wave's partial: sums over the quads (keys) of the accumulators, over 16 lanes (keys) of the weights
#pragma unroll
    for (int g = 0; g < R; ++g) {
        l[g] = row_sum(l[g]);
        // divided by the sum of the weights (up to 2^16 each, see above): a mean of V's values fits fp32, their sum may not
        const double inv_l = l[g] > 0.0 ? 1.0 / l[g] : 1.0;
#pragma unroll
        for (int c = 0; c < D / 64; ++c) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[g][c][e] = quad_sum(o[g][c][e]);
            if (quad == 0)
                *reinterpret_cast<float4*>(sm_o + (wave * R + g) * D + 64 * c + 4 * r16) =
                    float4{(float)(o[g][c][0] * inv_l), (float)(o[g][c][1] * inv_l), (float)(o[g][c][2] * inv_l),
                           (float)(o[g][c][3] * inv_l)};
        }
        if (lane == 0) {
            sm_m[wave * R + g] = m[g];
            sm_l[wave * R + g] = l[g];
        }
    }
    __syncthreads();

    // merge: thread -> (row, 4 columns)
    for (int it = threadIdx.x; it < kHeads * (D / 4); it += kWaves * 64) {
        const int g = it / (D / 4), c4 = it % (D / 4);
        if (g >= G) continue;
        const int first = (g / R) * R + g % R, step = R << (kHeads == 1 ? 0 : log2_groups);   // this row's partials: one per slot
        double M = -INFINITY, sum = 0.0, acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int p = 0; p < slots; ++p) M = __builtin_fmax(M, sm_m[first + p * step]);
        for (int p = 0; p < slots; ++p) {
            const double mp = sm_m[first + p * step], lp = sm_l[first + p * step];
            const double w = mp == -INFINITY ? lp : (double)exp2_of(mp - M) * lp;    // (no key seen: lp is 0, or NaN)
            const float4 v = *reinterpret_cast<const float4*>(sm_o + (first + p * step) * D + 4 * c4);
            sum += w;
            acc[0] += w * v.x;
            acc[1] += w * v.y;
            acc[2] += w * v.z;
            acc[3] += w * v.w;
        }
        if (nsplit > 1) {
            // component-major, device-scope stores: see the arrival below
            float* po = part + (unit * max_split + split) * kParts;
            const double inv = sum > 0.0 ? 1.0 / sum : 1.0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                __hip_atomic_store(po + e * (kHeads * D / 4) + it, (float)(acc[e] * inv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (c4 == 0) {
                double* ps = reinterpret_cast<double*>(po + kHeads * D) + 2 * g;
                __hip_atomic_store(ps, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(ps + 1, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            continue;
        }
        const double inv = len > 0 ? 1.0 / sum : 0.0;
        *reinterpret_cast<float4*>(out + (row0 + g) * D + 4 * c4) =
            float4{(float)(acc[0] * inv), (float)(acc[1] * inv), (float)(acc[2] * inv), (float)(acc[3] * inv)};
        if (lse && c4 == 0) lse[row0 + g] = len > 0 ? (float)(M * kLn2 + log(sum)) : -INFINITY;
    }
    if (nsplit == 1) return;

    // Arrival: every wave waits until its (write-through) stores are acknowledged, the barrier collects the waves, one
    // thread counts the workgroup in; the workgroup that finds nsplit - 1 earlier arrivals reads the partials, past the
    // caches that are not coherent across the chip, after its counting has returned.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) sm_last = arrival_count(counter, arrive_step, nsplit) ? 1u : 0u;
    __syncthreads();
    if (sm_last == 0u) return;
    // all partials at once: a thread adds up every J-th partial of its row and columns, J threads per piece of the output
    const float* pu = part + unit * max_split * kParts;
    __shared__ double sm_w[kF32MaxSplit * kHeads];
    __shared__ double sm_s[kHeads], sm_M[kHeads];
    __shared__ __attribute__((aligned(16))) double sm_a[kWaves * 64 * 4];
    for (int i = threadIdx.x; i < nsplit * G; i += kWaves * 64) {
        const double* ps = reinterpret_cast<const double*>(pu + (int64_t)(i / G) * kParts + kHeads * D) + 2 * (i % G);
        sm_w[i] = __hip_atomic_load(ps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sm_a[i] = __hip_atomic_load(ps + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if ((int)threadIdx.x < G) {                              // references -> weights, one row per thread
        double M = -INFINITY, sum = 0.0;
        for (int p = 0; p < nsplit; ++p) M = __builtin_fmax(M, sm_w[p * G + threadIdx.x]);
        for (int p = 0; p < nsplit; ++p) {
            const int i = p * G + threadIdx.x;
            const double lp = sm_a[i];
            const double w = sm_w[i] == -INFINITY ? lp : (double)exp2_of(sm_w[i] - M) * lp;
            sum += w;
            sm_w[i] = w;
        }
        sm_M[threadIdx.x] = M;
        sm_s[threadIdx.x] = sum;
    }
    __syncthreads();
    const int pieces = G * (D / 4);                          // at most 256
    const int J = kWaves * 64 / pieces, j = (int)threadIdx.x / pieces, piece = (int)threadIdx.x % pieces;
    const int mg = piece / (D / 4);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (j < J)
        for (int p = j; p < nsplit; p += J) {
            const float* pp = pu + (int64_t)p * kParts + piece;
            const double w = sm_w[p * G + mg];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] += w * (double)__hip_atomic_load(pp + e * (kHeads * D / 4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
    for (int e = 0; e < 4; ++e) sm_a[e * (kWaves * 64) + threadIdx.x] = acc[e];
    __syncthreads();
    if (threadIdx.x == 0) arrival_clear(counter);
    if ((int)threadIdx.x >= pieces) return;
    for (int k = 1; k < J; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += sm_a[e * (kWaves * 64) + k * pieces + threadIdx.x];
    const double sum = sm_s[mg], inv = len > 0 ? 1.0 / sum : 0.0;
    *reinterpret_cast<float4*>(out + (row0 + mg) * D + 4 * (piece % (D / 4))) =
        float4{(float)(acc[0] * inv), (float)(acc[1] * inv), (float)(acc[2] * inv), (float)(acc[3] * inv)};
    if (lse && piece % (D / 4) == 0) lse[row0 + mg] = len > 0 ? (float)(sm_M[mg] * kLn2 + log(sum)) : -INFINITY;
}

template <int D>
void launch_decode_f32_dim(const AttnArgs& a, hipStream_t stream)
{
    const int32_t G = a.num_q_heads / a.cache.num_kv_heads;
    constexpr int R = D == 64 ? 2 : 1;
    int32_t log2_groups = 0;
    while ((R << log2_groups) < G) ++log2_groups;
    auto kern = G == 1 ? paged_decode_f32_kernel<D, 1, 1> : paged_decode_f32_kernel<D, R, kF32MaxGroup>;
    hipLaunchKernelGGL(kern, dim3((uint32_t)(a.batch * a.short_nsplit), (uint32_t)a.cache.num_kv_heads), dim3(kWaves * 64), 0,
                       stream, a.cache, (const float*)a.q, (float*)a.out, a.lse, a.block_table, a.seq_lens, a.num_q_heads,
                       a.max_blocks, a.scale, log2_groups, a.short_nsplit, a.short_fill, a.short_chunk, a.short_part, a.short_arrive,
                       a.short_step, (const float*)a.k_new,
                       (const float*)a.v_new);
}

}  // namespace

bool attention_f32_supported(const AttnArgs& a)
{
    const int32_t d = a.cache.head_dim;
    return a.dtype == PA_DTYPE_F32 && (d == 64 || d == 128) && a.cache.page_size >= kKeys && !a.has_mods &&
           a.max_blocks > 0;
}

bool decode_f32_supported(const AttnArgs& a)
{
    // the vector kernel's rows: one query per sequence, up to 4 heads of a KV head (the grid's y extent is 16-bit)
    return attention_f32_supported(a) && !a.cu_q_lens && a.num_q_heads / a.cache.num_kv_heads <= kF32MaxGroup &&
           a.cache.num_kv_heads <= 65535 && (int64_t)a.batch * kF32MaxSplit <= 0x7fffffffLL;
}

int32_t decode_f32_tile_slots(const AttnArgs& a)
{
    const int32_t G = a.num_q_heads / a.cache.num_kv_heads, rows = G == 1 || a.cache.head_dim > 64 ? 1 : 2;
    int32_t slots = kWaves;
    for (int32_t n = rows; n < G; n *= 2) slots /= 2;
    return slots;
}

size_t decode_f32_part_floats(const AttnArgs& a, int32_t nsplit)
{
    const int32_t heads = a.num_q_heads == a.cache.num_kv_heads ? 1 : kF32MaxGroup;
    return nsplit > 1 ? (size_t)a.batch * a.cache.num_kv_heads * nsplit * heads * (a.cache.head_dim + 4) : 0;
}

pa_status launch_decode_f32(const AttnArgs& a, hipStream_t stream)
{
    if (a.short_nsplit > 1 && (a.short_nsplit > kF32MaxSplit || !a.short_part || !a.short_arrive)) return PA_ERR_INVALID_ARG;
    ProfileScope prof("paged_decode_f32_kernel", stream);
    if (a.cache.head_dim == 64) launch_decode_f32_dim<64>(a, stream);
    else launch_decode_f32_dim<128>(a, stream);
    return launch_status();
}

pa_status launch_attention_f32(const AttnArgs& a, hipStream_t stream)
{
    const int64_t G = a.num_q_heads / a.cache.num_kv_heads;
    // One workgroup per (row tile of the longest possible query range, sequence) where most of those exist, the heaviest
    // tiles of all sequences first; a compact grid of the row tiles that total_q allows where they do not (one prompt among
    // single queries, a loose max_q_len), since an empty workgroup costs its slot for a microsecond or two.  256 sequences
    // of 100 .. 400 tokens, four of them with 300 queries, 32 / 8 heads, head_dim 64: 371 / 113 us (portable kernel 310); 16
    // prompts of 100 .. 1000, 8 / 8 heads 202 / 145; 64 of 64 .. 2048, four with 300 queries 259 / 107.
    int64_t tiles = (a.max_q_len * G + kRows - 1) / kRows;
    if (tiles <= 0) return PA_OK;
    const int64_t compact = (int64_t)a.total_q * G / kRows + a.batch;
    int64_t blocks = tiles * a.batch;
    if (a.cu_q_lens && (blocks > 2 * compact || tiles * kRows > 0x7fffffffLL)) {
        blocks = compact;
        tiles = 0;
    }
    blocks *= (int64_t)a.cache.num_kv_heads * a.plan.nsplit;
    if (blocks * kWaves * 64 > 0xffffffffLL) return launch_attention_generic(a, stream);   // (a launch has 2^32 threads)
    ProfileScope prof("paged_attention_f32_kernel", stream);
    auto kern = a.cache.head_dim == 64 ? paged_attention_f32_kernel<64, kWaves> : paged_attention_f32_kernel<128, kWaves>;
    hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(kWaves * 64), 0, stream, a.cache, (const float*)a.q, (float*)a.out,
                       a.lse, a.cu_q_lens, a.block_table, a.seq_lens, a.batch, a.num_q_heads, a.max_blocks, a.scale,
                       a.cu_q_lens ? a.causal : 0, a.part_o, a.part_lse, a.plan.chunk, a.plan.nsplit, (int32_t)tiles,
                       (const float*)(a.cu_q_lens ? nullptr : a.k_new), (const float*)(a.cu_q_lens ? nullptr : a.v_new));
    return launch_status();
}

}  // namespace pa
