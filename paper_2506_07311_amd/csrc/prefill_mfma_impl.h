// Paged prefill (ragged packed queries, optional causal bound) for bf16 / fp16 pools with head_dim D = 128 or 64 on
// gfx950 (and D = 256, 80, 96, 112 for page sizes of 16 and more).  Internal header: the kernel templates; one translation unit
// per head_dim instantiates them.  The text below describes D = 128.  D = 64 is the same kernel with half the steps:
// LDS rows are 128 bytes (a load instruction brings 8 of them), the score product takes 4 steps instead of 8 and the value
// product covers 2 column blocks, not 4.  What a tile costs besides its matrix work then hides behind a third workgroup of a
// compute unit, for which there are registers (148; document masks and user modifications spill 4 to 6, see the kernel) and,
// with rows of their own size, LDS (32 KiB): 4 x 2048 with 32 / 8 heads
// 119 us with half-empty 256-byte rows and two workgroups, 102 like this, 1 x 8192 341 / 303, prompts of 2059 and 3146 tokens
// with a window 81 / 67, 1024 tokens of a 32768-token context 348 / 324; a fourth workgroup spills (158, 465, 102, -).
// D = 256 has
// 512-byte LDS rows (two swizzled 256-byte halves) and fills 128 KiB with its two tile buffers, so one workgroup per compute
// unit; it runs on eight waves of 16 rows (RowGeo), two a SIMD, because 32 rows of O and Q leave room for one wave a SIMD
// whose operand reads nothing hides: 1 x 8192 with 32 / 8 heads 1417 us with four waves of 32 rows, 1187 with eight of 16
// (32768 keys behind 1024 queries 1497 / 1200, 4 x 2048 429 / 365, prompts of 2059 and 3146 tokens with 16 / 8 heads, window
// 1024 and a soft cap 192 / 166, with slopes 433 / 336).  At D = 128, where 32 rows already fit twice, 16 rows lose: every
// operand read feeds half the matrix work (1 x 8192 505 / 568, 4 x 2048 154 / 173).
//
// Prefill is a dense contraction (about 590 flop per byte at 2048 tokens), so it runs on the matrix cores
// with v_mfma_f32_32x32x16_bf16 in the flash-attention arrangement: one workgroup of 4 waves owns 128
// consecutive ROWS of one (sequence, KV head); wave w owns 32 of them.  A row is a (query, query head) pair:
// the G query heads that share the KV head are packed next to each other (row = query * G + head; G a power of
// two up to 16, else one head per workgroup), so K and V are streamed once per KV head whatever G is and a
// call with few queries per sequence (decode rows, speculative tokens, short chunks) still fills the tile G
// times better.  "Query" below means such a row.  The context is walked in tiles of 64 keys; the launch may
// cut it into chunks (one workgroup per chunk, partials merged by the split-KV merge kernel) when the call has
// too few rows to fill the machine.  A tile's K and V rows are fetched page by page through the block table (Algorithm 1:
// page = block_table[s][j >> log2 P], slot = j & (P-1)) and written STRAIGHT INTO LDS by the load unit
// (global_load_lds_dwordx4: 16 bytes per lane, a wave fills 4 consecutive 256-byte rows per instruction), one
// tile ahead of the one being computed, into the other of two 32 KiB buffers -- no staging registers, no LDS
// store instructions, one barrier per tile.  Rows are unpadded (256 B = all 64 LDS banks); the 16-byte piece L
// of row r sits at piece L ^ swz(r), swz(r) = 4*(r%4) + (r/4)%4 (each lane simply fetches the piece that belongs
// at its LDS position), which makes both kinds of operand read conflict-free:
//   K rows are read as 16-byte MFMA operands (16 consecutive lanes = 16 consecutive rows, same logical piece:
//     swz takes 16 distinct values),
//   V rows are read TRANSPOSED with ds_read_b64_tr_b16, the LDS transpose load of gfx950 -- the contraction
//     index of P.V is the key while memory is contiguous along head_dim (32 lanes read 64 bytes of each of 4
//     consecutive rows: swz moves them to 4 different quarters of the banks).
// Both products are computed transposed so that every per-query quantity is lane-local (lane%32 = query):
//   S^T[key, q]  = K[key, :] . Q[q, :]^T        A = K from LDS, B = Q held in registers for the whole kernel
//   O^T[col, q] += V^T[col, key] . P^T[key, q]  A = V^T from LDS, B = P straight from the S^T accumulators
// The accumulator layout of S^T (lane holds keys 8a + 4h + b of its query) is, after packing to bf16, already
// the B-operand layout of the second product for a permuted key order, and the transpose loads fetch V in that
// same order.  Online softmax runs in the log2 domain; masking (length, causal, ragged rows) is by selection.
//
// Softmax weights enter the matrix cores as bf16.  With few keys the individual weights are large and their
// 2^-9 rounding shows in the output, so query tiles that see few keys -- at most kPreciseKeys, or fewer than
// kPreciseShare of the harmonic mean of the key counts of all the call's rows (precise_key_bound) -- carry the
// weights as two bf16 terms (p = hi + lo); over long contexts the rounding averages out.
#pragma once

#include <type_traits>

#include "prefill_tiles.h"

namespace pa {

namespace {

using namespace prefill;

// LDS row stride of a K or V row: 256 bytes (head_dims 80 to 128), 512 at head_dim 256, 128 at 64.  The swizzle permutes the 16
// pieces of a 256-byte half row among themselves (such a row starts at bank 0), or the 8 of a 128-byte row, of which every
// second one starts half way through the banks (row_swz).
template <int D>
struct RowGeo {
    static constexpr int kRowB = D > 128 ? 512 : D > 64 ? 256 : 128;
    static constexpr int kTileB = kBN * kRowB;        // K part of a tile buffer; the V part follows
    static constexpr int kBufB = 2 * kTileB;
    // Rows of a wave, and what follows from them: the lane groups that share a row (each takes four of every kStep
    // consecutive keys of S and columns of O), the waves of a workgroup.
    static constexpr int kRows = D > 128 ? 16 : 32;
    static constexpr int kGroups = 64 / kRows;
    static constexpr int kStep = 4 * kGroups;
    static constexpr int kWaves = kBM / kRows;
    static constexpr int kThreads = 64 * kWaves;
};
// head_dims 80, 96 and 112: rows hold 10, 12 or 14 pieces and the last column block of O is padded where D is not a
// multiple of 32.  Every tile carries two-term weights: the portable kernel, which served these head_dims, keeps its
// weights in fp32, and the second term (2^-17 of a weight) keeps the error at what the output's rounding leaves (see also
// Reference, which keeps their range, and half_pv_by_key).
// 2 prompts of 700 and 950 tokens, 32 / 32 heads, D = 96: 25 us for 9 GFLOP, bound by the start of a workgroup and its
// heaviest row tile like every short prompt here; 1065 us on the portable kernel, which reads K and V again per row.
template <int D>
constexpr bool kTwoTermOnly = D % 64 != 0;
// Swizzle of LDS row r.  16 rows a wave: a transpose load reads 32 bytes of 16 rows, 8 of them at a time, and an operand
// read one piece of 16 rows: both are free of conflicts if 8 consecutive rows differ in the upper three bits.
// head_dim 64: two rows share 256 bytes, so it is pairs of rows that differ; the two pairs of a transpose load's 4 rows in the
// upper bit, as it reads 4 of a row's 8 pieces.
template <int D>
__device__ __forceinline__ int row_swz(int r)
{
    return D == 64 ? ((r & 2) << 1) | ((r >> 2) & 3) : RowGeo<D>::kRows == 32 ? swz(r) : ((r & 7) << 1) | ((r >> 3) & 1);
}
// byte offset inside its row of logical 16-byte piece L of LDS row r
template <int D>
__device__ __forceinline__ int piece_pos(int L, int r) { return 16 * ((L & 16) | ((L & 15) ^ row_swz<D>(r))); }

// Tile fetch for 512-byte rows: one load-to-LDS instruction of a wave fills 2 consecutive rows (lane l: position
// l%32 of row l/32); wave w of eight issues, for i < 4, the K and V instructions of rows 16*i + 2*w, +1: one page each.
// lds = buffer + 2*w*512; row = 2*w + lane/32; lane_off = kv-head offset + this lane's logical piece (the swizzle repeats
// every 16 rows).
template <bool UNIFORM>
__device__ __forceinline__ void fetch_tile512(uint32_t lds, const PageIds& p, const CacheView& cache, int32_t t0, int32_t row,
                                              int32_t last_key, uint32_t lane_off)
{
    static_assert(UNIFORM, "two rows of a load share a page");
    constexpr int TB = RowGeo<256>::kTileB;
    const int32_t pg[4] = {p.p0, p.p1, p.p2, p.p3};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int32_t slot = min(t0 + 16 * i + row, last_key) & (cache.page_size - 1);
        int64_t page_off = (int64_t)pg[i] * cache.page_stride * 2;
        asm volatile("" : "+s"(page_off));                 // stays in scalar registers
        const uint32_t off32 = (uint32_t)slot * (uint32_t)(cache.token_stride * 2) + lane_off;
        load_to_lds16(lds, i * (16 * 512), reinterpret_cast<const char*>(cache.k) + page_off, off32);
        load_to_lds16(lds, i * (16 * 512) + TB, reinterpret_cast<const char*>(cache.v) + page_off, off32);
    }
}

__device__ __forceinline__ uint4 lds_frag(const char* p)
{
    return *reinterpret_cast<const uint4*>(p);
}

// V^T operand of the second product for 32 head_dim columns and one 16-key step, from row-major V.
// ds_read_b64_tr_b16 works on blocks of 16 lanes: lane i of a block receives element i%4 of the 8 bytes
// addressed by lanes i/4, i/4+4, i/4+8, i/4+12 of its block.  Lane x = q + 4*j of a block therefore points at
// key j of the step, columns 4q..4q+3 of the block's 16 columns, and lane i ends up with column i of 4 keys.
// The two loads fetch the keys of contraction slots 0-3 and 4-7 (8 rows apart; their swizzles differ).
struct tr_pair {
    s16x4 lo, hi;
};
__device__ __forceinline__ uint4 lds_frag_tr(const char* lo, const char* hi)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    tr_pair r;
    r.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lo));
    r.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(hi));
    return __builtin_bit_cast(uint4, r);
}

// Which rows need two-term weights.  A row that sees n keys carries a weight-rounding error of about
// 2^-9 * sqrt(sum p^2) ~ 1 / sqrt(n) in absolute terms, and the outputs of a call are judged against the RMS of the
// whole output tensor, which behaves as 1 / sqrt(H) with H the harmonic mean of n over all rows of the call.  A row
// whose n is well below H is therefore large compared with the scale it is measured on, whatever its own length:
// a short sequence batched beside long ones, or the first rows of a long causal prompt.  Every workgroup derives H
// from the lengths (one lane per sequence; sum over the rows of a causal sequence of 1/n = ln((hi+1/2)/(lo-1/2))
// for n = lo..hi, capped at the window) -- a few dozen instructions next to loads it needs anyway -- and tiles whose first row
// sees fewer than kPreciseShare * H keys take the two-term path.  Wave-uniform result.
constexpr float kPreciseShare = 0.9f;

__device__ __forceinline__ int32_t precise_key_bound(const int32_t* __restrict__ cu_q_lens,
                                                     const int32_t* __restrict__ seq_lens, int32_t batch,
                                                     int32_t causal, int32_t window, int lane)
{
    float rows = 0.f, inv = 0.f;
    for (int32_t i = lane; i < batch; i += 64) {
        const int32_t q_len = cu_q_lens[i + 1] - cu_q_lens[i];
        const int32_t len = seq_lens[i];
        if (q_len <= 0 || len <= 0) continue;
        const int32_t hi = len;                                       // keys of the last row
        const int32_t lo = causal ? max(len - q_len + 1, 1) : len;    // keys of the first row that sees any
        const int32_t cap = window > 0 ? (causal ? window : 2 * window - 1) : 0x7fffffff;
        const int32_t n_rows = causal ? hi - lo + 1 : q_len;
        rows += (float)n_rows;
        if (!causal) {
            inv += (float)q_len / (float)min(len, cap);
            continue;
        }
        const int32_t b = min(hi, cap);
        if (b >= lo) inv += __builtin_amdgcn_logf(((float)b + 0.5f) / ((float)lo - 0.5f)) * kLn2;
        const int32_t above = hi - max(lo, cap + 1) + 1;              // rows that see the whole window
        if (above > 0) inv += (float)above / (float)cap;
    }
    rows = wave_sum_moves(rows);
    inv = wave_sum_moves(inv);
    const float h = inv > 0.f ? rows / inv : 0.f;
    return max(kPreciseKeys, (int32_t)fminf(kPreciseShare * h, 1.0e9f));
}

// Operand reads of the 16-row products ahead of their use (a matrix instruction takes 16 cycles there).
// The order of the instructions around these reads is fixed by scheduling groups: left to itself the compiler clusters the
// reads of one base address and waits for nearly all of them at every step (1 x 8192 at head_dim 256 1312 -> 1199 us).
constexpr int kAheadK = 8, kAheadV = 6;

// Online-softmax update with the 32 keys of one half tile.  s holds raw scores on entry; the weights are
// returned in p.  The running statistic is a REFERENCE exponent m_ref (log2 domain) that may trail the true
// running max: weights are exp2(score - m_ref), and as long as a lane's weights (16, or 8 with
// 16 rows a wave) sum to at most kWeightSumMax
// every one of them is a number that fp32 sums and 16-bit operands carry without loss, and out = O / l does not
// depend on the reference.  So the common path takes no maximum at all: the weights are computed with the
// reference as it stands, and only when some lane's sum exceeds the bound (or is not a number: a fresh reference
// is -inf) -- always on a query's first keys, rarely later -- is the true maximum taken, the reference raised, O
// and l rescaled and the half's weights recomputed: a wave-uniform slow path that keeps the common path free of
// branches between the score and the value products.
// What the mask / score hooks need per row (this lane's).  Unused without their hook.
struct RowMods {
    int32_t lo;         // window: first visible key of this row
    int32_t lo_until;   // window: tiles that start before this key need the lower mask (wave-uniform)
    int32_t pos;        // score: the row's absolute position
    float slope2;       // score: bias slope * log2(e)
    float cap_in;       // score: 2 * log2(e) * scale / softcap
    float cap_out;      // score: softcap * log2(e)
    bool cap, bias;     // score: the call has a cap, slopes
    int32_t doc;        // document mask: the row's own document id
    pa_mod_ctx uc;      // user modification: what its hooks are told about the row
};

// A call with a soft cap and no slopes has a kernel of its own (beside the one with every score hook, whose wave-uniform
// tests cut the tile into pieces that the matrix and the vector work cannot be interleaved across), as has a window alone.
struct WindowCap : Mods<true, true, false> {
    static constexpr bool kCapOnly = true;
};
template <typename M, typename = void>
struct CapOnly : std::false_type {};
template <typename M>
struct CapOnly<M, std::enable_if_t<M::kCapOnly>> : std::true_type {};

// M: compile-time policy of the hooks.  With score hooks the scores are first rewritten in place as
// log2(e) * (cap(scale * s) + slope * (key - pos)) and the rest runs with a unit scale (a call with neither cap nor slopes
// keeps its scale).
// head_dims 80, 96, 112 keep what the portable kernel's fp32 weights gave them.  fp16: the reference
// stands 2^9 below the largest score, so that weights are lost from 2^-33 of the largest on and not from 2^-24 (8000 keys of
// which one leads by e^15: error 3.4e-3 with the reference at the maximum, 2.5e-4 like this and on the portable kernel).
// bf16: 2^14 above it and sums up to 1, so that no weight exceeds 1 and a weighted sum of finite values stays finite.
template <typename E, int D>
struct Reference {
    static constexpr bool kPadded = kTwoTermOnly<D>, kBf16 = E::kDtype == PA_DTYPE_BF16;
    static constexpr float kBelow = !kPadded ? 0.f : kBf16 ? -14.f : 9.f;
    static constexpr float kSumMax = kPadded && kBf16 ? 1.f : kWeightSumMax;
};
template <bool MASK, bool FIRST, typename E, typename M, int D, typename S, typename A, int T>
__device__ __forceinline__ void half_softmax(S& p, S& s, A (&o)[T], float& m_ref, float& l, float sc,
                                             int32_t key0, int32_t nk, const RowMods& rm, const int32_t* docs)
{
    constexpr int KS = D / 16;
    constexpr int kValu = ((CapOnly<M>::value ? 8 : 4) * kBN / 2 / RowGeo<D>::kGroups + 8) / KS;   // vector instructions a matrix instruction
    constexpr int kStep = RowGeo<D>::kStep, N = kBN / 2 / RowGeo<D>::kGroups;   // this lane's scores: four of every kStep keys
    // document mask: ids of this lane's keys (groups of 4 consecutive ones) from the tile's ids in LDS
    int4 ids[N / 4];
    if (M::kDoc) {
#pragma unroll
        for (int a = 0; a < N / 4; ++a) ids[a] = *reinterpret_cast<const int4*>(docs + kStep * a);
    }
    float shift = 0.f;               // score in the log2 domain = s * sc + shift
    if constexpr (CapOnly<M>::value) {
        // c * tanh(y / c) with tanh(z) = 1 - 2 / (1 + e^(2z)): s becomes -1 / (1 + e^(2z)), the rest goes into scale and shift
#pragma unroll
        for (int r = 0; r < N; ++r) s[r] = __builtin_amdgcn_rcpf(-1.f - __builtin_amdgcn_exp2f(s[r] * rm.cap_in));
        sc = 2.f * rm.cap_out;
        shift = rm.cap_out;
    } else if (M::kScore) {
        // Each hook's instructions are spent only on calls that have it (wave-uniform tests), and the cap takes five per score:
        // 2 x 1200 tokens, 32 / 8 heads, with a cap 68.3 -> 49.4 us, with a window alone 44.6 -> 38.4, 4 prompts of 1000 ..
        // 2000 with both 199 -> 148.
        if (rm.cap) {                // c * tanh(y / c) with tanh(z) = 1 - 2 / (1 + e^(2z)); cap_in carries 2 log2(e) / c
#pragma unroll
            for (int r = 0; r < N; ++r) {
                const float t = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(s[r] * rm.cap_in));
                s[r] = __builtin_fmaf(-2.f * rm.cap_out, t, rm.cap_out);
            }
            sc = 1.f;
        }
        if (rm.bias) {
            const float b0 = rm.slope2 * (float)(key0 - rm.pos);
#pragma unroll
            for (int r = 0; r < N; ++r)
                s[r] = s[r] * sc + __builtin_fmaf(rm.slope2, (float)(kStep * (r / 4) + (r % 4)), b0);
            sc = 1.f;
        }
    }
    if (M::kUser) {
        if (sc != 1.f) {
#pragma unroll
            for (int r = 0; r < N; ++r) s[r] *= sc;
            sc = 1.f;
        }   // (a user modification is compiled with the score hooks: the scores are in the log2 domain here)
#pragma unroll
        for (int r = 0; r < N; ++r)
            s[r] = user_score<M>(rm.uc, key0 + kStep * (r / 4) + (r % 4), s[r] * kLn2) * kLog2e;
    }
    // (16 rows a wave: a tile that a window cuts is a masked tile, so that no test stands between products and softmax)
    const bool below = RowGeo<D>::kRows == 32 && M::kWindow && key0 < rm.lo_until;      // wave-uniform up to the lane's 4-key offset
#pragma unroll
    for (int r = 0; r < N; ++r) {
        if (MASK && key0 + kStep * (r / 4) + (r % 4) >= nk) s[r] = -INFINITY;   // mask by selection
        if ((RowGeo<D>::kRows == 16 ? MASK && M::kWindow : below) && key0 + kStep * (r / 4) + (r % 4) < rm.lo) s[r] = -INFINITY;
        if (M::kDoc) {
            const int4 g = ids[r / 4];
            const int32_t id = (r % 4) == 0 ? g.x : (r % 4) == 1 ? g.y : (r % 4) == 2 ? g.z : g.w;
            if (id != rm.doc) s[r] = -INFINITY;
        }
    }
    // (an addition of no shift would not be free: it is an instruction beside the sign that the multiply-add has for nothing)
    auto less = [&](float ref) { return CapOnly<M>::value ? shift - ref : -ref; };
    float psum = 0.f;
    const float off = less(m_ref);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc, off));
        psum += p[r];
    }
    // keep the speculative weights ahead of the branch below (they are dead on its slow path, and the
    // optimiser would otherwise sink them behind the test, back onto the critical path)
    if constexpr (N == 8)
        asm volatile("" ::"v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7]));
    else
        asm volatile("" ::"v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7]), "v"(p[8]),
                     "v"(p[9]), "v"(p[10]), "v"(p[11]), "v"(p[12]), "v"(p[13]), "v"(p[14]), "v"(p[15]));
    if (FIRST && RowGeo<D>::kRows == 32) {
        // instruction order for the region that holds both score products and this half's softmax: the second
        // half's 8 matrix instructions are issued with the vector work of the first half's softmax in between
        // (KS = matrix instructions per score product)
        __builtin_amdgcn_sched_group_barrier(0x100, KS / 2, 0);
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        // (the region also holds the 4 * T transpose loads of the half's V fragments)
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i < KS / 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
        }
    }
    if (RowGeo<D>::kRows == 16) {
        if (FIRST) {
            __builtin_amdgcn_sched_group_barrier(0x100, kAheadK, 0);
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (i >= KS - kAheadK) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
            }
        }
    }
    typedef Reference<E, D> R;
    const bool jump = !(psum <= R::kSumMax);                  // also true for the NaN / inf of a fresh reference
    if (__any(jump)) {
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < N; ++r) tmax = fmaxf(tmax, s[r]);
        const float top = row_max<RowGeo<D>::kGroups>(tmax) * sc - (R::kBelow - shift);    // sc > 0: scaling commutes with the max
        const float m_new = fmaxf(m_ref, top);
        const float m_use = m_new == -INFINITY ? 0.f : m_new; // a query with no allowed key so far
        const float alpha = __builtin_amdgcn_exp2f(m_ref - m_use);
#pragma unroll
        for (int t = 0; t < T; ++t) o[t] *= alpha;
        l *= alpha;
        m_ref = m_new;
        psum = 0.f;
        const float off_use = less(m_use);
#pragma unroll
        for (int r = 0; r < N; ++r) {
            p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc, off_use));
            psum += p[r];
        }
    }
    l += psum;
}

// V^T operand fragments of half tile `half` (two 16-key steps x T column blocks), read ahead of their use: the
// transpose loads do not depend on the weights, so they are issued a phase early (under the score products and the
// softmax) and their latency never stands in front of the value product.
// vx[2t], vx[2t+1] = this lane's swizzled transpose-load offsets (slots 0-3 / 4-7) for the 32 columns t.
template <int T>
__device__ __forceinline__ void load_v_frags(uint4 (&va)[T], uint4 (&vb)[T], const char* vbuf, int half,
                                             const uint32_t (&vx)[2 * T])
{
    constexpr int RB = T > 2 ? 256 : 128;
    const char* v0 = vbuf + (32 * half) * RB;
#pragma unroll
    for (int t = 0; t < T; ++t) va[t] = lds_frag_tr(v0 + vx[2 * t], v0 + vx[2 * t + 1]);
#pragma unroll
    for (int t = 0; t < T; ++t) vb[t] = lds_frag_tr(v0 + 16 * RB + vx[2 * t], v0 + 16 * RB + vx[2 * t + 1]);
}

// The weights of 8 keys as a B operand (and their second 16-bit term: p = hi + lo, lo = round(p - hi)).
template <bool PRECISE, typename E, typename S>
__device__ __forceinline__ void pack_weights(uint4& w, uint4& wl, const S& s, int r0)
{
    w.x = E::pack(s[r0 + 0], s[r0 + 1]);
    w.y = E::pack(s[r0 + 2], s[r0 + 3]);
    w.z = E::pack(s[r0 + 4], s[r0 + 5]);
    w.w = E::pack(s[r0 + 6], s[r0 + 7]);
    if (PRECISE) {
        wl.x = E::pack(s[r0 + 0] - E::lo_of(w.x), s[r0 + 1] - E::hi_of(w.x));
        wl.y = E::pack(s[r0 + 2] - E::lo_of(w.y), s[r0 + 3] - E::hi_of(w.y));
        wl.z = E::pack(s[r0 + 4] - E::lo_of(w.z), s[r0 + 5] - E::hi_of(w.z));
        wl.w = E::pack(s[r0 + 6] - E::lo_of(w.w), s[r0 + 7] - E::hi_of(w.w));
    } else {
        wl = w;
    }
}

// O^T += V^T P^T for the 32 keys of a half tile whose fragments load_v_frags brought.  P^T as B operand of a step:
// elements e = 0..7 <-> weights 8*step + e.
template <bool PRECISE, typename E, int T>
__device__ __forceinline__ void half_pv_frags(f32x16 (&o)[T], const f32x16& s, const uint4 (&va)[T], const uint4 (&vb)[T])
{
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        uint4 w, wl;
        pack_weights<PRECISE, E>(w, wl, s, 8 * st);
        const uint4 (&cur)[T] = st ? vb : va;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            o[t] = E::mfma32(cur[t], w, o[t]);
            if (PRECISE) o[t] = E::mfma32(cur[t], wl, o[t]);
        }
    }
}

// The same product where V may hold values that are not finite: a masked key's weight is an exact zero, but zero times
// infinity is not, and an infinity times a weight's second term may undo the one times its first.  One key at a time (the
// other contraction slots zeroed on both sides), added only to the rows that see it, the second term only on finite values.
// base = first key of the half tile; weight r of lane half hh is key base + 8 (r / 4) + 4 hh + r % 4.
template <typename E, int T>
__device__ __forceinline__ void half_pv_by_key(f32x16 (&o)[T], const f32x16& s, const uint4 (&va)[T], const uint4 (&vb)[T],
                                               int32_t base, int32_t nk, int hh)
{
    constexpr uint32_t kExp = E::kDtype == PA_DTYPE_BF16 ? 0x7f80u : 0x7c00u;
    f32x16 p = s;
    if (E::kDtype == PA_DTYPE_F16) {                         // a weight that fp16 would drop still weighs an infinity
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = p[r] > 0.f && p[r] < 0x1p-24f ? 0x1p-24f : p[r];
    }
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        uint4 w, wl;
        pack_weights<true, E>(w, wl, p, 8 * st);
#pragma unroll 1
        for (int i = 0; i < 16; ++i) {
            const int e = i >> 1, h = i & 1;
            const bool seen = base + 8 * (2 * st + (e >> 2)) + 4 * h + (e & 3) < nk;
            const uint32_t half = hh != h ? 0u : (e & 1) ? 0xffff0000u : 0xffffu;
            const uint4 keep = {e >> 1 == 0 ? half : 0u, e >> 1 == 1 ? half : 0u, e >> 1 == 2 ? half : 0u, e >> 1 == 3 ? half : 0u};
            auto cut = [&](const uint4& v) { return uint4{v.x & keep.x, v.y & keep.y, v.z & keep.z, v.w & keep.w}; };
            auto finite = [&](uint32_t v) {
                if ((v & kExp) == kExp) v &= 0xffff0000u;
                if ((v & (kExp << 16)) == kExp << 16) v &= 0xffffu;
                return v;
            };
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint4 v = cut(st ? vb[t] : va[t]);
                f32x16 one = (f32x16)(0.f);
                one = E::mfma32(v, cut(w), one);
                one = E::mfma32(uint4{finite(v.x), finite(v.y), finite(v.z), finite(v.w)}, cut(wl), one);
#pragma unroll
                for (int r = 0; r < 16; ++r) o[t][r] = seen ? o[t][r] + one[r] : o[t][r];
                __builtin_amdgcn_sched_barrier(0);           // (one block's accumulators at a time)
            }
        }
    }
}

// S^T of half tile `half` (32 keys) against the wave's 32 queries: 8 chained matrix instructions, the K operand
// reads kept four ahead.  kx[ks] = this lane's swizzled operand offset for head_dim step ks.
template <typename E, int KS>
__device__ __forceinline__ void half_scores(f32x16& s, const char* kbuf, int half, const uint32_t (&kx)[KS],
                                            const uint4 (&qf)[KS])
{
    constexpr int RB = KS > 4 ? 256 : 128;
    s = (f32x16)(0.f);   // folded into the first matrix instruction's accumulator operand
    const char* kh = kbuf + (32 * half) * RB;
    uint4 ka[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ka[i] = lds_frag(kh + kx[i]);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
        s = E::mfma32(ka[i & 3], qf[i], s);
        if (i + 4 < KS) ka[i & 3] = lds_frag(kh + kx[i + 4]);
    }
}

// ---- 16 rows a wave (head_dim 256) ---------------------------------------------------------------------------------
// The same two products on 16 x 16 x 32 matrix instructions: lane%16 = query, lane/16 = group g of four.  S^T of a
// 16-key block leaves keys 4 g + r in lane group g; two blocks are the 8 contraction slots of a lane in the value product.
// kx / vx are LDS ADDRESSES in the tile's buffer (the other buffer is one bit away), swizzled, of the first 16 pieces of a
// row; everything else -- the second half row, key blocks, the V part -- is a constant that fits the instruction's offset.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) s16x4 lds_tr;

// S^T of half tile `half`: two blocks of 16 keys, D / 32 steps each, operand reads kept kAheadK ahead.
template <typename E, int D, int NK>
__device__ __forceinline__ void half_scores16(f32x8& s, int half, const uint32_t (&kx)[NK], const uint4 (&qf)[D / 32])
{
    constexpr int RB = RowGeo<D>::kRowB, N = 2 * (D / 32);
    auto frag = [&](int i) {
        return __builtin_bit_cast(uint4, *(lds_u32x4*)(uintptr_t)(kx[(i / 2) % NK] + (32 * half + 16 * (i & 1)) * RB + (i / 2 / NK) * 256));
    };
    mfma_f32x4 acc[2] = {(mfma_f32x4)(0.f), (mfma_f32x4)(0.f)};
    uint4 ka[kAheadK];
#pragma unroll
    for (int i = 0; i < kAheadK; ++i) ka[i] = frag(i);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        acc[i & 1] = E::mfma16(ka[i % kAheadK], qf[i / 2], acc[i & 1]);
        if (i + kAheadK < N) ka[i % kAheadK] = frag(i + kAheadK);
    }
    s = __builtin_shufflevector(acc[0], acc[1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// V^T operand of column block i % (D / 16) of half tile i / (D / 16).
template <int D, int NV>
__device__ __forceinline__ uint4 v_frag16(int i, const uint32_t (&vx)[NV])
{
    constexpr int RB = RowGeo<D>::kRowB, T = D / 16;
    const uint32_t p = vx[i % T % NV] + RowGeo<D>::kTileB + (i / T) * 32 * RB + (i % T / NV) * 256;
    tr_pair r;
    r.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr*)(uintptr_t)p);
    r.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr*)(uintptr_t)(p + 16 * RB));
    return __builtin_bit_cast(uint4, r);
}
// O^T += V^T P^T for the 32 keys of half tile HALF; va holds its first fragments on entry and, HALF == 0, those of the
// second half on return (kAheadV ahead of their use).
template <int HALF, bool PRECISE, typename E, int D, int T, int NV>
__device__ __forceinline__ void half_pv16(mfma_f32x4 (&o)[T], const f32x8& p, uint4 (&va)[kAheadV], const uint32_t (&vx)[NV])
{
    uint4 w, wl;
    pack_weights<PRECISE, E>(w, wl, p, 0);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int i = HALF * T + t;
        o[t] = E::mfma16(va[i % kAheadV], w, o[t]);
        if (PRECISE) o[t] = E::mfma16(va[i % kAheadV], wl, o[t]);
        if (i + kAheadV < 2 * T) va[i % kAheadV] = v_frag16<D>(i + kAheadV, vx);
    }
}

// One 64-key tile for one wave, processed as two half tiles of 32 keys so that, within the wave, the softmax of
// one half (vector ALU) runs under the matrix instructions of the other half:
//     matrix cores:  S(h0)   S(h1)          PV(h0)          PV(h1)
//     vector ALU:            softmax(h0)    softmax(h1)
// buf = tile buffer (K rows, then V rows); key0 = first key of the tile + 4 * (lane/32); nk = keys this lane's
// query may see (MASK only); sc = scale * log2(e) > 0.
// CAREFUL: values of V that are not finite stay with the rows that see them (see prefill_body).
template <bool PRECISE, bool MASK, bool CAREFUL, typename E, typename M, int D, typename A, int T, int KS, int NK, int NV>
__device__ __forceinline__ void attend_tile(const char* buf, const uint32_t (&kx)[NK], const uint32_t (&vx)[NV],
                                            const uint4 (&qf)[KS], A (&o)[T], float& m, float& l, float sc,
                                            int32_t key0, int32_t nk, const RowMods& rm, const int32_t* docs)
{
    const char* vbuf = buf + RowGeo<D>::kTileB;
    if constexpr (RowGeo<D>::kRows == 32) {
        f32x16 s0, s1, p;
        const int hh = (int)(threadIdx.x >> 5) & 1;
        uint4 va[T], vb[T];
        half_scores<E, KS>(s0, buf, 0, kx, qf);
        half_scores<E, KS>(s1, buf, 1, kx, qf);
        load_v_frags<T>(va, vb, vbuf, 0, vx);
        half_softmax<MASK, true, E, M, D>(p, s0, o, m, l, sc, key0, nk, rm, docs);
        if (CAREFUL) half_pv_by_key<E, T>(o, p, va, vb, key0 - 4 * hh, nk, hh);
        else half_pv_frags<PRECISE, E, T>(o, p, va, vb);
        load_v_frags<T>(va, vb, vbuf, 1, vx);
        half_softmax<MASK, false, E, M, D>(p, s1, o, m, l, sc, key0 + 32, nk, rm, docs + 32);
        if (CAREFUL) half_pv_by_key<E, T>(o, p, va, vb, key0 + 32 - 4 * hh, nk, hh);
        else half_pv_frags<PRECISE, E, T>(o, p, va, vb);
    } else {
        f32x8 s0, s1, p;
        uint4 va[kAheadV];
        half_scores16<E, D>(s0, 0, kx, qf);
        half_scores16<E, D>(s1, 1, kx, qf);
#pragma unroll
        for (int i = 0; i < kAheadV; ++i) va[i] = v_frag16<D>(i, vx);
        half_softmax<MASK, true, E, M, D>(p, s0, o, m, l, sc, key0, nk, rm, docs);
        half_pv16<0, PRECISE, E, D>(o, p, va, vx);
        half_softmax<MASK, false, E, M, D>(p, s1, o, m, l, sc, key0 + 32, nk, rm, docs + 32);
        half_pv16<1, PRECISE, E, D>(o, p, va, vx);
#pragma unroll
        for (int i = 0; i < T; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
        }
    }
}

// Where an item and its partial go.  (kLengthGrid: a plain grid in the order of contexts that are cut by their own lengths, or of
// the row tiles that there are: locate_live.)
constexpr int kPlainGrid = 0, kSlotList = 1, kEitherList = 2, kLengthGrid = 3;

// What a workgroup works on: sequence, its query range and context length, row tile, head group, and its chunk of the
// context (chunks == 1: all of it).
struct WorkItem {
    int32_t s, q_begin, q_end, len;
    int32_t tile, hg;
    int32_t split, chunks, chunk;
    int32_t slot;            // work-list mode: where a partial goes (-1: the plain layout)
};

// Returns whether the item has to be done again with CAREFUL (the same on every thread of the workgroup): at head_dims 80, 96
// and 112, which keep what the portable kernel, that never touches a key a row does not see, gave them.  An infinity or a NaN
// in V always leaves its mark on some accumulator of the row tile, so the tile loop need not look for it: the accumulators
// are looked at once, at the end (append + prefill of 2 prompts of 700 and 950 tokens, 32 / 32 heads, D = 96: 36.1 us, 38.0 with
// a test of V's fragments on every masked tile; 8 prompts of 33 .. 900, 8 / 2 heads, D = 112: 25.7, 30.5).
// LIST: the kind of list the item comes from (0: a plain grid).
template <bool PRECISE, bool UNIFORM, int LIST, bool CAREFUL, typename E, typename M, int D>
__device__ __forceinline__ bool prefill_body(
    char* buf0, char* buf1, int32_t* docs0, int32_t* docs1, const CacheView& cache, const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ block_table, int32_t num_q_heads, int32_t max_blocks, float scale, int32_t causal, const PrefillPlan& plan, int32_t precise_keys,
    const WorkItem& own, const int tid)
{
    typedef RowGeo<D> Geo;
    constexpr int R = Geo::kRows, RB = Geo::kRowB, STEP = Geo::kStep;
    constexpr int KS = D / (8 * Geo::kGroups);               // steps of a score product
    constexpr int T = (D + R - 1) / R;                       // R-column blocks of O
    const int lane = tid & 63, wave = tid >> 6;
    const int ql = lane & (R - 1), hh = lane / R;            // the lane's row in the wave, its group
    // Rows of a workgroup's 128-row tile are (query, head) pairs: the 2^log2_pack query heads packed into a tile
    // share one KV head, row r of a sequence is query r >> log2_pack, packed head r & (pack - 1).
    const int32_t lg = plan.log2_pack;
    const int32_t s = own.s, hg = own.hg, split = own.split;
    const int32_t q_begin = own.q_begin;                     // (this sequence's lengths: fetched by the kernel ahead of
    const int32_t q_len = own.q_end - own.q_begin;           //  everything else, see there)
    const int32_t n_rows = q_len << lg;
    const int32_t m0 = own.tile * kBM;
    if (m0 >= n_rows) return false;
    if (plan.skip_small && q_len * plan.group <= 16) return false;
    const int32_t len = own.len;
    // workgroup-wide key range; it also selects which instantiation handles this tile
    const int32_t q_last = (min(m0 + kBM, n_rows) - 1) >> lg;
    int32_t nk_wg = len;
    if (causal) nk_wg = min(len, len - q_len + q_last + 1);
    nk_wg = max(nk_wg, 0);
    // sliding window: |key - pos| < window.  The workgroup starts at the 64-aligned key before the window of its
    // first row and, without a causal bound, ends with the window of its last row.
    const int32_t window = (M::kWindow && plan.mods.window > 0) ? plan.mods.window : 0;
    int32_t k_lo = 0;
    if (window > 0) {
        k_lo = max(len - q_len + (m0 >> lg) - window + 1, 0) & ~(kBN - 1);
        if (!causal) nk_wg = max(min(nk_wg, len - q_len + q_last + window), 0);
    }
    // Few effective keys mean few, large weights whose 16-bit rounding shows: rows that see far fewer keys than the
    // call's rows do on (harmonic) average (precise_keys, see precise_key_bound), short contexts and windows, and any
    // position bias (a steep slope concentrates the weight on a handful of keys however long the context is).
    // (a document mask can leave a row a handful of keys out of any context)
    int32_t n_first = len;                                   // keys the tile's first row sees
    if (causal) n_first = min(len, len - q_len + (m0 >> lg) + 1);
    if (window > 0) n_first = min(n_first, causal ? window : 2 * window - 1);
    // (sequences with few queries carry two terms as they do on the decode kernel)
    const bool few_keys = kTwoTermOnly<D> || n_first <= precise_keys || q_len * plan.group <= 16 ||
                          (M::kScore && plan.mods.alibi_slopes != nullptr) || (M::kDoc && plan.mods.doc_ids != nullptr) ||
                          M::kUser;
    if (few_keys != PRECISE) return false;                        // the other instantiation handles this tile
    // this workgroup's chunk of the context; with a split, chunks without keys leave nothing behind (the merge
    // reads only the chunks that hold keys of a row)
    // (without a causal bound a window also cuts the END of a row's range, which the merge does not know: those
    // chunks must leave explicit empty partials, so the workgroup goes on with zero tiles)
    if (own.chunks > 1 && split * own.chunk >= nk_wg && !(window > 0 && !causal)) return false;
    const int32_t k_begin = max(split * own.chunk, k_lo);
    const int32_t k_end = min(nk_wg, split * own.chunk + own.chunk);

    const int32_t G = plan.group;
    const int32_t* table = block_table + (int64_t)s * max_blocks;

    // this lane's row: query, head, and key bound
    const int32_t r_lane = m0 + R * wave + ql;
    const bool q_valid = r_lane < n_rows;
    const int32_t r_c = min(r_lane, n_rows - 1);
    const int32_t qi_c = r_c >> lg;
    const int32_t h = (hg << lg) + (r_c & ((1 << lg) - 1));
    const int32_t kvh = (hg << lg) / G;
    const int32_t pos = len - q_len + qi_c;                  // the row's absolute position
    int32_t nk = len;                                        // keys 0 .. nk-1 are allowed
    if (causal) nk = min(len, pos + 1);
    else if (window > 0) nk = min(len, pos + window);
    nk = max(nk, 0);
    // per wave: the largest bound of its rows decides which tiles it can skip, the smallest which
    // tiles need no mask
    const int32_t pos_first = len - q_len + (min(m0 + R * wave, n_rows - 1) >> lg);
    const int32_t pos_last = len - q_len + (min(m0 + R * wave + R - 1, n_rows - 1) >> lg);
    int32_t nk_wave = len, nk_wave_min = len;
    if (causal) {
        nk_wave = min(len, pos_last + 1);
        nk_wave_min = min(len, pos_first + 1);
    } else if (window > 0) {
        nk_wave = min(len, pos_last + window);
        nk_wave_min = min(len, pos_first + window);
    }
    nk_wave = max(nk_wave, 0);
    nk_wave_min = max(nk_wave_min, 0);
    RowMods rm;
    rm.lo = 0;
    rm.lo_until = 0;
    rm.pos = pos;
    rm.slope2 = 0.f;
    rm.cap_in = 0.f;
    rm.cap_out = 0.f;
    rm.cap = rm.bias = false;
    rm.doc = 0;
    const int32_t* doc_row = nullptr;
    if (M::kDoc && plan.mods.doc_ids) {
        doc_row = plan.mods.doc_ids + (int64_t)s * plan.mods.doc_stride;
        rm.doc = doc_row[max(pos, 0)];
    }
    rm.uc = pa_mod_ctx{plan.mods.user_data, s, h, pos, len};
    int32_t lo_wave = 0;                                     // tiles that end at or before it hold nothing for the wave
    if (window > 0) {
        rm.lo = pos - window + 1;
        rm.lo_until = pos_last - window + 1;
        lo_wave = pos_first - window + 1;
    }
    if (M::kScore) {
        rm.bias = plan.mods.alibi_slopes != nullptr;
        if (rm.bias) rm.slope2 = plan.mods.alibi_slopes[h] * kLog2e;
        rm.cap = plan.mods.softcap > 0.f;
        if (rm.cap) {
            rm.cap_in = scale / plan.mods.softcap * (2.f * kLog2e);
            rm.cap_out = plan.mods.softcap * kLog2e;
        }
    }

    const int64_t row = (int64_t)(q_begin + qi_c) * num_q_heads + h;
    // Q as B operand: lane % R = query, step ks covers 8 head_dim elements of each lane group
    uint4 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qf[ks] = *reinterpret_cast<const uint4*>(q + row * D + 8 * Geo::kGroups * ks + 8 * hh);

    typename std::conditional<R == 32, f32x16, mfma_f32x4>::type o[T];
#pragma unroll
    for (int t = 0; t < T; ++t) o[t] = 0.f;
    float m = -INFINITY, l = 0.f;
    const float sc = scale * kLog2e;

    // swizzled LDS offsets of this lane's operands (see the header): K piece (2*ks + hh) of row ql,
    // V pieces of the 32 columns t for the lane's transpose-load row
    // (16 rows a wave: piece 4*ks + hh, V pieces of the 16 columns t; those of the second half row are not kept)
    constexpr int NK = R == 32 ? KS : 4, NV = R == 32 ? 2 * T : 8;
    uint32_t kx[NK], vx[NV];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) kx[ks] = ql * RB + piece_pos<D>(Geo::kGroups * ks + hh, ql);
    {
        // transpose-load rows of this lane: key 4*hh + j (+8 for slots 4-7) of a 16-key step, columns 4*qq..+3 of
        // the 16-column block dblk of the 32 columns t
        const int j = (lane & 15) >> 2, qq = lane & 3, dblk = (lane >> 4) & 1;
        if constexpr (R == 32) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int piece = 4 * t + 2 * dblk + (qq >> 1);
                vx[2 * t] = (4 * hh + j) * RB + piece_pos<D>(piece, 4 * hh + j) + 8 * (qq & 1);
                vx[2 * t + 1] = (4 * hh + j + 8) * RB + piece_pos<D>(piece, 4 * hh + j + 8) + 8 * (qq & 1);
            }
        } else {
            // key 4*hh + j of a 16-key block, columns 4*qq..+3 of the 16 columns t
#pragma unroll
            for (int t = 0; t < NV; ++t)
                vx[t] = lds_address(buf0) + (4 * hh + j) * RB + piece_pos<D>(2 * t + (qq >> 1), 4 * hh + j) + 8 * (qq & 1);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) kx[ks] += lds_address(buf0);
        }
    }
    // fetch role of this lane.  256-byte rows: position lane%16 of rows 16*i + frow holds logical piece
    // (lane%16) ^ swz(frow) (head_dims 80, 96 and 112 repeat their first pieces in the positions that they do not have, and the
    // columns of O beyond D that are computed from repeats are not stored).  512-byte rows: position lane%32 of rows
    // 16*i + frow.  128-byte rows: position lane%8 of rows 32*i + frow, one page each.
    const int frow = D > 128 ? 2 * wave + (lane >> 5) : D > 64 ? 4 * wave + (lane >> 4) : 8 * wave + (lane >> 3);
    const uint32_t head_off = (uint32_t)(kvh * cache.head_stride * 2);
    const int piece = (D > 128 ? lane & 16 : 0) | ((lane & (D > 64 ? 15 : 7)) ^ row_swz<D>(frow));
    const uint32_t lane_off = head_off + 16 * (D <= 128 && piece >= D / 8 ? piece - D / 8 : piece);
    const int32_t wrow = __builtin_amdgcn_readfirstlane(1024 * wave);    // (a load instruction fills 1 KiB)
    const int32_t second16 = D == 64 ? __builtin_amdgcn_readfirstlane(wave >> 1) : 0;
    const int32_t last_key = len - 1;
    const uint32_t lds0 = lds_address(buf0 + wrow), lds1 = lds_address(buf1 + wrow);
    auto fetch = [&](uint32_t lds, const PageIds& pg, int32_t t0) {
        if constexpr (D > 128) fetch_tile512<UNIFORM>(lds, pg, cache, t0, frow, last_key, lane_off);
        else if constexpr (D == 64) {
            constexpr int TB = Geo::kTileB;
            fetch_rows<UNIFORM, 0, TB>(lds, cache, UNIFORM && second16 ? pg.p1 : pg.p0, t0 + frow, last_key, lane_off);
            fetch_rows<UNIFORM, 32 * RB, TB>(lds, cache, UNIFORM && second16 ? pg.p3 : pg.p2, t0 + frow + 32, last_key, lane_off);
        } else fetch_tile<UNIFORM>(lds, pg, cache, t0, frow, last_key, lane_off);
    };

    // Document masks: wave 0 brings the 64 ids of the next tile (one per lane) and stores them next to the tile
    // buffer before the barrier that publishes the tile, together with their minimum and maximum (slots 64, 65).
    // A wave skips a tile whose id range misses the id range of its rows: always right, and it pays when documents
    // are contiguous runs of positions, as in packed batches.  (The tile is still fetched: deciding that ahead of
    // the fetch costs a dependent global load per tile, which was measured to cost more than the fetches it saves.)
    const bool doc_lane = M::kDoc && wave == 0;
    int32_t doc_next = 0;
    int32_t row_doc_min = rm.doc, row_doc_max = rm.doc;
    // minimum and maximum over the wave
    auto wave_range = [&](int32_t v, int32_t& mn, int32_t& mx) {
        mn = v;
        mx = v;
#define PA_RANGE_STEP(CTRL, ROWS)                                                                   \
        mn = min(mn, __builtin_amdgcn_update_dpp(mn, mn, CTRL, ROWS, 0xF, false));                  \
        mx = max(mx, __builtin_amdgcn_update_dpp(mx, mx, CTRL, ROWS, 0xF, false));
        PA_WAVE_FOLD(PA_RANGE_STEP)
#undef PA_RANGE_STEP
        mn = __builtin_amdgcn_readlane(mn, 63);
        mx = __builtin_amdgcn_readlane(mx, 63);
    };
    auto put_docs = [&](int32_t* dst, int32_t v) {           // wave 0: the tile's ids and their range
        int32_t mn, mx;
        wave_range(v, mn, mx);
        dst[lane] = v;
        if (lane < 2) dst[kBN + lane] = lane ? mx : mn;
    };
    auto docs_overlap = [&](const int32_t* d) -> bool {      // wave-uniform
        if (!M::kDoc) return true;
        const int32_t mn = __builtin_amdgcn_readfirstlane(d[kBN]);
        const int32_t mx = __builtin_amdgcn_readfirstlane(d[kBN + 1]);
        return mx >= row_doc_min && mn <= row_doc_max;
    };
    auto tile_ids = [&](int32_t t0) -> int32_t { return doc_row ? doc_row[min(t0 + lane, last_key)] : 0; };
    if (M::kDoc) wave_range(rm.doc, row_doc_min, row_doc_max);
    PageIds ids;
    const int32_t n_tiles = (max(k_end - k_begin, 0) + kBN - 1) / kBN;
    if (n_tiles > 0) {
        load_ids<UNIFORM>(ids, cache, table, k_begin, frow, last_key);
        fetch(lds0, ids, k_begin);
        if (doc_lane) put_docs(docs0, tile_ids(k_begin));
        if (n_tiles > 1) load_ids<UNIFORM>(ids, cache, table, k_begin + kBN, frow, last_key);
    }
    wait_tile_loads();                                       // (outside the test: the loop below must start from a
    __syncthreads();                                         //  state without pending loads on every path)
    if constexpr (R == 16) {
        // (one copy of the tile's code: the two buffers are one bit apart, and so are the addresses of their operands)
        for (int32_t t = 0; t < n_tiles; ++t) {
            const int32_t t0 = k_begin + t * kBN;
            if (t + 1 < n_tiles) {
                fetch(t & 1 ? lds0 : lds1, ids, t0 + kBN);
                if (doc_lane) doc_next = tile_ids(t0 + kBN);
                if (t + 2 < n_tiles) load_ids<UNIFORM>(ids, cache, table, t0 + 2 * kBN, frow, last_key);
            }
            int32_t* const docs = t & 1 ? docs1 : docs0;
            if (t0 < nk_wave && t0 + kBN > lo_wave && docs_overlap(docs)) {
                if (t0 + kBN > nk_wave_min || (M::kWindow && t0 < rm.lo_until))
                    attend_tile<PRECISE, true, CAREFUL, E, M, D>(nullptr, kx, vx, qf, o, m, l, sc, t0 + 4 * hh, nk, rm, docs + 4 * hh);
                else
                    attend_tile<PRECISE, false, CAREFUL, E, M, D>(nullptr, kx, vx, qf, o, m, l, sc, t0 + 4 * hh, nk, rm, docs + 4 * hh);
            }
            if (doc_lane && t + 1 < n_tiles) put_docs(t & 1 ? docs0 : docs1, doc_next);
            wait_tile_loads();
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NK; ++i) kx[i] ^= Geo::kBufB;
#pragma unroll
            for (int i = 0; i < NV; ++i) vx[i] ^= Geo::kBufB;
        }
    } else {
        // Two tiles per trip so that each buffer is a distinct LDS object for the compiler: while the matrix cores
        // read one, the load unit fills the other with the next tile; the page ids of the tile after that are requested
        // at the same time.  The barrier at the end of a tile waits for this wave's loads first.
        for (int32_t t = 0; t < n_tiles; t += 2) {
            const int32_t t0 = k_begin + t * kBN;
            if (t + 1 < n_tiles) {
                fetch(lds1, ids, t0 + kBN);
                if (doc_lane) doc_next = tile_ids(t0 + kBN);
                if (t + 2 < n_tiles) load_ids<UNIFORM>(ids, cache, table, t0 + 2 * kBN, frow, last_key);
            }
            if (t0 < nk_wave && t0 + kBN > lo_wave && docs_overlap(docs0)) {   // wave-uniform: else nothing for this wave here
                if (t0 + kBN > nk_wave_min)                      // wave-uniform: some score of this tile is masked
                    attend_tile<PRECISE, true, CAREFUL, E, M, D>(buf0, kx, vx, qf, o, m, l, sc, t0 + 4 * hh, nk, rm, docs0 + 4 * hh);
                else
                    attend_tile<PRECISE, false, CAREFUL, E, M, D>(buf0, kx, vx, qf, o, m, l, sc, t0 + 4 * hh, nk, rm, docs0 + 4 * hh);
            }
            if (doc_lane && t + 1 < n_tiles) put_docs(docs1, doc_next);
            wait_tile_loads();
            __syncthreads();
            if (t + 1 >= n_tiles) break;
            const int32_t t1 = t0 + kBN;
            if (t + 2 < n_tiles) {
                fetch(lds0, ids, t1 + kBN);
                if (doc_lane) doc_next = tile_ids(t1 + kBN);
                if (t + 3 < n_tiles) load_ids<UNIFORM>(ids, cache, table, t1 + 2 * kBN, frow, last_key);
            }
            if (t1 < nk_wave && t1 + kBN > lo_wave && docs_overlap(docs1)) {
                if (t1 + kBN > nk_wave_min)
                    attend_tile<PRECISE, true, CAREFUL, E, M, D>(buf1, kx, vx, qf, o, m, l, sc, t1 + 4 * hh, nk, rm, docs1 + 4 * hh);
                else
                    attend_tile<PRECISE, false, CAREFUL, E, M, D>(buf1, kx, vx, qf, o, m, l, sc, t1 + 4 * hh, nk, rm, docs1 + 4 * hh);
            }
            if (doc_lane && t + 2 < n_tiles) put_docs(docs0, doc_next);
            wait_tile_loads();
            __syncthreads();
        }
    }

    if constexpr (kTwoTermOnly<D> && !CAREFUL) {
        bool odd = false;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) odd |= !(__builtin_fabsf(o[t][r]) <= 3.402823466e38f);
        const bool any = __any(odd);
        if (lane == 0) docs0[wave] = any ? 1 : 0;            // (no document masks here: the array is free)
        __syncthreads();
        if (docs0[0] | docs0[1] | docs0[2] | docs0[3]) return true;
    }
    if (R == 16) l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (!q_valid) return false;
    const float inv = l > 0.f ? 1.f / l : 0.f;
    // (a NaN among the scores makes l and the LSE NaN, in a partial too: the merge hands it on)
    const float row_lse = l <= 0.f ? -INFINITY : (m + __builtin_amdgcn_logf(l)) * kLn2;
    // four columns STEP*i + 4*hh .. +3 of this lane's query: o[t][r] is column 32*t + 8*(r/4) + 4*hh + r%4, or with 16
    // rows a wave column 16*t + 4*hh + r
    constexpr int NC = T * (R / STEP);
    auto cols = [&](int i) {
        if constexpr (R == 32)
            return float4{o[i / 4][4 * (i % 4) + 0] * inv, o[i / 4][4 * (i % 4) + 1] * inv, o[i / 4][4 * (i % 4) + 2] * inv,
                          o[i / 4][4 * (i % 4) + 3] * inv};
        else return float4{o[i][0] * inv, o[i][1] * inv, o[i][2] * inv, o[i][3] * inv};
    };
    if (LIST != kPlainGrid && own.slot >= 0) {
        // work-list mode: normalised accumulators lane by lane (whole cache lines per store), LSE per row.  The layout is
        // that of 32 rows a wave: 16-byte piece i of lane (row, group of two), piece = 8 columns.
        float4* po = reinterpret_cast<float4*>(plan.list_o) + (int64_t)own.slot * (list_slot_floats(D) / 4) +
                     (R * wave / 32) * (list_slot_floats(D) / 16);
        if constexpr (R == 32) po += lane;
        else po += (hh >> 1) * 64 + (hh & 1) * 32 + (16 * wave + ql) % 32;
#pragma unroll
        for (int i = 0; i < NC; ++i) po[i * (R == 32 ? 64 : 128)] = cols(i);
        if (hh == 0) plan.list_lse[(int64_t)own.slot * kBM + R * wave + ql] = row_lse;
        return false;
    }
    if (LIST != kSlotList && own.chunks > 1) {
        // partial of this chunk: normalised output in fp32 and the natural-log LSE over the chunk's keys
        const int64_t pidx = row * plan.nsplit + split;
        float* prow = plan.part_o + pidx * D;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (STEP * i >= D) continue;                     // columns that pad the last block
            *reinterpret_cast<float4*>(prow + STEP * i + 4 * hh) = cols(i);
        }
        if (hh == 0) plan.part_lse[pidx] = row_lse;
        return false;
    }
    uint16_t* orow = out + row * D;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        if (STEP * i >= D) continue;
        const float4 c = cols(i);
        *reinterpret_cast<uint2*>(orow + STEP * i + 4 * hh) = uint2{E::pack(c.x, c.y), E::pack(c.z, c.w)};
    }
    if (lse && hh == 0) lse[row] = row_lse;
    return false;
}

__device__ __forceinline__ WorkList scan_plan_list(const PrefillPlan& plan, const int32_t* __restrict__ cu_q_lens,
                                                   const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_q_heads)
{
    return scan_list(cu_q_lens, seq_lens, batch, plan.log2_pack, plan.skip_small ? plan.group : kNoSmallGroup,
                     num_q_heads >> plan.log2_pack, (int)(threadIdx.x & 63));
}

// The work-list mode of prefill_tiles.h: items first, first + step, ... of the call's list (as scan_plan_list left it).  LIST: kSlotList (partials by slot) or
// kEitherList (also, with chunk_unit, contexts cut by their own lengths and partials by row, as a plain grid leaves them).
template <bool UNIFORM, int LIST, typename E, typename M, int D>
__device__ __forceinline__ void list_body(
    char* buf0, char* buf1, int32_t* docs0, int32_t* docs1, const CacheView& cache, const uint16_t* __restrict__ q,
    uint16_t* __restrict__ out, float* __restrict__ lse, const int32_t* __restrict__ cu_q_lens,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_q_heads,
    int32_t max_blocks, float scale, int32_t causal, const PrefillPlan& plan, WorkList& list, uint32_t first, uint32_t step)
{
    WorkItem own;
    const int32_t heads = num_q_heads >> plan.log2_pack;
    // A workgroup steps over the list by `step`.  Between two items nothing has to be waited for: a
    // tile loop ends with the barrier behind its last read of LDS.  The thread index is made opaque for each item:
    // what the body derives from it would otherwise be kept in registers across the loop, which spills.
    constexpr bool kByLength = LIST == kEitherList;
    cut_list(list, cu_q_lens, seq_lens, plan.list_unit, D, (int)(threadIdx.x & 63));
    list.nsplit = plan.nsplit;
    list.unit = plan.chunk_unit;
    int32_t precise_keys = 0;
    if constexpr (!kTwoTermOnly<D>)
        precise_keys = precise_key_bound(cu_q_lens, seq_lens, batch, causal, 0, (int)(threadIdx.x & 63));
    for (uint32_t index = first;; index += step) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        ListItem it;
        if (!list_locate<false, kByLength>(it, list, cu_q_lens, seq_lens, (int32_t)(index / (uint32_t)heads), tid & 63)) return;
        own.s = it.s;
        own.hg = (int32_t)(index % (uint32_t)heads);
        own.tile = it.tile;
        own.split = it.split;
        own.chunks = it.chunks;
        own.slot = it.chunks > 1 && !(kByLength && list.unit > 0) ? list_slot(it, it.split, heads, own.hg) : -1;
        own.q_begin = cu_q_lens[it.s];
        own.q_end = cu_q_lens[it.s + 1];
        own.len = seq_lens[it.s];
        own.chunk = list_chunk<kByLength>(list, own.len);
        if constexpr (!kTwoTermOnly<D>)
            prefill_body<false, UNIFORM, LIST, false, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table,
                                                        num_q_heads, max_blocks, scale, causal, plan, precise_keys, own,
                                                        tid);
        const bool again =
            prefill_body<true, UNIFORM, LIST, false, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table,
                                                              num_q_heads, max_blocks, scale, causal, plan, precise_keys,
                                                              own, tid);
        if constexpr (kTwoTermOnly<D>)
            if (again)
                prefill_body<true, UNIFORM, LIST, true, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table,
                                                                 num_q_heads, max_blocks, scale, causal, plan,
                                                                 precise_keys, own, tid);
    }
}

// precise_key_bound from a lane's own sequence.  (A text of its own: sharing one changed the plain kernel's code, whose start and
// tile loop answer to such changes with up to 10 %.)
struct RowSums {
    float rows, inv;     // rows, and the sum of 1 / n over them
};
__device__ __forceinline__ void add_rows(RowSums& r, int32_t q_len, int32_t len, int32_t causal, int32_t window)
{
    if (q_len <= 0 || len <= 0) return;
    const int32_t hi = len;                                       // keys of the last row
    const int32_t lo = causal ? max(len - q_len + 1, 1) : len;    // keys of the first row that sees any
    const int32_t cap = window > 0 ? (causal ? window : 2 * window - 1) : 0x7fffffff;
    const int32_t n_rows = causal ? hi - lo + 1 : q_len;
    r.rows += (float)n_rows;
    if (!causal) {
        r.inv += (float)q_len / (float)min(len, cap);
        return;
    }
    const int32_t b = min(hi, cap);
    if (b >= lo) r.inv += __builtin_amdgcn_logf(((float)b + 0.5f) / ((float)lo - 0.5f)) * kLn2;
    const int32_t above = hi - max(lo, cap + 1) + 1;              // rows that see the whole window
    if (above > 0) r.inv += (float)above / (float)cap;
}
__device__ __forceinline__ int32_t precise_keys_of(const RowSums& r)   // (every lane's rows)
{
    const float rows = wave_sum_moves(r.rows), inv = wave_sum_moves(r.inv);
    const float h = inv > 0.f ? rows / inv : 0.f;
    return max(kPreciseKeys, (int32_t)fminf(kPreciseShare * h, 1.0e9f));
}

// Row tile number `index` of those that the call has, from the last ones of every sequence to the first (at most 64 sequences).
// Without it the grid has a workgroup for every tile of the longest query range in every sequence, and the ones that a shorter
// sequence does not have come first: they end at once, but workgroups go to the shader engines of a chiplet in turn and each
// waits for room on its own, so the compute units that empty workgroups leave stand by while the others are full.
// The lengths that every lane brings (one sequence each) serve the two-term rule as well.
__device__ __forceinline__ bool locate_live(WorkItem& own, int32_t& precise_keys, int32_t index, int32_t num_tiles,
                                            const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ seq_lens,
                                            int32_t batch, int32_t causal, int32_t window, const PrefillPlan& plan)
{
    const int32_t lane = (int32_t)(threadIdx.x & 63), s = min(lane, batch - 1);
    const int32_t q_begin = cu_q_lens[s], q_end = cu_q_lens[s + 1], len = seq_lens[s], q_len = q_end - q_begin;
    int32_t n = min(((max(q_len, 0) << plan.log2_pack) + kBM - 1) / kBM, num_tiles);
    if (lane >= batch || (plan.skip_small && q_len * plan.group <= 16)) n = 0;
    // lo: the last tile index of which, and of those above, there are more than `index`; above: tiles of the indexes beyond it
    int32_t lo = -1, above = 0;
    if (num_tiles <= 64 && batch <= 16) {                    // (a lane for every tile index)
        int32_t f = 0;
        for (int32_t i = 0; i < batch; ++i) f += max(__builtin_amdgcn_readlane(n, i) - lane, 0);
        lo = 63 - __clzll((unsigned long long)__ballot(f > index));
        if (lo < 63) above = __builtin_amdgcn_readlane(f, lo + 1);
    } else {
        for (int32_t hi = num_tiles; hi - lo > 1;) {
            const int32_t mid = (lo + hi) >> 1, f = wave_total_moves(max(n - mid, 0));
            if (f > index) {
                lo = mid;
            } else {
                hi = mid;
                above = f;
            }
        }
    }
    if (lo < 0) return false;
    RowSums rows = {0.f, 0.f};
    if (lane < batch) add_rows(rows, q_len, len, causal, window);
    precise_keys = precise_keys_of(rows);
    const uint64_t have = __ballot(n > lo);
    const int32_t rank = (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(have >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)have, 0));
    const int at = __ffsll((unsigned long long)__ballot(n > lo && rank == index - above)) - 1;
    own.s = at;
    own.tile = lo;
    own.q_begin = __builtin_amdgcn_readlane(q_begin, at);
    own.q_end = __builtin_amdgcn_readlane(q_end, at);
    own.len = __builtin_amdgcn_readlane(len, at);
    return true;
}

// Both instantiations live in one kernel as two separate code paths (each with its own tile loop); a
// workgroup runs exactly one of them, decided by its context length.
// LIST: kSlotList, the work-list mode of prefill_tiles.h; kPlainGrid (kByTile); or kLengthGrid (the other orders; an instantiation of its own: deciding it
// here scattered the first loads and cost a prompt of 128 tokens 0.4 us of 9).
// Waves a SIMD: two, three at head_dim 64.  Hooks that keep more state spill under that bound: document masks and user
// modifications 4 - 6 registers at head_dim 64, 12 and 24 at 256, slopes 7 at 256, and nothing at 128.  us for 4 x 2048, 2 x 1200 and
// 1 x 500 tokens (32 / 8 heads, 16 / 8 at 256), one wave less and no spill / like this: at head_dim 64 documents 105 / 89,
// 34.0 / 34.8, 19.0 / 18.7, prefix-LM 504 / 399, 142 / 96, 35 / 35; at 256, where that is four waves of 32 rows, documents
// 191 / 173, 72 / 53, 35 / 32, prefix-LM 725 / 638, 226 / 198, 56 / 47, slopes 350 / 270, 100 / 77, 46 / 37.
template <bool UNIFORM, typename E, typename M, int D, int LIST = kPlainGrid>
__global__ __launch_bounds__(RowGeo<D>::kThreads, D > 64 ? 2 : 3) void paged_prefill_mfma_kernel(
    CacheView cache, const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_tiles, int32_t num_q_heads, int32_t max_blocks,
    float scale, int32_t causal, PrefillPlan plan)
{
    // two tile buffers; with 16 rows a wave they are one object, aligned to its size, so that one address bit tells them apart
    constexpr bool kPair = RowGeo<D>::kRows == 16;
    constexpr int kOne = kPair ? 2 * RowGeo<D>::kBufB : RowGeo<D>::kBufB;
    static_assert(!kPair || (RowGeo<D>::kBufB & (RowGeo<D>::kBufB - 1)) == 0, "the buffers of a pair are one bit apart");
    __shared__ __attribute__((aligned(kPair ? kOne : 1024))) char buf0[kOne];
    __shared__ __attribute__((aligned(1024))) char other[kPair ? 16 : RowGeo<D>::kBufB];
    char* const buf1 = kPair ? buf0 + RowGeo<D>::kBufB : other;
    __shared__ __attribute__((aligned(16))) int32_t docs0[kBN + 4];
    __shared__ __attribute__((aligned(16))) int32_t docs1[kBN + 4];
    // The workgroup's own lengths are requested first (scalar loads), the scan of every sequence's lengths for the
    // two-term rule right behind them (vector loads): one round trip to memory instead of three in a row in front
    // of the query and block-table loads that depend on them.
    if constexpr (LIST == kSlotList) {
        WorkList list = scan_plan_list(plan, cu_q_lens, seq_lens, batch, num_q_heads);
        list_body<UNIFORM, kSlotList, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, cu_q_lens, block_table, seq_lens,
                                               batch, num_q_heads, max_blocks, scale, causal, plan, list, blockIdx.x, gridDim.x);
    } else {
        // Workgroups are dispatched in blockIdx.x order: the row-tile index is the slowest-varying part and runs
        // backwards, so the whole grid is handed out heaviest (latest causal tiles) first.  With chunks (kLengthGrid) all row
        // tiles of a context chunk precede the next chunk's, whose first ones have no keys there: chunk beside chunk those would
        // recur at one place in every few workgroups (see locate_live; 3000 tokens in two chunks, 16 / 8 heads, head_dim 256, 169
        // -> 145 us, 20 sequences of which two have 128 queries with a cap 231 -> 224; launch_prefill_mfma says where
        // another order is taken).  Where contexts are cut by their own lengths (kLengthGrid) they are much longer than the query
        // ranges and no tile is heavy: there the sequence is the slowest part, so that the workgroups with keys stand side by
        // side and get a compute unit each, whatever is empty between them (128 queries on 32768 keys and on 2000 three times
        // 206 -> 119 us, 256 on 32768 and on 16000 285 -> 224, 500 on 2048 in a call for up to 32768 65 -> 42).  In a
        // sequence the chunks of a tile follow each other if it is alone, so that a compute unit's workgroups walk the same
        // keys (1024 queries on 32768 with the append 506 us, tile after tile in a chunk 510); in batches tile after tile
        // (four with 128 queries on 32768 300, chunk after chunk 313; 256 on 16000 and on 1500 with 8 / 8 heads 43 and 51).
        WorkItem own;
        const int32_t heads = num_q_heads >> plan.log2_pack;
        constexpr bool kByLength = LIST == kLengthGrid;
        const int32_t hb = heads * (kByLength ? 1 : batch);
        const int32_t slow = (int32_t)(blockIdx.x / (uint32_t)hb);
        const int32_t rest = (int32_t)(blockIdx.x % (uint32_t)hb);
        own.hg = rest % heads;
        own.chunks = plan.nsplit;
        own.chunk = plan.chunk;
        own.slot = -1;
        int32_t precise_keys = 0;
        if constexpr (kByLength) {
            if (plan.order == kLiveTiles) {
                own.split = 0;
                if (!locate_live(own, precise_keys, slow, num_tiles, cu_q_lens, seq_lens, batch, causal,
                                 (M::kWindow && plan.mods.window > 0) ? plan.mods.window : 0, plan)) return;
            } else {
                const int32_t each = num_tiles * plan.nsplit;    // (by length: row tiles and chunks of a sequence)
                const int32_t of_all = slow / batch;
                own.s = plan.chunk_unit > 0 ? slow / each : slow - of_all * batch;
                own.q_begin = cu_q_lens[own.s];
                own.q_end = cu_q_lens[own.s + 1];
                own.len = seq_lens[own.s];
                if (plan.chunk_unit > 0) {
                    own.chunk = sequence_chunk(own.len, plan.chunk, plan.nsplit, plan.chunk_unit);
                    const int32_t live = max((own.len + own.chunk - 1) / own.chunk, 1), part = slow - own.s * each;
                    const int32_t per = batch == 1 ? live : num_tiles, quot = part / per, rem = part - quot * per;
                    own.tile = num_tiles - 1 - (batch == 1 ? quot : rem);
                    own.split = batch == 1 ? rem : quot;
                    if (own.tile < 0) return;                    // (beyond a single sequence's chunks)
                } else {
                    const int32_t quot = of_all / num_tiles;
                    own.split = plan.order == kLastChunkFirst ? plan.nsplit - 1 - quot : quot;
                    own.tile = num_tiles - 1 - (of_all - quot * num_tiles);
                }
            }
        } else {
            own.s = rest / heads;
            own.tile = num_tiles - 1 - slow / plan.nsplit;
            own.split = slow % plan.nsplit;
            own.q_begin = cu_q_lens[own.s];
            own.q_end = cu_q_lens[own.s + 1];
            own.len = seq_lens[own.s];
        }
        if constexpr (!kTwoTermOnly<D>) {
            if (!kByLength || plan.order != kLiveTiles)
                precise_keys = precise_key_bound(cu_q_lens, seq_lens, batch, causal,
                                                 (M::kWindow && plan.mods.window > 0) ? plan.mods.window : 0,
                                                 (int)(threadIdx.x & 63));
            prefill_body<false, UNIFORM, kPlainGrid, false, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table, num_q_heads,
                                                        max_blocks, scale, causal, plan, precise_keys, own, (int)threadIdx.x);
        }
        const bool again =
            prefill_body<true, UNIFORM, kPlainGrid, false, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table,
                                                              num_q_heads, max_blocks, scale, causal, plan, precise_keys, own,
                                                              (int)threadIdx.x);
        if constexpr (kTwoTermOnly<D>)
            if (again)
                prefill_body<true, UNIFORM, kPlainGrid, true, E, M, D>(buf0, buf1, docs0, docs1, cache, q, out, lse, block_table,
                                                                 num_q_heads, max_blocks, scale, causal, plan, precise_keys,
                                                                 own, (int)threadIdx.x);
    }
}

}  // namespace

// The plain grid's kernel in the order that the plan asks for.
#define PA_GRID_KERNEL(UNIFORM, E, M)                                                                                  \
    (plan.order != kByTile ? paged_prefill_mfma_kernel<UNIFORM, E, M, D, kLengthGrid> : paged_prefill_mfma_kernel<UNIFORM, E, M, D>)

// Every kernel instantiation of one head_dim; defined in that head_dim's translation unit.
template <int D>
pa_status launch_prefill_mfma_dim(const AttnArgs& a, const PrefillPlan& plan, int64_t blocks, int64_t tiles,
                                  hipStream_t stream)
{
    const dim3 grid((uint32_t)blocks, 1, 1);
    if constexpr (kTwoTermOnly<D>) {   // (prefill_mfma_supported takes no hooks and no pages below 16 tokens here)
        if (a.has_mods || a.cache.page_size < 16) return PA_ERR_UNSUPPORTED;
        auto kern = a.dtype == PA_DTYPE_BF16
                        ? (plan.list_items > 0 ? paged_prefill_mfma_kernel<true, ElemBf16, NoMods, D, kSlotList>
                                               : PA_GRID_KERNEL(true, ElemBf16, NoMods))
                        : (plan.list_items > 0 ? paged_prefill_mfma_kernel<true, ElemF16, NoMods, D, kSlotList>
                                               : PA_GRID_KERNEL(true, ElemF16, NoMods));
        hipLaunchKernelGGL(kern, grid, dim3(RowGeo<D>::kThreads), 0, stream, a.cache, (const uint16_t*)a.q, (uint16_t*)a.out, a.lse,
                           a.cu_q_lens, a.block_table, a.seq_lens, a.batch, (int32_t)tiles, a.num_q_heads, a.max_blocks,
                           a.scale, a.causal, plan);
        return launch_status();
    } else {
    // page sizes of 16 and more make the page of a 16-key group wave-uniform (scalar page translation)
    const bool uniform = a.cache.page_size >= 16;
    if (D > 128 && !uniform) return PA_ERR_UNSUPPORTED;   // 512-byte rows: two rows per load must share a page
    constexpr bool kLargePagesOnly = D > 128;             // (no kernels for smaller pages then)
    typedef Mods<true, true, false> WindowScore;
    // (a window alone and a soft cap have kernels of their own at head_dim 256 only: prompts of 2059 and 3146 tokens, 16 / 8
    // heads, window 1024 with the shared kernel / the own one 178 / 157 us, with a cap 193 / 166; 32 / 8 heads at head_dim
    // 128 104.4 / 103.9 and 128.1 / 127.1, at 64 74.5 / 77.1 and 103.9 / 103.8)
    typedef std::conditional_t<(D > 128), Mods<true, false, false>, WindowScore> Window;
    typedef std::conditional_t<(D > 128), WindowCap, WindowScore> Cap;
    const bool windowed = D > 128 && a.has_mods && !a.mods.alibi_slopes && !(a.mods.softcap > 0.f);
    const bool capped = D > 128 && a.mods.softcap > 0.f && !a.mods.alibi_slopes;
    auto kern = PA_GRID_KERNEL(true, ElemBf16, NoMods);
    if (plan.list_items > 0) {                            // (prefill_list_supported)
        if (a.has_mods || !uniform) return PA_ERR_UNSUPPORTED;
        kern = a.dtype == PA_DTYPE_BF16 ? paged_prefill_mfma_kernel<true, ElemBf16, NoMods, D, kSlotList>
                                        : paged_prefill_mfma_kernel<true, ElemF16, NoMods, D, kSlotList>;
    } else if (a.mods.user_mod) {                         // a user modification: one instantiation per listed struct
        bool found = false;
#define PA_USER_CASE(U)                                                                                     \
        if (a.mods.user_mod == U::kId) {                                                                    \
            typedef Mods<true, true, true, U> UM;                                                           \
            found = true;                                                                                   \
            if (a.dtype == PA_DTYPE_BF16)                                                                   \
                kern = uniform ? PA_GRID_KERNEL(true, ElemBf16, UM)                           \
                               : PA_GRID_KERNEL(kLargePagesOnly, ElemBf16, UM);                         \
            else                                                                                            \
                kern = uniform ? PA_GRID_KERNEL(true, ElemF16, UM)                            \
                               : PA_GRID_KERNEL(kLargePagesOnly, ElemF16, UM);                          \
        }
        PA_USER_MODS(PA_USER_CASE)
#undef PA_USER_CASE
        if (!found) return PA_ERR_INVALID_ARG;
    } else if (a.has_mods && a.mods.doc_ids) {
        if (a.dtype == PA_DTYPE_BF16)
            kern = uniform ? PA_GRID_KERNEL(true, ElemBf16, AllMods)
                           : PA_GRID_KERNEL(kLargePagesOnly, ElemBf16, AllMods);
        else
            kern = uniform ? PA_GRID_KERNEL(true, ElemF16, AllMods)
                           : PA_GRID_KERNEL(kLargePagesOnly, ElemF16, AllMods);
    } else if (a.dtype == PA_DTYPE_BF16) {
        if (windowed) kern = PA_GRID_KERNEL(true, ElemBf16, Window);
        else if (capped) kern = PA_GRID_KERNEL(true, ElemBf16, Cap);
        else if (a.has_mods) kern = uniform ? PA_GRID_KERNEL(true, ElemBf16, WindowScore)
                                       : PA_GRID_KERNEL(kLargePagesOnly, ElemBf16, WindowScore);
        else if (!uniform) kern = PA_GRID_KERNEL(kLargePagesOnly, ElemBf16, NoMods);
    } else {
        if (windowed) kern = PA_GRID_KERNEL(true, ElemF16, Window);
        else if (capped) kern = PA_GRID_KERNEL(true, ElemF16, Cap);
        else if (a.has_mods) kern = uniform ? PA_GRID_KERNEL(true, ElemF16, WindowScore)
                                       : PA_GRID_KERNEL(kLargePagesOnly, ElemF16, WindowScore);
        else kern = uniform ? PA_GRID_KERNEL(true, ElemF16, NoMods)
                            : PA_GRID_KERNEL(kLargePagesOnly, ElemF16, NoMods);
    }
    hipLaunchKernelGGL(kern, grid, dim3(RowGeo<D>::kThreads), 0, stream, a.cache, (const uint16_t*)a.q, (uint16_t*)a.out, a.lse,
                       a.cu_q_lens, a.block_table, a.seq_lens, a.batch, (int32_t)tiles, a.num_q_heads, a.max_blocks,
                       a.scale, a.causal, plan);
    return launch_status();
    }
}

#undef PA_GRID_KERNEL

}  // namespace pa
