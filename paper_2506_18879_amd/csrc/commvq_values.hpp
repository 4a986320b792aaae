// Value and output stage of indexed values in one kernel (included by commvq.hip).
#pragma once
#include "commvq_internal.hpp"

namespace {

// 64-bit words of a codeword's row of bins (a word per pair of heads and codebook, repeated to fill the row), and bytes of
// the bins of one slot.
template <int G, int CB, int S>
constexpr int values_words()
{
    constexpr int own = (G >= 2 ? G / 2 : 1) * CB, row = S == 1 && G >= 4 ? 32 : 16;
    return own > row ? own : row;
}
template <int G, int CB, int S>
constexpr int values_slot() { return kK * values_words<G, CB, S>() * 8; }
// LDS of a workgroup: the slots' bins or, later, the wavefronts' sums; behind them, for more than one span, the sums of the spans before
// (two floats per word of a row without copies), and three numbers per slot and head and two more per span.
template <int G, int CB, int S, int NCS, int NT>
constexpr int values_bins()
{
    constexpr int red = NT / 64 * S * G * (kD / NCS) * 4, bins = S * values_slot<G, CB, S>();
    return bins > red ? bins : red;
}
template <int G, int CB, int S, int NCS, int NT>
constexpr int values_lds(int spans)
{
    return values_bins<G, CB, S, NCS, NT>() + (spans > 1 ? kK * (G >= 2 ? G / 2 : 1) * CB * 8 : 0) + (3 + 2 * spans) * S * G * 4;
}

// Units of a fixed-point sum per 1: with n numbers of sum l, each rounded to a whole number of them, the sum stays below 2^32 (2^-14 covers
// what l and the numbers, computed apart, differ by, and a second rounding of such sums another 2^-14).
__device__ __forceinline__ float units_per_one(float l, int n, float margin)
{
    return l >= 1e-30f ? fminf((4294967296.f * (1.f - margin) - (float)n) * __builtin_amdgcn_rcpf(l), 0x1p120f) : 1.f;
}
__device__ __forceinline__ float unit_of(float per)        // its reciprocal, to a rounding
{
    const float r = __builtin_amdgcn_rcpf(per);
    return __builtin_fmaf(r, __builtin_fmaf(-per, r, 1.f), r);
}

struct ValuesArgs {
    const uint8_t *val_codes;
    const void *val_cb;       // [Hkv][M][K][d] bf16 or fp32
    const int32_t *cu;
    const float *scores;
    const float2 *sstat;      // [B * Hq][nsplit] (max, sum of exp(logit - max)) of the score stage
    unsigned *bins;           // mode 1 writes, mode 2 reads: [B * Hkv][ranges][ncg][K][pairs][CB][2 heads]
    float *vscale, *lsum;     // [B * Hq][ranges]
    float *partial;           // [B * Hq][ranges][ncg][d]
    int Hq, Hkv, M;
    int nsplit, split_len;    // statistics tiles of the score stage
    int batch, ncg;
    Divisor by_hkv, by_ncg, by_batch, by_span;
    int split_shift;          // log2 split_len
    int ranges, range_len;    // token ranges of a sequence (S > 1: one)
    int span, spans;          // tokens of a range that share a fixed-point unit (S > 1: all); spans of a range
    int mode;                 // 0: everything; 1: up to the bins, which go to memory; 2: from there on
};

// x in whole units (numbers on [0, 2^32)): rounded to nearest, NaN to 0.
__device__ __forceinline__ unsigned whole_units(float x, float per)
{
    unsigned r;
    const float y = __builtin_fmaf(x, per, 0.5f);
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(y));        // (truncates; saturates, which C++ leaves open)
    return r;
}

// x + y after exchanging the odd 16-lane rows of x with the even rows of y (row r of the result:
// r even: x[r] + x[r+1], r odd: y[r-1] + y[r]), and the same with 32-lane halves.
__device__ __forceinline__ float swap16_add(float x, float y)
{
    auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float swap32_add(float x, float y)
{
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// Softmax(A) S_V of Eq. optimized_v and its product with the value codebook, without the bins' trip through memory.  A
// workgroup takes CB of the M value codebooks of a KV head, for a range of a sequence's tokens or (S > 1) for S whole
// sequences side by side, and leaves one unnormalised output row per head and range, which k_out_final adds.
//
// Bins.  w = exp(logit - max of the sequence) is added in whole units with integer LDS atomics.  The score stage has
// left the exp-sum l of every statistics tile; a unit of l / 2^32 (a little more: units_per_one), l of the tiles that a span of tokens touches,
// keeps every bin below 2^32 and the rounding below (tokens) 2^-33 of l.  A span is two value splits of the plan at most, so that
// weights are as fine as with a unit of l / 2^31 per split.  A range of several spans is added up in fp32 between them, each with its unit, and at
// its end made whole numbers once more: 0.8 us a span (three of them in a range at 32K, 32 codebooks: 55.7 -> 58.7 us a call, with one unit for the
// range), where ranges of one span would each read the codebook rows again.  (logit - max) is taken before the product with log2 e and the
// unit after the exponential: both in one sum of up to 32 took 4e-7 of a weight.  Error against 64 bits, codebooks of mean zero, one unit per range
// of 2^30 to 2^31 and one sum -> now: 32K of 8 x 4 heads 1.2e-6 -> 3.2e-7, 64K of 64 x 4 heads 7.7e-6 -> 1.5e-6 (a unit per split and
// one sum: 1.1e-6 and 2.4e-6).  Heads 2 p and 2 p + 1 share a 64-bit word (no carry crosses).  A 64-bit LDS
// atomic is served 16 lanes at a time, so a codeword's row is [copy][pair][codebook] with at least 16 words and
// lane l starts at (copy, pair, codebook) l mod 16 and walks pairs and codebooks by exclusive or: 16 lanes are on 16 bank pairs
// at every step, whatever their codes, and lanes with the same code do not meet either.
//
// Product.  The bins of CB codebooks are a (heads x CB K) x (CB K x d) matrix product.  A bin is an integer of four 8-bit
// digits, each exact in bf16, so that digit x head fill the 16 rows of v_mfma_f32_16x16x32_bf16 (4 heads; two tiles for 8) and
// the exact bins are multiplied, not their 24 leading bits; the digits' sums are scaled by 256^(digit - 4) at the end.  The
// wavefronts share the k-steps; a lane loads 16 bytes of 8 rows (256 bytes of a row per 16 lanes) and interleaves them in
// registers, column 8 n + t of lane n for tile t, so the codebook needs no other layout.  fp32 rows are multiplied by vector
// instructions, four columns per lane.
//
// What bounds it, by clocks at the phases' ends, 128K tokens of the 8B layer at 16 codebooks (16 us in the workgroups of 20.4 under the
// tracer, the rest is its launch and end; 20.9 while the score kernels left 17 MB of logits dirty in the L2s, which they now write
// through): 2 until the first token is worked on, 10.8 for the tokens (the atomics alone are
// 7.3 at 8.2 lanes a clock, the vector instructions of four wavefronts as much), 0.4 for the copies' sums, 1.3 for the rows of the product,
// 1.2 for the digits and 0.5 for the wavefronts' sums.  The statistics are asked for before the sequence's length is known and ahead of
// the tokens, and the workgroup's indices take no division: with both behind the length the phase before the tokens was 3.1 us (whole
// calls, with the same change to k_out_final: 8B 2-bit 1237 tokens 19.8 -> 18.5, 1-bit 128K 86.6 -> 84.3, position-free 36.8 -> 34.3, one
// fp32 head of 4096 tokens 16.9 -> 15.0).  The bins' way through memory
// that it replaces (16 MB out of one kernel and into the next at that size, 67 MB for 64 chats) and one launch less, whole call:
// one fp32 head of 4096 tokens 23.9 -> 19.8 us; 8B 2-bit 1237 tokens 31.1 -> 24.8, 32K 69.8 -> 56.9, 8 x 8K..64K 483 -> 469, 64 x
// 512..1024 136 -> 118; 8B 1-bit 128K 92.8 -> 88.6, position-free 39.5 -> 36.0; 70B 4 x 128K 559 -> 553.  Not kept: equal chunks of the whole batch
// instead of ranges per sequence (more products: 8 x 8K..64K 456 -> 480), rows touched early to have them in L2 (no change, with
// codebooks that were there from the call before).  Eight heads with 8 codebooks take the k-steps in
// a loop: unrolled, the sums move from register to register and 9 of them spill (4 x 128K 498.5 -> 494.7 us, 6 x 15000..30000 152.8 -> 150.2, 40 x
// 1500..3000 184.1 -> 179.5).
template <int G, int CB, int S, int NCS, int NT, bool BF16>
__global__ __launch_bounds__(NT, S > 1 ? 2 : 4) void k_values(const ValuesArgs a)
{
    constexpr int NP = G >= 2 ? G / 2 : 1;                 // head pairs, a 64-bit word each
    constexpr int WORDS = values_words<G, CB, S>(), ROWB = WORDS * 8, SLOT = values_slot<G, CB, S>(), COPIES = WORDS / (NP * CB);
    constexpr int PX = CB * COPIES < 16 ? 16 / (CB * COPIES) : 1;  // pairs that the lanes walk by exclusive or; the others are offsets
    static_assert((ROWB == 128 || ROWB == 256) && (CB == 4 || CB == 8), "rows of bins of one or half an LDS bank row");
    static_assert(BF16 || S == 1, "fp32 rows: one slot");
    constexpr int CD = CB / 4;                             // code dwords of a token
    constexpr int NW = NT / 64;
    constexpr int KS = CB * kK / 32 / NW;                  // k-steps of a wavefront
    constexpr int NX = (G + 3) / 4;                        // first-operand tiles: 4 heads x 4 digits
    constexpr int COLS = kD / NCS, NCT = COLS / 16;        // columns of the workgroup, tiles of 16
    constexpr int ND = NCT / 2;                            // dwords of a codebook row that a lane loads
    constexpr int DEPTH = S == 1 ? (CB * NP <= 8 ? 4 : 2) : S == 2 ? 2 : 1;  // tokens whose codes and logits are in flight, per slot
    extern __shared__ __attribute__((aligned(128))) unsigned char lds[];
    constexpr int ROW = NP * CB;                           // words of a row of bins without copies
    constexpr bool SPANS = S == 1 && !(CB == 8 && NT == 512);  // (value_shape: these have one)
    const int spans = SPANS ? a.spans : 1;
    float2 *const sums = reinterpret_cast<float2 *>(lds + values_bins<G, CB, S, NCS, NT>());
    float *const max_s = reinterpret_cast<float *>(sums) + (spans > 1 ? 2 * kK * ROW : 0);  // maximum of the sequence
    float *const unit_s = max_s + S * G, *const per_s = unit_s + S * G;  // the last bins' unit, units per 1
    float *const span_s = per_s + S * G, *const own_s = span_s + spans * S * G;  // [span] units per 1; exp-sum
    float *red = reinterpret_cast<float *>(lds);           // [NW][S][G][COLS]

    const int id0 = blockIdx.x, id1 = quotient(id0, a.by_hkv), id2 = quotient(id1, a.by_ncg);
    const int g = id0 - id1 * a.Hkv;                       // (head = index mod Hkv: with 8 KV heads an XCD serves one head)
    const int cg = id1 - id2 * a.ncg;
    const int cs = id2 % NCS, grp = id2 / NCS;
    const int rng = S == 1 ? quotient(grp, a.by_batch) : 0, b0 = S == 1 ? grp - rng * a.batch : grp * S;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // The statistics that the wavefront looks at first are asked for before anything that takes the sequence's length (which
    // is on its way meanwhile), as many as a sequence of the longest length has.
    const int first = rng * a.range_len;                   // first token (S > 1: 0)
    auto job_stats = [&](int job, int &v0) -> const float2 * __attribute__((always_inline)) {
        v0 = first + (SPANS ? job / (S * G) * a.span : 0);
        return a.sstat + ((size_t)min(b0 + job / G % S, a.batch - 1) * a.Hq + (size_t)g * G + job % G) * a.nsplit;
    };
    RangeStats stats;
    if (a.mode != 2 && wave < spans * (S * G)) {
        int v0;
        const float2 *st = job_stats(wave, v0);
        stats.request(st, a.nsplit, v0 >> a.split_shift, min((v0 + a.span + a.split_len - 1) >> a.split_shift, a.nsplit), lane);
    }
    __builtin_amdgcn_sched_barrier(0);

    const int mshift = a.M == 32 ? 5 : 4;                  // (16 or 32 codebooks)
    int sb[S], sv0[S], sv1[S], sL[S], scu[S];              // sequence, first and last token + 1, length, offset of the slots
    bool any = false;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int b = b0 + s;
        sb[s] = b < a.batch ? b : 0;
        scu[s] = a.cu[sb[s]];
        sL[s] = a.cu[sb[s] + 1] - scu[s];
        sv0[s] = first;
        sv1[s] = S == 1 ? min(sv0[s] + a.range_len, sL[s]) : b < a.batch ? sL[s] : 0;
        any |= sv0[s] < sv1[s];
    }
    if (!any) return;

    // the first tokens' codes and logits
    // (buffer loads: one offset per lane, reads past the sequence return zeros)
    unsigned cnext[S][DEPTH][CD];
    float snext[S][DEPTH][G];
    auto fetch = [&](int s, int d, int t) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t codes = make_rsrc(a.val_codes + ((size_t)scu[s] * a.Hkv + (size_t)g * sL[s]) * a.M, (unsigned)sL[s] * (unsigned)a.M);
        const __amdgpu_buffer_rsrc_t rows = make_rsrc(a.scores + (size_t)scu[s] * a.Hq + (size_t)g * G * sL[s], (unsigned)sL[s] * (unsigned)(G * 4));
        const unsigned i = (unsigned)(t + tid), at = i << mshift;
        if constexpr (CD == 1) {
            cnext[s][d][0] = __builtin_amdgcn_raw_buffer_load_b32(codes, at, (unsigned)(cg * CB), 0);
        } else {
            const uint2_t c = __builtin_amdgcn_raw_buffer_load_b64(codes, at, (unsigned)(cg * CB), 0);
            cnext[s][d][0] = c[0];
            cnext[s][d][1] = c[1];
        }
#pragma unroll
        for (int hh = 0; hh < G; ++hh)
            snext[s][d][hh] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, i * 4u, (unsigned)(hh * 4) * (unsigned)sL[s], 0));
    };
    if (a.mode != 2) {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int d = 0; d < DEPTH; ++d)
                if (sv0[s] + d * NT < sv1[s]) fetch(s, d, sv0[s] + d * NT);
    }
    for (int x = tid; x < S * SLOT / 16; x += NT) reinterpret_cast<uint4 *>(lds)[x] = make_uint4(0u, 0u, 0u, 0u);

    // (maximum of the sequence, exp-sum) of every span, slot and head
    const int live = spans > 1 ? quotient(sv1[0] - sv0[0] + a.span - 1, a.by_span) : 1;  // spans that have tokens
    for (int job = wave; job < live * (S * G); job += NW) {
        const int s = job / G % S, hh = job % G, span = job / (S * G);
        int b = 0, v0 = 0, v1 = 0, L = 0;
#pragma unroll
        for (int k = 0; k < S; ++k)
            if (s == k) { b = sb[k]; v0 = sv0[k]; v1 = sv1[k]; L = sL[k]; }
        if (v0 >= v1) continue;
        const float2 *st = job_stats(job, v0);
        if constexpr (SPANS) v1 = min(v1, v0 + a.span);
        const size_t at = ((size_t)b * a.Hq + (size_t)g * G + hh) * a.ranges + rng;
        if (a.mode == 2) {
            if (lane == 0 && span == 0) unit_s[job] = a.vscale[at];
            continue;
        }
        const int ns = min((L + a.split_len - 1) >> a.split_shift, a.nsplit);
        // the exp-sum l of all tiles that the span touches bounds every bin; what it reports towards the softmax denominator is lown
        const int ta = v0 >> a.split_shift, tb = min((v1 + a.split_len - 1) >> a.split_shift, ns);
        if (job != wave) stats.request(st, ns, ta, tb, lane);
        float mx, l, lown;
        stats.finish(st, ns, ta, tb, a.split_len, v0, lane, mx, l, lown);
        if (lane == 0) {
            const float per = units_per_one(l, v1 - v0, 0x1p-14f);
            span_s[job] = per;
            own_s[job] = lown;
            if (span == 0) max_s[job] = mx;
            if (live == 1) {
                unit_s[job] = unit_of(per);
                if (cg == 0 && cs == 0) {
                    a.lsum[at] = lown;
                    if (a.mode == 1) a.vscale[at] = unit_of(per);
                }
            }
        }
    }
    __syncthreads();
    if (SPANS && live > 1 && a.mode != 2 && tid < G) {    // of the whole range
        float own = 0.f, all = 0.f;
        for (int k = 0; k < live; ++k) {
            const float per = span_s[k * G + tid];
            own += own_s[k * G + tid];
            all += per == 1.f ? 0.f : (4294967296.f * (1.f - 0x1p-14f)) * unit_of(per);  // (no less than the span's exp-sum; 1: nothing in it rounds to a unit)
        }
        const float per = units_per_one(all, sv1[0] - sv0[0], 0x1p-13f);
        per_s[tid] = per;
        unit_s[tid] = unit_of(per);
        if (cg == 0 && cs == 0) {
            const size_t at = ((size_t)sb[0] * a.Hq + (size_t)g * G + tid) * a.ranges + rng;
            a.lsum[at] = own;
            if (a.mode == 1) a.vscale[at] = unit_of(per);
        }
    }

    // the wavefront's codebook rows, k-step by k-step: the first ones travel while the tokens are worked on
    // (addresses: a uniform base per codebook and k-step, one offset per lane)
    const char *cb0 = static_cast<const char *>(a.val_cb) + (((size_t)g * a.M + (size_t)cg * CB) * (size_t)(kK * kD) + cs * COLS) * 2;
    constexpr int RB = S * NX == 1 ? 2 : 1;            // k-steps whose rows are in flight
    constexpr int CL = 8 / CB;                         // codewords of a lane's eight rows
    unsigned R[RB][8][ND];
    auto load_rows = [&](int j, unsigned(&r)[8][ND]) __attribute__((always_inline)) {
        const int ln = fresh_lane();
        const unsigned off = (unsigned)((ln >> 4) * CL * kD + (ln & 15) * NCT) * 2u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int code = (wave * KS + j) * (32 / CB) + e / CB, cb = e % CB;
            const unsigned *p = reinterpret_cast<const unsigned *>(cb0 + (size_t)(cb * kK + code) * (size_t)(kD * 2) + off);
            if constexpr (ND == 4) {
                typedef unsigned u4u __attribute__((ext_vector_type(4), aligned(4)));  // (the caller's codebook: any alignment that its elements have)
                const u4u v = *reinterpret_cast<const u4u *>(p);
                r[e][0] = v[0]; r[e][1] = v[1]; r[e][2] = v[2]; r[e][3] = v[3];
            } else {
                static_assert(ND == 4 || ND == 1, "16 or 4 bytes of a row");
                r[e][0] = p[0];
            }
        }
    };
    __builtin_amdgcn_sched_barrier(0);
    if (BF16 && a.mode != 1) load_rows(0, R[0]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");

    typedef __attribute__((address_space(3))) unsigned long long *lds_u64_ptr;  // (dynamic LDS begins at LDS address 0: there is no other)
    if (a.mode != 2) {
        const int cbl = lane & (CB - 1);                   // codebook of step k: cbl ^ k
        const int copy = lane / CB % COPIES;
        const int pr = lane / (CB * COPIES) % PX;          // pair of step kp: kp ^ pr
        unsigned sel[CD];                              // byte selectors: the codes in the order of the steps
#pragma unroll
        for (int v = 0; v < CD; ++v) {
            sel[v] = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) sel[v] |= (unsigned)(cbl ^ (4 * v + j)) << (8 * j);
        }
        const unsigned lanepart = (unsigned)(copy * NP * CB + pr * CB + cbl) * 8u;
        auto copies_sum = [&](int x) __attribute__((always_inline)) {  // (no carry between the halves: their sums stay below 2^32)
            const unsigned long long *row = reinterpret_cast<const unsigned long long *>(lds) + x / ROW * WORDS + x % ROW;
            unsigned long long v = 0;
#pragma unroll
            for (int k = 0; k < COPIES; ++k) v += row[((k + x / ROW) & (COPIES - 1)) * ROW];  // (neighbouring rows on different banks)
            return v;
        };
        // what to do with the sums of the spans up to this one, word by word of the first slot, a few of the thread's at a time (NT is a
        // multiple of ROW: they are of two heads)
        constexpr int OWN = kK * ROW / NT, AT_ONCE = OWN < 4 ? OWN : G == 8 ? 2 : 4;
        const int head0 = tid % ROW / CB * 2, head1 = min(head0 + 1, G - 1);
        auto add_span = [&](int span, auto put) __attribute__((always_inline)) {
            const float unit0 = unit_of(span_s[span * G + head0]), unit1 = unit_of(span_s[span * G + head1]);
#pragma unroll 1
            for (int x0 = tid; x0 < kK * ROW; x0 += AT_ONCE * NT) {
                uint2_t v[AT_ONCE];
                float2 t[AT_ONCE];
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) {
                    v[i] = __builtin_bit_cast(uint2_t, copies_sum(x0 + i * NT));
                    t[i] = span > 0 ? sums[x0 + i * NT] : make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i)
                    put(x0 + i * NT, make_float2(__builtin_fmaf((float)v[i][0], unit0, t[i].x), __builtin_fmaf((float)v[i][1], unit1, t[i].y)));
            }
        };
        auto next_span = [&](int span) __attribute__((always_inline)) {  // the bins to the sums, and empty for the next span
            // (This barrier stands at the head of the loop; the compiler has left out its own wait there, with atomics of the
            // iteration before under way.)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();
            add_span(span, [&](int x, float2 t) __attribute__((always_inline)) {
                sums[x] = t;
#pragma unroll
                for (int k = 0; k < COPIES; ++k)           // (in copies_sum's order)
                    reinterpret_cast<unsigned long long *>(lds)[x / ROW * WORDS + x % ROW + ((k + x / ROW) & (COPIES - 1)) * ROW] = 0;
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();
        };
        auto uniform = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); };
#pragma unroll
        for (int s = 0; s < S; ++s) {
            unsigned lane_k[CB];
#pragma unroll
            for (int k = 0; k < CB; ++k) lane_k[k] = (unsigned)(s * SLOT) + (lanepart ^ (unsigned)(k * 8));
            float mx[G], per[G];                           // (uniform)
#pragma unroll
            for (int hh = 0; hh < G; ++hh) {
                mx[hh] = uniform(max_s[s * G + hh]);
                per[hh] = uniform(span_s[s * G + hh]);
            }
            int span = 0, next = live > 1 ? sv0[s] + a.span : -1;  // (a span is a whole number of rounds of NT tokens)
            for (int t0 = sv0[s]; t0 < sv1[s]; t0 += DEPTH * NT) {
#pragma unroll
                for (int d = 0; d < DEPTH; ++d) {
                    const int t = t0 + d * NT;
                    if (t < sv1[s]) {
                        if (SPANS && t == next) {
                            next_span(span);
                            ++span;
                            next += a.span;
#pragma unroll
                            for (int hh = 0; hh < G; ++hh) per[hh] = uniform(span_s[span * G + hh]);
                        }
                        unsigned p[G], cw[CD];
#pragma unroll
                        for (int v = 0; v < CD; ++v) cw[v] = __builtin_amdgcn_perm(cnext[s][d][CD - 1], cnext[s][d][0], sel[v]);
#pragma unroll
                        for (int hh = 0; hh < G; ++hh)
                            p[hh] = whole_units(__builtin_amdgcn_exp2f((snext[s][d][hh] - mx[hh]) * kLog2e), per[hh]);
                        if (S == 1 || t + DEPTH * NT < sv1[s]) fetch(s, d, t + DEPTH * NT);
                        asm volatile("" ::: "memory");     // keeps the compiler from sinking the fetch below the atomics
                        unsigned long long pp[NP];
                        if (G == 1) {
                            pp[0] = p[0];
                        } else {
#pragma unroll
                            for (int hp = 0; hp < NP; ++hp) pp[hp] = (unsigned long long)p[(2 * hp) % G] | (unsigned long long)p[(2 * hp + 1) % G] << 32;
                        }
#pragma unroll
                        for (int st = 1; st < PX; st *= 2) {  // pp[kp] <- pp[kp ^ pr]
                            unsigned long long q[NP];
#pragma unroll
                            for (int hp = 0; hp < NP; ++hp) q[hp] = (pr & st) ? pp[hp ^ st] : pp[hp];
#pragma unroll
                            for (int hp = 0; hp < NP; ++hp) pp[hp] = q[hp];
                        }
                        if (t + tid < sv1[s]) {
#pragma unroll
                            for (int k = 0; k < CB; ++k) {
                                const unsigned c = (cw[k / 4] >> (8 * (k % 4))) & 0xffu;
                                const unsigned ad = ROWB == 256 ? __builtin_amdgcn_perm(cw[k / 4], lane_k[k], 0x03020000u | (unsigned)(4 + k % 4) << 8)
                                                                : (c << 7) | lane_k[k];
#pragma unroll
                                for (int hp = 0; hp < NP; ++hp)
                                    __hip_atomic_fetch_add(reinterpret_cast<lds_u64_ptr>((ad ^ (unsigned)(hp % PX * CB * 8)) + (unsigned)(hp / PX * PX * CB * 8)), pp[hp],
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();
        if (SPANS && live > 1) {                          // the spans' sums in whole units of the range
            const float per0 = per_s[head0], per1 = per_s[head1];
            add_span(live - 1, [&](int x, float2 t) __attribute__((always_inline)) {
                reinterpret_cast<unsigned long long *>(lds)[x / ROW * WORDS + x % ROW] =
                    (unsigned long long)whole_units(t.x, per0) | (unsigned long long)whole_units(t.y, per1) << 32;
            });
            __syncthreads();
        } else if constexpr (COPIES > 1) {                 // the copies' sums, in copy 0
            for (int x = tid; x < S * kK * ROW; x += NT) reinterpret_cast<unsigned long long *>(lds)[x / ROW * WORDS + x % ROW] = copies_sum(x);
            __syncthreads();
        }
    }
    if (a.mode != 0) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (sv0[s] >= sv1[s]) continue;
            // (one head: its half of the words only)
            const size_t first = ((((size_t)sb[s] * a.Hkv + g) * a.ranges + rng) * a.ncg + cg) * (size_t)(kK * ROW);
            unsigned long long *mem = reinterpret_cast<unsigned long long *>(a.bins) + first, *own = reinterpret_cast<unsigned long long *>(lds + s * SLOT);
            for (int x = tid; x < kK * ROW; x += NT) {
                unsigned long long *row = own + x / ROW * WORDS + x % ROW;
                if (a.mode == 1) {
                    if (cs == 0 && G == 1) a.bins[first + x] = (unsigned)row[0];
                    if (cs == 0 && G > 1) mem[x] = row[0];
                } else {
                    row[0] = G == 1 ? a.bins[first + x] : mem[x];
                }
            }
        }
        __syncthreads();
    }

    if (a.mode != 1) {
        if constexpr (BF16) {
            auto convert = [&](int s, int x, int ks) __attribute__((always_inline)) {
                const int ln = fresh_lane(), hh = 4 * x + (ln & 3);
                const unsigned dsh = (unsigned)(ln & 12) * 2u;  // the lane's digit of the weight
                const unsigned char *at = lds + s * SLOT + (ks * (32 / CB) + (ln >> 4) * CL) * ROWB + (hh >> 1) * (CB * 8) + (hh & 1) * 4;
                unsigned f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned v = *reinterpret_cast<const unsigned *>(at + e / CB * ROWB + e % CB * 8);
                    const float d = (float)((v >> dsh) & 0xffu);
                    f[e] = __builtin_bit_cast(unsigned, G % 4 != 0 && hh >= G ? 0.f : d);
                }
                uint4_t w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = __builtin_amdgcn_perm(f[2 * e + 1], f[2 * e], 0x07060302u);
                return __builtin_bit_cast(bf16x8_t, w);
            };
            __builtin_amdgcn_sched_barrier(0);
            floatx4_t acc[S][NX][NCT];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int x = 0; x < NX; ++x)
#pragma unroll
                    for (int t = 0; t < NCT; ++t) acc[s][x][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll NX == 2 && CB == 8 && S == 1 ? 1 : KS
            for (int j = 0; j < KS; ++j) {
                if (RB == 2 && j + 1 < KS) load_rows(j + 1, R[(j + 1) % RB]);
                bf16x8_t A[S][NX];
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        A[s][x] = convert(s, x, wave * KS + j);
                        if (S * NX > 1) __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                for (int t = 0; t < NCT; ++t) {
                    uint4_t w;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = __builtin_amdgcn_perm(R[j % RB][2 * e + 1][t / 2], R[j % RB][2 * e][t / 2], t & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
                    for (int s = 0; s < S; ++s)
#pragma unroll
                        for (int x = 0; x < NX; ++x)
                            acc[s][x][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[s][x], __builtin_bit_cast(bf16x8_t, w), acc[s][x][t], 0, 0, 0);
                    if (S * NX > 1) __builtin_amdgcn_sched_barrier(0);
                }
                if (RB == 1 && j + 1 < KS) load_rows(j + 1, R[0]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int ln = fresh_lane(), n = ln & 15, kg = ln >> 4;
            // digits combined: lane (n, kg) keeps head 4 x + kg of column NCT n + t.  (Bins as fractions of 2^32, so that no sum is larger than the
            // codebook's rows; a wavefront's own, of digits, overflow for codebooks beyond 5e33.)
            const float dscale = kg == 0 ? 0x1p-32f : kg == 1 ? 0x1p-24f : kg == 2 ? 0x1p-16f : 0x1p-8f;
            float sums[S][NX][NCT];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int x = 0; x < NX; ++x)
#pragma unroll
                    for (int t = 0; t < NCT; ++t) {
                        const floatx4_t v = acc[s][x][t] * dscale;
                        sums[s][x][t] = swap16_add(swap32_add(v[0], v[2]), swap32_add(v[1], v[3]));
                    }
            __syncthreads();                           // the bins have been read
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int x = 0; x < NX; ++x)
#pragma unroll
                    for (int t = 0; t < NCT; ++t)
                        if (4 * x + kg < G) red[((wave * S + s) * G + 4 * x + kg) * COLS + n * NCT + t] = sums[s][x][t];
        } else {
            // a lane takes four columns of every RPL-th row of the wavefront's share
            constexpr int LPR = COLS / 4, RPL = 64 / LPR, NR = CB * kK / NW;
            const int cl = lane % LPR, rl = lane / LPR;
            const float *rows = static_cast<const float *>(a.val_cb) + ((size_t)g * a.M + (size_t)cg * CB) * (size_t)(kK * kD) + cs * COLS + 4 * cl;
            float sum[G][4];
#pragma unroll
            for (int hh = 0; hh < G; ++hh)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[hh][e] = 0.f;
            typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
            auto row_at = [&](int r) __attribute__((always_inline)) { return *reinterpret_cast<const f4u *>(rows + (size_t)(wave * NR + r * RPL + rl) * kD); };
            auto add_row = [&](int r, const f4u &c) __attribute__((always_inline)) {
                const int row = wave * NR + r * RPL + rl, cb = row / kK, code = row % kK;
                const unsigned char *at = lds + code * ROWB + cb * 8;
#pragma unroll
                for (int hh = 0; hh < G; ++hh) {
                    const float w = (float)*reinterpret_cast<const unsigned *>(at + hh / 2 * (CB * 8) + (hh & 1) * 4) * 0x1p-32f;
                    sum[hh][0] += w * c.x; sum[hh][1] += w * c.y; sum[hh][2] += w * c.z; sum[hh][3] += w * c.w;
                }
            };
            if constexpr (G == 8 && NCS == 1) {
                // Sixteen rows asked for at once: left to itself the compiler orders this loop for six wavefronts on a SIMD (there are four), and
                // a wavefront waits for every row.  Whole calls in microseconds, so -> now: 16 x 8 heads, 40 sequences of 900 tokens 383.7 -> 353.4,
                // 2 x 8 heads, 40 of 16927 559 -> 520, 4 x 8 heads, 3 of 265 37.8 -> 26.5.  (Fewer heads, or a quarter of the columns a
                // workgroup: the loop is in that order already; eight at a time and a barrier 1 to 2 % slower.)
                constexpr int AT = 16;
                static_assert(NR / RPL % AT == 0, "whole groups of rows");
#pragma unroll 1
                for (int r = 0; r < NR / RPL; r += AT) {
                    f4u c[AT];
#pragma unroll
                    for (int k = 0; k < AT; ++k) c[k] = row_at(r + k);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < AT; ++k) add_row(r + k, c[k]);
                }
            } else {
#pragma unroll 8
                for (int r = 0; r < NR / RPL; ++r) add_row(r, row_at(r));
            }
#pragma unroll
            for (int m = LPR; m < 64; m *= 2)
#pragma unroll
                for (int hh = 0; hh < G; ++hh)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[hh][e] += __shfl_xor(sum[hh][e], m);
            __syncthreads();                           // the bins have been read
            if (rl == 0)
#pragma unroll
                for (int hh = 0; hh < G; ++hh)
                    *reinterpret_cast<float4 *>(red + (wave * G + hh) * COLS + 4 * cl) = make_float4(sum[hh][0], sum[hh][1], sum[hh][2], sum[hh][3]);
        }
        __syncthreads();
        // the wavefronts' sums
        for (int o = tid; o < S * G * COLS; o += NT) {
            const int s = o / (G * COLS), hh = o / COLS % G, col = o % COLS;
            int b = 0, v0 = 0, v1 = 0;
#pragma unroll
            for (int k = 0; k < S; ++k)
                if (s == k) { b = sb[k]; v0 = sv0[k]; v1 = sv1[k]; }
            if (v0 >= v1) continue;
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += red[w * (S * G * COLS) + o];
            a.partial[((((size_t)b * a.Hq + (size_t)g * G + hh) * a.ranges + rng) * a.ncg + cg) * kD + cs * COLS + col] = sum * (unit_s[s * G + hh] * 4294967296.f);
        }
    }
}

}  // namespace
