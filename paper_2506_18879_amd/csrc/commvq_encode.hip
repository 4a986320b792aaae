// libcommvq: key encoding for cache append (residual nearest-centre search), hand-written for gfx950.
#include "commvq_internal.hpp"

#include <algorithm>

namespace {

// ------------------------------------------------------------------ key encoding (cache append)
// Residual nearest-centre search (Sec. 4.2: the E step's assignment, level by level on the error of the
// previous levels; App. A.1 for the paired centres).  ||res - c||^2 = ||res||^2 - 2 res.c + ||c||^2, so a
// level needs the dot products of the residual with that level's rows and a table of squared norms:
//   norms[g][level][K]            ||C[g][level][c]||^2
//   cross[g][level][K][K]         paired only: 2 C[a] . (i C[b])   (K = 64), so that a paired centre costs
//                                 norms[a] + norms[b] + cross[a][b] - 2 (res.C[a] + res.(i C[b]))
template <bool BF16>
__global__ __launch_bounds__(256) void k_encode_tables(const void *__restrict__ cb, float *__restrict__ norms,
                                                       float *__restrict__ cross, int rows_total, int K, int paired)
{
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t < (size_t)rows_total) {
        float acc = 0.f;
        for (int e = 0; e < kD; ++e) {
            const float v = cb_elem<BF16>(cb, t * kD + e);
            acc = __builtin_fmaf(v, v, acc);
        }
        norms[t] = acc;
    }
    if (paired && t < (size_t)rows_total * K) {
        const size_t level = t / ((size_t)K * K);   // g * R + r
        const int a = (int)(t / K % K), b = (int)(t % K);
        const size_t ra = (level * K + a) * kD, rb = (level * K + b) * kD;
        float acc = 0.f;
        for (int j = 0; j < kJ; ++j) {  // (x_a, y_a) . (-y_b, x_b)
            const float xa = cb_elem<BF16>(cb, ra + 2 * j), ya = cb_elem<BF16>(cb, ra + 2 * j + 1);
            const float xb = cb_elem<BF16>(cb, rb + 2 * j), yb = cb_elem<BF16>(cb, rb + 2 * j + 1);
            acc = __builtin_fmaf(ya, xb, __builtin_fmaf(-xa, yb, acc));
        }
        cross[t] = 2.f * acc;
    }
}

// The lower of the minima that lanes l, l ^ 16, l ^ 32 and l ^ 48 hold, and its index (the lower one on ties): every one
// of the four lanes receives both.
__device__ __forceinline__ void min4(float &best, int &index)
{
    auto lower = [&](unsigned b0, unsigned b1, unsigned i0, unsigned i1) {
        const float f0 = __builtin_bit_cast(float, b0), f1 = __builtin_bit_cast(float, b1);
        const bool second = f1 < f0 || (f1 == f0 && (int)i1 < (int)i0);
        best = second ? f1 : f0;
        index = second ? (int)i1 : (int)i0;
    };
    unsigned b = __builtin_bit_cast(unsigned, best), i = (unsigned)index;
    auto b16 = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    auto i16 = __builtin_amdgcn_permlane16_swap(i, i, false, false);
    lower(b16[0], b16[1], i16[0], i16[1]);
    b = __builtin_bit_cast(unsigned, best);
    i = (unsigned)index;
    auto b32 = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    auto i32 = __builtin_amdgcn_permlane32_swap(i, i, false, false);
    lower(b32[0], b32[1], i32[0], i32[1]);
}

// The same over the two halves of a wavefront, lanes l and l ^ 32; returns which of them held it.
__device__ __forceinline__ bool min2_halves(float &best, int &index)
{
    const unsigned b = __builtin_bit_cast(unsigned, best), i = (unsigned)index;
    auto b32 = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    auto i32 = __builtin_amdgcn_permlane32_swap(i, i, false, false);
    const float f0 = __builtin_bit_cast(float, (unsigned)b32[0]), f1 = __builtin_bit_cast(float, (unsigned)b32[1]);
    const bool second = f1 < f0 || (f1 == f0 && (int)i32[1] < (int)i32[0]);
    best = second ? f1 : f0;
    index = second ? (int)i32[1] : (int)i32[0];
    return second;
}

// a token's largest and second largest value, from those of its lanes 16 (32) apart
__device__ __forceinline__ void two_largest(unsigned b0, unsigned b1, unsigned s0, unsigned s1, float &best, float &second)
{
    const float f0 = __builtin_bit_cast(float, b0), f1 = __builtin_bit_cast(float, b1);
    second = fmaxf(fminf(f0, f1), fmaxf(__builtin_bit_cast(float, s0), __builtin_bit_cast(float, s1)));
    best = fmaxf(f0, f1);
}
__device__ __forceinline__ void two_largest16(float &best, float &second)
{
    const unsigned b = __builtin_bit_cast(unsigned, best), s = __builtin_bit_cast(unsigned, second);
    const auto b16 = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    const auto s16 = __builtin_amdgcn_permlane16_swap(s, s, false, false);
    two_largest(b16[0], b16[1], s16[0], s16[1], best, second);
}
__device__ __forceinline__ void two_largest32(float &best, float &second)
{
    const unsigned b = __builtin_bit_cast(unsigned, best), s = __builtin_bit_cast(unsigned, second);
    const auto b32 = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    const auto s32 = __builtin_amdgcn_permlane32_swap(s, s, false, false);
    two_largest(b32[0], b32[1], s32[0], s32[1], best, second);
}
__device__ __forceinline__ float sum4(float v)  // over the four lanes of a token
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned w = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, (unsigned)r16[0]) + __builtin_bit_cast(float, (unsigned)r16[1]));
    const auto r32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return __builtin_bit_cast(float, (unsigned)r32[0]) + __builtin_bit_cast(float, (unsigned)r32[1]);
}
typedef float floatx2_t __attribute__((ext_vector_type(2)));
// The least of the 64 lanes' non-negative indices, in every lane.
__device__ __forceinline__ int wave_min_index(int v)
{
    auto other = [&](float f) { v = min(v, __builtin_bit_cast(int, f)); };
    other(dpp_mov<0xB1>(__builtin_bit_cast(float, v)));
    other(dpp_mov<0x4E>(__builtin_bit_cast(float, v)));
    other(dpp_mov<0x141>(__builtin_bit_cast(float, v)));
    other(dpp_mov<0x140>(__builtin_bit_cast(float, v)));
    auto r16 = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = min((int)r16[0], (int)r16[1]);
    auto r32 = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return min((int)r32[0], (int)r32[1]);
}

struct EncodeDims {
    int Hkv, levels, K, key_bf16, record_bytes;
    long long token_stride, head_stride;
};

// Index-form keys, fp32 codebooks: one workgroup per (token, KV head), one thread per centre of the level, rows
// straight from L2.  Ties go to the lowest index.  (bf16 codebooks: k_encode_rows below.)
__global__ __launch_bounds__(256) void k_encode(const void *__restrict__ keys, const float *__restrict__ cb,
                                                const float *__restrict__ norms, uint8_t *__restrict__ out, const EncodeDims a)
{
    __shared__ float res[kD];
    __shared__ float wbest[4];
    __shared__ int wcand[4];
    __shared__ int chosen[32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x % a.Hkv;
    const size_t tok = blockIdx.x / a.Hkv;
    const int K = a.K;  // 256 = the workgroup size
    if (tid < kD) {
        const size_t i = (tok * a.Hkv + g) * kD + tid;
        res[tid] = a.key_bf16 ? __builtin_bit_cast(float, (unsigned)static_cast<const uint16_t *>(keys)[i] << 16)
                              : static_cast<const float *>(keys)[i];
    }
    __syncthreads();
    for (int l = 0; l < a.levels; ++l) {
        const size_t level = (size_t)g * a.levels + l;
        const size_t base = level * K * kD;
        float acc = 0.f;
#pragma unroll 16
        for (int e = 0; e < kD; ++e) acc = __builtin_fmaf(res[e], cb[base + (size_t)tid * kD + e], acc);
        const float best = norms[level * K + tid] - 2.f * acc;
        // argmin over the workgroup, lowest index on ties
        const float wm = -wave_max(-best);
        int wc = best == wm ? tid : 0x7fffffff;
        for (int off = 32; off > 0; off >>= 1) wc = min(wc, __shfl_xor(wc, off));
        if (lane == 0) { wbest[wave] = wm; wcand[wave] = wc; }
        __syncthreads();
        float m = wbest[0];
        int c = wcand[0];
        for (int w = 1; w < 4; ++w)
            if (wbest[w] < m || (wbest[w] == m && wcand[w] < c)) { m = wbest[w]; c = wcand[w]; }
        c &= K - 1;  // no candidate if every distance is NaN: any row, but one of the codebook's
        if (tid == 0) chosen[l] = c;
        if (tid < kD) res[tid] -= cb[base + (size_t)c * kD + tid];
        __syncthreads();
    }
    if (tid < a.levels) out[tok * a.token_stride + (long long)g * a.head_stride + tid] = (uint8_t)chosen[tid];
}

// Index-form vectors, bf16 codebooks.  The dot products of a level are a (256 rows x 128) x (128 x tokens) matrix
// product, so they run on the matrix cores, for one token as for thousands.  The fp32 residual of a token is split
// EXACTLY into three bf16 parts (its 24 mantissa bits are 8 + 8 + 8: truncate, subtract, truncate, subtract), each
// multiplied with the exact bf16 rows and accumulated in fp32: the same dot product as an fp32 FMA chain up to
// summation order.
//   first operand : 16 rows x 32 elements from LDS
//   second operand: lane (n, g) supplies elements 32 kc + 8 g .. + 7 of token n, the part of the residual it keeps
//   result        : lane (n, g) receives rows 4 g .. 4 g + 3 of the row tile for token n
// The levels are a dependent chain, but the rows of level l + 1 do not depend on the residual: they travel from memory
// straight into LDS (16 bytes per lane, no register destination) while level l is searched, into the other half of a
// double buffer.  Piece x of row t sits in slot x xor (t mod 16) of its row: the operand reads are free of bank
// conflicts, and a load instruction (64 lanes -> 64 consecutive slots) still covers 1 KiB of contiguous memory.
// Eight wavefronts: 8 / RS sets of 16 tokens, the 256 rows of a level shared by the RS wavefronts of a set, which
// exchange their minima through LDS.  With a split and an update per wavefront instead of shared ones a level of RS = 8 (16 tokens) took
// 2.1 us instead of 1.5.  RS = 4 and 8 leave the sending to two wavefronts more: eight sends of every wavefront before it can
// go on held it up for as long as its products take (1000 tokens, 32 levels 75.6 -> 64 us, 500 tokens 52 -> 47.6, 16 levels 40.3 -> 34.2
// and 27.7 -> 25.1; RS = 2, whose level is longer: no change, so its wavefronts send for themselves).
// The images sit at LDS address 0: no static LDS here.
constexpr int er_threads(int rs) { return rs >= 4 ? 640 : 512; }
constexpr int kErImg = 16 * kK;  // 16-byte pieces of one level's rows
constexpr int kErNorms = 2 * kErImg * 16;              // [2][256] floats
constexpr int kErPart = kErNorms + 2 * kK * 4;         // [8 wavefronts][16 tokens] minimum and its row
constexpr int kErSplit = kErPart + 8 * 16 * 8;         // RS >= 4: [sets][3 parts][4 kc][64 lanes] operands of the token sets
constexpr int er_chosen(int rs) { return kErSplit + (rs >= 4 ? 8 / rs * 12 * 64 * 16 : 0); }  // [tokens][32 levels] bytes
constexpr int er_lds(int rs) { return er_chosen(rs) + 128 / rs * 32; }
static_assert(er_lds(2) <= 163840 && er_lds(4) <= 163840 && er_lds(8) <= 163840, "LDS of a compute unit");
template <int RS>
__global__ __launch_bounds__(er_threads(RS)) void k_encode_rows(const void *__restrict__ keys, const uint4 *__restrict__ cb,
                                                            const float *__restrict__ norms, uint8_t *__restrict__ out,
                                                            const EncodeDims a, int n_tokens)
{
    extern __shared__ __attribute__((aligned(16))) uint4 er_mem[];
    char *lds = reinterpret_cast<char *>(er_mem);
    uint8_t *chosen = reinterpret_cast<uint8_t *>(lds + er_chosen(RS));
    constexpr int kSets = 8 / RS, kTiles = 16 / RS;
    constexpr bool kSenders = RS >= 4;         // two wavefronts more, for the rows of the next level
    constexpr bool kShare = RS >= 4;           // the wavefronts of a set share the update and the split of its residuals
    constexpr int kOwn = kShare ? 32 / RS : 32;  // elements of its token that a lane keeps: from `own` of its 4 kc x 8
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, gk = lane >> 4;
    const int set = wave % kSets, rs = wave / kSets;
    const int own = kShare ? rs * kOwn : 0;
    uint4_t *split = reinterpret_cast<uint4_t *>(lds + kErSplit) + (kShare ? set * 12 * 64 : 0);
    const int g = blockIdx.x % a.Hkv;
    const int tl = set * 16 + n;  // token within the workgroup
    const long long tok = (long long)(blockIdx.x / a.Hkv) * (16 * kSets) + tl;
    const size_t tokc = (size_t)(tok < n_tokens ? tok : n_tokens - 1);
    const uint4 *rows = cb + (size_t)g * a.levels * kErImg;
    const float *nrows = norms + (size_t)g * a.levels * kK;
    auto send = [&](int l, int first, auto count) __attribute__((always_inline)) {  // an instruction: four rows
        const uint4 *src = rows + (size_t)l * kErImg;
#pragma unroll
        for (int i = 0; i < decltype(count)::value; ++i) {
            const int r0 = first + 4 * i, t = r0 + gk;
            lds_dma16(src, (unsigned)(t * 16 + ((lane ^ t) & 15)) * 16u, (unsigned)((l & 1) * kErImg + r0 * 16) * 16u);
        }
    };
    auto send_norms = [&](int l) { lds_dma16(nrows + (size_t)l * kK, (unsigned)lane * 16u, (unsigned)(kErNorms + (l & 1) * kK * 4)); };
    auto send_share = [&](int l) __attribute__((always_inline)) {  // RS = 2: a wavefront's share
        send(l, 32 * wave, std::integral_constant<int, 8>());
        if (wave == 0) send_norms(l);
    };
    if (kSenders && wave >= 8) {
        auto send_half = [&](int l, int half) __attribute__((always_inline)) {
            send(l, half * 128 + (wave - 8) * 64, std::integral_constant<int, 16>());
            if (half && wave == 8) send_norms(l);
        };
        send_half(0, 0);
        send_half(0, 1);
        for (int l = 0; l < a.levels; ++l) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // level l has landed
            __syncthreads();
            if (l + 1 < a.levels) send_half(l + 1, 0);
            __syncthreads();
            if (l + 1 < a.levels) send_half(l + 1, 1);
        }
        __syncthreads();
        return;
    }
    if (!kSenders) send_share(0);
    float res[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; i += 4) {  // elements 32 kc + 8 gk .. + 7 of the token, four at a time
        const int f = own + i;
        const size_t at = (tokc * a.Hkv + g) * kD + (f >> 3) * 32 + 8 * gk + (f & 7);
        if (a.key_bf16) {
            const uint2 v = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(keys) + at);
            res[i] = bf16_lo(v.x); res[i + 1] = bf16_hi(v.x);
            res[i + 2] = bf16_lo(v.y); res[i + 3] = bf16_hi(v.y);
        } else {
            const float4 v = *reinterpret_cast<const float4 *>(static_cast<const float *>(keys) + at);
            res[i] = v.x; res[i + 1] = v.y; res[i + 2] = v.z; res[i + 3] = v.w;
        }
    }
    for (int l = 0; l < a.levels; ++l) {
        const int buf = l & 1;
        const char *img = lds + buf * kErImg * 16;
        const float *nrm = reinterpret_cast<const float *>(lds + kErNorms) + buf * kK;
        // exact three-way bf16 split of the residuals, packed as MFMA operands
        unsigned mine[3][kOwn / 2];
#pragma unroll
        for (int i = 0; i < kOwn / 2; ++i) {
            float v0 = res[2 * i], v1 = res[2 * i + 1];
#pragma unroll
            for (int s3 = 0; s3 < 3; ++s3) {
                const unsigned u0 = __builtin_bit_cast(unsigned, v0), u1 = __builtin_bit_cast(unsigned, v1);
                mine[s3][i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);  // the upper halves
                v0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
                v1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
            }
        }
        if (kShare) {
#pragma unroll
            for (int s3 = 0; s3 < 3; ++s3) {
                uint4_t *dst = split + (s3 * 4 + (own >> 3)) * 64 + lane;
                if constexpr (RS == 4) *dst = uint4_t{mine[s3][0], mine[s3][1], mine[s3][2], mine[s3][3]};
                if constexpr (RS == 8) reinterpret_cast<uint2_t *>(dst)[rs & 1] = uint2_t{mine[s3][0], mine[s3][1]};
            }
        }
        if (!kSenders) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's rows of level l have landed
        __syncthreads();                                   // ... and everybody's; the other image is no longer read
        if (!kSenders && l + 1 < a.levels) send_share(l + 1);
        uint4_t part[3][4];
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                if constexpr (kShare) part[s3][kc] = split[(s3 * 4 + kc) * 64 + lane];
                else part[s3][kc] = uint4_t{mine[s3][4 * kc], mine[s3][4 * kc + 1], mine[s3][4 * kc + 2], mine[s3][4 * kc + 3]};
            }
        float best = INFINITY;
        int brow = 0;
#pragma unroll 2
        for (int t = 0; t < kTiles; ++t) {
            const int rt = rs * kTiles + t;
            floatx4_t D = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                const uint4 pc = *reinterpret_cast<const uint4 *>(img + (rt * 16 + n) * 256 + ((4 * kc + gk) ^ n) * 16);
                const uint4_t pv = {pc.x, pc.y, pc.z, pc.w};
                const bf16x8_t A = __builtin_bit_cast(bf16x8_t, pv);
#pragma unroll
                for (int s3 = 0; s3 < 3; ++s3) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, __builtin_bit_cast(bf16x8_t, part[s3][kc]), D, 0, 0, 0);
            }
            const float4 nr = *reinterpret_cast<const float4 *>(nrm + rt * 16 + 4 * gk);
            const float nv[4] = {nr.x, nr.y, nr.z, nr.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float sc = nv[r] - 2.f * D[r];
                if (sc < best) { best = sc; brow = rt * 16 + 4 * gk + r; }  // rows come in increasing order: ties keep the lowest
            }
        }
        min4(best, brow);  // the four lanes of a token hold the minima of disjoint row sets
        {  // ... and so do the RS wavefronts of a token set
            float2 *pm = reinterpret_cast<float2 *>(lds + kErPart);
            if (gk == 0) pm[wave * 16 + n] = make_float2(best, __builtin_bit_cast(float, brow));
            __syncthreads();
            float2 m = pm[set * 16 + n];
#pragma unroll
            for (int w = 1; w < RS; ++w) {
                const float2 o = pm[(w * kSets + set) * 16 + n];
                if (o.x < m.x) m = o;  // rows come in increasing order
            }
            brow = __builtin_bit_cast(int, m.y);
        }
        if (gk == 0 && rs == 0) chosen[tl * 32 + l] = (uint8_t)brow;
        // residual -= chosen row (the lane's elements of it)
#pragma unroll
        for (int i = 0; i < kOwn; i += 4) {
            const int f = own + i;
            const uint2 w = *reinterpret_cast<const uint2 *>(img + brow * 256 + ((4 * (f >> 3) + gk) ^ (brow & 15)) * 16 + (f & 4) * 2);
            res[i] -= bf16_lo(w.x); res[i + 1] -= bf16_hi(w.x);
            res[i + 2] -= bf16_lo(w.y); res[i + 3] -= bf16_hi(w.y);
        }
    }
    __syncthreads();
    if (tok < n_tokens && rs == 0) {
        uint8_t *dst = out + tok * a.token_stride + (long long)g * a.head_stride;
        for (int l = gk; l < a.levels; l += 4) dst[l] = chosen[tl * 32 + l];
    }
}

// Index-form vectors, few at a time (a decode step appends one token per sequence): the matrix product of k_encode_rows, shaped
// for the latency of a level, since the levels are a dependent chain.  The exact three-way split of up to five residuals is
// 15 columns of ONE second operand, so a level costs a wavefront (32 of the 256 rows) 8 matrix instructions and 12 operand
// reads of LDS, where k_encode_rows<8> takes a part after the other: 24 and 20; the sums of a token's three parts are added by
// two row shifts.  Two more wavefronts do nothing but send the next level's rows (64 KiB, memory -> LDS): 8 sends of every
// wavefront in a row hold it up for as long as its products take.
// Per level: products, minimum over a lane's 8 rows, the 32 minima of a token through LDS; then wavefront w < 5 (two elements of
// token w's residual a lane) finds the least, subtracts the row and leaves the parts of the next level's operand.
// Second operand: lane (n, g) supplies elements 32 kc + 8 g .. + 7 of column n; piece s = 4 kc + g of column n sits in slot n xor s
// of 16, so that neither the reads nor the writes of a token's 64 lanes collide.  The images sit at LDS address 0.
// What bounds it: the rows' way into one compute unit's LDS, 64 KiB in 0.95 us.  64 vectors, 16 levels, codebook in the L2: 18.2 us
// (k_encode_rows<8> 24.8; rows sent by the eight wavefronts themselves 22.5; loaded into registers straight from memory in operand order,
// 64 cache lines an instruction, 38), 32 levels 33.8 (47.2).  Up to 160 tokens of 8 heads (one round of workgroups): 37.1 (48.4).
// The codebook of a layer is seldom in the L2 when its turn comes, and a level from the last-level cache takes 0.25 us more.  So where the
// launch leaves compute units idle, they get workgroups that read a word of every cache line of the levels to come: 22.3 -> 18.9 (in the
// L2 already: 18.4 -> 18.9).  A head's have the head's place in the numbering, with 8 or 16 heads that is the same L2.  Asked for by the
// workgroups that need them, the same words stand in the way of the rows: 26.
constexpr int kFewTok = 5, kFewThreads = 640;
constexpr int kFewParts = 2 * kErImg * 16;             // [16 pieces][16 slots] 16 bytes
constexpr int kFewMin = kFewParts + 16 * 16 * 16;      // [5 tokens][8 wavefronts][4] least cost of 8 rows, its row, the second least
constexpr int kFewTop = kFewMin + kFewTok * 32 * 16;   // [2] the largest |c|^2 of a level and its root
constexpr int kFewLds = kFewTop + 2 * 8;
static_assert(kFewLds <= 163840, "LDS of a compute unit");
__global__ __launch_bounds__(kFewThreads) void k_encode_few(const void *__restrict__ keys, const uint4 *__restrict__ cb,
                                                            const float *__restrict__ norms, uint8_t *__restrict__ out,
                                                            const EncodeDims a, int n_tokens, int workers)
{
    extern __shared__ __attribute__((aligned(16))) uint4 few_mem[];
    char *lds = reinterpret_cast<char *>(few_mem);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, gk = lane >> 4;
    const int g = blockIdx.x % a.Hkv;
    const uint4 *rows = cb + (size_t)g * a.levels * kErImg;
    const float4 *all_norms = reinterpret_cast<const float4 *>(norms + (size_t)g * a.levels * kK);  // 64 a level
    if ((int)blockIdx.x >= workers) {                      // reads ahead: a word of each of a level's 512 + 8 cache lines
        for (int l = 1 + ((int)blockIdx.x - workers) / a.Hkv; l < a.levels; l += ((int)gridDim.x - workers) / a.Hkv) {
            const unsigned *line = tid < 512 ? reinterpret_cast<const unsigned *>(rows + (size_t)l * kErImg + 8 * tid)
                                             : reinterpret_cast<const unsigned *>(all_norms + l * 64 + 8 * ((tid - 512) & 7));
            const unsigned word = *line;
            asm volatile("" : : "v"(word));
        }
        return;
    }
    float2 *tops = reinterpret_cast<float2 *>(lds + kFewTop);
    if (wave >= 8) {                                       // the senders: slots as in k_encode_rows
        auto send = [&](int l, int half) __attribute__((always_inline)) {
            const uint4 *src = rows + (size_t)l * kErImg;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int r0 = half * 128 + (wave - 8) * 64 + 4 * i, t = r0 + gk;
                lds_dma16(src, (unsigned)(t * 16 + ((lane ^ t) & 15)) * 16u, (unsigned)((l & 1) * kErImg + r0 * 16) * 16u);
            }
        };
        float4 nq = all_norms[lane];
        send(0, 0);
        send(0, 1);
        for (int l = 0; l < a.levels; ++l) {
            const float top = wave_max(fmaxf(fmaxf(nq.x, nq.y), fmaxf(nq.z, nq.w)));  // of level l
            if (wave == 8 && lane == 0) tops[l & 1] = make_float2(top, __builtin_amdgcn_sqrtf(top + 1e-34f));  // (of level l - 2 nothing is read any more)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // level l has landed
            __syncthreads();
            nq = all_norms[(l + 1 < a.levels ? l + 1 : l) * 64 + lane];
            if (l + 1 < a.levels) send(l + 1, 0);
            __syncthreads();
            if (l + 1 < a.levels) send(l + 1, 1);
        }
        return;
    }
    const long long tok = (long long)(blockIdx.x / a.Hkv) * kFewTok + wave;  // the token whose residual the wavefront keeps
    const bool owner = wave < kFewTok;
    const float4 *nrows = all_norms + 8 * wave + gk;
    float4 next_norm[2] = {nrows[0], nrows[4]};
    float r0 = 0.f, r1 = 0.f;                              // elements 2 lane, 2 lane + 1
    if (owner && tok < n_tokens) {
        const size_t at = ((size_t)tok * a.Hkv + g) * kD + 2 * lane;
        if (a.key_bf16) {
            const uint16_t *k = static_cast<const uint16_t *>(keys) + at;
            r0 = __builtin_bit_cast(float, (unsigned)k[0] << 16);
            r1 = __builtin_bit_cast(float, (unsigned)k[1] << 16);
        } else {
            const float *k = static_cast<const float *>(keys) + at;
            r0 = k[0];
            r1 = k[1];
        }
    }
    auto put_parts = [&]() __attribute__((always_inline)) {
        const int piece = lane >> 2;
        float v0 = r0, v1 = r1;
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const unsigned u0 = __builtin_bit_cast(unsigned, v0), u1 = __builtin_bit_cast(unsigned, v1);
            reinterpret_cast<unsigned *>(lds + kFewParts)[(piece * 16 + ((3 * wave + s3) ^ piece)) * 4 + (lane & 3)] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
            v0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
            v1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
        }
    };
    float whole2 = wave_sum(r0 * r0 + r1 * r1) * 1.0001f + 1e-34f;  // at least the squared norm of the residual
    if (owner) put_parts();
    else if (wave == kFewTok && lane < 16) reinterpret_cast<uint4 *>(lds + kFewParts)[lane * 16 + (15 ^ lane)] = make_uint4(0u, 0u, 0u, 0u);
    unsigned keep = 0u;                                    // lane l: the row chosen in level l
    float4 *pm = reinterpret_cast<float4 *>(lds + kFewMin);
    for (int l = 0; l < a.levels; ++l) {
        const char *img = lds + (l & 1) * kErImg * 16;
        __syncthreads();                                   // the rows and the operand are there
        uint4_t A[2][4], B[4];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            B[kc] = *reinterpret_cast<const uint4_t *>(lds + kFewParts + ((4 * kc + gk) * 16 + (n ^ (4 * kc + gk))) * 16);
#pragma unroll
            for (int t = 0; t < 2; ++t) A[t][kc] = *reinterpret_cast<const uint4_t *>(img + (32 * wave + 16 * t + n) * 256 + ((4 * kc + gk) ^ n) * 16);
        }
        const float nv[2][4] = {{next_norm[0].x, next_norm[0].y, next_norm[0].z, next_norm[0].w}, {next_norm[1].x, next_norm[1].y, next_norm[1].z, next_norm[1].w}};
        floatx4_t D[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                D[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A[t][kc]), __builtin_bit_cast(bf16x8_t, B[kc]), D[t], 0, 0, 0);
        float best = INFINITY, second = INFINITY;
        int brow = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float d = D[t][r], dot = d + (dpp_mov<0x101>(d) + dpp_mov<0x102>(d));  // columns n + 1, n + 2: the smaller parts
                const float sc = nv[t][r] - 2.f * dot;
                second = __builtin_amdgcn_fmed3f(best, second, sc);
                if (sc < best) { best = sc; brow = 32 * wave + 16 * t + 4 * gk + r; }  // rows come in increasing order: ties keep the lowest
            }
        const int tk = n / 3;
        if (n < 15 && n == 3 * tk) pm[(tk * 8 + wave) * 4 + gk] = make_float4(best, __builtin_bit_cast(float, brow), second, 0.f);
        {
            const int next = l + 1 < a.levels ? l + 1 : l;
            next_norm[0] = nrows[next * (kK / 4)];
            next_norm[1] = nrows[next * (kK / 4) + 4];
        }
        __syncthreads();
        if (owner) {
            const float4 o = pm[wave * 32 + (lane & 31)];  // lanes 32 .. 63 as 0 .. 31
            const float2 longest = tops[l & 1];
            const float cc = longest.x, m = -wave_max(-o.x);
            const int win = __builtin_ctz((unsigned)__ballot(o.x == m) | 0x80000000u);
            const float up = -wave_max(-((lane & 31) == win ? o.z : o.x));  // (of two equal ones: the same again)
            int row = __builtin_amdgcn_readlane(__builtin_bit_cast(int, o.y), win);
            // The sums here and in k_encode_rows are of the same products: 5 and 12 roundings of at most |r| |c| each, twice in a
            // cost, and one of the cost itself.  If the second least cost is within what that can amount to for two rows, or
            // something overflows or is not a number, the row tiles of the candidates are taken again in the order of
            // k_encode_rows: its codes, bit for bit.
            // (The norms' product, not the root of their squares' product: that leaves the range of fp32 for rows and vectors of 2^-32 or 2^31.)
            const float rc = 1.01f * __builtin_amdgcn_sqrtf(whole2) * longest.y, bound = 9e-6f * rc + 5e-7f * cc;
            const float left = __builtin_fmaf(whole2, 1.000001f, m + 2.f * bound);  // |r - c|^2 = |r|^2 + (|c|^2 - 2 r c)
            whole2 = left < 1e-34f ? 1e-34f : left;        // (not fmaxf: NaN has to stay)
            // (A level of zeros, as whoever has fewer levels than the format fills it up, needs no second look: 32 of them, 8 tokens: 156 -> 34 us.)
            const bool zeros = cc == 0.f && m == 0.f && up == 0.f;
            if (__any(!((up - m > bound || zeros) && rc < 1e37f))) {
                uint4_t part[3][4];
#pragma unroll
                for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc)
                        part[s3][kc] = *reinterpret_cast<const uint4_t *>(lds + kFewParts + ((4 * kc + gk) * 16 + ((3 * wave + s3) ^ (4 * kc + gk))) * 16);
                unsigned tiles = 0u;
                const unsigned some = (unsigned)__ballot(!(o.x > m + bound));
                if (__any(!(rc < 1e37f)) || __builtin_popcount(some) > 12) {
                    tiles = 0xffffu;
                } else {                                   // a lane's 8 rows are of two tiles: both, if two of the rows are candidates.  (32 levels of 8 tokens,
                                                           // every row with a twin next to it: 54 us, with all tiles then 156; k_encode_rows<8> 47)
                    const unsigned both = (unsigned)__ballot(!(o.z > m + bound));
                    for (unsigned hold = some; hold; hold &= hold - 1) {
                        const int at = __builtin_ctz(hold), t = __builtin_amdgcn_readlane(__builtin_bit_cast(int, o.y), at) >> 4 & 15;
                        tiles |= both >> at & 1 ? 3u << (t & 14) : 1u << t;
                    }
                }
                float least = INFINITY;
                row = 0;
                while (tiles) {                            // two at a time; rows come in increasing order: ties keep the lowest
                    int t[2];
                    t[0] = __builtin_ctz(tiles);
                    tiles &= tiles - 1;
                    t[1] = tiles ? __builtin_ctz(tiles) : t[0];
                    tiles &= tiles - 1;
                    float4 nr[2];
                    floatx4_t E[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        nr[e] = all_norms[(unsigned)(l * 64 + 4 * t[e] + gk)];
                        E[e] = floatx4_t{0.f, 0.f, 0.f, 0.f};
                    }
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc) {
                        uint4_t x[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) x[e] = *reinterpret_cast<const uint4_t *>(img + (16 * t[e] + n) * 256 + ((4 * kc + gk) ^ n) * 16);
#pragma unroll
                        for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                            for (int e = 0; e < 2; ++e)
                                E[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[e]), __builtin_bit_cast(bf16x8_t, part[s3][kc]), E[e], 0, 0, 0);
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float ev[4] = {nr[e].x, nr[e].y, nr[e].z, nr[e].w};
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float sc = ev[r] - 2.f * E[e][r];
                            if (sc < least) { least = sc; row = 16 * t[e] + 4 * gk + r; }
                        }
                    }
                }
                min4(least, row);
                row = __builtin_amdgcn_readfirstlane(row);
            }
            keep = lane == l ? (unsigned)row : keep;
            const unsigned v = *reinterpret_cast<const unsigned *>(img + row * 256 + (((lane >> 2) ^ row) & 15) * 16 + (lane & 3) * 4);
            r0 -= bf16_lo(v);
            r1 -= bf16_hi(v);
            put_parts();
        }
    }
    if (owner && tok < n_tokens && lane < a.levels) out[tok * a.token_stride + (long long)g * a.head_stride + lane] = (uint8_t)keep;
}

// Index-form vectors, many at a time: the choices of k_encode_rows, 128 tokens per workgroup, from two thirds of its products.
// The third part of a residual decides next to nothing.  So the costs are screened with the first two (the second rounded
// instead of truncated), from -|c|^2 / 2 as the accumulator's start, and a row costs three vector instructions: its number
// goes into the last six bits of r c - |c|^2 / 2, and two medians keep the largest and the second largest.  What all that can
// be off by is bounded; where a token's second best is within the bound of its best (0.2 to 0.3 % of a Gaussian token's levels),
// the row tiles that hold its candidates are taken again exactly as k_encode_rows does.  The codes are the same, bit for bit.
// A level takes 7900 clk: the matrix unit needs 4200 of them (two wavefronts a SIMD, 128 products of 16 clk each; between
// two products of a wavefront there is room for two vector instructions, and they are placed so), the choice 700, the
// update 600, the split 650, the second look 700 on average.  4000 tokens, 8 heads, 32 levels: 136 us, with all three parts and
// the compiler's order 177 us.  The two wavefronts of a SIMD half a level apart (a barrier for each half) took 155: a
// wavefront by itself issues an instruction every 5 clk, and that bounds its products at 26 clk each.  Two workgroups of four
// wavefronts with an image each, 147.
// Where rows have twins (a trained codebook with merged codewords) the screen decides nothing.  A wavefront that has had to repeat every tile for five
// tokens, of one level or of several, takes the next 15 levels without a screen, and 31 after each further try.  Every row with a twin, 32 levels:
// 259 -> 165 us (all three parts throughout: 168); a tenth of the rows: 234 -> 183 (178).  The next residual is split without need in those levels:
// a branch around it costs the codebooks without twins 3 us.
constexpr int kManyThreads = 512, kManyTokens = 128;
constexpr int kManyNorms = 2 * kErImg * 16;              // [2][256] -|c|^2 / 2
constexpr int kManyWhole = kManyNorms + 2 * kK * 4;        // [2][256] |c|^2
constexpr int kManyTops = kManyWhole + 2 * kK * 4;         // [2][4] the largest |c|^2 / 2 of 64 rows
constexpr int kManyChosen = kManyTops + 2 * 4 * 4;         // [128 tokens][32 levels] bytes
constexpr int kManyLds = kManyChosen + kManyTokens * 32;
static_assert(kManyLds <= 163840, "LDS of a compute unit");
__global__ __launch_bounds__(kManyThreads, 2) void k_encode_many(const void *__restrict__ keys, const uint4 *__restrict__ cb,
                                                               const float *__restrict__ norms, uint8_t *__restrict__ out,
                                                               const EncodeDims a, int n_tokens)
{
    extern __shared__ __attribute__((aligned(16))) uint4 many_mem[];
    char *lds = reinterpret_cast<char *>(many_mem);
    uint8_t *chosen = reinterpret_cast<uint8_t *>(lds + kManyChosen);
    float *tops = reinterpret_cast<float *>(lds + kManyTops);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, gk = lane >> 4;
    const bool norms_too = wave < 4;                       // (these are through with a level's products first)
    const int g = blockIdx.x % a.Hkv;
    const int tl = wave * 16 + n;  // token within the workgroup
    const long long tok = (long long)(blockIdx.x / a.Hkv) * kManyTokens + tl;
    const size_t tokc = (size_t)(tok < n_tokens ? tok : n_tokens - 1);
    const uint4 *rows = cb + (size_t)g * a.levels * kErImg;
    const float *nrows = norms + (size_t)g * a.levels * kK;
    auto fetch_rows = [&](int l, int buf, int i) __attribute__((always_inline)) {  // rows 32 wave + 4 i .. + 3, slots as in k_encode_rows
        const int r0 = 32 * wave + 4 * i, t = r0 + gk;
        lds_dma16(rows + (size_t)l * kErImg, (unsigned)(t * 16 + ((lane ^ t) & 15)) * 16u, (unsigned)(buf * kErImg + r0 * 16) * 16u);
    };
    float norm = 0.f;
    auto put_norms = [&](int buf) __attribute__((always_inline)) {  // wavefronts 0 to 3
        const float half = 0.5f * norm, top = wave_max(half);
        reinterpret_cast<float *>(lds + kManyNorms)[buf * kK + tid] = -half;
        reinterpret_cast<float *>(lds + kManyWhole)[buf * kK + tid] = norm;
        if (lane == 0) tops[buf * 4 + wave] = top;
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) fetch_rows(0, 0, i);
    if (norms_too) {
        norm = nrows[tid];
        put_norms(0);
    }
    float res[32];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {  // elements 32 kc + 8 gk .. + 7 of the token
        const size_t at = (tokc * a.Hkv + g) * kD + 32 * kc + 8 * gk;
        if (a.key_bf16) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint2 v = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(keys) + at + 4 * i);
                res[8 * kc + 4 * i] = bf16_lo(v.x); res[8 * kc + 4 * i + 1] = bf16_hi(v.x);
                res[8 * kc + 4 * i + 2] = bf16_lo(v.y); res[8 * kc + 4 * i + 3] = bf16_hi(v.y);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float4 v = *reinterpret_cast<const float4 *>(static_cast<const float *>(keys) + at + 4 * i);
                res[8 * kc + 4 * i] = v.x; res[8 * kc + 4 * i + 1] = v.y; res[8 * kc + 4 * i + 2] = v.z; res[8 * kc + 4 * i + 3] = v.w;
            }
        }
    }
    uint4_t part[2][4];
    float third, whole2 = 0.f;  // the third part's norm and the squared norm of the residual are at most this
#pragma unroll
    for (int i = 0; i < 32; ++i) whole2 = __builtin_fmaf(res[i], res[i], whole2);
    whole2 = sum4(whole2) * 1.0001f + 1e-34f;
    auto split = [&]() __attribute__((always_inline)) {
        float rest2[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float v0 = res[2 * i], v1 = res[2 * i + 1];
            const unsigned u0 = __builtin_bit_cast(unsigned, v0), u1 = __builtin_bit_cast(unsigned, v1);
            const unsigned hi = __builtin_amdgcn_perm(u1, u0, 0x07060302u);  // the upper halves
            v0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
            v1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
            const floatx2_t rest = {v0, v1};
            const unsigned mid = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, bf16x2_t));
            rest2[0] = __builtin_fmaf(v0, v0, rest2[0]);
            rest2[1] = __builtin_fmaf(v1, v1, rest2[1]);
            part[0][i >> 2][i & 3] = hi;
            part[1][i >> 2][i & 3] = mid;
        }
        // what rounding to the second part leaves is at most 2^-8 of it; 1 % covers this sum's own rounding
        third = 0.00395f * __builtin_amdgcn_sqrtf(sum4(rest2[0] + rest2[1]) + 1e-34f);
    };
    split();
    const unsigned keep = opaque_sgpr(0xffffffc0u);
    const float inf = __builtin_bit_cast(float, opaque_sgpr(0x7f800000u));
    // Levels to come without a screen, how many when next it does not pay, and what tells: 4 for each near token of a screen that repeated
    // every tile, 1 less for each that did not.
    int plain = 0, stretch = 15, in_vain = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // level 0 has landed
    __syncthreads();
    for (int l = 0; l < a.levels; ++l) {
        const char *img = lds + (l & 1) * kErImg * 16;
        const float *nrm = reinterpret_cast<const float *>(lds + kManyNorms) + (l & 1) * kK;
        auto rows_of = [&](int t, int kc) __attribute__((always_inline)) {
            return *reinterpret_cast<const uint4_t *>(img + (t * 16 + n) * 256 + ((4 * kc + gk) ^ n) * 16);
        };
        auto mul = [&](const uint4_t &r, const uint4_t &x, const floatx4_t &d) __attribute__((always_inline)) {
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, r), __builtin_bit_cast(bf16x8_t, x), d, 0, 0, 0);
        };
        const int next = l + 1 < a.levels ? l + 1 : l;     // (the last level is sent once more, to nobody)
        norm = nrows[(unsigned)(next * kK + (tid & (kK - 1)))];
        int brow = 0;
        bool near = true;
        unsigned tiles = 0xffffu;
        const bool searched = plain > 0;
        if (searched) {
            --plain;
#pragma unroll
            for (int i = 0; i < 8; ++i) fetch_rows(next, (l + 1) & 1, i);
        } else {
            // multiply: two row tiles at a time, with the medians of the two before them between the matrix instructions
            uint4_t A[2][4][2];
            floatx4_t D[2][2], start[2];
            auto norms_of = [&](int t) __attribute__((always_inline)) { return *reinterpret_cast<const floatx4_t *>(nrm + t * 16 + 4 * gk); };
#pragma unroll
            for (int e = 0; e < 2; ++e) start[e] = norms_of(e);
#pragma unroll
            for (int kc = 0; kc < 4; ++kc)
#pragma unroll
                for (int e = 0; e < 2; ++e) A[0][kc][e] = rows_of(e, kc);
            float best = -INFINITY, second = -INFINITY, sc = 0.f;
#pragma unroll
            for (int t = 0; t <= 16; t += 2) {
                const int cur = (t >> 1) & 1, old = cur ^ 1;
#pragma unroll
                for (int m = 0; m < 16; ++m) {                 // a matrix instruction (16 clk), one or two vector ones, a read or none
                    const int st = m >> 1, kc = st >> 1, e = m & 1;
                    if (t < 16) D[cur][e] = mul(A[cur][kc][e], part[st & 1][kc], st == 0 ? start[e] : D[cur][e]);
                    if (t > 0)
#pragma unroll
                        for (int u = (24 * m) / 16; u < (24 * m + 24) / 16; ++u) {
                            const int i = u / 3;
                            const float d = D[old][i >> 2][i & 3];  // (a bit cast of the element itself would read element 0)
                            if (u % 3 == 0) sc = __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, d) & keep) | (unsigned)(4 * (t - 2) + i));
                            if (u % 3 == 1) second = __builtin_amdgcn_fmed3f(best, second, sc);
                            if (u % 3 == 2) best = __builtin_amdgcn_fmed3f(best, sc, inf);  // the larger one
                        }
                    if (t < 14) {
                        if (!(m & 1)) A[old][m >> 2][(m >> 1) & 1] = rows_of(t + 2 + ((m >> 1) & 1), m >> 2);
                        if (m == 3 || m == 5) start[(m >> 1) - 1] = norms_of(t + 2 + (m >> 1) - 1);
                    }
                    if (t < 16 && m == 7) fetch_rows(next, (l + 1) & 1, t >> 1);
                    if (t > 0) asm volatile("" : "+v"(best), "+v"(second), "+v"(sc));  // here, not where they are used
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (norms_too) put_norms((l + 1) & 1);
            const float4 t4 = *reinterpret_cast<const float4 *>(tops + (l & 1) * 4);
            // choose
            float lo = best, up = second;
            two_largest16(lo, up);
            two_largest32(lo, up);
            const unsigned long long who = __ballot(best == lo);  // one lane of the token's four
            const unsigned w0 = (unsigned)who >> n, w1 = (unsigned)(who >> 32) >> n;
            const int at = (int)(__builtin_bit_cast(unsigned, lo) & 63u);
            brow = (at >> 2) * 16 + 4 * (int)(((w0 >> 16) & 1u) + 2u * (w1 & 1u) + 3u * ((w1 >> 16) & 1u)) + (at & 3);
            // A cost is off by the third part, |r''| |c|; by the last six bits, 2^-17 of it; and by the roundings of the sums, 8 here
            // and 13 in k_encode_rows, of at most |c|^2 / 2 + |r| |c|.  Overflow and NaN fail a comparison.
            const float top = fmaxf(fmaxf(t4.x, t4.y), fmaxf(t4.z, t4.w)), cmax = __builtin_amdgcn_sqrtf(2.f * top + 1e-34f), rc = 1.01f * __builtin_amdgcn_sqrtf(whole2) * cmax;
            const float bound = 2.f * third * cmax + 1.6e-5f * fabsf(lo) + 7.7e-6f * (top + rc);
            const float left = __builtin_fmaf(whole2, 1.000001f, 4.f * bound - 2.f * lo);  // |r - c|^2 = |r|^2 - 2 (r c - |c|^2 / 2)
            whole2 = left < 1e-34f ? 1e-34f : left;            // (not fmaxf: NaN has to stay, and to fail the comparison below)
            near = !(lo - up > bound && rc < 1e37f);
            tiles = 0u;
            if (__any(near)) {
                // the row tiles that hold a near token's candidates: the lanes' best, or all tiles if a lane's second best is one too
                if (__any(near && !(second < lo - bound && rc < 1e37f))) {
                    tiles = 0xffffu;
                } else {
                    for (unsigned long long hold = __ballot(near && best >= lo - bound); hold; hold &= hold - 1)
                        tiles |= 1u << (__builtin_amdgcn_readlane(__builtin_bit_cast(int, best), __builtin_ctzll(hold)) >> 2 & 15);
                }
            }
            in_vain = tiles == 0xffffu ? in_vain + __builtin_popcountll(__ballot(near)) : max(in_vain - 1, 0);
            if (in_vain >= 20) {
                plain = stretch;
                stretch = 31;
            }
        }
        if (tiles) {
            uint4_t exact[3][4];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float v0 = res[2 * i], v1 = res[2 * i + 1];
#pragma unroll
                for (int s3 = 0; s3 < 3; ++s3) {
                    const unsigned u0 = __builtin_bit_cast(unsigned, v0), u1 = __builtin_bit_cast(unsigned, v1);
                    exact[s3][i >> 2][i & 3] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
                    v0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
                    v1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
                }
            }
            float least = INFINITY;
            int row = 0;
            auto take = [&](const int (&t)[2]) __attribute__((always_inline)) {  // two tiles; rows come in increasing order: ties keep the lowest
                floatx4_t nr[2], E[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    nr[e] = *reinterpret_cast<const floatx4_t *>(lds + kManyWhole + ((l & 1) * kK + t[e] * 16 + 4 * gk) * 4);
                    E[e] = floatx4_t{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int kc = 0; kc < 4; ++kc) {
                    const uint4_t r[2] = {rows_of(t[0], kc), rows_of(t[1], kc)};
#pragma unroll
                    for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                        for (int e = 0; e < 2; ++e) E[e] = mul(r[e], exact[s3][kc], E[e]);
                }
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float sc = nr[e][r] - 2.f * E[e][r];
                        if (sc < least) { least = sc; row = t[e] * 16 + 4 * gk + r; }
                    }
            };
            if (tiles == 0xffffu) {
#pragma unroll
                for (int e = 0; e < 16; e += 2) take({e, e + 1});
            } else {
                while (tiles) {
                    int t[2];
                    t[0] = __builtin_ctz(tiles);
                    tiles &= tiles - 1;
                    t[1] = tiles ? __builtin_ctz(tiles) : t[0];
                    tiles &= tiles - 1;
                    take(t);
                }
            }
            min4(least, row);
            brow = near ? row : brow;
            if (searched && norms_too) put_norms((l + 1) & 1);
        }
        if (gk == 0) chosen[tl * 32 + l] = (uint8_t)brow;
        // residual -= chosen row (the lane's elements of it)
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const uint4 w = *reinterpret_cast<const uint4 *>(img + brow * 256 + ((4 * kc + gk) ^ (brow & 15)) * 16);
            const unsigned ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                res[8 * kc + 2 * i] -= bf16_lo(ws[i]);
                res[8 * kc + 2 * i + 1] -= bf16_hi(ws[i]);
            }
        }
        split();
        if (searched && !plain) {
            whole2 = 0.f;
#pragma unroll
            for (int i = 0; i < 32; ++i) whole2 = __builtin_fmaf(res[i], res[i], whole2);
            whole2 = sum4(whole2) * 1.0001f + 1e-34f;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's rows of level l + 1 have landed
        __syncthreads();                                   // ... and everybody's, and level l is no longer read
    }
    if (tok < n_tokens) {
        uint8_t *dst = out + tok * a.token_stride + (long long)g * a.head_stride;
        for (int l = gk; l < a.levels; l += 4) dst[l] = chosen[tl * 32 + l];
    }
}

// Paired-format keys, many tokens at once.  A level is two sets of 64 dot products, P[a] = res . C[a] and
// Q[b] = res . (i C[b]), on the matrix cores with the exact split of k_encode_rows, and a scan of the 64 x 64 centres:
//   ||c_ab||^2 - 2 res . c_ab = U[a] + (V[b] + X[a][b]),  U = N[a] - 2 P[a],  V = N[b] - 2 Q[b]
// The scan is a minimum over b of V[b] + X[a][b] for every a and token.  The sums are matrix instructions too: for one a
// and 32 tokens, result[b][token] = V[b][token] + x0 * 1 + x1 * 1 + x2 * 1 with V in the accumulator operand and the exact
// bf16 parts of X[a][b] along k.  (Measured: one rounded addition of V and X while their exponents are within 2 of each
// other, otherwise up to a unit in the last place beside it.)  That is 1024 sums in 32 clk where vector adds take 64, and a cross term is read from LDS
// once for 32 tokens; what is left to the vector unit is half a three-way minimum per centre.
// Four wavefronts, one per SIMD: 4 / RS sets of 32 tokens.  The RS wavefronts of a set share the rows a of the scan (and
// compute only their part of P); residual, split and Q are each wavefront's own: handing them round through LDS, with
// eight wavefronts and the residuals split between two, cost more than it saved (8.9 us a level at RS = 1's sizes).
// A level takes 7.5 us with RS = 1 (128 tokens), 5.8 (2) and 4.9 (4), of which a row of the scan is 45 ns: two matrix
// instructions (64 clk) and 21 vector ones (90 clk) that hide in each other only where they alternate in the program, so
// the order is fixed below (left to the compiler: 90 ns).  32768 vectors, 21 levels: 160 us, 8192 vectors 103; with the
// scan's sums on the vector unit and cross terms read per 16 tokens 258 and 165.
//   32 x 32 operands: lane (n, h) supplies row / token n and elements 8 h .. + 7 of a chunk of 16 (scan: 4 h .. + 3 of 8)
//   32 x 32 result  : lane (n, h) receives, in register i, row 8 (i / 4) + 4 h + i % 4 for token n
// A level's tables do not depend on the residual: rows, cross terms and norms of the next level travel from memory straight into the other of
// two buffers while this one is searched; what is made of them (i C, the terms' parts) takes the place of the last level's.  Through registers
// they were 33 of 256 for the whole level, 16 of which spilled, and one LDS write more: keys at 21 levels and values at 16 of 4000
// tokens 247.6 -> 238.7 us, 300 tokens 137.6 -> 132.8; keys at 11 levels, 1000 tokens 93.7 -> 90.7, 2500 160.2 -> 154.4.  (Addresses made anew
// at every level instead of held: 244.1, 139.9, 94.7, 160.9.  512 registers: the compiler moves half of them to and fro, 314.)
// With a wait that the compiler had put into every level for the keys loaded ahead of them, and so for all of the next level's tables, 2 to 4 us
// more (300 tokens 130.8 -> 126.3, 1000 90.1 -> 87.6, 4000 235.6 -> 233.0); with the scan's operands read one row ahead instead of two another
// 7 at 4000 tokens (238.7 -> 231.7), 2 at 300.
constexpr int kEpThreads = 256;
constexpr int kEpImage = 64 * 256;                  // C and the cross terms, of two levels in turn: 64 rows of 256 bytes, 16-byte piece x of row t in
constexpr int kEpRows = 0;                          // slot x xor (t mod 16)
constexpr int kEpTurned = 2 * kEpImage;             // i C, likewise
constexpr int kEpParts = kEpTurned + kEpImage;      // [64 a][64 b] x0, x1, x2, 0 of the cross terms, 8 bytes each
constexpr int kEpCross = kEpParts + 4096 * 8;
constexpr int kEpNorms = kEpCross + 2 * kEpImage;   // [2][64]
constexpr int kEpMin = kEpNorms + 2 * 64 * 4;           // [4 wavefronts][32 tokens] minimum, its row and that row's U
constexpr int kEpChosen = kEpMin + 4 * 32 * 16;     // [tokens][32 levels][2]
constexpr int ep_lds(int rs) { return kEpChosen + 128 / rs * 64; }
static_assert(ep_lds(1) <= 163840, "LDS of a compute unit");
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef short shortx4_t __attribute__((ext_vector_type(4)));
template <int RS>
__global__ __launch_bounds__(kEpThreads, 2) void k_encode_pairs(const void *__restrict__ keys, const uint4 *__restrict__ cb,
                                                             const float *__restrict__ norms, const float *__restrict__ cross,
                                                             uint8_t *__restrict__ out, const EncodeDims a, int n_tokens)
{
    extern __shared__ __attribute__((aligned(16))) uint4 ep_mem[];
    char *lds = reinterpret_cast<char *>(ep_mem);
    uint8_t *chosen = reinterpret_cast<uint8_t *>(lds + kEpChosen);
    constexpr int kSets = 4 / RS, kTiles = RS == 1 ? 2 : 1, kPairs = 32 / RS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int set = wave % kSets, rs = wave / kSets;
    const int a0 = 64 / RS * rs;  // the wavefront's first row a; its tile of P begins at a0 & 32
    const int g = blockIdx.x % a.Hkv;
    float res[8][8];  // dimensions 16 kc + 8 h .. + 7
    const size_t tokc = (size_t)min((long long)(blockIdx.x / a.Hkv) * (32 * kSets) + set * 32 + n, (long long)n_tokens - 1);
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
        const size_t i = (tokc * a.Hkv + g) * kD + 16 * kc + 8 * h;
        if (a.key_bf16) {
            const uint4 v = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(keys) + i);
            const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) { res[kc][2 * e] = bf16_lo(w[e]); res[kc][2 * e + 1] = bf16_hi(w[e]); }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) res[kc][e] = static_cast<const float *>(keys)[i + e];
        }
    }
    auto fetch_level = [&](int l) {
        const size_t level = (size_t)g * a.levels + l;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int p0 = (wave * 4 + x) * 64, p = p0 + lane, t = p >> 4, at = (t * 16 + ((p ^ t) & 15)) * 16;
            lds_dma16(cb + level * 64 * 16, (unsigned)at, (unsigned)(kEpRows + (l & 1) * kEpImage + p0 * 16));
            lds_dma16(cross + level * 4096, (unsigned)at, (unsigned)(kEpCross + (l & 1) * kEpImage + p0 * 16));
        }
        if (wave == 0 && fresh_lane() < 16) lds_dma16(norms + level * 64, (unsigned)fresh_lane() * 16u, (unsigned)(kEpNorms + (l & 1) * 256));
    };
    auto park_level = [&](int l) {
        const char *rows = lds + kEpRows + (l & 1) * kEpImage, *terms = lds + kEpCross + (l & 1) * kEpImage;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int p = x * 256 + tid, t = p >> 4;
            const uint4 row = *reinterpret_cast<const uint4 *>(rows + p * 16);
            const unsigned w[4] = {row.x, row.y, row.z, row.w};
            unsigned r[4];  // (x, y) -> (-y, x)
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_alignbit(w[e], w[e], 16) ^ 0x8000u;
            *reinterpret_cast<uint4 *>(lds + kEpTurned + p * 16) = make_uint4(r[0], r[1], r[2], r[3]);
            const float4 term = *reinterpret_cast<const float4 *>(terms + (t * 16 + ((p ^ t) & 15)) * 16);
            const float xv[4] = {term.x, term.y, term.z, term.w};
            unsigned pr[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned u0 = __builtin_bit_cast(unsigned, xv[e]);
                const float v1 = xv[e] - __builtin_bit_cast(float, u0 & 0xffff0000u);
                const unsigned u1 = __builtin_bit_cast(unsigned, v1);
                const float v2 = v1 - __builtin_bit_cast(float, u1 & 0xffff0000u);
                pr[2 * e] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
                pr[2 * e + 1] = __builtin_bit_cast(unsigned, v2) >> 16;
            }
            uint4 *pd = reinterpret_cast<uint4 *>(lds + kEpParts + p * 32);
            pd[0] = make_uint4(pr[0], pr[1], pr[2], pr[3]);
            pd[1] = make_uint4(pr[4], pr[5], pr[6], pr[7]);
        }
    };
    // three ones along k in the lanes of the lower half, nothing in the upper: every cross term enters once
    const uint2_t ones_bits = h ? uint2_t{0u, 0u} : uint2_t{0x3f803f80u, 0x3f80u};
    const shortx4_t ones = __builtin_bit_cast(shortx4_t, ones_bits);
    fetch_level(0);
    // (the keys: the compiler would wait for them in the loop, in every level, and with them for what is on its way for the next)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    for (int l = 0; l < a.levels; ++l) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's part of the level has landed
        __syncthreads();                                   // ... and everybody's, and the previous level's tables are no longer read
        park_level(l);
        if (l + 1 < a.levels) fetch_level(l + 1);
        __syncthreads();
        const char *const img = lds + kEpRows + (l & 1) * kEpImage, *const terms = lds + kEpCross + (l & 1) * kEpImage;
        const float *const nrm = reinterpret_cast<const float *>(lds + kEpNorms + (l & 1) * 256);
        floatx16_t P[kTiles], V[2];
#pragma unroll
        for (int t = 0; t < kTiles; ++t) P[t] = floatx16_t{0.f};
        V[0] = V[1] = floatx16_t{0.f};
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) {
            uint4_t part[3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v0 = res[kc][2 * e], v1 = res[kc][2 * e + 1];
#pragma unroll
                for (int s3 = 0; s3 < 3; ++s3) {
                    const unsigned u0 = __builtin_bit_cast(unsigned, v0), u1 = __builtin_bit_cast(unsigned, v1);
                    part[s3][e] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);  // the upper halves
                    v0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
                    v1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
                }
            }
            bf16x8_t A[kTiles + 2];
#pragma unroll
            for (int t = 0; t < kTiles + 2; ++t) {
                const int row = (t < kTiles ? (RS == 1 ? 32 * t : (a0 & 32)) : 32 * (t - kTiles)) + n;
                const uint4 pc = *reinterpret_cast<const uint4 *>((t < kTiles ? img : lds + kEpTurned) + row * 256 + ((2 * kc + h) ^ (n & 15)) * 16);
                const uint4_t pv = {pc.x, pc.y, pc.z, pc.w};
                A[t] = __builtin_bit_cast(bf16x8_t, pv);
            }
#pragma unroll
            for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                for (int t = 0; t < kTiles + 2; ++t) {
                    floatx16_t &d = t < kTiles ? P[t] : V[t - kTiles];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t], __builtin_bit_cast(bf16x8_t, part[s3]), d, 0, 0, 0);
                }
        }
        float U[kPairs];  // of row a0 + 8 (i / 4) + 4 h + i % 4
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 nr = *reinterpret_cast<const float4 *>(nrm + 8 * q + 4 * h);
            const float nv[4] = {nr.x, nr.y, nr.z, nr.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) V[q >> 2][4 * (q & 3) + e] = nv[e] - 2.f * V[q >> 2][4 * (q & 3) + e];
        }
#pragma unroll
        for (int q = 0; q < kPairs / 4; ++q) {
            const float4 nr = *reinterpret_cast<const float4 *>(nrm + a0 + 8 * q + 4 * h);
            const float nv[4] = {nr.x, nr.y, nr.z, nr.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float p;
                if constexpr (RS == 1) p = P[q >> 2][4 * (q & 3) + e];
                else if constexpr (RS == 2) p = P[0][4 * q + e];
                else p = rs & 1 ? P[0][8 + 4 * q + e] : P[0][4 * q + e];
                U[4 * q + e] = nv[e] - 2.f * p;
            }
        }
        // stage one: the row a of the nearest centre.  The sums of a row are issued before the minimum of the row
        // before it is taken; a pair of rows (r, r + 4) gives each half of the wavefront one of them to finish.
        float best = INFINITY, ubest = U[0];  // (and the row's U)
        int bi = 0;
        {
            const uint2_t *xs = reinterpret_cast<const uint2_t *>(lds + kEpParts) + a0 * 64 + n;
            auto row_of = [](int k) { return 8 * (k >> 3) + ((k >> 1) & 3) + 4 * (k & 1); };  // k-th row in the order of the pairs
            // the minimum as the median with -inf: fminf of values that might be NaN is preceded by a quieting of each
            const float low = __builtin_bit_cast(float, opaque_sgpr(0xff800000u));
            auto least = [&](float x, float y) { return __builtin_amdgcn_fmed3f(x, y, low); };
            floatx16_t D[2][2];
            uint2_t x[2][2] = {{xs[0], xs[32]}, {xs[row_of(1) * 64], xs[row_of(1) * 64 + 32]}};  // (two rows ahead: the LDS takes longer than one)
            float half[2] = {0.f, 0.f}, m0 = 0.f, m1 = 0.f;
#pragma unroll
            for (int k = 0; k <= 2 * kPairs; ++k) {
                const int cur = k & 1, old = cur ^ 1;
                if (k < 2 * kPairs) D[cur][0] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(shortx4_t, x[cur][0]), ones, V[0], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (k > 0) {
                    m0 = least(D[old][0][0], D[old][0][1]);
#pragma unroll
                    for (int i = 2; i < 16; i += 2) m0 = fminf(fminf(m0, D[old][0][i]), D[old][0][i + 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (k < 2 * kPairs) {
                    D[cur][1] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(shortx4_t, x[cur][1]), ones, V[1], 0, 0, 0);
                    if (k + 2 < 2 * kPairs) { x[cur][0] = xs[row_of(k + 2) * 64]; x[cur][1] = xs[row_of(k + 2) * 64 + 32]; }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (k > 0) {
                    m1 = least(D[old][1][0], D[old][1][1]);
#pragma unroll
                    for (int i = 2; i < 16; i += 2) m1 = fminf(fminf(m1, D[old][1][i]), D[old][1][i + 1]);
                    half[old] = least(m0, m1);
                    if (!cur) {
                        const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, half[0]), __builtin_bit_cast(unsigned, half[1]), false, false);
                        const int i = (k >> 1) - 1;
                        const float sc = U[i] + least(__builtin_bit_cast(float, (unsigned)sw[0]), __builtin_bit_cast(float, (unsigned)sw[1]));
                        if (sc < best) { best = sc; bi = i; ubest = U[i]; }  // a lane's rows come in increasing order
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        int ca = a0 + 8 * (bi >> 2) + 4 * h + (bi & 3);
        {
            const bool second = min2_halves(best, ca);
            const auto u32 = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, ubest), __builtin_bit_cast(unsigned, ubest), false, false);
            ubest = __builtin_bit_cast(float, second ? (unsigned)u32[1] : (unsigned)u32[0]);
        }
        if (RS > 1) {
            float4 *pm = reinterpret_cast<float4 *>(lds + kEpMin);
            if (h == 0) pm[wave * 32 + n] = make_float4(best, __builtin_bit_cast(float, ca), ubest, 0.f);
            __syncthreads();
            float4 m = pm[set * 32 + n];
#pragma unroll
            for (int w = 1; w < RS; ++w) {
                const float4 o = pm[(w * kSets + set) * 32 + n];
                if (o.x < m.x) m = o;  // rows come in increasing order
            }
            ca = __builtin_bit_cast(int, m.y);
            ubest = m.z;
        }
        // stage two: the partner b of row ca, the lowest of those whose whole cost is the least.  (V + X alone would tell apart
        // costs that are equal in fp32, and give a vector another code than k_encode_one does; it would save 3 us of 179.)
        float bestb = INFINITY;
        int cb2 = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b0 = 32 * t + 8 * q + 4 * h;
                const float4 x4 = *reinterpret_cast<const float4 *>(terms + ca * 256 + (((b0 >> 2) ^ ca) & 15) * 16);
                const float xv[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sc = ubest + (V[t][4 * q + e] + xv[e]);
                    if (sc < bestb) { bestb = sc; cb2 = b0 + e; }
                }
            }
        min2_halves(bestb, cb2);
        if (h == 0 && rs == 0) { chosen[((set * 32 + n) * 32 + l) * 2] = (uint8_t)ca; chosen[((set * 32 + n) * 32 + l) * 2 + 1] = (uint8_t)cb2; }
        // residual -= C[a] + i C[b]
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) {
            const int piece = 2 * kc + h;
            const uint4 pa = *reinterpret_cast<const uint4 *>(img + ca * 256 + (piece ^ (ca & 15)) * 16);
            const uint4 pb = *reinterpret_cast<const uint4 *>(lds + kEpTurned + cb2 * 256 + (piece ^ (cb2 & 15)) * 16);
            const unsigned wa[4] = {pa.x, pa.y, pa.z, pa.w}, wb[4] = {pb.x, pb.y, pb.z, pb.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                res[kc][2 * e] -= bf16_lo(wa[e]) + bf16_lo(wb[e]);
                res[kc][2 * e + 1] -= bf16_hi(wa[e]) + bf16_hi(wb[e]);
            }
        }
    }
    __syncthreads();
    const int last_lane = fresh_lane(), tl = set * 32 + (last_lane & 31);
    const long long tok = (long long)(blockIdx.x / a.Hkv) * (32 * kSets) + tl;
    if (tok < n_tokens) {
        uint8_t *dst = out + tok * a.token_stride + (long long)g * a.head_stride;
        for (int byte = 2 * rs + (last_lane >> 5); byte < a.record_bytes; byte += 2 * RS) {
            unsigned v = 0;
            for (int r = (8 * byte) / 12; r < a.levels && 12 * r < 8 * byte + 8; ++r) {
                const unsigned pr = (unsigned)chosen[(tl * 32 + r) * 2] | (unsigned)chosen[(tl * 32 + r) * 2 + 1] << 6;
                const int sh = 12 * r - 8 * byte;
                v |= sh >= 0 ? pr << sh : pr >> -sh;
            }
            dst[byte] = (uint8_t)(v & 0xffu);
        }
    }
}

// Paired-format keys, few vectors (a decode step appends one token per sequence): one workgroup per (token, KV head),
// shaped for the latency of a level, since the levels are a dependent chain.  The rows and cross terms of level l + 1
// travel from memory into the other half of a double buffer while level l is searched, the rows in the layout of
// k_encode_rows.  Four lanes share a dot product (32 of its 128 elements each, summed by quad permutes): 512 threads for 64
// rows and two products of each.  Their sums come back through LDS, and wavefront w scans the rows a = 8 w .. + 7, lane b.
// Ties go to the lowest index.  11 levels, 64 vectors: 18.5 us (31 us with 256 threads, the next level fetched through
// registers and the products re-added from LDS by every candidate), 512 vectors 26 us (37).  The same shape for the 256
// rows of an index-form level takes 1.95 us a level, k_encode_rows 1.5.
// No static LDS: the images sit at LDS address 0.
constexpr int kOneThreads = 512;
constexpr int kOneResFloats = kD + 4 * 8;  // 8 unused after every 32: the four lanes of a dot product hit different banks
constexpr int kOneImage = 64 * 256, kOneCross = 2 * kOneImage, kOneTail = kOneCross + 2 * 4096 * 4;
constexpr int kOneLds = kOneTail + kOneResFloats * 4 + 128 * 4 + 8 * 8 + 32 * 4;
__global__ __launch_bounds__(kOneThreads) void k_encode_one(const void *__restrict__ keys, const uint4 *__restrict__ cb,
                                                            const float *__restrict__ norms, const float *__restrict__ cross,
                                                            uint8_t *__restrict__ out, const EncodeDims a)
{
    constexpr int K = 64, kWaves = kOneThreads / 64;
    extern __shared__ __attribute__((aligned(16))) uint4 one_mem[];
    char *lds = reinterpret_cast<char *>(one_mem);
    float *res = reinterpret_cast<float *>(lds + kOneTail);              // element e at e + 8 (e / 32)
    float *uv = res + kOneResFloats;                                  // [U 64][V 64]
    float2 *part = reinterpret_cast<float2 *>(uv + 128);              // [wavefronts] minimum and its index
    int *chosen = reinterpret_cast<int *>(part + kWaves);             // [32]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % a.Hkv;
    const size_t tok = blockIdx.x / a.Hkv;
    const int q = tid & 3, row = (tid >> 2) & (K - 1);
    const bool second = wave >= kWaves / 2;  // the products with i C
    const uint4 *rows = cb + (size_t)g * a.levels * K * 16;
    const float *nrows = norms + (size_t)g * a.levels * K;
    const float *xrows = cross + (size_t)g * a.levels * 4096;
    auto fetch_level = [&](int l, int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int p0 = (wave * 2 + i) * 64, p = p0 + lane, t = p >> 4;
            lds_dma16(rows + (size_t)l * K * 16, (unsigned)(t * 16 + ((p ^ t) & 15)) * 16u, (unsigned)(buf * kOneImage + p0 * 16));
            lds_dma16(xrows + (size_t)l * 4096, (unsigned)p * 16u, (unsigned)(kOneCross + buf * 4096 * 4 + p0 * 16));
        }
    };
    fetch_level(0, 0);
    float mine = 0.f;  // threads below 128: an element of the residual each
    if (tid < kD) {
        const size_t i = (tok * a.Hkv + g) * kD + tid;
        mine = a.key_bf16 ? __builtin_bit_cast(float, (unsigned)static_cast<const uint16_t *>(keys)[i] << 16)
                          : static_cast<const float *>(keys)[i];
        res[tid + (tid >> 5) * 8] = mine;
    }
    float nrm = nrows[row];
    for (int l = 0; l < a.levels; ++l) {
        const int buf = l & 1;
        const char *img = lds + buf * kOneImage;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's part of level l has landed
        __syncthreads();                                   // ... and everybody's; the residual is up to date
        float nrm_next = 0.f;
        if (l + 1 < a.levels) {
            nrm_next = nrows[(size_t)(l + 1) * K + row];
            fetch_level(l + 1, buf ^ 1);
        }
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 pc = *reinterpret_cast<const uint4 *>(img + row * 256 + ((4 * q + i) ^ (row & 15)) * 16);
            const unsigned w[4] = {pc.x, pc.y, pc.z, pc.w};
            const float4 r0 = *reinterpret_cast<const float4 *>(res + 40 * q + 8 * i), r1 = *reinterpret_cast<const float4 *>(res + 40 * q + 8 * i + 4);
            const float rx[4] = {r0.x, r0.z, r1.x, r1.z}, ry[4] = {r0.y, r0.w, r1.y, r1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = bf16_lo(w[e]), y = bf16_hi(w[e]);
                if (second) { s0 = __builtin_fmaf(ry[e], x, s0); s1 = __builtin_fmaf(-rx[e], y, s1); }
                else { s0 = __builtin_fmaf(rx[e], x, s0); s1 = __builtin_fmaf(ry[e], y, s1); }
            }
        }
        float dot = s0 + s1;
        dot += dpp_mov<0xB1>(dot);
        dot += dpp_mov<0x4E>(dot);
        if (q == 0) uv[tid >> 2] = nrm - 2.f * dot;
        __syncthreads();
        const float4 u0 = *reinterpret_cast<const float4 *>(uv + 8 * wave), u1 = *reinterpret_cast<const float4 *>(uv + 8 * wave + 4);
        const float u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        const float v = uv[64 + lane];
        const float *xs = reinterpret_cast<const float *>(lds + kOneCross) + buf * 4096 + 8 * wave * 64 + lane;
        float best = INFINITY;
        int cand = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float sc = u[k] + (v + xs[k * 64]);
            if (sc < best) { best = sc; cand = (8 * wave + k) * 64 + lane; }
        }
        const float wm = -wave_max(-best);
        const int wc = wave_min_index(best == wm ? cand : 0x7fffffff);
        if (lane == 0) part[wave] = make_float2(wm, __builtin_bit_cast(float, wc));
        __syncthreads();
        if (tid < kD) {
            float m = INFINITY;
            int c = 0x7fffffff;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {  // the wavefronts hold increasing indices
                const float2 o = part[w];
                if (o.x < m) { m = o.x; c = __builtin_bit_cast(int, o.y); }
            }
            c &= 4095;  // always in range for finite input
            auto element = [&](int r, int e) {
                return __builtin_bit_cast(float, (unsigned)*reinterpret_cast<const uint16_t *>(img + r * 256 + (((e >> 3) ^ r) & 15) * 16 + (e & 7) * 2) << 16);
            };
            const float va = element(c >> 6, tid), vb = element(c & 63, tid ^ 1);  // C[a] + i C[b], i (x, y) = (-y, x)
            mine -= tid & 1 ? va + vb : va - vb;
            res[tid + (tid >> 5) * 8] = mine;
            if (tid == 0) chosen[l] = c;
        }
        nrm = nrm_next;
    }
    __syncthreads();
    uint8_t *dst = out + tok * a.token_stride + (long long)g * a.head_stride;
    if (tid < a.record_bytes) {
        unsigned v = 0;
        for (int r = (8 * tid) / 12; r < a.levels && 12 * r < 8 * tid + 8; ++r) {
            const unsigned pr = (unsigned)(chosen[r] >> 6) | (unsigned)(chosen[r] & 63) << 6;
            const int sh = 12 * r - 8 * tid;
            v |= sh >= 0 ? pr << sh : pr >> -sh;
        }
        dst[tid] = (uint8_t)(v & 0xffu);
    }
}

}  // namespace

namespace {

// What is encoded: the keys (the configured key format) or the values (always index form, m_val codebooks).
struct EncodeWhat {
    bool paired;
    int levels, K, rec;
};
EncodeWhat encode_what(const commvq_config &c, bool values)
{
    EncodeWhat w;
    w.paired = !values && c.key_format == COMMVQ_KEYS_PAIRED;
    w.levels = values ? c.m_val : w.paired ? c.key_levels : c.m_key;
    w.K = w.paired ? 64 : kK;
    w.rec = w.paired ? (12 * w.levels + 7) / 8 : w.levels;
    return w;
}

commvq_status encoder_table_bytes(const commvq_handle *h, bool values, size_t *bytes)
{
    if (!h || !bytes) return COMMVQ_ERR_NULL;
    const EncodeWhat w = encode_what(h->cfg, values);
    *bytes = (size_t)h->cfg.n_kv_heads * w.levels * w.K * sizeof(float) * (w.paired ? 1 + w.K : 1);
    return COMMVQ_OK;
}

commvq_status encoder_prepare(commvq_handle *h, bool values, const void *cb, void *tables, void *stream)
{
    if (!h || !cb || !tables) return COMMVQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(tables) & 15u) return COMMVQ_ERR_SHAPE;
    if (h->device < 0) return COMMVQ_ERR_NO_DEVICE;
    const commvq_config &c = h->cfg;
    const EncodeWhat w = encode_what(c, values);
    const int rows = c.n_kv_heads * w.levels * w.K;
    float *norms = static_cast<float *>(tables), *cross = norms + rows;
    const size_t n = w.paired ? (size_t)rows * w.K : (size_t)rows;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (c.codebook_dtype == COMMVQ_BF16)
        hipLaunchKernelGGL(k_encode_tables<true>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cb, norms, cross, rows, w.K, w.paired ? 1 : 0);
    else
        hipLaunchKernelGGL(k_encode_tables<false>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cb, norms, cross, rows, w.K, w.paired ? 1 : 0);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status launch_encode_one(const void *keys, const void *cb, const float *norms, const float *cross, uint8_t *out,
                                const EncodeDims &d, int n_tokens, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_encode_one, kOneLds, lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_encode_one, dim3((unsigned)(n_tokens * d.Hkv)), dim3(kOneThreads), kOneLds, s, keys,
                       static_cast<const uint4 *>(cb), norms, cross, out, d);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

template <int RS>
commvq_status launch_encode_rows(const void *keys, const void *cb, const float *norms, uint8_t *out, const EncodeDims &d, int n_tokens,
                                 hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_encode_rows<RS>, er_lds(RS), lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    constexpr int per_wg = 16 * (8 / RS);
    hipLaunchKernelGGL(k_encode_rows<RS>, dim3((unsigned)((n_tokens + per_wg - 1) / per_wg * d.Hkv)), dim3(er_threads(RS)), er_lds(RS), s, keys,
                       static_cast<const uint4 *>(cb), norms, out, d, n_tokens);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status launch_encode_few(const void *keys, const void *cb, const float *norms, uint8_t *out, const EncodeDims &d, int n_tokens, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_encode_few, kFewLds, lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    const int workers = (n_tokens + kFewTok - 1) / kFewTok * d.Hkv, ahead = std::min(d.levels - 1, std::max(0, 256 - workers) / d.Hkv) * d.Hkv;
    hipLaunchKernelGGL(k_encode_few, dim3((unsigned)(workers + ahead)), dim3(kFewThreads), kFewLds, s, keys,
                       static_cast<const uint4 *>(cb), norms, out, d, n_tokens, workers);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status launch_encode_many(const void *keys, const void *cb, const float *norms, uint8_t *out, const EncodeDims &d, int n_tokens, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_encode_many, kManyLds, lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_encode_many, dim3((unsigned)((n_tokens + kManyTokens - 1) / kManyTokens * d.Hkv)), dim3(kManyThreads), kManyLds, s, keys,
                       static_cast<const uint4 *>(cb), norms, out, d, n_tokens);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status encode_rows(const void *keys, const void *cb, const float *norms, uint8_t *out, const EncodeDims &d, int n_tokens,
                          hipStream_t s)
{
    // A compute unit holds one workgroup, so a launch of up to 256 is one round, and a round is the cheaper the more
    // wavefronts share a token set: 32 levels of 8 heads take 34 to 37 us with k_encode_few (up to 160 tokens), 47 with
    // RS = 8 (512), 64 (4; 1024), 112 (2; 2048), 136 with k_encode_many (4096).  So full rounds go to the latter, and the rest to the first of them that
    // needs one round.
    const int64_t round = 128 * (int64_t)std::max(1, 256 / d.Hkv);
    const int full = (int)(n_tokens / round * round), rest = n_tokens - full;
    if (full) {
        const commvq_status st = launch_encode_many(keys, cb, norms, out, d, full, s);
        if (st != COMMVQ_OK || !rest) return st;
        keys = static_cast<const char *>(keys) + (size_t)full * d.Hkv * kD * (d.key_bf16 ? 2 : 4);
        out += full * d.token_stride;
    }
    auto one_round = [&](int per_wg) { return (int64_t)(rest + per_wg - 1) / per_wg * d.Hkv <= 256; };
    if (one_round(kFewTok)) return launch_encode_few(keys, cb, norms, out, d, rest, s);
    if (one_round(16)) return launch_encode_rows<8>(keys, cb, norms, out, d, rest, s);
    if (one_round(32)) return launch_encode_rows<4>(keys, cb, norms, out, d, rest, s);
    if (one_round(64)) return launch_encode_rows<2>(keys, cb, norms, out, d, rest, s);
    return launch_encode_many(keys, cb, norms, out, d, rest, s);
}

template <int RS>
commvq_status launch_encode_pairs(const void *keys, const void *cb, const float *norms, const float *cross, uint8_t *out,
                                  const EncodeDims &d, int n_tokens, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_encode_pairs<RS>, ep_lds(RS), lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    constexpr int per_wg = 128 / RS;
    hipLaunchKernelGGL(k_encode_pairs<RS>, dim3((unsigned)((n_tokens + per_wg - 1) / per_wg * d.Hkv)), dim3(kEpThreads), ep_lds(RS), s, keys,
                       static_cast<const uint4 *>(cb), norms, cross, out, d, n_tokens);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status encode_pairs(const void *keys, const void *cb, const float *norms, const float *cross, uint8_t *out, const EncodeDims &d,
                           int n_tokens, hipStream_t s)
{
    // As in encode_rows: full rounds of one workgroup per compute unit go to RS = 1, and the rest to what needs one round.
    // 21 levels of 8 heads take 103 us with RS = 4 (up to 1024 tokens), 118 (2; 2048), 160 (1; 4096).  A workgroup per
    // vector takes 33 to 46 us while the vectors fit the chip, two workgroups per compute unit.
    const int64_t round = 128 * (int64_t)std::max(1, 256 / d.Hkv);
    const int full = (int)(n_tokens / round * round), rest = n_tokens - full;
    if (full) {
        const commvq_status st = launch_encode_pairs<1>(keys, cb, norms, cross, out, d, full, s);
        if (st != COMMVQ_OK || !rest) return st;
        keys = static_cast<const char *>(keys) + (size_t)full * d.Hkv * kD * (d.key_bf16 ? 2 : 4);
        out += full * d.token_stride;
    }
    auto one_round = [&](int per_wg) { return (int64_t)(rest + per_wg - 1) / per_wg * d.Hkv <= 256; };
    if ((int64_t)rest * d.Hkv <= 512) return launch_encode_one(keys, cb, norms, cross, out, d, rest, s);
    if (one_round(32)) return launch_encode_pairs<4>(keys, cb, norms, cross, out, d, rest, s);
    if (one_round(64)) return launch_encode_pairs<2>(keys, cb, norms, cross, out, d, rest, s);
    return launch_encode_pairs<1>(keys, cb, norms, cross, out, d, rest, s);
}

commvq_status encode_vectors(commvq_handle *h, bool values, const void *keys, int32_t n_tokens, const void *key_cb, const void *tables,
                             uint8_t *codes_out, int64_t token_stride, int64_t head_stride, void *stream)
{
    if (!h || !keys || !key_cb || !tables || !codes_out) return COMMVQ_ERR_NULL;
    const commvq_config &c = h->cfg;
    const EncodeWhat w = encode_what(c, values);
    const bool paired = w.paired;
    const int levels = w.levels, K = w.K, rec = w.rec;
    if (n_tokens < 1 || (int64_t)n_tokens * c.n_kv_heads > (int64_t)1 << 30) return COMMVQ_ERR_SHAPE;
    if (head_stride < rec || token_stride < rec) return COMMVQ_ERR_SHAPE;  // records must not overlap
    if ((reinterpret_cast<uintptr_t>(tables) | reinterpret_cast<uintptr_t>(keys) | reinterpret_cast<uintptr_t>(key_cb)) & 15u)
        return COMMVQ_ERR_SHAPE;
    EncodeDims d;
    d.Hkv = c.n_kv_heads; d.levels = levels; d.K = K; d.key_bf16 = c.q_dtype == COMMVQ_BF16; d.record_bytes = rec;
    d.token_stride = token_stride; d.head_stride = head_stride;
    const int rows = c.n_kv_heads * levels * K;
    const float *norms = static_cast<const float *>(tables), *cross = norms + rows;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool bf16 = c.codebook_dtype == COMMVQ_BF16;
    if (paired && !bf16) return COMMVQ_ERR_CONFIG;
    if (h->device < 0) return COMMVQ_ERR_NO_DEVICE;
    if (paired) {
        return encode_pairs(keys, key_cb, norms, cross, codes_out, d, n_tokens, s);
    } else if (bf16) {
        return encode_rows(keys, key_cb, norms, codes_out, d, n_tokens, s);
    } else {
        hipLaunchKernelGGL(k_encode, dim3((unsigned)(n_tokens * c.n_kv_heads)), dim3(256), 0, s, keys, static_cast<const float *>(key_cb), norms,
                           codes_out, d);
    }
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

}  // namespace

extern "C" {

commvq_status commvq_encoder_table_bytes(const commvq_handle *h, size_t *bytes) { return encoder_table_bytes(h, false, bytes); }
// a free binary value code has no greedy stand-in here: its only producer is the trained encoder of Sec. 4.1
static bool binary_values(const commvq_handle *h) { return h && h->cfg.value_format == COMMVQ_VALUES_BINARY; }

commvq_status commvq_value_encoder_table_bytes(const commvq_handle *h, size_t *bytes)
{
    if (binary_values(h)) return COMMVQ_ERR_CONFIG;
    return encoder_table_bytes(h, true, bytes);
}

commvq_status commvq_encoder_prepare(commvq_handle *h, const void *key_cb, void *tables, void *stream)
{
    return encoder_prepare(h, false, key_cb, tables, stream);
}
commvq_status commvq_value_encoder_prepare(commvq_handle *h, const void *val_cb, void *tables, void *stream)
{
    if (binary_values(h)) return COMMVQ_ERR_CONFIG;
    return encoder_prepare(h, true, val_cb, tables, stream);
}

commvq_status commvq_encode_keys(commvq_handle *h, const void *keys, int32_t n_tokens, const void *key_cb, const void *tables,
                                 uint8_t *codes_out, int64_t token_stride, int64_t head_stride, void *stream)
{
    return encode_vectors(h, false, keys, n_tokens, key_cb, tables, codes_out, token_stride, head_stride, stream);
}
commvq_status commvq_encode_values(commvq_handle *h, const void *values, int32_t n_tokens, const void *val_cb, const void *tables,
                                   uint8_t *codes_out, int64_t token_stride, int64_t head_stride, void *stream)
{
    if (binary_values(h)) return COMMVQ_ERR_CONFIG;
    return encode_vectors(h, true, values, n_tokens, val_cb, tables, codes_out, token_stride, head_stride, stream);
}

}  // extern "C"
