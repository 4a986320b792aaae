// Shared by the translation units of libcommvq: constants, the handle, vector types and wavefront helpers.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <new>
#include <utility>
#include <vector>

#include "commvq.h"
#include "commvq_launch.hpp"

namespace {

constexpr int kD = 128;         // head_dim
constexpr int kJ = 64;          // 2-D sub-spaces = lanes of a wavefront
constexpr int kK = 256;         // codewords per codebook
constexpr int kLoBits = 6;      // relative position = hi * 64 + lo
constexpr int kLo = 1 << kLoBits;
constexpr int kScoreMaxTpt = 4;      // tiles of k_score_lut: at most 4 x 1024 tokens
constexpr int kStreamPasses = 8;     // k_score_stream: passes of a workgroup at most
constexpr int kPassTokens = 512;     // tokens of a pass: 16 wavefronts x 32
constexpr int kStreamSlices = kD / 8;  // codebook slices: 8 elements of every codeword each
constexpr int kScoreMinWgs = 2048;   // row-gather score kernel: tiles are halved until this many workgroups exist
constexpr int kScoreThreads = 256;
constexpr int kFewTokens = kScoreThreads / 16;  // tokens of a workgroup of k_score_few, the smallest tile of the row-gather kernels
constexpr int kOutThreads = 256;
constexpr int kOutRows = 64;    // codebook rows per k_out workgroup
constexpr int kOutMfmaRows = 256;   // codebook rows per k_out_mfma workgroup (batched output stage)
constexpr int kOutMfmaMinRows = 16;  // batch * (query heads per KV head) from which the batched output kernel is used
constexpr int kLdsBytes = 160 * 1024;  // LDS of a compute unit
constexpr int kProfRing = 64;
constexpr float kLog2e = 1.4426950408889634f;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Quotients of workgroup indices by numbers that the host knows: a multiplication instead of the 40 dependent instructions of a
// division, which every wavefront would run before its first load.  With s = ceil(log2 d) and m = floor(2^(31 + s) / d) + 1 the
// product n m / 2^(31 + s) is n / d and less than 1 / d more for every n below 2^31, so that its whole part is the quotient.
struct Divisor {
    unsigned mul, shift;
};
inline Divisor divisor(unsigned d)
{
    unsigned s = 0;
    while (s < 31 && 1u << s < d) ++s;
    return Divisor{(unsigned)(((uint64_t)1 << (31 + s)) / d + 1), s};
}
__host__ __device__ inline int quotient(int n, Divisor d) { return (int)((unsigned)(((uint64_t)(2u * (unsigned)n) * d.mul) >> 32) >> d.shift); }

}  // namespace

struct commvq_handle {
    commvq_config cfg;
    int G;
    float scale;
    int n_hi;
    int device;      // device ordinal of the phase tables; -1 for a planner handle (no device resources)
    float2 *tbl_hi;  // [n_hi][64]  exp(i * theta_j * 64 * hi)
    float2 *tbl_lo;  // [64][64]    exp(i * theta_j * lo)
    void *static_scratch;  // this device's copy of the library's static scratch array (commvq_decode_attn_static)
    int prof_every, prof_calls;  // stage events on every prof_every-th call (0: never)
    int prof_head, prof_count;
    hipEvent_t prof_ev[kProfRing][4];
    bool prof_ev_made;
    // key codebooks that the caller has had re-laid once (commvq_pack_key_codebooks): source pointer -> packed copy
    std::vector<std::pair<const void *, const uint4 *>> packed_keys;
    // value codebooks re-laid once for the batched output kernel (commvq_pack_value_codebooks): source -> packed copy
    std::vector<std::pair<const void *, const uint4 *>> packed_vals;
};

namespace {

typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x16_t __attribute__((ext_vector_type(16)));
typedef unsigned uint8v_t __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ device helpers
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// The lane's index, made anew wherever it is asked for: what depends on it is then neither hoisted out of a loop nor kept in
// registers (or spilled) across it.
__device__ __forceinline__ int fresh_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Sum over the 64 lanes of a wavefront; every lane receives the total.
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);  // row_half_mirror
    v += dpp_mov<0x140>(v);  // row_mirror: every lane now holds its 16-lane row sum
    unsigned u = __builtin_bit_cast(unsigned, v);
    auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __builtin_bit_cast(float, (unsigned)r16[0]) + __builtin_bit_cast(float, (unsigned)r16[1]);
    u = __builtin_bit_cast(unsigned, v);
    auto r32 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (unsigned)r32[0]) + __builtin_bit_cast(float, (unsigned)r32[1]);
}

__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_mov<0xB1>(v));
    v = fmaxf(v, dpp_mov<0x4E>(v));
    v = fmaxf(v, dpp_mov<0x141>(v));
    v = fmaxf(v, dpp_mov<0x140>(v));
    unsigned u = __builtin_bit_cast(unsigned, v);
    auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = fmaxf(__builtin_bit_cast(float, (unsigned)r16[0]), __builtin_bit_cast(float, (unsigned)r16[1]));
    u = __builtin_bit_cast(unsigned, v);
    auto r32 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__builtin_bit_cast(float, (unsigned)r32[0]), __builtin_bit_cast(float, (unsigned)r32[1]));
}

// element i of a bf16 or fp32 array, widened exactly
template <bool BF16>
__device__ __forceinline__ float cb_elem(const void *cb, size_t i)
{
    if (BF16) return __builtin_bit_cast(float, (unsigned)static_cast<const uint16_t *>(cb)[i] << 16);
    return static_cast<const float *>(cb)[i];
}

// 16 bytes per lane from global memory straight into LDS (no register destination): lane l of the wavefront lands at
// LDS byte address lds_byte_addr_uniform + 16 l.  Issued from inline asm, so the compiler makes no later access wait
// for it: the kernel waits itself (s_waitcnt vmcnt(0)) before the data is used.
__device__ __forceinline__ void lds_dma16(const void *gptr, unsigned lds_byte_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_byte_addr_uniform), "v"(gptr) : "memory");
}

// the same from a wavefront-uniform address plus a byte offset per lane
__device__ __forceinline__ void lds_dma16(const void *base_uniform, unsigned offset, unsigned lds_byte_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_byte_addr_uniform), "v"(offset), "s"(base_uniform) : "memory");
}

// Raw buffer descriptor over [base, base + bytes): loads take a per-lane byte offset plus a
// wave-uniform (scalar) byte offset, and reads past the end return zero instead of faulting.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}

// Stores that do not stay in the writer's L2.  What a kernel leaves there is written back once it has ended, before the next
// one begins: for results of megabytes (logits, bins, partial sums) several microseconds in which nothing else runs, and the
// next kernel's workgroups, on all eight L2s, read them from memory either way.  Whole calls, kept -> written through: 8B
// layer at 128K 85.5 -> 83.9 us, paired keys and binary values 116.8 -> 113.3, 32K at 2 bits 57.7 -> 56.5, 70B 4 x 128K 544.5 -> 539.2.
constexpr int kThrough = 16;  // cache policy of the buffer instructions: visible to the whole GPU
__device__ __forceinline__ void store_through(uint4_t v, __amdgpu_buffer_rsrc_t r, unsigned offset) { __builtin_amdgcn_raw_buffer_store_b128(v, r, offset, 0, kThrough); }
__device__ __forceinline__ void store_through(float v, __amdgpu_buffer_rsrc_t r, unsigned offset) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, offset, 0, kThrough); }

// Softmax statistics of one head over tokens v0 .. of a sequence, by a wavefront, from the (max, sum of exp(logit - max)) of the ns
// score tiles of split_len tokens: the maximum of the sequence, the exp-sum of the tiles ta .. tb - 1 that the range touches, and
// of those that BEGIN inside it (a tile shared by two ranges is counted once).  Every load is requested before
// the first is waited for.  128K tokens have 256 tiles: four rounds of 64 for the maximum and as many again for the sums, each
// after the one before, took k_values 20.8 us instead of 19.7, k_vbits 24.0 instead of 22.7; one fp32 head of 4096 tokens, in tiles
// of 16, 7.0 instead of 5.9.
struct RangeStats {
    float2 first[4], own;
    __device__ __forceinline__ void request(const float2 *st, int ns, int ta, int tb, int lane)
    {
        const int k = ta + ((lane - ta) & 63);
        own = k < tb ? st[k] : make_float2(-INFINITY, 0.f);
#pragma unroll
        for (int i = 0; i < 4; ++i) first[i] = lane + 64 * i < ns ? st[lane + 64 * i] : make_float2(-INFINITY, 0.f);
    }
    // (the sequence's own ns and tb, which may be less than what was asked for)
    __device__ __forceinline__ void finish(const float2 *st, int ns, int ta, int tb, int split_len, int v0, int lane, float &mx, float &l, float &lown) const
    {
        mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, lane + 64 * i < ns ? first[i].x : -INFINITY);
        for (int k = lane + 256; k < ns; k += 64) mx = fmaxf(mx, st[k].x);
        mx = wave_max(mx);
        l = lown = 0.f;
        float2 s = own;
        for (int k = ta + ((lane - ta) & 63); k < tb; k += 64) {
            if (k >= ta + 64) s = st[k];
            const float t = s.y * __builtin_amdgcn_exp2f((s.x - mx) * kLog2e);
            l += t;
            if (k * split_len >= v0) lown += t;
        }
        l = wave_sum(l);
        lown = wave_sum(lown);
    }
};

__device__ __forceinline__ float bf16_lo(unsigned v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float bf16_hi(unsigned v) { return __builtin_bit_cast(float, v & 0xffff0000u); }

// acc + low / high bf16 half of a packed pair, in one v_dot2c_f32_bf16 each: the other half
// is multiplied by zero, so this is an exact fp32 add of the widened value.  The selector
// (1.0 in one half, 0 in the other) is passed through an opaque register so that it is never
// encoded as an inline constant, whose meaning for packed bf16 operands is ambiguous.
__device__ __forceinline__ unsigned opaque_sgpr(unsigned v)
{
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ float add_bf16_sel(unsigned v, unsigned sel, float acc)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, v), __builtin_bit_cast(bf16x2_t, sel), acc, false);
}

}  // namespace
