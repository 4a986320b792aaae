// libcommvq: EM-like learner of the RoPE-commutative key codebook (Sec. 4.2, Algorithm 1; App. A.2),
// one iteration for J independent 2-D sub-spaces, hand-written for gfx950.
//
// A sub-space has N_c' parameter pairs phi = (x_l, y_l) and N_c'^2 clustering centres
// c_ab = (x_a - y_b, y_a + x_b) (Eq. def_center).  One iteration:
//   E step   W_i,ab = softmax_ab(-D_i,ab / T), D the Euclidean distance of point i to centre ab
//            (soft assignment with temperature, Eq. W);
//   M step   the minimiser of sum_ab N_ab ||c_ab(phi) - m_ab||^2 with N_ab = sum_i W_i,ab and m_ab the
//            weighted mean of the points of centre ab.  The paper writes it with a constant matrix T as
//            phi* = (T^T S T)^-1 T^T S m; T^T S T and T^T S m are formed here directly from their
//            entries (derivatives of the objective with respect to x_a and y_a):
//              A[x_a][x_a] = A[y_a][y_a] = sum_b (N_ab + N_ba)
//              A[x_a][y_b] = A[y_b][x_a] = N_ba - N_ab
//              rhs[x_a] = sum_b (Sx_ab + Sy_ba),   rhs[y_a] = sum_b (Sy_ab - Sx_ba)
//            with (Sx, Sy)_ab = sum_i W_i,ab k_i = N_ab m_ab, and solved by Cholesky factorisation.
// Three kernels: k_em_norm (per point: nearest distance and softmax denominator), k_em_accum (per centre:
// N_ab and S_ab, points streamed through LDS, summed in a fixed order), k_em_solve (one workgroup per
// sub-space, the 2 N_c' x 2 N_c' system in LDS).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cstdint>

#include "commvq.h"
#include "commvq_internal.hpp"

namespace {

constexpr int kEmMaxNc = 64;
constexpr int kEmTile = 1024;  // points per LDS tile in k_em_accum
constexpr float kLog2eEm = 1.4426950408889634f;

inline size_t em_align(size_t v) { return (v + 255) / 256 * 256; }

// v_sqrt_f32 as it is (1 ulp): the library square root adds a scaling and a correction step per call, and the
// E step takes one per (point, centre) pair.
__device__ __forceinline__ float em_sqrt(float v) { return __builtin_amdgcn_sqrtf(v); }

// dmin[j][i] = min_ab D_i,ab ;  zsum[j][i] = sum_ab exp(-(D_i,ab - dmin) / T)
__global__ __launch_bounds__(256) void k_em_norm(const float2 *__restrict__ data, const float2 *__restrict__ phi,
                                                 float *__restrict__ dmin, float *__restrict__ zsum, int N, int Nc, float inv_t)
{
    __shared__ float2 ph[kEmMaxNc];
    const int j = blockIdx.y;
    if (threadIdx.x < Nc) ph[threadIdx.x] = phi[(size_t)j * Nc + threadIdx.x];
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const float2 k = data[(size_t)j * N + i];
    // two sweeps over the centres: the nearest squared distance first (no square root, no exponential), then the
    // denominator -- one v_sqrt_f32 and one v_exp_f32 per pair, the quarter-rate instructions that bound this kernel
    // (a single sweep with a running minimum computes a second exponential per pair for the rescaling)
    float dm2 = INFINITY;
    for (int a = 0; a < Nc; ++a)
        for (int b = 0; b < Nc; ++b) {
            const float ex = k.x - (ph[a].x - ph[b].y), ey = k.y - (ph[a].y + ph[b].x);
            dm2 = fminf(dm2, ex * ex + ey * ey);
        }
    const float dm = em_sqrt(dm2), sc = inv_t * kLog2eEm;
    float z = 0.f;
    for (int a = 0; a < Nc; ++a)
        for (int b = 0; b < Nc; ++b) {
            const float ex = k.x - (ph[a].x - ph[b].y), ey = k.y - (ph[a].y + ph[b].x);
            z += __builtin_amdgcn_exp2f((dm - em_sqrt(ex * ex + ey * ey)) * sc);
        }
    dmin[(size_t)j * N + i] = dm;
    zsum[(size_t)j * N + i] = z;
}

// One thread per centre ab of sub-space j; all points pass by in LDS tiles, in index order.
__global__ __launch_bounds__(256) void k_em_accum(const float2 *__restrict__ data, const float2 *__restrict__ phi,
                                                  const float *__restrict__ dmin, const float *__restrict__ zsum,
                                                  float *__restrict__ nab, float2 *__restrict__ sab, int N, int Nc, float inv_t)
{
    __shared__ float2 pts[kEmTile];
    __shared__ float2 nz[kEmTile];  // (dmin, 1 / zsum) of the tile's points
    const int j = blockIdx.y;
    const int ab = blockIdx.x * 256 + threadIdx.x;
    const bool live = ab < Nc * Nc;
    float cx = 0.f, cy = 0.f;
    if (live) {
        const float2 pa = phi[(size_t)j * Nc + ab / Nc], pb = phi[(size_t)j * Nc + ab % Nc];
        cx = pa.x - pb.y;
        cy = pa.y + pb.x;
    }
    float n = 0.f, sx = 0.f, sy = 0.f;
    const float sc = inv_t * kLog2eEm;
    for (int t0 = 0; t0 < N; t0 += kEmTile) {
        const int cnt = min(kEmTile, N - t0);
        __syncthreads();
        for (int x = threadIdx.x; x < cnt; x += 256) {
            pts[x] = data[(size_t)j * N + t0 + x];
            nz[x] = make_float2(dmin[(size_t)j * N + t0 + x], 1.f / zsum[(size_t)j * N + t0 + x]);
        }
        __syncthreads();
        if (live) {
#pragma unroll 4
            for (int x = 0; x < cnt; ++x) {
                const float2 k = pts[x];
                const float ex = k.x - cx, ey = k.y - cy;
                const float w = __builtin_amdgcn_exp2f((nz[x].x - em_sqrt(ex * ex + ey * ey)) * sc) * nz[x].y;
                n += w;
                sx = __builtin_fmaf(w, k.x, sx);
                sy = __builtin_fmaf(w, k.y, sy);
            }
        }
    }
    if (live) {
        nab[(size_t)j * Nc * Nc + ab] = n;
        sab[(size_t)j * Nc * Nc + ab] = make_float2(sx, sy);
    }
}

// Blocked Cholesky A = L L^T in place (lower triangle of A [np][ld] in LDS; np a multiple of 16, the rows and
// columns past the system's size n hold the identity), 16 columns per step.  The 16 x 16 diagonal block is
// factored by wavefront 0 with a row per lane, columns exchanged through v_readlane (constant lanes: scalar
// broadcasts, no LDS round trips); the same lanes then invert the triangular block, so that everything below --
// the panel's rows here, the right-hand sides in em_substitute -- is a product with inv(L_kk) by independent
// threads instead of a 16-step chain per thread.  Dinv [np / 16][16][16] receives the inverses.
constexpr int kEmNb = 16;
__device__ __forceinline__ int em_pad(int n) { return (n + kEmNb - 1) / kEmNb * kEmNb; }
__device__ __forceinline__ float em_lane(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ float em_rcp(float d)
{
    const float x = __builtin_amdgcn_rcpf(d);
    return x * (2.f - d * x);
}
template <int NT>
__device__ __forceinline__ void em_cholesky(float *A, int ld, int np, float *Dinv, int tid)
{
    for (int k0 = 0; k0 < np; k0 += kEmNb) {
        float *Di = Dinv + (k0 / kEmNb) * (kEmNb * kEmNb);
        if (tid < 64) {
            const int t = tid & (kEmNb - 1);  // lanes 16..63 repeat lanes 0..15 and store nothing
            float row[kEmNb], isd[kEmNb];
#pragma unroll
            for (int c = 0; c < kEmNb; ++c) row[c] = c <= t ? A[(k0 + t) * ld + k0 + c] : 0.f;
#pragma unroll
            for (int c = 0; c < kEmNb; ++c) {
                const float d = __builtin_sqrtf(em_lane(row[c], c));
                isd[c] = em_rcp(d);
                row[c] = t == c ? d : row[c] * isd[c];  // entries above the diagonal are never read
#pragma unroll
                for (int cc = c + 1; cc < kEmNb; ++cc) row[cc] -= row[c] * em_lane(row[c], cc);  // L[t][c] L[cc][c]
            }
            // column t of X = inv(L_kk):  X[i][t] = (delta_it - sum_{k < i} L[i][k] X[k][t]) / L[i][i]
            float x[kEmNb];
#pragma unroll
            for (int i = 0; i < kEmNb; ++i) {
                float v = i == t ? 1.f : 0.f;
#pragma unroll
                for (int k = 0; k < i; ++k) v -= em_lane(row[k], i) * x[k];
                x[i] = i >= t ? v * isd[i] : 0.f;
            }
            if (tid < kEmNb) {
#pragma unroll
                for (int c = 0; c < kEmNb; ++c) {
                    if (c <= t) A[(k0 + t) * ld + k0 + c] = row[c];
                    Di[c * kEmNb + t] = x[c];
                }
            }
        }
        __syncthreads();
        for (int r = k0 + kEmNb + tid; r < np; r += NT) {  // x L_kk^T = a for the rows below: x = a inv(L_kk)^T
            float av[kEmNb], xv[kEmNb];
#pragma unroll
            for (int e = 0; e < kEmNb; ++e) av[e] = A[r * ld + k0 + e];
#pragma unroll
            for (int c = 0; c < kEmNb; ++c) {
                float v = 0.f;
#pragma unroll
                for (int e = 0; e <= c; ++e) v += av[e] * Di[c * kEmNb + e];
                xv[c] = v;
            }
#pragma unroll
            for (int c = 0; c < kEmNb; ++c) A[r * ld + k0 + c] = xv[c];
        }
        __syncthreads();
        // rest -= panel panel^T (lower triangle): 32 lanes walk a row's columns, the row's panel entries in registers
        for (int r = k0 + kEmNb + tid / 32; r < np; r += NT / 32) {
            float pr[kEmNb];
#pragma unroll
            for (int e = 0; e < kEmNb; ++e) pr[e] = A[r * ld + k0 + e];
            for (int cc = k0 + kEmNb + tid % 32; cc <= r; cc += 32) {
                float sum = 0.f;
#pragma unroll
                for (int e = 0; e < kEmNb; ++e) sum += pr[e] * A[cc * ld + k0 + e];
                A[r * ld + cc] -= sum;
            }
        }
        __syncthreads();
    }
}

// L Z = R, then L^T X = Z, for the nr columns of R [np][nr] in LDS (16 nr <= NT), blocked like em_cholesky: thread
// (c, j) forms entry c of a block's solution for column j as a product with the inverted diagonal block, then
// every thread takes one (row, column) of what remains and subtracts the block's contribution.
template <int NT>
__device__ __forceinline__ void em_substitute(const float *A, int ld, int np, const float *Dinv, float *R, int nr, int tid)
{
    const bool act = tid < kEmNb * nr;
    const int c = tid / nr, j = tid % nr;
    for (int k0 = 0; k0 < np; k0 += kEmNb) {
        const float *Di = Dinv + (k0 / kEmNb) * (kEmNb * kEmNb);
        float v = 0.f;
        if (act) {
#pragma unroll
            for (int e = 0; e < kEmNb; ++e)
                if (e <= c) v += Di[c * kEmNb + e] * R[(k0 + e) * nr + j];
        }
        __syncthreads();
        if (act) R[(k0 + c) * nr + j] = v;
        __syncthreads();
        for (int x = tid; x < (np - k0 - kEmNb) * nr; x += NT) {
            const int r = k0 + kEmNb + x / nr, jj = x % nr;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < kEmNb; ++e) sum += A[r * ld + k0 + e] * R[(k0 + e) * nr + jj];
            R[r * nr + jj] -= sum;
        }
        __syncthreads();
    }
    for (int k0 = np - kEmNb; k0 >= 0; k0 -= kEmNb) {
        const float *Di = Dinv + (k0 / kEmNb) * (kEmNb * kEmNb);
        float v = 0.f;
        if (act) {
#pragma unroll
            for (int e = 0; e < kEmNb; ++e)
                if (e >= c) v += Di[e * kEmNb + c] * R[(k0 + e) * nr + j];  // inv(L_kk)^T
        }
        __syncthreads();
        if (act) R[(k0 + c) * nr + j] = v;
        __syncthreads();
        for (int x = tid; x < k0 * nr; x += NT) {
            const int r = x / nr, jj = x % nr;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < kEmNb; ++e) sum += A[(k0 + e) * ld + r] * R[(k0 + e) * nr + jj];
            R[r * nr + jj] -= sum;
        }
        __syncthreads();
    }
}

// One workgroup per sub-space: build the 2Nc x 2Nc normal equations, Cholesky, two triangular solves.
__global__ __launch_bounds__(256) void k_em_solve(const float *__restrict__ nab, const float2 *__restrict__ sab,
                                                  float2 *__restrict__ phi, int Nc)
{
    extern __shared__ float em_lds[];
    const int n2 = 2 * Nc, np = em_pad(n2);
    float *A = em_lds;                 // [np][np + 1]: padded rows; identity past n2
    float *rhs = A + np * (np + 1);    // [np]
    float *Dinv = rhs + np;            // [np / 16][16][16]
    const int ld = np + 1;
    const int j = blockIdx.x, tid = threadIdx.x;
    const float *Nj = nab + (size_t)j * Nc * Nc;
    const float2 *Sj = sab + (size_t)j * Nc * Nc;
    for (int x = tid; x < np * ld; x += 256) A[x] = 0.f;
    if (tid < np) rhs[tid] = 0.f;
    __syncthreads();
    if (tid >= n2 && tid < np) A[tid * ld + tid] = 1.f;
    // off-diagonal blocks: A[x_a][y_b] = A[y_b][x_a] = N_ba - N_ab  (unknown order x_0, y_0, x_1, y_1, ...)
    for (int x = tid; x < Nc * Nc; x += 256) {
        const int a = x / Nc, b = x % Nc;
        const float v = Nj[b * Nc + a] - Nj[a * Nc + b];
        A[(2 * a) * ld + 2 * b + 1] = v;
        A[(2 * b + 1) * ld + 2 * a] = v;
    }
    __syncthreads();
    if (tid < Nc) {
        const int a = tid;
        float d = 0.f, rx = 0.f, ry = 0.f;
        for (int b = 0; b < Nc; ++b) {
            d += Nj[a * Nc + b] + Nj[b * Nc + a];
            rx += Sj[a * Nc + b].x + Sj[b * Nc + a].y;
            ry += Sj[a * Nc + b].y - Sj[b * Nc + a].x;
        }
        A[(2 * a) * ld + 2 * a] = d;
        A[(2 * a + 1) * ld + 2 * a + 1] = d;
        rhs[2 * a] = rx;
        rhs[2 * a + 1] = ry;
    }
    __syncthreads();
    em_cholesky<256>(A, ld, np, Dinv, tid);
    em_substitute<256>(A, ld, np, Dinv, rhs, 1, tid);
    if (tid < Nc) phi[(size_t)j * Nc + tid] = make_float2(rhs[2 * tid], rhs[2 * tid + 1]);
}

// ------------------------------------------------------------------ one code shared by a group of sub-spaces
// Sec. 4.2 groups g consecutive sub-spaces under one quantized value, so a clustering centre is the pair (a, b)
// applied in all g sub-spaces and the E step weighs whole vectors:  D_i,ab^2 = sum_j ||k_i^j - c_ab^j||^2
//   = ||k_i||^2 + (N_a - 2 P_i[a]) + (N_b - 2 Q_i[b]) + X_ab,   P_i[a] = k_i . C[a],  Q_i[b] = k_i . (i C[b]),
//   N_a = ||C[a]||^2,  X_ab = 2 C[a] . (i C[b])     (C[a] = the row (x_a^j, y_a^j)_j; i C = (-y, x) per sub-space)
// -- the tables of the key encoder.  The M step is App. A.2's closed form in every sub-space with the common W:
// one matrix T^T S T (it only holds N_ab = sum_i W_i,ab) and one right-hand side per sub-space, which needs
// only the marginals of W:  rhs_j[x_a] = sum_i k_i^jx Wa_i[a] + k_i^jy Wb_i[a],  rhs_j[y_a] = sum_i k_i^jy Wa_i[a] -
// k_i^jx Wb_i[a],  Wa_i[a] = sum_b W_i,ab,  Wb_i[a] = sum_b W_i,ba.
//
// Three kernels: k_ems_accumulate (per workgroup a range of points: N_ab and rhs partials), k_ems_reduce (their sums
// in a fixed order), k_ems_solve.  Index range padded to NP = 8 NB (16, 32 or 64) centres: X_ab = INFINITY there, so the
// weights are exact zeros.
constexpr int kEmsPts = 32;       // points per pass of a workgroup of k_ems_accumulate
constexpr int kEmsThreads = 512;  // 2 wavefronts per SIMD: the 2 NB^2 registers of weights and sums leave no room for more
constexpr int kEmsMaxWg = 256;    // one workgroup per compute unit

typedef float em_f4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ float em_dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppRor8 = 0x128, kDppBcast = 0x150;
// x + y where x's odd 16-lane rows and y's even rows change places (and the same with 32-lane halves): with x == y a
// step of an all-lanes sum, otherwise two sums at once, x's in the even rows and y's in the odd ones
__device__ __forceinline__ float em_swap16_add(float x, float y)
{
    auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float em_swap32_add(float x, float y)
{
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float em_swap_min(float v)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned w = __builtin_bit_cast(unsigned, fminf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])));
    auto t = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return fminf(__builtin_bit_cast(float, (unsigned)t[0]), __builtin_bit_cast(float, (unsigned)t[1]));
}
__device__ __forceinline__ float em_sum8(float v)  // over 8 consecutive lanes
{
    v += em_dpp<kDppXor1>(v);
    v += em_dpp<kDppXor2>(v);
    return v + em_dpp<kDppHalfMirror>(v);
}
__device__ __forceinline__ float em_min8(float v)
{
    v = fminf(v, em_dpp<kDppXor1>(v));
    v = fminf(v, em_dpp<kDppXor2>(v));
    return fminf(v, em_dpp<kDppHalfMirror>(v));
}

// Sizes shared by host and device.
struct EmsDims {
    int np, j2, j16, ps;   // padded centres; sub-spaces padded to 2 and to 16; floats per point row in LDS
    __host__ __device__ EmsDims(int J, int NP) : np(NP), j2((J + 1) & ~1), j16((J + 15) & ~15), ps(2 * ((J + 15) & ~15) + 4) {}
    __host__ __device__ int part() const { return np * np + 2 * j16 * np; }  // floats of a workgroup's partial sums
    __host__ __device__ int lds() const
    {
        const int all = np * np + 2 * kEmsPts * (np + 4) + 9 * np + kEmsPts + kEmsPts * ps + 2 * j2 * np;
        return (all > 4 * np * np ? all : 4 * np * np) * 4;  // the end of the kernel needs 4 planes of N_ab
    }
};

// Workgroup = a range of P points, 32 at a time.  The contractions (X, then P and Q, then the right-hand sides) are fp32
// matrix instructions out of LDS.  The sweep over the centre pairs in between gives a wavefront one point: lane (al, bl)
// holds the pairs a = NB al + .., b = NB bl + .., so that the distances, the weights, both marginals and the
// denominator come from ONE evaluation of each pair, kept in registers until the denominator is known.
//   bound: the quarter-rate v_sqrt_f32 and v_exp_f32, one each per (point, pair), and 8 more operations of the
// vector unit per pair.
// 8192 points, 64 x 64 pairs, 64 sub-spaces: 29 us, of which the sweep 14 and the contractions 9; as separate passes over
// the points (tables, four evaluations of each pair, right-hand sides from the stored marginals) it was 196 us.
template <int NB>
__global__ __launch_bounds__(kEmsThreads) void k_ems_accumulate(const float2 *__restrict__ data, const float2 *__restrict__ phi,
                                                                float *__restrict__ part, int N, int J, int Nc, int P, float c)
{
    constexpr int NP = 8 * NB, NT = NP / 16, US = NP + 4;
    extern __shared__ __attribute__((aligned(16))) float ems_lds[];
    const EmsDims dm(J, NP);
    float *xl = ems_lds;                       // X in the sweep's order: [NB^2 / 4][64 lanes][4]
    float *us = xl + NP * NP;                  // [32][US] N_a - 2 P[a], then Wa
    float *vs = us + kEmsPts * US;             // [32][US] N_b - 2 Q[b], then Wb
    float *na = vs + kEmsPts * US;             // [NP]
    float *nap = na + NP;                      // [8][NP]
    float *kk = nap + 8 * NP;                  // [32] ||k||^2
    float *pts = kk + kEmsPts;                 // [32][ps] (x, y) of the sub-spaces; zeros past J
    float *ph = pts + kEmsPts * dm.ps;         // [j2][NP] (x, y); zeros past J and Nc
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4, gh = g >> 1, gl = g & 1;
    const int first = blockIdx.x * P, last = min(N, first + P);
    {   // every load of the codebook (at most NB a thread) and of the first points under way before the first is used
        float2 pv[NB];
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int x = tid + e * kEmsThreads, j = x / NP, a = x % NP;
            pv[e] = phi[(size_t)min(j, J - 1) * Nc + min(a, Nc - 1)];
            if (j >= J || a >= Nc) pv[e] = make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int x = tid + e * kEmsThreads;
            if (x < dm.j2 * NP) *reinterpret_cast<float2 *>(ph + 2 * x) = pv[e];
        }
    }
    float nacc[NB * NB];
#pragma unroll
    for (int e = 0; e < NB * NB; ++e) nacc[e] = 0.f;
    em_f4 racc[2][2] = {};
    for (int i0 = first; i0 < last; i0 += kEmsPts) {
        const int cnt = min(kEmsPts, last - i0), cnt8 = (cnt + 7) & ~7;
        float2 kv[kEmsPts / 8];
#pragma unroll
        for (int e = 0; e < kEmsPts / 8; ++e) {
            const int i = wave + 8 * e;
            kv[e] = data[(size_t)(i0 + min(i, cnt - 1)) * J + min(lane, J - 1)];
            if (i >= cnt || lane >= J) kv[e] = make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int e = 0; e < kEmsPts / 8; ++e) {
            const int i = wave + 8 * e;
            if (lane < dm.j16) *reinterpret_cast<float2 *>(pts + i * dm.ps + 2 * lane) = kv[e];
            float s = kv[e].x * kv[e].x + kv[e].y * kv[e].y;
            s = em_sum8(s);
            s += em_dpp<kDppRor8>(s);
            s = em_swap16_add(s, s);
            s = em_swap32_add(s, s);
            if (lane == 0) kk[i] = s;
        }
        __syncthreads();
        if (i0 == first) {
            // X_ab = 2 sum_j (y_a x_b - x_a y_b): rows a, columns b, contraction over (j, component); lane (n, g) supplies
            // component g & 1 of sub-space j + (g >> 1)
            constexpr int TW = NT * NT > 8 ? NT * NT / 8 : 1;  // tiles of a wavefront, all of one row of tiles
            if (wave * TW < NT * NT) {
                const int ta = wave * TW / NT, tb = wave * TW % NT;
                const float *pa = ph + 2 * (gh * NP + 16 * ta + n) + 1 - gl, *pb = ph + 2 * (gh * NP + 16 * tb + n) + gl;
                const float sign = gl ? -2.f : 2.f;
                em_f4 acc[TW] = {};
#pragma unroll 8
                for (int j = 0; j < dm.j2; j += 2) {
                    const float av = sign * pa[2 * j * NP];
#pragma unroll
                    for (int e = 0; e < TW; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, pb[2 * j * NP + 32 * e], acc[e], 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < TW; ++e) {
                    const int b = 16 * (tb + e) + n, bl = b / NB, bi = b % NB;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int a = 16 * ta + 4 * g + r, al = a / NB, f = (a % NB) * NB + bi;
                        xl[((f >> 2) * 64 + al * 8 + bl) * 4 + (f & 3)] = a < Nc && b < Nc ? acc[e][r] : INFINITY;
                    }
                }
            }
            for (int x = tid; x < 8 * NP; x += kEmsThreads) {
                const int a = x % NP;
                float s = 0.f;
#pragma unroll 8
                for (int j = x / NP; j < J; j += 8) {
                    const float2 v = *reinterpret_cast<const float2 *>(ph + 2 * (j * NP + a));
                    s += v.x * v.x + v.y * v.y;
                }
                nap[x] = s;
            }
            __syncthreads();
            if (tid < NP) {
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) s += nap[e * NP + tid];
                na[tid] = s;
            }
            __syncthreads();
        }
        // P[i][a] = sum_j k.x x_a + k.y y_a and Q[i][b] = sum_j k.y x_b - k.x y_b: the same right operand
        for (int t = wave; t < (cnt + 15) / 16 * NT; t += 8) {
            const int ti = t / NT, ta = t % NT;
            const float *row = pts + (16 * ti + n) * dm.ps + 2 * gh, *pb = ph + 2 * (gh * NP + 16 * ta + n) + gl;
            em_f4 accp = {}, accq = {};
#pragma unroll 8
            for (int j = 0; j < dm.j2; j += 2) {
                const float kx = row[2 * j], ky = row[2 * j + 1], b = pb[2 * j * NP];
                accp = __builtin_amdgcn_mfma_f32_16x16x4f32(gl ? ky : kx, b, accp, 0, 0, 0);
                accq = __builtin_amdgcn_mfma_f32_16x16x4f32(gl ? -kx : ky, b, accq, 0, 0, 0);
            }
            const float nv = na[16 * ta + n];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * ti + 4 * g + r;
                us[i * US + 16 * ta + n] = nv - 2.f * accp[r];
                vs[i * US + 16 * ta + n] = nv - 2.f * accq[r];
            }
        }
        __syncthreads();
        for (int i = wave; i < cnt8; i += 8) {
            const int al = lane >> 3, bl = lane & 7;
            float *urow = us + i * US + NB * al, *vrow = vs + i * US + NB * bl;
            if (i >= cnt) {  // no point here: zero weights for the contraction below
                if (bl == 0)
                    for (int e = 0; e < NB; ++e) urow[e] = 0.f;
                if (al == 0)
                    for (int e = 0; e < NB; ++e) vrow[e] = 0.f;
                continue;
            }
            float u[NB], v[NB], e[NB * NB];
            const float ki = kk[i];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                u[x] = ki + urow[x];
                v[x] = vrow[x];
            }
#pragma unroll
            for (int q = 0; q < NB * NB / 4; ++q) {
                const em_f4 x4 = *reinterpret_cast<const em_f4 *>(xl + (q * 64 + lane) * 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) e[4 * q + r] = x4[r];
            }
            float d2m = INFINITY;
#pragma unroll
            for (int f = 0; f < NB * NB; ++f) {
                e[f] = u[f / NB] + (v[f % NB] + e[f]);
                d2m = fminf(d2m, e[f]);
            }
            d2m = em_min8(d2m);
            d2m = fminf(d2m, em_dpp<kDppRor8>(d2m));
            d2m = em_swap_min(d2m);
            if (d2m < 0.f) {  // a point on a centre, by rounding
#pragma unroll
                for (int f = 0; f < NB * NB; ++f) e[f] = fmaxf(e[f], 0.f);
                d2m = 0.f;
            }
            // The difference first: the nearest centre's weight is exactly 1 at every temperature.  One fused multiply-add with
            // dmin c would carry the rounding of dmin c, up to 2^-24 dmin c, into every exponent: once T is below some 1e-9 dmin
            // all weights of a point are then 0 or infinity.  (8192 points, 64 x 64 pairs: 44.2 us an iteration against 43.2 with the
            // fused form, 45.2 with a branch between the two.)
            const float dmin = em_sqrt(d2m);
            float row[NB], col[NB];
#pragma unroll
            for (int f = 0; f < NB * NB; ++f) {
                const float w = __builtin_amdgcn_exp2f((dmin - em_sqrt(e[f])) * c);
                e[f] = w;
                row[f / NB] = f % NB == 0 ? w : row[f / NB] + w;
                col[f % NB] = f < NB ? w : col[f % NB] + w;
            }
            float z = 0.f;
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                row[x] = em_sum8(row[x]);
                z += row[x];
            }
            z += em_dpp<kDppRor8>(z);
            z = em_swap16_add(z, z);
            z = em_swap32_add(z, z);
            const float rz = em_rcp(z);
#pragma unroll
            for (int f = 0; f < NB * NB; ++f) nacc[f] = __builtin_fmaf(e[f], rz, nacc[f]);
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                col[x] += em_dpp<kDppRor8>(col[x]);
                col[x] = em_swap16_add(col[x], col[x]);
                col[x] = em_swap32_add(col[x], col[x]);
            }
            if (bl == 0) {
#pragma unroll
                for (int x = 0; x < NB; ++x) urow[x] = row[x] * rz;
            }
            if (al == 0) {
#pragma unroll
                for (int x = 0; x < NB; ++x) vrow[x] = col[x] * rz;
            }
        }
        __syncthreads();
        // rhs_j[x_a] += k.x Wa + k.y Wb, rhs_j[y_a] += k.y Wa - k.x Wb: rows j, columns a, contraction over (point, Wa or Wb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int unit = wave + 8 * t, tj = unit / NT, ta = unit % NT;
            if (tj < dm.j16 / 16) {
                const float *kp = pts + gh * dm.ps + 2 * (16 * tj + n), *wp = (gl ? vs : us) + gh * US + 16 * ta + n;
#pragma unroll 4
                for (int i = 0; i < cnt8; i += 2) {
                    const float2 k = *reinterpret_cast<const float2 *>(kp + i * dm.ps);
                    const float w = wp[i * US];
                    racc[t][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(gl ? k.y : k.x, w, racc[t][0], 0, 0, 0);
                    racc[t][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(gl ? -k.x : k.y, w, racc[t][1], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    // N_ab of the 8 wavefronts, in the sweep's order
    float *slot = ems_lds + (wave & 3) * NP * NP;
    if (wave >= 4) {
#pragma unroll
        for (int q = 0; q < NB * NB / 4; ++q)
            *reinterpret_cast<em_f4 *>(slot + (q * 64 + lane) * 4) = em_f4{nacc[4 * q], nacc[4 * q + 1], nacc[4 * q + 2], nacc[4 * q + 3]};
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll
        for (int q = 0; q < NB * NB / 4; ++q)
            *reinterpret_cast<em_f4 *>(slot + (q * 64 + lane) * 4) += em_f4{nacc[4 * q], nacc[4 * q + 1], nacc[4 * q + 2], nacc[4 * q + 3]};
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t mine = make_rsrc(part + (size_t)blockIdx.x * dm.part(), (unsigned)dm.part() * 4u);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int unit = wave + 8 * t, tj = unit / NT, ta = unit % NT;
        if (tj < dm.j16 / 16) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    store_through(racc[t][x][r], mine, (unsigned)(NP * NP + (x * dm.j16 + 16 * tj + 4 * g + r) * NP + 16 * ta + n) * 4u);
        }
    }
    for (int x = tid; x < NP * NP; x += kEmsThreads)
        store_through((ems_lds[x] + ems_lds[NP * NP + x]) + (ems_lds[2 * NP * NP + x] + ems_lds[3 * NP * NP + x]), mine, (unsigned)x * 4u);
}

// Sums of the workgroups' partials in a fixed order: 16 threads per 4 neighbouring sums take every 16th workgroup.
// Bound by the read of 12.6 MB that the launch before has just written (256 workgroups, largest shape): 4.5 us, and 0.8 less between the
// two launches since those are written through.
__global__ __launch_bounds__(256) void k_ems_reduce(const float *__restrict__ part, float *__restrict__ sums, int n_wg, int len)
{
    __shared__ em_f4 red[16][16];
    const int l = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int at = blockIdx.x * 64 + 4 * l;
    em_f4 s = {};
#pragma unroll 8
    for (int w = q; w < n_wg; w += 16) s += *reinterpret_cast<const em_f4 *>(part + (size_t)w * len + at);
    red[q][l] = s;
    __syncthreads();
    if (q == 0) {
#pragma unroll
        for (int e = 1; e < 16; ++e) s += red[e][l];
        *reinterpret_cast<em_f4 *>(sums + at) = s;
    }
}

// In-place inverse of a symmetric positive definite 16 x 16 block by Gauss-Jordan elimination in one wavefront: lane
// (r, g) holds a[e] = A[r][4 g + e].  Rows and columns travel by DPP and lane swaps: about 120 cycles a pivot.
template <int K>
__device__ __forceinline__ void em_pivot(float (&a)[4], int r, int g)
{
    const float p = em_lane(a[K % 4], K + K / 4 * 16);
    const unsigned own = __builtin_bit_cast(unsigned, a[K % 4]);
    auto s = __builtin_amdgcn_permlane16_swap(own, own, false, false);
    const unsigned w = (unsigned)s[(K / 4) & 1];
    auto t = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const bool is = r == K;
    const float f = is ? -1.f : __builtin_bit_cast(float, (unsigned)t[(K / 4) >> 1]);  // A[r][K] in all four lanes of row r
    const float x = __builtin_amdgcn_rcpf(p), c = 2.f - p * x;  // 1 / p = x c
    const float m = (f * x) * c;
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = __builtin_fmaf(-m, em_dpp<kDppBcast + K>(a[e]), is ? 0.f : a[e]);
    if (g == K / 4) a[K % 4] = -m;  // row K: 1 / p
}
__device__ __forceinline__ void em_invert16(float (&a)[4], int r, int g)
{
    em_pivot<0>(a, r, g), em_pivot<1>(a, r, g), em_pivot<2>(a, r, g), em_pivot<3>(a, r, g);
    em_pivot<4>(a, r, g), em_pivot<5>(a, r, g), em_pivot<6>(a, r, g), em_pivot<7>(a, r, g);
    em_pivot<8>(a, r, g), em_pivot<9>(a, r, g), em_pivot<10>(a, r, g), em_pivot<11>(a, r, g);
    em_pivot<12>(a, r, g), em_pivot<13>(a, r, g), em_pivot<14>(a, r, g), em_pivot<15>(a, r, g);
}

// Solutions for 16 sub-spaces per workgroup.  With the unknowns ordered (x_0 .. x_n, y_0 .. y_n) the system is
//   [D V; V^T D] [x; y] = [rx; ry],   D = diag(sum_b N_ab + N_ba),  V_ab = N_ba - N_ab = -V_ba,
// so the first half of a Cholesky factorisation is a division by D, and what remains is half the order:
//   (D + V D^-1 V) y = ry + V D^-1 rx,   x = D^-1 (rx - V y).
// It is eliminated in blocks of 16 (block Gauss-Jordan: the diagonal blocks' inverses by one wavefront, the rest matrix
// instructions).  Every workgroup repeats the factorisation, a chain that one workgroup runs as fast as many.
// All matrices lie in LDS row by row, right-hand sides one row per sub-space, and the matrix instructions take the
// contraction index in the order 16 s + 4 (lane / 16) + step: operands are float4 reads along a row, a result's lanes
// hold what the next product needs as an operand, and symmetric tiles are stored transposed, again as float4.
//   bound: the chain of NP pivots.  64 x 64 pairs, 64 sub-spaces: 10 us (a Cholesky
// factorisation of the whole system with substitution on the vector unit: 71 us).
constexpr int kEmsSolveThreads = 1024;  // 16 wavefronts: the 14 tiles of the largest reduced system at once
template <int NB>
__global__ __launch_bounds__(kEmsSolveThreads) void k_ems_solve(const float *__restrict__ sums, float2 *__restrict__ phi, int J, int Nc)
{
    constexpr int NP = 8 * NB, NT = NP / 16, LD = NP + 4;
    __shared__ __attribute__((aligned(16))) float nm[NP * LD], vm[NP * LD], rx[16 * LD], ry[16 * LD], pinv[NT * 16 * 20],
        dsum[NP], dinv[NP], dp[8 * NP];
    float *sm = nm;  // the matrix of the reduced system, once N_ab has been read
    const EmsDims dm(J, NP);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int j0 = blockIdx.x * 16;
    {
        constexpr int NE = (NP * NP + kEmsSolveThreads - 1) / kEmsSolveThreads;
        const bool in = tid < 16 * NP;
        const int j = tid / NP, ja = tid % NP;
        const float *rp = sums + NP * NP + (in ? (j0 + j) * NP + ja : 0);
        const float vx = rp[0], vy = rp[dm.j16 * NP];
        float v[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) v[e] = sums[min(tid + e * kEmsSolveThreads, NP * NP - 1)];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int x = tid + e * kEmsSolveThreads, l = (x >> 2) & 63, f = (x >> 8) * 4 + (x & 3);
            if (x < NP * NP) nm[(NB * (l >> 3) + f / NB) * LD + NB * (l & 7) + f % NB] = v[e];
        }
        if (in) {
            rx[j * LD + ja] = vx;
            ry[j * LD + ja] = vy;
        }
    }
    __syncthreads();
    for (int x = tid; x < NP * NP; x += kEmsSolveThreads) {
        const int a = x / NP, b = x % NP;
        vm[a * LD + b] = nm[b * LD + a] - nm[a * LD + b];
    }
    if (tid < 8 * NP) {
        const int a = tid % NP, b0 = tid / NP;
        float s = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) s += nm[a * LD + b0 + 8 * b] + nm[(b0 + 8 * b) * LD + a];
        dp[tid] = s;
    }
    __syncthreads();
    if (tid < NP) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += dp[e * NP + tid];
        s = tid < Nc ? s : 1.f;
        dsum[tid] = s;
        dinv[tid] = 1.f / s;
    }
    __syncthreads();
    // C + A B over all NP, A's rows at ap, B's columns at bp; two chains, since each step waits for the one before
    auto product = [&](em_f4 acc, const float *ap, const float *bp, auto scale) {
        em_f4 acc2 = {};
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            const em_f4 av = *reinterpret_cast<const em_f4 *>(ap + 16 * s + 4 * g);
            const em_f4 bv = *reinterpret_cast<const em_f4 *>(bp + 16 * s + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                em_f4 &to = r & 1 ? acc2 : acc;
                to = __builtin_amdgcn_mfma_f32_16x16x4f32(av[r], scale(16 * s + 4 * g + r) * bv[r], to, 0, 0, 0);
            }
        }
        return acc + acc2;
    };
    // tiles (ti, tj), ti <= tj < NT: D + V D^-1 V (V[k][b] = -V[b][k]), as tile [tj][ti]; tj = NT: ry + V D^-1 rx
    int unit = 0;
#pragma unroll
    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
        for (int tj = ti; tj <= NT; ++tj) {
            if (unit++ != wave) continue;
            float *row = tj < NT ? sm + (16 * tj + n) * LD : ry + n * LD;
            em_f4 acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int a = 16 * ti + 4 * g + r;
                acc[r] = tj == NT ? row[a] : a == 16 * tj + n ? dsum[a] : 0.f;
            }
            acc = product(acc, vm + (16 * ti + n) * LD, tj < NT ? vm + (16 * tj + n) * LD : rx + n * LD,
                          [&](int k) { return tj < NT ? -dinv[k] : dinv[k]; });
            *reinterpret_cast<em_f4 *>(row + 16 * ti + 4 * g) = acc;
        }
    __syncthreads();
    // Stage k: S_ij -= S_ik P_k S_kj, P_k = S_kk^-1, for every i other than k and j > k (j = NT: the right-hand sides).  i < k
    // takes the place of a back substitution; tile (i, j) is kept as [j][i].  Wavefront 0 takes (k + 1, k + 1), which
    // leaves the matrix unit in the order that the inversion starts from, and inverts it while the others update.
    auto update = [&](int k, int i, int j) {
        const em_f4 pv = *reinterpret_cast<const em_f4 *>(pinv + (k * 16 + n) * 20 + 4 * g);
        em_f4 iv;
        if (i > k) {
            iv = *reinterpret_cast<const em_f4 *>(sm + (16 * i + n) * LD + 16 * k + 4 * g);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) iv[r] = sm[(16 * k + 4 * g + r) * LD + 16 * i + n];
        }
        float *row = j < NT ? sm + (16 * j + n) * LD : ry + n * LD;
        const em_f4 jv = *reinterpret_cast<const em_f4 *>(row + 16 * k + 4 * g);
        em_f4 acc = *reinterpret_cast<const em_f4 *>(row + 16 * i + 4 * g), acc2 = {}, m = {}, m2 = {};
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            m = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[r], iv[r], m, 0, 0, 0);
            m2 = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[r + 1], iv[r + 1], m2, 0, 0, 0);
        }
        m += m2;
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-m[r], jv[r], acc, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(-m[r + 1], jv[r + 1], acc2, 0, 0, 0);
        }
        return acc + acc2;
    };
    auto invert = [&](int k, em_f4 blk) {
        float a[4] = {blk[0], blk[1], blk[2], blk[3]};
        em_invert16(a, n, g);
        *reinterpret_cast<em_f4 *>(pinv + (k * 16 + n) * 20 + 4 * g) = em_f4{a[0], a[1], a[2], a[3]};
    };
    if (wave == 0) invert(0, *reinterpret_cast<const em_f4 *>(sm + n * LD + 4 * g));
    __syncthreads();
    for (int k = 0; k < NT; ++k) {
        if (wave == 0) {
            if (k + 1 < NT) invert(k + 1, update(k, k + 1, k + 1));
        } else {
            int left = wave - 1;  // the unit of this wavefront among the stage's (i, j)
            for (int i = 0; i < NT; ++i) {
                if (i == k) continue;
                const int from = i < k ? k + 1 : i == k + 1 ? i + 1 : i;
                if (left <= NT - from) {
                    const int j = from + left;
                    const em_f4 acc = update(k, i, j);
                    *reinterpret_cast<em_f4 *>((j < NT ? sm + (16 * j + n) * LD : ry + n * LD) + 16 * i + 4 * g) = acc;
                    break;
                }
                left -= NT - from + 1;
            }
        }
        __syncthreads();
    }
    if (wave < NT) {  // y_k = P_k ry_k
        float *yp = ry + n * LD + 16 * wave + 4 * g;
        const em_f4 pv = *reinterpret_cast<const em_f4 *>(pinv + (wave * 16 + n) * 20 + 4 * g), yv = *reinterpret_cast<const em_f4 *>(yp);
        em_f4 acc = {};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[r], yv[r], acc, 0, 0, 0);
        *reinterpret_cast<em_f4 *>(yp) = acc;
    }
    __syncthreads();
    if (wave < NT) {  // x = D^-1 (rx - V y)
        const em_f4 acc = product(*reinterpret_cast<const em_f4 *>(rx + n * LD + 16 * wave + 4 * g), vm + (16 * wave + n) * LD,
                                  ry + n * LD, [](int) { return -1.f; });
        if (j0 + n < J) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int a = 16 * wave + 4 * g + r;
                if (a < Nc) phi[(size_t)(j0 + n) * Nc + a] = make_float2(acc[r] * dinv[a], ry[n * LD + a]);
            }
        }
    }
}

// Points per workgroup: a wavefront has one at a time, and up to 256 workgroups (one per compute unit) share the points
// before any of them gets a second round of 8.
struct EmsLayout {
    int n_wg, per, np, len;
    size_t part, sums, bytes;
};
inline EmsLayout ems_layout(int J, int N, int Nc)
{
    EmsLayout l;
    l.np = Nc <= 16 ? 16 : Nc <= 32 ? 32 : 64;
    l.per = ((N + kEmsMaxWg - 1) / kEmsMaxWg + 7) / 8 * 8;
    l.n_wg = (N + l.per - 1) / l.per;
    l.len = EmsDims(J, l.np).part();
    l.part = 0;
    l.sums = em_align((size_t)l.n_wg * l.len * 4);
    l.bytes = l.sums + em_align((size_t)l.len * 4);
    return l;
}

template <int NB>
inline commvq_status ems_launch(const EmsLayout &l, const float2 *data, float2 *phi, float *part, float *sums, int N, int J, int Nc,
                                float c, hipStream_t s)
{
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_ems_accumulate<NB>, EmsDims(64, 8 * NB).lds(), lds_ok) != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_ems_accumulate<NB>, dim3((unsigned)l.n_wg), dim3(kEmsThreads), EmsDims(J, 8 * NB).lds(), s, data, phi, part,
                       N, J, Nc, l.per, c);
    if (hipGetLastError() != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_ems_reduce, dim3((unsigned)(l.len / 64)), dim3(256), 0, s, part, sums, l.n_wg, l.len);
    if (hipGetLastError() != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_ems_solve<NB>, dim3((unsigned)((J + 15) / 16)), dim3(kEmsSolveThreads), 0, s, sums, phi, J, Nc);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

}  // namespace

extern "C" {

commvq_status commvq_em_workspace_bytes(int32_t n_subspaces, int32_t n_points, int32_t n_centres, size_t *bytes)
{
    if (!bytes) return COMMVQ_ERR_NULL;
    // sub-spaces are the y dimension of the launch grids (at most 65535); point indices are 32-bit
    if (n_subspaces < 1 || n_subspaces > 65535 || n_points < 1 || n_points > (1 << 24) || n_centres < 1 || n_centres > kEmMaxNc)
        return COMMVQ_ERR_SHAPE;
    const size_t pts = (size_t)n_subspaces * n_points, cen = (size_t)n_subspaces * n_centres * n_centres;
    *bytes = 2 * em_align(pts * 4) + em_align(cen * 4) + em_align(cen * 8);
    return COMMVQ_OK;
}

commvq_status commvq_em_step(const float *data, int32_t n_subspaces, int32_t n_points, int32_t n_centres,
                             float temperature, float *phi, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!data || !phi || !workspace) return COMMVQ_ERR_NULL;
    size_t need = 0;
    commvq_status st = commvq_em_workspace_bytes(n_subspaces, n_points, n_centres, &need);
    if (st != COMMVQ_OK) return st;
    if (!(temperature > 0.f)) return COMMVQ_ERR_CONFIG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need) return COMMVQ_ERR_WORKSPACE;
    const size_t pts = (size_t)n_subspaces * n_points, cen = (size_t)n_subspaces * n_centres * n_centres;
    char *w = static_cast<char *>(workspace);
    float *dmin = reinterpret_cast<float *>(w);
    float *zsum = reinterpret_cast<float *>(w + em_align(pts * 4));
    float *nab = reinterpret_cast<float *>(w + 2 * em_align(pts * 4));
    float2 *sab = reinterpret_cast<float2 *>(w + 2 * em_align(pts * 4) + em_align(cen * 4));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const float inv_t = std::min(1.f / temperature, FLT_MAX / 2.f);  // finite, and times log2 e too: the nearest centre's exponent is 0 times it
    const float2 *d2 = reinterpret_cast<const float2 *>(data);
    float2 *p2 = reinterpret_cast<float2 *>(phi);
    hipLaunchKernelGGL(k_em_norm, dim3((unsigned)((n_points + 255) / 256), (unsigned)n_subspaces), dim3(256), 0, s, d2, p2,
                       dmin, zsum, n_points, n_centres, inv_t);
    if (hipGetLastError() != hipSuccess) return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_em_accum, dim3((unsigned)((n_centres * n_centres + 255) / 256), (unsigned)n_subspaces), dim3(256), 0, s,
                       d2, p2, dmin, zsum, nab, sab, n_points, n_centres, inv_t);
    if (hipGetLastError() != hipSuccess) return COMMVQ_ERR_LAUNCH;
    const int np = (2 * n_centres + 15) / 16 * 16;  // the system padded to whole 16-column blocks
    const int lds = (np * (np + 1) + np + np * 16) * 4;
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(&k_em_solve, (2 * kEmMaxNc * (2 * kEmMaxNc + 1) + 2 * kEmMaxNc + 2 * kEmMaxNc * 16) * 4, lds_ok) != hipSuccess)
        return COMMVQ_ERR_LAUNCH;
    hipLaunchKernelGGL(k_em_solve, dim3((unsigned)n_subspaces), dim3(256), lds, s, nab, sab, p2, n_centres);
    return hipGetLastError() == hipSuccess ? COMMVQ_OK : COMMVQ_ERR_LAUNCH;
}

commvq_status commvq_em_shared_workspace_bytes(int32_t group, int32_t n_points, int32_t n_centres, size_t *bytes)
{
    if (!bytes) return COMMVQ_ERR_NULL;
    if (group < 1 || group > 64 || n_points < 1 || n_points > (1 << 24) || n_centres < 1 || n_centres > kEmMaxNc) return COMMVQ_ERR_SHAPE;
    *bytes = ems_layout(group, n_points, n_centres).bytes;
    return COMMVQ_OK;
}

commvq_status commvq_em_step_shared(const float *data, int32_t group, int32_t n_points, int32_t n_centres, float temperature,
                                    float *phi, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!data || !phi || !workspace) return COMMVQ_ERR_NULL;
    size_t need = 0;
    commvq_status st = commvq_em_shared_workspace_bytes(group, n_points, n_centres, &need);
    if (st != COMMVQ_OK) return st;
    if (!(temperature > 0.f)) return COMMVQ_ERR_CONFIG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need) return COMMVQ_ERR_WORKSPACE;
    const int J = group, N = n_points, Nc = n_centres;
    const EmsLayout l = ems_layout(J, N, Nc);
    char *w = static_cast<char *>(workspace);
    float *part = reinterpret_cast<float *>(w + l.part), *sums = reinterpret_cast<float *>(w + l.sums);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const float2 *d2 = reinterpret_cast<const float2 *>(data);
    float2 *p2 = reinterpret_cast<float2 *>(phi);
    // A normal, finite number for every T > 0: 0 (T = infinity) would make NaN of the padding's infinite distances, infinity
    // of the nearest centre's zero.  At either end the weights are what they would be beyond it: all alike, or one centre's.
    const float c = std::min(std::max(kLog2eEm / temperature, FLT_MIN), FLT_MAX);
    switch (l.np) {
        case 16: return ems_launch<2>(l, d2, p2, part, sums, N, J, Nc, c, s);
        case 32: return ems_launch<4>(l, d2, p2, part, sums, N, J, Nc, c, s);
        default: return ems_launch<8>(l, d2, p2, part, sums, N, J, Nc, c, s);
    }
}

}  // extern "C"
